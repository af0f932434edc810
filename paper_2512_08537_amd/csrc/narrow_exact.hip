// The narrow-tile GEMM (narrow.hip) for the products a round spends most of its launches on: K a whole number of
// 32-k steps per wave (K slice = 128 NS with NS in {8, 10, 12, 16}) and one of a dozen epilogues, both fixed at compile time.
//
// What bounds such a launch is not memory but its own instruction stream: a workgroup runs once, on a cold instruction
// cache.  Time stamps in the general kernel (8 rows x 1024 x 1024, one of a chain of dependent launches, weights in HBM;
// 4.8 us a launch, 1.2 of it the gap to the next): the first kernel argument 0.4 us after the wave starts, the last operand
// load issued at 1.3, the last epilogue operand requested at 2.2 - when the operands themselves have long arrived - and
// 0.5-1.0 from the last MFMA to the store.  So here
//   - the arguments that the operand loads need come first and fit the preloaded scalar registers;
//   - every address is a uniform base plus one 32-bit lane offset; strides that depend on the layout (row-major or tile
//     order) come from the host as numbers, not as branches;
//   - nothing branches before the operands, the epilogue's operands and the device-side row count are all requested: absent
//     bias or row count is a select on a loaded value;
//   - only the waves that write (MT NT of the four) request the epilogue's operands.
// K shares: 1024, 1280 and 1536 are the model widths this was measured at, 2048 the share of a wave's 16 steps, the most that
// the tiles hold.  A further share is 18 to 29 instances more; other multiples of 128 stay with the general kernel, unmeasured.
// Measured over whole rounds, general kernel -> this one: one sample of 24 layers of 1024 3.31 -> 2.97 ms (566 launches), eight
// samples of 40 layers of 5120 with its 12-block head 16.8 -> 15.5 ms, four rounds of 32 samples of 1024 16.0 -> 14.2 ms.
#include "gemm.h"

namespace fard {

namespace {

enum NarrowMode {
  NM_STORE,        // bf16 rows
  NM_GELU,         // bf16 gelu
  NM_SILU,         // bf16 silu
  NM_F32,          // fp32 rows
  NM_RESID,        // fp32 +=
  NM_RESID_COPY,   // fp32 += and a bf16 copy of the updated rows
  NM_GATE,         // fp32 += gate *
  NM_PARTIAL,      // fp32 plane of a K slice
  NM_LNF_GELU,     // bf16 gelu of a product of raw rows, norm folded in (GemmArgs::ln_cs)
  NM_ADA_SILU,     // bf16 silu, modulated norm folded in (GemmArgs::ada_mom)
  NM_ADA_GATE,     // NM_GATE + bf16 rows times (1 + copy_scale) + tile moments (GemmArgs::copy_scale, mom_out)
};

struct NarrowTail {                  // what follows the preloaded arguments
  const int* m_dev;                  // device-side row count, or any readable address (has_m = 0)
  const float* bias;                 // [N], or any readable N floats (has_bias = 0)
  void* out;
  const float* x0;                   // gate [M, ldx] | column sums of the folded norm [N] | c1 [M, ldx]
  const float* x1;                   // c0 [M, ldx] | copy_scale [M, ldx1]
  float* mom;                        // tile moments, read (ADA_SILU) or written (ADA_GATE)
  bf16* copy;
  unsigned ldo, ldx, ldx1, mom_ld;   // elements
  unsigned o_hi, o_lo, o_c32, o_c8;  // bf16 output: element strides of a 16-row tile, a row in it, 32 columns, 8 columns
  unsigned plane;                    // NM_PARTIAL: floats between planes
  float eps;
  int has_m, has_bias, rms;
};

template <int MT, int NT, int NS, int MODE>
__global__ __launch_bounds__(256, (MT == 2 && NT == 4) ? 2 : 1) void gemm_narrow_exact_kernel(
    const char* __restrict__ W, const char* __restrict__ A, unsigned a_hi, unsigned a_lo, unsigned a_kg, unsigned a_step, int Mh,
    unsigned kb16, NarrowTail t) {
  constexpr bool LNF = MODE == NM_LNF_GELU, ADA_IN = MODE == NM_ADA_SILU, ADA_OUT = MODE == NM_ADA_GATE;
  constexpr bool GATE = MODE == NM_GATE || ADA_OUT;
  constexpr bool RMW = GATE || MODE == NM_RESID || MODE == NM_RESID_COPY;
  constexpr bool OUT16 = MODE == NM_STORE || MODE == NM_GELU || MODE == NM_SILU || LNF || ADA_IN;
  constexpr int ACT = (MODE == NM_GELU || LNF) ? ACT_GELU : ((MODE == NM_SILU || ADA_IN) ? ACT_SILU : ACT_NONE);
  constexpr int ROWS = 16 * MT, CG = 4 * NT, RPP = 256 / CG, EP = (ROWS + RPP - 1) / RPP, LDT = 16 * NT + 4;
  constexpr unsigned WAVES_OUT = MT * NT < 4 ? MT * NT : 4;   // waves that hold output rows
  constexpr int TPR = 256 / ROWS, MOMT = 8 * NS / TPR;        // threads that share a row's tile moments; moments a thread
  __shared__ __attribute__((aligned(16))) float red[4 * ROWS * LDT];
  __shared__ float stat[LNF ? 4 * ROWS * 2 : 1];
  __shared__ float rowstat[ADA_IN ? ROWS * 2 : 1];

  const unsigned tid = threadIdx.x, lane = tid & 63u, kw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned kg = lane >> 4, l16 = lane & 15u;
  const unsigned row_tile = blockIdx.y * MT, m0 = row_tile * 16;
  const unsigned n0 = blockIdx.x * 16 * NT;
  const unsigned s0 = (MODE == NM_PARTIAL ? blockIdx.z * (4 * NS) : 0) + kw;   // this wave's first 32-k step; then every fourth

  // operands: steps s0, s0 + 4, ... of the packed weights (2 KiB a step and 32 columns) and of the rows
  const unsigned wl = (lane >> 5) * 1024 + (kg & 1u) * 512 + l16 * 16;
  bf16x8 breg[NS][NT], areg[NS][MT];
  {
    const char* wb[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const unsigned c16 = blockIdx.x * NT + j;
      wb[j] = W + (size_t)(c16 >> 1) * kb16 * 1024 + (c16 & 1u) * 256 + s0 * 2048;
    }
    const char* ab[MT];
    unsigned al[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const unsigned last = (unsigned)Mh - 1;
      unsigned tile = row_tile + i;                        // (a workgroup's last row tile may lie past the matrix)
      if (MT > 1) tile = tile < (last >> 4) ? tile : (last >> 4);
      const unsigned top = last - tile * 16;
      ab[i] = A + (size_t)tile * a_hi + (size_t)s0 * a_step;
      al[i] = (l16 < top ? l16 : top) * a_lo + kg * a_kg;
    }
    unsigned w_step = 8192;                                // opaque: the bases advance in scalar registers
    asm("" : "+s"(w_step));
#pragma unroll
    for (int p = 0; p < NS; ++p) {
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        breg[p][j] = *(const bf16x8*)(wb[j] + wl);
        wb[j] += w_step;
      }
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        areg[p][i] = *(const bf16x8*)(ab[i] + al[i]);
        ab[i] += 4 * a_step;
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // operands of the epilogue: thread -> 4 columns of rows er, er + RPP, ...
  const unsigned er = tid / CG, ec = (tid % CG) * 4;
  f32x4 bias4, cs4, gate[EP], old[EP], c1[EP], c0[EP];
  float mom_m[ADA_IN ? MOMT : 1], mom_q[ADA_IN ? MOMT : 1], pivot = 0.f;
  const int m_read = *t.m_dev;
  if constexpr (ADA_IN) {
    unsigned r = m0 + tid / TPR;
    r = r < (unsigned)Mh ? r : (unsigned)Mh - 1;
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2* mp = (const f32x2*)t.mom;
    const unsigned mo = r * t.mom_ld, t0 = tid % TPR;
    pivot = mp[mo][0];
#pragma unroll
    for (int i = 0; i < MOMT; ++i) {
      const f32x2 q = mp[mo + t0 + TPR * i];
      mom_m[i] = q[0];
      mom_q[i] = q[1];
    }
  }
  if (WAVES_OUT == 4 || kw < WAVES_OUT) {
    bias4 = *(const f32x4*)(t.bias + (n0 + ec));
    if constexpr (LNF) cs4 = *(const f32x4*)(t.x0 + (n0 + ec));
#pragma unroll
    for (int i = 0; i < EP; ++i) {
      unsigned r = m0 + er + RPP * i;
      r = r < (unsigned)Mh ? r : (unsigned)Mh - 1;
      if constexpr (RMW) old[i] = *(const f32x4*)((const float*)t.out + (r * t.ldo + n0 + ec));
      if constexpr (GATE) gate[i] = *(const f32x4*)(t.x0 + (r * t.ldx + n0 + ec));
      if constexpr (ADA_IN) {
        c1[i] = *(const f32x4*)(t.x0 + (r * t.ldx + n0 + ec));
        c0[i] = *(const f32x4*)(t.x1 + (r * t.ldx + n0 + ec));
      }
      if constexpr (ADA_OUT) c1[i] = *(const f32x4*)(t.x1 + (r * t.ldx1 + n0 + ec));
    }
  }
  const int M = (t.has_m && m_read < Mh) ? m_read : Mh;
  if ((int)m0 >= M) return;                                // (uniform over the workgroup)
  __builtin_amdgcn_sched_barrier(0);

  f32x4 acc[MT][NT];
  float s1[MT], s2[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    s1[i] = s2[i] = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int g = 0; g < NS; ++g) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const bf16x8 af = areg[g][i];
      if constexpr (LNF) {
        // sum x and sum x^2 of the fragment's 8 values, two per instruction (v_dot2c_f32_bf16: fp32 accumulate)
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        bf16x2 ones;
        ones[0] = (bf16)1.0f;
        ones[1] = (bf16)1.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bf16x2 pr;
          pr[0] = af[2 * e];
          pr[1] = af[2 * e + 1];
          s1[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, s1[i], false);
          s2[i] = __builtin_amdgcn_fdot2_f32_bf16(pr, pr, s2[i], false);
        }
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, breg[g][j], acc[i][j], 0, 0, 0);
    }
  }

  // ---- the four waves' partial tiles meet in LDS
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) red[(kw * ROWS + 16 * i + 4 * kg + e) * LDT + 16 * j + l16] = acc[i][j][e];
  if constexpr (LNF) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      s1[i] = xor32_sum(xor16_sum(s1[i]));
      s2[i] = xor32_sum(xor16_sum(s2[i]));
      if (lane < 16) {
        stat[(kw * ROWS + 16 * i + lane) * 2] = s1[i];
        stat[(kw * ROWS + 16 * i + lane) * 2 + 1] = s2[i];
      }
    }
  }
  if constexpr (ADA_IN) {
    // mean and 1 / std of the rows from the tile moments (pairwise update of Chan et al. for equal counts, about the first
    // tile's mean)
    float sd = 0.f, sd2 = 0.f, sq = 0.f;
#pragma unroll
    for (int i = 0; i < MOMT; ++i) {
      const float d = mom_m[i] - pivot;
      sd += d;
      sd2 = fmaf(d, d, sd2);
      sq += mom_q[i];
    }
    auto sum = [](float v) {
      v += dpp_move<DPP_SWAP1>(v);
      v += dpp_move<DPP_SWAP2>(v);
      v += dpp_move<DPP_HALF_MIRROR>(v);
      if (TPR == 16) v += dpp_move<DPP_MIRROR>(v);
      return v;
    };
    sd = sum(sd); sd2 = sum(sd2); sq = sum(sq);
    if (tid % TPR == 0) {
      constexpr float inv_t = 1.0f / (8 * NS);
      const float m2 = sq + 16.0f * fmaxf(sd2 - sd * sd * inv_t, 0.f);
      rowstat[(tid / TPR) * 2] = pivot + sd * inv_t;
      rowstat[(tid / TPR) * 2 + 1] = 1.0f / sqrtf(m2 / (float)(128 * NS) + t.eps);
    }
  }
  __syncthreads();
  if (WAVES_OUT < 4 && kw >= WAVES_OUT) return;
#pragma unroll
  for (int i = 0; i < EP; ++i) {
    const unsigned row = er + RPP * i, gr = m0 + row;
    if ((int)gr >= M) continue;
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) v += *(const f32x4*)(red + (k * ROWS + row) * LDT + ec);
    if constexpr (LNF) {
      float a1 = 0.f, a2 = 0.f;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a1 += stat[(k * ROWS + row) * 2];
        a2 += stat[(k * ROWS + row) * 2 + 1];
      }
      constexpr float inv_k = 1.0f / (128 * NS);
      const float mean = t.rms ? 0.f : a1 * inv_k;
      const float rstd = rsqrtf(fmaxf(a2 * inv_k - mean * mean, 0.f) + t.eps);
      v = (v - cs4 * mean) * rstd;
    }
    if constexpr (ADA_IN) v = (v - c1[i] * rowstat[row * 2]) * rowstat[row * 2 + 1] + c0[i];
    if (t.has_bias && (MODE != NM_PARTIAL || blockIdx.z == 0)) v += bias4;
    if constexpr (OUT16) {
      bf16x4 b;
#pragma unroll
      for (int e = 0; e < 4; ++e) b[e] = (bf16)apply_act<true>(v[e], ACT);
      const unsigned gc = n0 + ec;
      const unsigned o = (row_tile + (row >> 4)) * t.o_hi + (row & 15u) * t.o_lo + (gc >> 5) * t.o_c32 + ((gc >> 3) & 3u) * t.o_c8 + (gc & 7u);
      *(bf16x4*)((bf16*)t.out + o) = b;
    } else {
      const unsigned o = gr * t.ldo + n0 + ec;
      if constexpr (MODE == NM_PARTIAL) {
        *(f32x4*)((float*)t.out + (size_t)blockIdx.z * t.plane + o) = v;
      } else if constexpr (!RMW) {
        *(f32x4*)((float*)t.out + o) = v;
      } else {
        f32x4 nv;
        if constexpr (GATE) nv = old[i] + gate[i] * v; else nv = old[i] + v;
        *(f32x4*)((float*)t.out + o) = nv;
        if constexpr (MODE == NM_RESID_COPY || ADA_OUT) {
          bf16x4 b;
#pragma unroll
          for (int e = 0; e < 4; ++e) b[e] = (bf16)(ADA_OUT ? nv[e] * (1.0f + c1[i][e]) : nv[e]);
          const unsigned gc = n0 + ec;
          const unsigned oc = (row_tile + (row >> 4)) * t.o_hi + (row & 15u) * t.o_lo + (gc >> 5) * t.o_c32 + ((gc >> 3) & 3u) * t.o_c8 + (gc & 7u);
          *(bf16x4*)(t.copy + oc) = b;
        }
        if constexpr (ADA_OUT) {
          // moments of the updated row over this 16-column tile: its 4 threads are one quad of lanes (the quad shares the
          // row, so it is whole or skipped as one)
          float sm = (nv[0] + nv[1]) + (nv[2] + nv[3]);
          sm += dpp_move<DPP_SWAP1>(sm);
          sm += dpp_move<DPP_SWAP2>(sm);
          const float mean = sm * (1.0f / 16.0f);
          float q = 0.f;
#pragma unroll
          for (int e = 0; e < 4; ++e) { const float d = nv[e] - mean; q = fmaf(d, d, q); }
          q += dpp_move<DPP_SWAP1>(q);
          q += dpp_move<DPP_SWAP2>(q);
          typedef float f32x2 __attribute__((ext_vector_type(2)));
          if ((tid & 3u) == 0) *((f32x2*)t.mom + (gr * t.mom_ld + ((n0 + ec) >> 4))) = f32x2{mean, q};
        }
      }
    }
  }
}

// The epilogue of a as a mode of the kernel above, -1 where it has none.
int narrow_mode(const GemmArgs& a) {
  const bool ada_in = a.ada_mom != nullptr, lnf = a.ln_cs != nullptr;
  if ((a.copy_scale != nullptr) != (a.mom_out != nullptr) || (ada_in && (lnf || a.mom_out != nullptr))) return -1;
  switch (a.epi) {
    case EPI_STORE:
      if (ada_in) return a.act == ACT_SILU ? NM_ADA_SILU : -1;
      if (lnf) return a.act == ACT_GELU ? NM_LNF_GELU : -1;
      return a.act == ACT_GELU ? NM_GELU : (a.act == ACT_SILU ? NM_SILU : NM_STORE);
    case EPI_STORE_F32: return (ada_in || lnf || a.act != ACT_NONE) ? -1 : NM_F32;
    case EPI_RESID: return (ada_in || lnf || a.mom_out != nullptr) ? -1 : (a.copy_bf16 != nullptr ? NM_RESID_COPY : NM_RESID);
    case EPI_GATE_RESID:
      if (ada_in || lnf) return -1;
      return a.mom_out != nullptr ? (a.copy_bf16 != nullptr ? NM_ADA_GATE : -1) : (a.copy_bf16 != nullptr ? -1 : NM_GATE);
    case EPI_PARTIAL: return NM_PARTIAL;
    default: return -1;
  }
}

}  // namespace

bool launch_narrow_exact(hipStream_t s, const GemmArgs& a, hipError_t* err) {
  const int kz = (a.epi == EPI_PARTIAL && a.k_slices > 1) ? a.k_slices : 1;
  if (a.K % (128 * kz) != 0) return false;
  const int ns = a.K / (128 * kz), mode = narrow_mode(a);
  if (mode < 0) return false;
  // every offset below is 32-bit
  const size_t lim = (size_t)1 << 30;
  const size_t rows = (size_t)a.M + 32;
  if (rows * (size_t)a.lda >= lim || rows * (size_t)a.ldo >= lim || rows * (size_t)a.N >= lim || rows * (size_t)a.K >= lim ||
      rows * (size_t)a.ldg >= lim || rows * (size_t)a.ada_ld >= lim || rows * (size_t)a.copy_ld >= lim ||
      rows * (size_t)(a.mom_ld + a.ada_mom_ld) >= lim || a.part_stride >= lim)
    return false;
  NarrowTail t{};
  t.has_m = a.m_dev != nullptr;
  t.m_dev = t.has_m ? a.m_dev : (const int*)a.W;
  t.has_bias = a.bias != nullptr;
  t.bias = t.has_bias ? a.bias : (const float*)a.W;          // (K >= 128 rows of N bf16: at least N floats)
  t.out = a.out;
  t.ldo = (unsigned)a.ldo;
  t.copy = (bf16*)a.copy_bf16;
  const bool tiled = a.out_tiled != 0;
  t.o_hi = tiled ? (unsigned)a.N * 16 : (unsigned)a.ldo * 16;
  t.o_lo = tiled ? 8 : (unsigned)a.ldo;
  t.o_c32 = tiled ? 512 : 32;
  t.o_c8 = tiled ? 128 : 8;
  t.plane = (unsigned)a.part_stride;
  if (mode == NM_GATE || mode == NM_ADA_GATE) { t.x0 = a.gate; t.ldx = (unsigned)a.ldg; }
  if (mode == NM_ADA_GATE) { t.x1 = a.copy_scale; t.ldx1 = (unsigned)a.copy_ld; t.mom = a.mom_out; t.mom_ld = (unsigned)a.mom_ld; }
  if (mode == NM_LNF_GELU) { t.x0 = a.ln_cs; t.eps = a.ln_eps; t.rms = a.ln_rms; }
  if (mode == NM_ADA_SILU) {
    t.x0 = a.ada_c1; t.x1 = a.ada_c0; t.ldx = (unsigned)a.ada_ld; t.eps = a.ada_eps;
    t.mom = (float*)a.ada_mom; t.mom_ld = (unsigned)a.ada_mom_ld;
  }
  const unsigned a_hi = a.a_tiled ? (unsigned)a.K * 32 : (unsigned)a.lda * 32, a_lo = a.a_tiled ? 16 : (unsigned)a.lda * 2;
  const unsigned a_kg = a.a_tiled ? 256 : 16, a_step = a.a_tiled ? 1024 : 64;
#define FARD_NX(MTV, NTV, NSV, MODEV)                                                                                          \
  case MODEV:                                                                                                                  \
    gemm_narrow_exact_kernel<MTV, NTV, NSV, MODEV><<<dim3(a.N / (16 * NTV), (a.M + 16 * MTV - 1) / (16 * MTV), kz), 256, 0, s>>>( \
        (const char*)a.W, (const char*)a.A, a_hi, a_lo, a_kg, a_step, a.M, (unsigned)a.K >> 4, t);                             \
    break
#define FARD_NX_ALL(MTV, NTV, NSV)                                                                              \
  FARD_NX(MTV, NTV, NSV, NM_STORE); FARD_NX(MTV, NTV, NSV, NM_GELU); FARD_NX(MTV, NTV, NSV, NM_F32);            \
  FARD_NX(MTV, NTV, NSV, NM_RESID); FARD_NX(MTV, NTV, NSV, NM_RESID_COPY); FARD_NX(MTV, NTV, NSV, NM_PARTIAL);  \
  FARD_NX(MTV, NTV, NSV, NM_LNF_GELU)
#define FARD_NX_HEAD(MTV, NTV, NSV) FARD_NX(MTV, NTV, NSV, NM_SILU); FARD_NX(MTV, NTV, NSV, NM_GATE)
#define FARD_NX_ADA(MTV, NTV, NSV) FARD_NX(MTV, NTV, NSV, NM_ADA_SILU); FARD_NX(MTV, NTV, NSV, NM_ADA_GATE)
#define FARD_NX_SHAPE(...)        \
  do {                            \
    switch (mode) {               \
      __VA_ARGS__;                \
      default: return false;      \
    }                             \
  } while (0)
  // the tiles are those of launch_gemm_narrow (measured there)
  if (a.M <= 64) {
    if (a.N >= 2048 && mode != NM_ADA_SILU && mode != NM_ADA_GATE) {
      if (ns == 8) FARD_NX_SHAPE(FARD_NX_ALL(1, 2, 8));
      else if (ns == 10) FARD_NX_SHAPE(FARD_NX_ALL(1, 2, 10));
      else if (ns == 12) FARD_NX_SHAPE(FARD_NX_ALL(1, 2, 12));
      else if (ns == 16) FARD_NX_SHAPE(FARD_NX_ALL(1, 2, 16));
      else return false;
    } else {
      if (ns == 8) FARD_NX_SHAPE(FARD_NX_ALL(1, 1, 8); FARD_NX_HEAD(1, 1, 8); FARD_NX_ADA(1, 1, 8));
      else if (ns == 10) FARD_NX_SHAPE(FARD_NX_ALL(1, 1, 10); FARD_NX_HEAD(1, 1, 10); FARD_NX_ADA(1, 1, 10));
      else if (ns == 12) FARD_NX_SHAPE(FARD_NX_ALL(1, 1, 12); FARD_NX_HEAD(1, 1, 12); FARD_NX_ADA(1, 1, 12));
      else if (ns == 16) FARD_NX_SHAPE(FARD_NX_ALL(1, 1, 16));
      else return false;
    }
  } else {
    if (ns == 8 && a.N % 64 == 0) FARD_NX_SHAPE(FARD_NX_ALL(2, 4, 8); FARD_NX_HEAD(2, 4, 8));
    else if (ns == 10) FARD_NX_SHAPE(FARD_NX_ALL(2, 2, 10); FARD_NX_HEAD(2, 2, 10));
    else if (ns == 12) FARD_NX_SHAPE(FARD_NX_ALL(2, 2, 12); FARD_NX_HEAD(2, 2, 12));
    else return false;
  }
#undef FARD_NX_SHAPE
#undef FARD_NX_ADA
#undef FARD_NX_HEAD
#undef FARD_NX_ALL
#undef FARD_NX
  *err = hipGetLastError();
  return true;
}

}  // namespace fard
