// Training-side losses of the draft model: the attention-entropy loss L_entropy (Sec. 3; S2.1) with its gradients
// with respect to the queries and keys of the layer it is taken on, and the Smooth-L1 feature regression loss.
//
// L_entropy = -(1 / (B N R)) sum_{b,h,r} H_{b,h,r},  H_r = -sum_c Omega_{r,c} ln Omega_{r,c},
// Omega_r = softmax over the causal row r of s_{r,c} = q_r . k_c / sqrt(d_head) (c <= r).
// dL/ds_{r,c} = Omega_{r,c} (ln Omega_{r,c} + H_r) / (B N R); dq_r = sum_c dL/ds k_c / sqrt(d); dk_c = sum_r dL/ds q_r / sqrt(d).
//
// Two kernels over 32 x 32 score tiles, none of which writes a score to memory (v_mfma_f32_32x32x16_bf16):
//  1. rows: a wave owns 32 queries of one head.  A first walk over the key blocks up to the diagonal keeps a running
//     (max, sum e^t, sum e^t t) and leaves ln sum exp and H per row; a second walk rebuilds the tile of dL/ds and multiplies
//     it with the keys (dq);
//  2. dk: a wave owns 32 keys of one kv head and walks the query blocks from the diagonal on, over every query head of its
//     group; dL/ds is rebuilt with queries and keys in swapped roles and multiplied with the queries.
// No atomics: every output element has one owner.
//
// A workgroup is four waves with adjacent 32-row blocks.  The rows that they walk over (keys, or queries) go to LDS once per
// workgroup, 64 at a time, by direct-to-LDS loads into one of two buffers while the other is worked on; they serve both
// products: the scores read rows (16 bytes a lane), the gradients read the same tile transposed (ds_read_b64_tr_b16: a
// group of 16 lanes reads 4 rows x 16 columns and gets a column of 4 a lane).  Bound: the vector instructions around the exponentials (about 7 an
// element and walk) and the LDS reads beside the MFMAs.  With a wave fetching its fragments from memory by itself, a row a
// lane, and transposed copies of q and k written beforehand, the grouped 8 x 40 (8) x 1024 x 128 loss took 285 us for the
// statistics, 564 for dq, 810 for dk and 59 for the copies; now 180 (statistics and dq) and 164 (medians of kernel traces).  32 x
// 16 x 256 x 64: 20 + 34 + 40 + 11 us, now 21 and 16.
//
// Layouts.  Register e of lane half hh of a score tile holds row 8 (e / 4) + 4 hh + e % 4 of the operand whose rows are in the
// registers.  Registers 8 t .. 8 t + 7 are, as they stand, an operand fragment of the second product: its contraction slot
// (hh, j) is row 16 t + 8 (j / 4) + 4 hh + j % 4, which is what two transposed reads of four rows each deliver for the other
// operand.  The 16-byte pieces of a row are stored XOR-ed with twr(row), so that neither kind of read meets bank conflicts.
#include "kernels.h"

#include <algorithm>

namespace fard {

namespace {

typedef const __attribute__((address_space(1))) void* gptr;
typedef __attribute__((address_space(3))) void* lptr;
typedef __attribute__((address_space(3))) bf16x4* ltr;

constexpr float LOG2E = 1.44269504088896341f, LN2 = 0.69314718055994531f;
constexpr float MASKED = -3e38f;      // score of a masked pair: finite, so that its 0 probability times it is 0
constexpr float M_START = -3e37f;     // running maximum before the first score: above MASKED times s2 >= 0.1275 (128-wide heads)
constexpr int WR = 64;                // rows walked over per LDS tile
constexpr int GR = 128;               // rows owned by a workgroup

__device__ __forceinline__ int twr(int r) { return 2 * (r & 3) + ((r >> 2) & 1); }

template <int DH>
struct Frag {
  bf16x8 f[DH / 16];
};

// rows of a [R][DH] matrix as MFMA operand: lane -> row `row` (clamped), k-slots 16 s + 8 hh
template <int DH>
__device__ __forceinline__ void load_rows(Frag<DH>& fr, const bf16* __restrict__ base, int row, int R, int hh) {
  const int rr = row < R ? row : R - 1;
  const bf16* p = base + (size_t)rr * DH + 8 * hh;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) fr.f[s] = *(const bf16x8*)(p + 16 * s);
}

// rows r0 .. r0 + 63 of a [R][DH] matrix to LDS (rows past R: row R - 1, masked by the caller), a quarter per wave
template <int DH>
__device__ __forceinline__ void walk_load(char* buf, const bf16* __restrict__ base, int r0, int R, int wave, int lane) {
  constexpr int P = DH / 8;                                  // 16-byte pieces of a row
#pragma unroll
  for (int i = 0; i < DH / 32; ++i) {
    const int n = (wave * (DH / 32) + i) * 64 + lane, row = n / P;
    const int piece = (n & (P - 1)) ^ (twr(row) & (P - 1));
    int gr = r0 + row;
    gr = gr < R ? gr : R - 1;
    __builtin_amdgcn_global_load_lds((gptr)(base + (size_t)gr * DH + piece * 8), (lptr)(buf + (wave * (DH / 32) + i) * 1024), 16, 0, 0);
  }
}

// scores of 32 walked rows (from LDS row r0 on: the registers) and the wave's own 32 rows (the lanes)
template <int DH>
__device__ __forceinline__ f32x16 score_tile(const char* buf, int r0, const Frag<DH>& own, int lane) {
  constexpr int P = DH / 8;
  const int row = r0 + (lane & 31), x = twr(lane & 31) & (P - 1), hh = lane >> 5;
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) {
    const bf16x8 f = *(const bf16x8*)(buf + row * (DH * 2) + (((2 * s + hh) ^ x) << 4));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, own.f[s], acc, 0, 0, 0);
  }
  return acc;
}

// out[own row, d] += sum over 32 walked rows of g[walked row, own row] walked[row, d]
template <int DH>
__device__ __forceinline__ void grad_product(const char* buf, int r0, const bf16x8 (&g)[2], f32x16 (&out)[DH / 32], int lane) {
  constexpr int P = DH / 8;
  const int i = lane & 15, hh = lane >> 5;
  const int x = (2 * (i >> 2) + hh) & (P - 1);               // twr of the rows this lane addresses
  const int pc = 2 * ((lane >> 4) & 1) + ((i & 3) >> 1);     // piece inside a 32-column block
  const char* at = buf + (r0 + 4 * hh + (i >> 2)) * (DH * 2) + (i & 1) * 8;
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const char* p = at + 16 * t * (DH * 2) + (((4 * d + pc) ^ x) << 4);
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((ltr)p);
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((ltr)(p + 8 * (DH * 2)));
      out[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[t], __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7), out[d], 0, 0, 0);
    }
}

// the tile that `buf` receives has arrived for all waves, and all are done with the other buffer
__device__ __forceinline__ void tile_sync() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0070);                        // vmcnt(0) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Calls f(buf, r0) for the 64-row tiles r0 = first, first + 64, .. < end of `base`: the next tile is on its way while one is
// worked on.  The loads stand under no condition (past the end they re-read row R - 1 into a tile that nobody uses):
// under one, the compiler would wait for all loads before every LDS read.
#define ENT_WALK(first, end, issue, body)                \
  do {                                                        \
    issue(b0, first);                                         \
    for (int r_ = (first); r_ < (end); r_ += 2 * WR) {        \
      tile_sync();                                            \
      issue(b1, r_ + WR);                                     \
      body(b0, r_);                                           \
      tile_sync();                                            \
      issue(b0, r_ + 2 * WR);                                 \
      if (r_ + WR < (end)) body(b1, r_ + WR);                 \
    }                                                         \
    tile_sync();                                              \
  } while (0)

// ---- rows: statistics, and dq.  Four waves x 32 queries of one (b, h); a wave past R only loads.  SHORT, up to 32 rows: a wave has
// a (b, h) and its keys to itself, or three of four waves would have no queries (64 x 40 (8) x 24 x 128, statistics alone: 18.6 us
// with one (b, h) per workgroup, 13.0 with the unstaged kernels described above, 8.5 now).
template <int DH, bool SHORT>
__global__ __launch_bounds__(256, 3) void ent_rows_kernel(const bf16* __restrict__ q, const bf16* __restrict__ k, int BH, int H, int Hkv,
                                                          int R, int Rp, float scale, float cc, float* __restrict__ lse2,
                                                          float* __restrict__ cch, float* __restrict__ partial,
                                                          float* __restrict__ h_out, float* __restrict__ dq) {
  __shared__ __attribute__((aligned(1024))) char b0[WR * DH * 2];
  __shared__ __attribute__((aligned(1024))) char b1[WR * DH * 2];
  __shared__ float part[4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the longest walks first
  const int n_groups = Rp / GR, slot = SHORT ? 4 * blockIdx.x + wave : blockIdx.x % BH;
  const bool live = slot < BH;
  const int bh = live ? slot : BH - 1, grp = SHORT ? 0 : n_groups - 1 - blockIdx.x / BH;
  const int b = bh / H, h = bh - b * H, bkv = b * Hkv + h / (H / Hkv);
  const int c = lane & 31, hh = lane >> 5;
  const int q0 = SHORT ? 0 : grp * GR + 32 * wave, query = q0 + c;
  const int last = q0 < R ? q0 : -1;                         // first row of the last key block
  const int end = grp * GR + GR < R ? grp * GR + GR : R;     // keys that this workgroup's queries see
  const bf16* kbase = k + (size_t)bkv * R * DH;
  const float s2 = scale * LOG2E;
  Frag<DH> qf;
  load_rows<DH>(qf, q + (size_t)bh * R * DH, query, R, hh);

  auto issue = [&](char* buf, int r0) __attribute__((always_inline)) { walk_load<DH>(buf, kbase, r0, R, wave, lane); };
  // scores of 32 keys from key0 on (buffer row sub), masked on the diagonal
  auto scores = [&](const char* buf, int sub, int key0) __attribute__((always_inline)) {
    f32x16 acc = score_tile<DH>(buf, sub, qf, lane);
    if (key0 == q0) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (8 * (e >> 2) + 4 * hh + (e & 3) > c) acc[e] = MASKED;
    }
    return acc;
  };

  // base-2 units: t = s log2 e - m
  float m = M_START, l = 0.f, a = 0.f;
  auto stats = [&](const char* buf, int r0) __attribute__((always_inline)) {
#pragma unroll 1
    for (int sub = 0; sub < (SHORT ? 32 : WR); sub += 32) {
      if (r0 + sub > last) break;
      const f32x16 acc = scores(buf, sub, r0 + sub);
      float mx = acc[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, acc[e]);
      const float mn = fmaxf(m, mx * s2), d = mn - m, f = __builtin_amdgcn_exp2f(-d);
      a = (a - d * l) * f;
      l *= f;
      m = mn;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float t = fmaxf(fmaf(acc[e], s2, -m), -1e30f), p = __builtin_amdgcn_exp2f(t);
        l += p;
        a = fmaf(p, t, a);
      }
    }
  };
  char* own_keys = (wave < 2 ? b0 : b1) + (wave & 1) * (32 * DH * 2);
  if constexpr (SHORT) {
    walk_load<DH>(own_keys, kbase, 0, R, 0, lane);           // rows 0 .. 15
    walk_load<DH>(own_keys, kbase, 0, R, 1, lane);
    tile_sync();
    stats(own_keys, 0);
  } else {
    ENT_WALK(0, end, issue, stats);
  }
  {
    const float mo = other_half(m), lo = other_half(l), ao = other_half(a);
    const float mn = fmaxf(m, mo), d1 = mn - m, d2 = mn - mo;
    const float f1 = __builtin_amdgcn_exp2f(-d1), f2 = __builtin_amdgcn_exp2f(-d2);
    a = (l > 0.f ? (a - d1 * l) * f1 : 0.f) + (lo > 0.f ? (ao - d2 * lo) * f2 : 0.f);
    l = l * f1 + lo * f2;
    m = mn;
  }
  const float ll = __builtin_amdgcn_logf(l);
  const bool valid = live && query < R;
  const float hv = valid ? LN2 * (ll - a / l) : 0.f;
  const float ls = valid ? m + ll : 1e30f;                   // rows past R: probability 0 in the second kernel
  // (SHORT: the second halves of the waves fill the rest of the 64-row tile that the dk kernel reads)
  if (SHORT ? live : hh == 0) {
    lse2[(size_t)bh * Rp + query + 32 * hh] = hh == 0 ? ls : 1e30f;
    cch[(size_t)bh * Rp + query + 32 * hh] = hh == 0 ? cc * hv : 0.f;
  }
  if (hh == 0 && valid && h_out) h_out[(size_t)bh * R + query] = hv;
  const float hs = wave_sum(hh == 0 ? hv : 0.f);
  if (lane == 0) part[wave] = hs;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
  if (!dq) return;

  f32x16 out[DH / 32];
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[d][e] = 0.f;
  const float c1 = cc * LN2, c2 = cc * hv;
  auto grads = [&](const char* buf, int r0) __attribute__((always_inline)) {
#pragma unroll 1
    for (int sub = 0; sub < (SHORT ? 32 : WR); sub += 32) {
      if (r0 + sub > last) break;
      const f32x16 acc = scores(buf, sub, r0 + sub);
      bf16x8 g[2];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float t = fmaf(acc[e], s2, -ls);
        g[e >> 3][e & 7] = (bf16)(__builtin_amdgcn_exp2f(t) * fmaf(t, c1, c2));
      }
      grad_product<DH>(buf, sub, g, out, lane);
    }
  };
  if constexpr (SHORT) grads(own_keys, 0);
  else ENT_WALK(0, end, issue, grads);
  float* dq_b = dq + (size_t)bh * R * DH;
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = q0 + 8 * (e >> 2) + 4 * hh + (e & 3);
      if (live && row < R) dq_b[(size_t)row * DH + 32 * d + c] = out[d][e];
    }
}

// ---- dk.  Four waves x 32 keys of one (b, kv head).
template <int DH>
__global__ __launch_bounds__(256, DH == 128 ? 2 : 3) void ent_dk_kernel(const bf16* __restrict__ q, const bf16* __restrict__ k, int BHkv, int H, int Hkv,
                                                        int R, int Rp, float scale, float cc, const float* __restrict__ lse2,
                                                        const float* __restrict__ cch, float* __restrict__ dk) {
  constexpr int TILE = WR * DH * 2;                          // then 64 ln sum exp and 64 cc H of the tile's queries
  __shared__ __attribute__((aligned(1024))) char b0[TILE + 512];
  __shared__ __attribute__((aligned(1024))) char b1[TILE + 512];
  // the first half of the workgroups takes the long walks, longest first, the second half the short ones, shortest first: the
  // two that meet on a compute unit add up to about the same
  const int n_groups = Rp / GR, half = (n_groups + 1) / 2;
  const int bkv = blockIdx.x % BHkv, o = blockIdx.x / BHkv;
  const int grp = o < half ? o : n_groups - 1 - (o - half);
  const int b = bkv / Hkv, hkv = bkv - b * Hkv, G = H / Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, hh = lane >> 5;
  const int k0 = grp * GR + 32 * wave;
  const int own = k0 < R ? k0 : 1 << 30;                     // first row of the first query block; a wave past R only loads
  const float s2 = scale * LOG2E, c1 = cc * LN2;
  Frag<DH> kf;
  load_rows<DH>(kf, k + (size_t)bkv * R * DH, k0 + c, R, hh);
  f32x16 out[DH / 32];
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) out[d][e] = 0.f;

  const int first = grp * GR;
#pragma unroll 1
  for (int gi = 0; gi < G; ++gi) {
    const int bh = b * H + hkv * G + gi;
    const bf16* qbase = q + (size_t)bh * R * DH;
    // (waves of the same parity fetch the same 64 values to the same place)
    const float* st = ((wave & 1) ? cch : lse2) + (size_t)bh * Rp + lane;
    auto issue = [&](char* buf, int r0) __attribute__((always_inline)) {
      walk_load<DH>(buf, qbase, r0, R, wave, lane);
      const int rs = r0 < Rp ? r0 : Rp - WR;                 // (Rp % 64 == 0)
      __builtin_amdgcn_global_load_lds((gptr)(st + rs), (lptr)(buf + TILE + (wave & 1) * 256), 4, 0, 0);
    };
    auto grads = [&](const char* buf, int r0) __attribute__((always_inline)) {
#pragma unroll 1
      for (int sub = 0; sub < WR; sub += 32) {
        if (r0 + sub < own) continue;
        f32x16 acc = score_tile<DH>(buf, sub, kf, lane);
        if (r0 + sub == k0) {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (8 * (e >> 2) + 4 * hh + (e & 3) < c) acc[e] = MASKED;
        }
        bf16x8 g[2];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          const f32x4 ls = *(const f32x4*)(buf + TILE + (sub + 8 * n + 4 * hh) * 4);
          const f32x4 c2 = *(const f32x4*)(buf + TILE + 256 + (sub + 8 * n + 4 * hh) * 4);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int e = 4 * n + j;
            const float t = fmaf(acc[e], s2, -ls[j]);
            g[e >> 3][e & 7] = (bf16)(__builtin_amdgcn_exp2f(t) * fmaf(t, c1, c2[j]));
          }
        }
        grad_product<DH>(buf, sub, g, out, lane);
      }
    };
    ENT_WALK(first, R, issue, grads);
  }
#undef ENT_WALK
  float* dk_b = dk + (size_t)bkv * R * DH;
#pragma unroll
  for (int d = 0; d < DH / 32; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = k0 + 8 * (e >> 2) + 4 * hh + (e & 3);
      if (row < R) dk_b[(size_t)row * DH + 32 * d + c] = out[d][e];
    }
}

// Smooth-L1: per-workgroup partial sums (fixed order), gradient per element.  Bound: the memory's read and write of 8 to 12
// bytes an element.  VEC elements a lane and step: 16 bytes of input where all pointers allow that and n is large, else one
// (42 M bf16 elements: 141 us with one, 72 us, 4.7 TB/s, with eight).
template <typename T, int VEC>
__global__ __launch_bounds__(256) void smooth_l1_kernel(const T* __restrict__ pred, const T* __restrict__ target, long n, float beta,
                                                        float* __restrict__ partial, float* __restrict__ dpred) {
  typedef T tvec __attribute__((ext_vector_type(VEC)));
  typedef float fvec __attribute__((ext_vector_type(VEC < 4 ? VEC : 4)));   // (the gradient is 16-byte aligned, no more)
  constexpr int GV = VEC < 4 ? VEC : 4;
  __shared__ float part[4];
  float s = 0.f;
  const float inv_n = 1.0f / (float)n;
  auto one = [&](float p, float t) __attribute__((always_inline)) {
    const float d = p - t, a = fabsf(d);
    const bool quad = a < beta;
    s += quad ? 0.5f * d * d / beta : a - 0.5f * beta;
    return (quad ? d / beta : copysignf(1.0f, d)) * inv_n;
  };
  const long nv = n / VEC, step = (long)gridDim.x * 256;
  const long i0 = (long)blockIdx.x * 256 + threadIdx.x;
  for (long i = i0; i < nv; i += step) {
    const tvec p = ((const tvec*)pred)[i], t = ((const tvec*)target)[i];
    fvec g[VEC / GV];
#pragma unroll
    for (int e = 0; e < VEC; ++e) g[e / GV][e % GV] = one(to_f32(p[e]), to_f32(t[e]));
    if (dpred) {
#pragma unroll
      for (int h = 0; h < VEC / GV; ++h) ((fvec*)dpred)[i * (VEC / GV) + h] = g[h];
    }
  }
  if (VEC > 1 && i0 < n - nv * VEC) {
    const long i = nv * VEC + i0;
    const float g = one(to_f32(pred[i]), to_f32(target[i]));
    if (dpred) dpred[i] = g;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
__global__ __launch_bounds__(1024) void sum_partials_kernel(const float* __restrict__ partial, int n_part, float inv_n, float* __restrict__ loss) {
  __shared__ float part[16];
  float s = 0.f;
  for (int i = threadIdx.x; i < n_part; i += 1024) s += partial[i];
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x < 64) {
    s = wave_sum(threadIdx.x < 16 ? part[threadIdx.x] : 0.f);
    if (threadIdx.x == 0) *loss = s * inv_n;
  }
}

template <int DH>
hipError_t entropy_loss_t(hipStream_t s, const bf16* q, const bf16* k, int B, int H, int Hkv, int R, void* scratch, float* loss,
                          float* h_rows, float* dq, float* dk) {
  const EntLossScratch lay = entropy_loss_scratch(B, H, Hkv, R, DH);
  const int Rp = (R + GR - 1) / GR * GR, n_groups = Rp / GR;
  char* base = (char*)scratch;
  float* lse2 = (float*)(base + lay.lse);
  float* cch = (float*)(base + lay.hrow);
  float* partial = (float*)(base + lay.partial);
  const float scale = 1.0f / sqrtf((float)DH);
  const float cc = scale / ((float)B * (float)H * (float)R);
  const int n_part = R <= 32 ? (B * H + 3) / 4 : B * H * n_groups;
  if (R <= 32) ent_rows_kernel<DH, true><<<n_part, 256, 0, s>>>(q, k, B * H, H, Hkv, R, Rp, scale, cc, lse2, cch, partial, h_rows, dq);
  else ent_rows_kernel<DH, false><<<n_part, 256, 0, s>>>(q, k, B * H, H, Hkv, R, Rp, scale, cc, lse2, cch, partial, h_rows, dq);
  sum_partials_kernel<<<1, 1024, 0, s>>>(partial, n_part, -1.0f / (float)((long)B * H * R), loss);
  if (dk)
    ent_dk_kernel<DH><<<B * Hkv * n_groups, 256, 0, s>>>(q, k, B * Hkv, H, Hkv, R, Rp, scale, cc, lse2, cch, dk);
  return hipGetLastError();
}

}  // namespace

EntLossScratch entropy_loss_scratch(int B, int H, int Hkv, int R, int dh) {
  const size_t Rp = (size_t)((R + GR - 1) / GR * GR);
  EntLossScratch l;
  l.lse = 0;
  l.hrow = l.lse + (size_t)B * H * Rp * 4;
  l.partial = l.hrow + (size_t)B * H * Rp * 4;
  l.bytes = l.partial + (size_t)B * H * (Rp / GR) * 4;
  return l;
}

hipError_t launch_entropy_loss(hipStream_t s, const void* q, const void* k, int B, int H, int Hkv, int R, int dh, void* scratch,
                               float* loss, float* h_rows, float* dq, float* dk) {
  if (B < 1 || H < 1 || Hkv < 1 || H % Hkv != 0 || R < 1) return hipErrorInvalidValue;
  if (dh == 32) return entropy_loss_t<32>(s, (const bf16*)q, (const bf16*)k, B, H, Hkv, R, scratch, loss, h_rows, dq, dk);
  if (dh == 64) return entropy_loss_t<64>(s, (const bf16*)q, (const bf16*)k, B, H, Hkv, R, scratch, loss, h_rows, dq, dk);
  if (dh == 128) return entropy_loss_t<128>(s, (const bf16*)q, (const bf16*)k, B, H, Hkv, R, scratch, loss, h_rows, dq, dk);
  return hipErrorInvalidValue;
}

hipError_t launch_smooth_l1(hipStream_t s, int is_bf16, const void* pred, const void* target, long n, float beta, float* partial,
                            int n_part, float* loss, float* dpred) {
  if (n < 1 || n_part < 1 || !(beta > 0.f)) return hipErrorInvalidValue;
  const uintptr_t in = (uintptr_t)pred | (uintptr_t)target;
  // Below two workgroups of 16-byte pieces per compute unit the lanes' serial elements cost more than narrow accesses: 20000 bf16
  // elements 5.6 us with eight a lane, 4.8 with one; 131072 5.7 and 4.8, 524288 6.0 and 5.8, 1 M 6.6 and 6.6, 3 M 9.0 and 9.8.
  const int per = is_bf16 ? 8 : 4;
  const bool vec = (in & 15) == 0 && ((uintptr_t)dpred & 15) == 0 && n / per > 512 * 256;
  if (vec) n_part = (int)std::min<long>(n_part, (n / per + 255) / 256);
#define FARD_L1(T, VEC) smooth_l1_kernel<T, VEC><<<n_part, 256, 0, s>>>((const T*)pred, (const T*)target, n, beta, partial, dpred)
  if (is_bf16) {
    if (vec) FARD_L1(bf16, 8); else FARD_L1(bf16, 1);
  } else {
    if (vec) FARD_L1(float, 4); else FARD_L1(float, 1);
  }
#undef FARD_L1
  sum_partials_kernel<<<1, 1024, 0, s>>>(partial, n_part, 1.0f / (float)n, loss);
  return hipGetLastError();
}

}  // namespace fard
