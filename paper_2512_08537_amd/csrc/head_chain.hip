// All residual blocks of one sampler step of the diffusion head in one launch, for a few rows (Sec. 3.2's AdaLN MLP).
//
// As separate launches a block is two dependent products of a few rows with 2-5 MB of weights, each a launch that costs
// 1.6 us of dispatch (2.5 when another queue waits on this one) and 1.5-2 us of cold start for well under a microsecond
// of work.  Here one workgroup per 16 or 32 columns and 16 rows stays for all blocks: its slice of the fp32 residual rows lives
// in registers, the weights of the next product are requested while the current one runs, and the bf16 rows that every
// product needs whole pass between the workgroups through memory.
//
// The exchange has no barrier, counter or fence: what passes are 8-byte words {payload, tag} (two bf16 or one fp32, and the
// number of the exchange), written and read at agent scope, so that a reader knows from the word alone whether it is fresh
// and simply reads again.  Two buffers alternate (rows v in, hidden rows a2 out of a block's first product): a workgroup
// writes an exchange only after all its waves have read the previous one, and that needs every workgroup's words of it, so
// no word is overwritten before its last reader is through.  Tags go on from a count of decodes that the kernel before this one
// advances; where they start over, after 2^20 decodes, it clears the words: words of earlier launches never match.
//
// From the second block on the modulated norm is folded around the first product as in narrow_exact.hip (NM_ADA_SILU,
// NM_ADA_GATE): v = (h - m)(1 + scale), tile moments of h beside it, rstd, mean - m, c1 and c0 applied in the epilogue; m is the
// row's mean a block earlier, which every workgroup knows, so that the rounding of v does not grow with the rows' mean.  The
// first block's rows are whole in memory when the launch starts: every workgroup takes their statistics itself and passes on
// the normalised rows.
//
// All workgroups of the launch have to be resident together: head_chain_tiles keeps the grid so small that this holds with a
// given number of such launches on the chip at once, and the context takes this path only on streams that have the whole chip
// and share the counted hardware queues (api.hip).  Where the count is wrong all the same (more processes on the GPU than it was
// told of), every wait is bounded in time: a workgroup that gives up marks the state, so that those which start after it and
// every later launch do not wait, and a word in host memory, which the context's next call returns as an error; the rows are NaN.
#include "kernels.h"

namespace fard {

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// agent-scope 16-byte accesses (sc1): past this XCD's L2, where other XCDs' stores would not show
constexpr int AUX_AGENT = 16;
__device__ __forceinline__ u32x4 load_agent(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, AUX_AGENT));
}
__device__ __forceinline__ void store_agent(__amdgpu_buffer_rsrc_t r, unsigned voff, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, 0, AUX_AGENT);
}

// low word of the steady counter, as a scalar
__device__ __forceinline__ unsigned steady_now() { return __builtin_amdgcn_readfirstlane((unsigned)__builtin_readsteadycounter()); }

// R: rows that a launch reads per 16-row group (4, 8 or 16).  What bounds a read of an exchange is the compute unit's 64
// bytes a clock from the vector cache: rows that are not there are not read, and up to 8 rows go through LDS (a wave stores
// its own share of k and reads it back as operands) instead of every lane reading its row's copy.
// CT: 16-column tiles of a workgroup; wave j < CT holds tile j's slice of the rows and writes for it.
template <int NS, int R, int CT>                           // w = 128 NS
__global__ __launch_bounds__(256, 2) void head_chain_kernel(HeadChainArgs a) {
  constexpr int W_COLS = 128 * NS;
  constexpr bool STAGE = R < 16;
  constexpr int NP = NS * R / 8;                           // 16-byte pieces a lane reads of an exchange
  constexpr int TPR = 256 / R;                             // threads that share a row's tile moments: lanes of one wave
  constexpr int NM = (8 * NS + TPR - 1) / TPR;             // moments a thread reads
  constexpr int LDT = 20;
  __shared__ __attribute__((aligned(16))) float red[2][CT][4 * 16 * LDT];
  __shared__ __attribute__((aligned(16))) char stage[STAGE ? 4 * NS * 64 * R : 16];
  __shared__ float rowstat[32];

  const unsigned tid = threadIdx.x, lane = tid & 63u, kw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned kg = lane >> 4, l16 = lane & 15u;
  const unsigned m0 = blockIdx.y * 16, n0 = blockIdx.x * (16 * CT);
  const int n = eff_rows(a.n, a.n_dev);
  if ((int)m0 >= n) return;                                // (uniform over the workgroups of a row group)
  const unsigned rows = (unsigned)n - m0 < (unsigned)R ? (unsigned)n - m0 : (unsigned)R;
  const unsigned st_decodes = a.state->decodes, st_gave_up = a.state->gave_up;   // (used behind the first loads)
  bool dead = false;

  // this row group's exchange area: rows in, a2 (4 R w bytes each: [32-k step][half][k group][row] pieces of 4 columns),
  // moments (R w bytes: [row][16-column tile])
  constexpr unsigned XA = 0, XB = 4 * R * W_COLS, XM = 8 * R * W_COLS, AREA = 9 * R * W_COLS;
  char* area = (char*)a.xch + (size_t)blockIdx.y * AREA;
  __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)area, 0, AREA, 0x00020000);
  // readers: pieces of the steps kw, kw + 4, ...; lane l of read i takes piece (64 i + l) of the wave's share
  unsigned rd[STAGE ? NP : 1], rdm[NM];
  if constexpr (STAGE) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const unsigned q = 64 * i + lane, r = q % R, hk = (q / R) & 7u, p = q / (8 * R);
      rd[i] = ((kw + 4 * p) * 8 + hk) * (16 * R) + (r < rows ? r : rows - 1) * 16;
    }
  } else {
    rd[0] = kg * 256 + (l16 < rows ? l16 : rows - 1) * 16 + kw * 2048;
  }
  const unsigned mr = tid / TPR, mt = tid % TPR;           // moments: thread -> row, tiles mt, mt + TPR, ...
#pragma unroll
  for (int i = 0; i < NM; ++i) {
    const unsigned t = mt + TPR * i;
    rdm[i] = XM + ((mr < rows ? mr : rows - 1) * (8 * NS) + (t < 8 * NS ? t : 0)) * 16;
  }
  // writers: 4 columns of a row
  const bool out_wave = kw < CT;
  const unsigned er = lane >> 2, ec = (lane & 3u) * 4, own = out_wave ? kw : 0, col = n0 + 16 * own + ec;
  const bool mine = out_wave && er < rows;
  const unsigned wr = (((col >> 5) * 8 + ((col >> 2) & 1u) * 4 + ((col >> 3) & 3u)) * R + er) * 16;
  const unsigned wrm = XM + (er * (8 * NS) + blockIdx.x * CT + own) * 16;
  const unsigned gr = m0 + (er < rows ? er : rows - 1);

  // weights: packed fragments of this 16-column tile, step s
  const unsigned wl = (lane >> 5) * 1024 + (kg & 1u) * 512 + l16 * 16;
  const unsigned t0 = blockIdx.x * CT;
  const size_t wtile = (size_t)(t0 >> 1) * (W_COLS / 16) * 1024 + (t0 & 1u) * 256 + kw * 2048;
  auto load_w = [&](const void* Wm, bf16x8 (&b)[CT][NS]) {
    const char* p = (const char*)Wm + wtile;
    unsigned step = 8192;
    asm("" : "+s"(step));
#pragma unroll
    for (int i = 0; i < NS; ++i) {
#pragma unroll
      for (int j = 0; j < CT; ++j) b[j][i] = *(const bf16x8*)(p + wl + j * 256);
      p += step;
    }
  };
  // An exchange's words, read until all are there.  The waves that do not write wait 64 x 20-24 cycles first: the words
  // cannot be there sooner, and their reads would stand in the way of the writers' stores (w = 1536, 8 rows, a block: 5.7 us
  // without that wait, 5.35 with 8, 4.8 with 20, 5.0 with 28).
  u32x4 x[NP], xm[NM];
  auto get = [&](unsigned base, unsigned tag, bool moments) {
    bool ok = dead;
    unsigned since = 0;
    if (!out_wave) __builtin_amdgcn_s_sleep(R < 16 ? 20 : 24);
    for (unsigned it = 0;; ++it) {
      if (it > 0) __builtin_amdgcn_s_sleep(1);
      asm volatile("" ::: "memory");                       // (every turn reads memory again)
      if (!ok) {
#pragma unroll
        for (int i = 0; i < NP; ++i)
          x[i] = STAGE ? load_agent(rx, rd[STAGE ? i : 0], base) : load_agent(rx, rd[0], base + (i >> 1) * 8192 + (i & 1) * 1024);
        if (moments) {
#pragma unroll
          for (int i = 0; i < NM; ++i) xm[i] = load_agent(rx, rdm[i], 0);
        }
        unsigned bad = 0;
#pragma unroll
        for (int i = 0; i < NP; ++i) bad |= (x[i][1] ^ tag) | (x[i][3] ^ tag);
        if (moments) {
#pragma unroll
          for (int i = 0; i < NM; ++i) bad |= (xm[i][1] ^ tag) | (xm[i][3] ^ tag);
        }
        asm("" : "+v"(bad));                               // (one vector chain, not dozens of compares joined in scalar registers)
        ok = bad == 0;
      }
      if (__all(ok)) break;
      if ((it & 255u) == 255u) {
        const unsigned now = steady_now();
        if (it == 255u) since = now;
        else if (now - since >= a.limit) { dead = true; break; }
      }
    }
  };
  f32x4 acc[CT];
  auto product = [&](const bf16x8 (&b)[CT][NS]) {
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (STAGE) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      char* st = stage + kw * (NS * 64 * R);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const unsigned q = 64 * i + lane, r = q % R, hk = (q / R) & 7u, p = q / (8 * R);
        *(u32x2*)(st + ((p * 4 + (hk & 3u)) * R + r) * 16 + (hk >> 2) * 8) = u32x2{x[i][0], x[i][2]};
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
      for (int p = 0; p < NS; ++p) {
        const bf16x8 f = *(const bf16x8*)(st + ((p * 4 + kg) * R + (l16 % R)) * 16);
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, b[j][p], acc[j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int p = 0; p < NS; ++p) {
        const u32x4 f = {x[2 * p][0], x[2 * p][2], x[2 * p + 1][0], x[2 * p + 1][2]};
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), b[j][p], acc[j], 0, 0, 0);
      }
    }
    if (dead) {
#pragma unroll
      for (int j = 0; j < CT; ++j) acc[j] = f32x4{1.f, 1.f, 1.f, 1.f} * __builtin_nanf("");
    }
  };
  auto to_lds = [&](float (&r)[CT][4 * 16 * LDT]) {
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) r[j][(kw * 16 + 4 * kg + e) * LDT + l16] = acc[j][e];
  };
  auto from_lds = [&](const float (&r)[CT][4 * 16 * LDT]) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 4; ++k) v += *(const f32x4*)(r[own] + (k * 16 + er) * LDT + ec);
    return v;
  };
  auto put4 = [&](unsigned base, f32x4 v, unsigned tag) {
    bf16x4 b;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = (bf16)v[e];
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 q = __builtin_bit_cast(u32x2, b);
    store_agent(rx, base + wr, u32x4{q[0], tag, q[1], tag});
  };
  // v and the tile moments of the rows h, as exchange `tag`
  auto put_rows = [&](f32x4 h, f32x4 scale, float centre, unsigned tag) {
    put4(XA, (h - centre) * (1.0f + scale), tag);
    float sm = (h[0] + h[1]) + (h[2] + h[3]);
    sm += dpp_move<DPP_SWAP1>(sm);
    sm += dpp_move<DPP_SWAP2>(sm);
    const float mean = sm * (1.0f / 16.0f);
    float q = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) { const float d = h[e] - mean; q = fmaf(d, d, q); }
    q += dpp_move<DPP_SWAP1>(q);
    q += dpp_move<DPP_SWAP2>(q);
    if ((lane & 3u) == 0) store_agent(rx, wrm, u32x4{__float_as_uint(mean), tag, __float_as_uint(q), tag});
  };

  const float* mrow = a.mod + ((size_t)gr * a.ldm + col);  // this thread's row and columns of the step's modulations
  f32x4 h = {0.f, 0.f, 0.f, 0.f}, b1, c1, c0, b2, gate, scn;
  float centre = 0.f;
  bf16x8 wt[CT][NS];
  HeadBlockW blk = a.blocks[0];
  load_w(blk.w1, wt);
  if (out_wave) {
    h = *(const f32x4*)(a.hh + (size_t)gr * W_COLS + col);
    c0 = *(const f32x4*)mrow;                              // shift and scale of the first block
    c1 = *(const f32x4*)(mrow + W_COLS);
    b1 = *(const f32x4*)(blk.b1 + col);
  }
  {
    // mean and 1 / std of the rows: a wave takes R / 4 of them, about the row's first element (as the norm kernel does)
    f32x4 hv[R / 4][NS / 2];
#pragma unroll
    for (int r = 0; r < R / 4; ++r) {
      const unsigned row = kw * (R / 4) + r;
      const float* p = a.hh + (size_t)(m0 + (row < rows ? row : rows - 1)) * W_COLS;
#pragma unroll
      for (int i = 0; i < NS / 2; ++i) hv[r][i] = *(const f32x4*)(p + 256 * i + lane * 4);
    }
#pragma unroll
    for (int r = 0; r < R / 4; ++r) {
      const float pivot = lane_value(hv[r][0][0], 0);
      float s = 0.f, q = 0.f;
#pragma unroll
      for (int i = 0; i < NS / 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float d = hv[r][i][e] - pivot; s += d; q = fmaf(d, d, q); }
      const float m1 = wave_sum(s) / (float)W_COLS, m2 = wave_sum(q) / (float)W_COLS;
      if (lane == 0) {
        rowstat[(kw * (R / 4) + r) * 2] = pivot + m1;
        rowstat[(kw * (R / 4) + r) * 2 + 1] = 1.0f / sqrtf(fmaxf(m2 - m1 * m1, 0.f) + 1e-6f);
      }
    }
  }
  const unsigned tag0 = __builtin_amdgcn_readfirstlane(st_decodes) * 4096u + (unsigned)a.tag_base;
  dead = __builtin_amdgcn_readfirstlane(st_gave_up) != 0;  // (an earlier launch has given up)
  __syncthreads();
  if (out_wave) {
    centre = rowstat[er * 2];
    if (mine) put4(XA, (h - centre) * rowstat[er * 2 + 1] * (1.0f + c1) + c0, tag0);
  }
  for (int j = 0; j < a.n_blocks; ++j) {
    const unsigned tag = tag0 + 2 * j;
    const bool more = j + 1 < a.n_blocks;
    const HeadBlockW next = a.blocks[more ? j + 1 : j];    // (asked for long before it is needed)
    // ---- a2 = silu(LN(h)(1 + scale) W1 + shift W1 + b1)
    get(XA, tag, j > 0);
    product(wt);
    if (!out_wave) load_w(blk.w2, wt);                     // (the writers ask for theirs behind the exchange's words)
    to_lds(red[0]);
    if (j > 0) {
      // mean and 1 / std of the rows from the tile moments (pairwise update of Chan et al. for equal counts, about the
      // row's first tile)
      const float first = __uint_as_float(xm[0][0]);
      float pivot;
      if constexpr (TPR == 16) pivot = dpp_move<DPP_ROW_FIRST>(first);
      else if constexpr (TPR == 32) pivot = (lane & 32u) ? lane_value(first, 32) : lane_value(first, 0);
      else pivot = lane_value(first, 0);
      float sd = 0.f, sd2 = 0.f, sq = 0.f;
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        if (mt + TPR * i < 8 * NS) {
          const float d = __uint_as_float(xm[i][0]) - pivot;
          sd += d;
          sd2 = fmaf(d, d, sd2);
          sq += __uint_as_float(xm[i][2]);
        }
      }
      auto sum = [](float v) { return TPR == 16 ? row16_sum(v) : (TPR == 32 ? half_sum(v) : wave_sum(v)); };
      sd = sum(sd); sd2 = sum(sd2); sq = sum(sq);
      if (mt == 0) {
        constexpr float inv_t = 1.0f / (8 * NS), inv_w = 1.0f / W_COLS;
        const float m2 = sq + 16.0f * fmaxf(sd2 - sd * sd * inv_t, 0.f);
        rowstat[mr * 2] = pivot + sd * inv_t;
        rowstat[mr * 2 + 1] = 1.0f / sqrtf(fmaf(m2, inv_w, 1e-6f));
      }
    }
    __syncthreads();
    if (out_wave) {
      f32x4 v = from_lds(red[0]);
      if (j > 0) {
        const float mean = rowstat[er * 2];
        v = (v - c1 * (mean - centre)) * rowstat[er * 2 + 1] + c0;
        centre = mean;
      }
      v += b1;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = silu<true>(v[e]);
      if (mine) put4(XB, v, tag + 1);
      __builtin_amdgcn_sched_barrier(0);
      load_w(blk.w2, wt);
      const float* m = mrow + 3 * W_COLS * j;
      b2 = *(const f32x4*)(blk.b2 + col);
      gate = *(const f32x4*)(m + 2 * W_COLS);
      if (more) scn = *(const f32x4*)(m + 4 * W_COLS);
    }
    // ---- h += gate (a2 W2 + b2)
    get(XB, tag + 1, false);
    product(wt);
    if (!out_wave && more) load_w(next.w1, wt);
    to_lds(red[1]);
    __syncthreads();
    if (out_wave) {
      f32x4 v = from_lds(red[1]);
      v += b2;
      h = h + gate * v;
      if (more) {
        if (mine) put_rows(h, scn, centre, tag + 2);
        __builtin_amdgcn_sched_barrier(0);
        load_w(next.w1, wt);
        const float* m = mrow + a.fold_base + 2 * W_COLS * (j + 1);
        c0 = *(const f32x4*)m;
        c1 = *(const f32x4*)(m + W_COLS);
        b1 = *(const f32x4*)(next.b1 + col);
      }
    }
    blk = next;
  }
  if (mine) *(f32x4*)(a.hh + (size_t)gr * W_COLS + col) = h;
  if (dead) {
    // (workgroups that only start when this one makes room see it; all lanes store the same words)
    __hip_atomic_store(&a.state->gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(a.state->host_gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Rows that the kernel is compiled for per 16-row group: the smallest that holds a launch of n.
int head_chain_rows(int n) { return n <= 4 ? 4 : (n <= 8 ? 8 : 16); }

}  // namespace

size_t head_chain_bytes(int rows, int w) { return (size_t)((rows + 15) / 16) * 16 * 9 * w; }

// Every workgroup has to be resident while any of them waits: two fit a compute unit (registers), and `launches` of them may be
// on the chip side by side.  Workgroups of one 16-column tile while that holds, else of
// two, which read as much of the exchange for twice the columns (a decode of 2 steps, launch per product -> resident: 33 rows of
// 6 x 1024 140 -> 103 us, 64 rows 144 -> 105; 17 rows of 8 x 1280 183 -> 138, 48 rows 196 -> 151; one tile at 32 and 16 rows of
// these 97 and 128).  At a width of 1536 two tiles do not fit the registers.  The widths are those it was measured at; others keep
// a launch per product.
int head_chain_tiles(int n, int w, int n_blocks, int n_steps, int compute_units, int launches) {
  if (w != 1024 && w != 1280 && w != 1536) return 0;
  if (n < 1 || n_blocks < 1 || n_steps < 1 || (long)2 * n_blocks * n_steps >= 4095 || launches < 1) return 0;
  const long one = (long)(w / 16) * ((n + 15) / 16) * launches;
  if (one <= 2L * compute_units) return 1;
  return w <= 1280 && one <= 4L * compute_units ? 2 : 0;
}

hipError_t launch_head_chain(hipStream_t s, const HeadChainArgs& a, int w, int tiles, bool short_of_one) {
  if (a.n < 1 || a.n_blocks < 1 || a.tag_base < 1 || a.tag_base + 2 * a.n_blocks > 4096 || a.state == nullptr)
    return hipErrorInvalidValue;
  if (tiles != 1 && (tiles != 2 || w > 1280)) return hipErrorInvalidValue;
  const dim3 grid(w / (16 * tiles) - (short_of_one ? 1 : 0), (a.n + 15) / 16);
  const int R = head_chain_rows(a.n);
#define FARD_HC(NSV)                                                                \
  case 128 * NSV:                                                                   \
    if (tiles == 2) {                                                               \
      if constexpr (NSV <= 10) head_chain_kernel<NSV, 16, 2><<<grid, 256, 0, s>>>(a); \
    } else if (R == 4) {                                                            \
      head_chain_kernel<NSV, 4, 1><<<grid, 256, 0, s>>>(a);                         \
    } else if (R == 8) {                                                            \
      head_chain_kernel<NSV, 8, 1><<<grid, 256, 0, s>>>(a);                         \
    } else {                                                                        \
      head_chain_kernel<NSV, 16, 1><<<grid, 256, 0, s>>>(a);                        \
    }                                                                               \
    break
  switch (w) {
    FARD_HC(8);
    FARD_HC(10);
    FARD_HC(12);
    default: return hipErrorInvalidValue;
  }
#undef FARD_HC
  return hipGetLastError();
}

}  // namespace fard
