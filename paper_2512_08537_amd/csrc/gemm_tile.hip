// GEMM of many rows: out = epilogue(A[M,K] * W[K,N]) on 128 x 128 to 256 x 256 tiles (bf16 MFMA, fp32 accumulation).
//
// For prefill passes and the verify stage of large batches (hundreds to thousands of rows).  A workgroup is four waves (2 x 2)
// of 32 WI x 32 WJ outputs each.  What the tile size trades: a 128 x 256 tile of the streaming kernel (gemm.hip) asks its XCD's
// L2 for 48 B per clock and compute unit of the 64 that it has, a 256 x 256 tile for 32; per 128 clocks of MFMAs the LDS
// moves 75 % of what it can for 256 x 256 tiles (with eight waves of 128 x 64 it was full: 5 % slower), 125 % for
// 192 x 128 and 150 % for 128 x 128.  The small tiles are ahead all the same where the large ones leave compute units idle, and
// with a short K, since two of their workgroups share a compute unit and one's first loads and last stores overlap the other's
// MFMAs.  With one workgroup per compute unit they keep three 64-k stages in flight instead of one.
//  * both operands go from memory to LDS by direct-to-LDS loads, 64 k a stage, NS stages: the next NS - 1 are in
//    flight for the whole of the present one;
//  * the weights keep their fragment order (a fragment is 1 KiB of consecutive LDS); the 16-byte pieces of an activation
//    row are stored XOR-ed with the row's low bits, by permuting which piece a lane fetches, so that fragment reads of 32
//    rows spread over all banks;
//  * the fragments of a k-step are read between the MFMAs of the step before, across the stage boundary as well: the one
//    barrier of a stage stands before its last k-step, when the stage's reads are all done, so that its buffer can be
//    refilled at once.  The buffers are separate LDS objects, and waits go through the builtin: otherwise the compiler
//    waits for every outstanding load before each LDS read.
// What bounds it: 256 x 256 tiles on full-range inputs the card's clock under MFMA load (1.65 us per stage with all compute
// units at work, 1.1 us for a lone tile; a library product of the same size and kind measured 1140-1210 TFLOP/s beside it);
// the small tiles the LDS, and the ~4 us before the first and after the last MFMA of a tile that has no neighbour.
#include "gemm.h"

#include <algorithm>
#include <cmath>

namespace fard {

namespace {

// WI x WJ: 32 x 32 accumulator blocks of a wave; the four waves stand 2 x 2
constexpr int TBK = 64;                                      // k per stage
constexpr int stage_bytes(int wi, int wj) { return 64 * (wi + wj) * TBK * 2; }
// accumulator blocks along M that leave per pass: 64 columns of a wave's outputs fit its quarter of the two stages
constexpr int out_blocks(int wi, int wj) {
  return 32 * wi * 64 * 4 * 4 <= 2 * stage_bytes(wi, wj) ? wi : wi % 2 == 0 ? wi / 2 : 1;
}

// s_waitcnt operand: vmcnt in bits 3:0 and 15:14, expcnt 6:4 (7: not waited for), lgkmcnt 11:8
constexpr int wait_vm(int n) { return 0x0070 | (n & 15) | ((n >> 4) << 14); }   // vmcnt(n) lgkmcnt(0)

typedef const __attribute__((address_space(1))) void* gptr;
typedef __attribute__((address_space(3))) void* lptr;

// ROWS x 64 outputs of a wave leaves through the wave's own share of the LDS as 16-byte stores of consecutive
// columns; no barrier.  Value (row, c) is at row * 64 + (c ^ 32 for rows with bit 2 set), which puts the two rows of an
// accumulator register on different banks.  The row loop stays rolled: a workgroup runs this code once or twice, and unrolled
// over rows it was fetched from memory for longer than it ran (20 us of a 44 us launch of one tile per compute unit).
__device__ __forceinline__ f32x4 half_read(const float* half, int row, int c) {
  return *(const f32x4*)(half + row * 64 + (c ^ ((row & 4) << 3)));
}
template <int KIND, int ROWS>
__device__ __forceinline__ void half_out(const GemmArgs& a, const float* half, int mb, int M, int n0, int lane) {
  if constexpr (KIND == EPI_SWIGLU) {
    // packed columns: 32 gate, 32 up -> 32 outputs; lane -> (row, 8 columns)
    const int c = (lane & 3) * 8;
    bf16* out = (bf16*)a.out + (n0 >> 1) + c;
#pragma unroll 1
    for (int row = lane >> 2; row < ROWS && mb + row < M; row += 16) {
      bf16x8 o;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 g = half_read(half, row, c + 4 * h), u = half_read(half, row, 32 + c + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[4 * h + e] = (bf16)(silu<true>(g[e]) * u[e]);
      }
      *(bf16x8*)(out + (size_t)(mb + row) * a.ldo) = o;
    }
  } else if constexpr (KIND == EPI_STORE) {
    const int c = (lane & 7) * 8;
    if (n0 + c >= a.N) return;
    f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = b0;
    if (a.bias) { b0 = *(const f32x4*)(a.bias + n0 + c); b1 = *(const f32x4*)(a.bias + n0 + c + 4); }
#pragma unroll 1
    for (int row = lane >> 3; row < ROWS && mb + row < M; row += 8) {
      f32x4 v0 = half_read(half, row, c) + b0, v1 = half_read(half, row, c + 4) + b1;
      if (a.act == ACT_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v0[e] = gelu_erf<true>(v0[e]); v1[e] = gelu_erf<true>(v1[e]); }
      } else if (a.act == ACT_SILU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v0[e] = silu<true>(v0[e]); v1[e] = silu<true>(v1[e]); }
      }
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) { o[e] = (bf16)v0[e]; o[4 + e] = (bf16)v1[e]; }
      *(bf16x8*)((bf16*)a.out + (size_t)(mb + row) * a.ldo + n0 + c) = o;
    }
  } else {
    const int c = (lane & 15) * 4;
    if (n0 + c >= a.N) return;
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (a.bias) b = *(const f32x4*)(a.bias + n0 + c);
    if constexpr (KIND == EPI_STORE_F32) {
#pragma unroll 1
      for (int row = lane >> 4; row < ROWS && mb + row < M; row += 4) {
        f32x4 v = half_read(half, row, c) + b;
        if (a.act != ACT_NONE) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], a.act);
        }
        *(f32x4*)((float*)a.out + (size_t)(mb + row) * a.ldo + n0 + c) = v;
      }
    } else {
      // eight rows of old values are requested before the first is used
#pragma unroll 1
      for (int row = lane >> 4; row < ROWS && mb + row < M; row += 32) {
        f32x4 old[8], g[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int gr = mb + row + 4 * p < M ? mb + row + 4 * p : M - 1;
          old[p] = *(const f32x4*)((const float*)a.out + (size_t)gr * a.ldo + n0 + c);
          if constexpr (KIND == EPI_GATE_RESID) g[p] = *(const f32x4*)(a.gate + (size_t)gr * a.ldg + n0 + c);
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          f32x4 v = half_read(half, row + 4 * p, c) + b;
          if constexpr (KIND == EPI_GATE_RESID) v *= g[p];
          if (mb + row + 4 * p < M) *(f32x4*)((float*)a.out + (size_t)(mb + row + 4 * p) * a.ldo + n0 + c) = old[p] + v;
        }
      }
    }
  }
}

template <int KIND, int WI, int WJ, int NS>
__global__ __launch_bounds__(256, 2 * NS * stage_bytes(WI, WJ) <= 160 * 1024 ? 2 : 1) void gemm_tile_kernel(GemmArgs a, int n_tiles,
                                                                                                       int m_tiles, int xm) {
  constexpr int TBM = 64 * WI, TBN = 64 * WJ;
  constexpr int ABYTES = TBM * TBK * 2, STAGE = stage_bytes(WI, WJ);
  constexpr int OB = out_blocks(WI, WJ);
  static_assert(2 * WI % WJ == 0 && WJ % 2 == 0 && 3 * WJ >= WI + WJ && WI % OB == 0,
                "loads and fragment reads divide over the column blocks, rows over the passes of the epilogue");
  __shared__ __attribute__((aligned(1024))) char s0[STAGE];
  __shared__ __attribute__((aligned(1024))) char s1[STAGE];
  __shared__ __attribute__((aligned(1024))) char s2[NS > 2 ? STAGE : 1];
  __shared__ __attribute__((aligned(1024))) char s3[NS > 2 ? STAGE : 1];

  // workgroup id % 8 is the XCD; the XCDs form xm groups along M times 8 / xm along N (as in gemm_bf16_kernel)
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int xn = 8 / xm;
  const int mt_per = (m_tiles + xm - 1) / xm;
  const int pq = slot / mt_per, mt = (xcd % xm) * mt_per + (slot - pq * mt_per);
  const int nt = pq * xn + xcd / xm;
  if (nt >= n_tiles || mt >= m_tiles) return;
  const int M = eff_rows(a.M, a.m_dev);
  const int m0 = mt * TBM;
  if (m0 >= M) return;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int kb16 = a.K >> 4, nblocks = a.N >> 5;
  const int n_stages = a.K / TBK;

  // what this wave fetches of a stage: 16 WI activation rows (8 rows of 128 B per load) and 2 WJ KiB of weight fragments
  const bf16* ga[2 * WI];
  const int piece = (lane & 7) ^ (lane >> 3);
#pragma unroll
  for (int i = 0; i < 2 * WI; ++i) {
    int row = m0 + 16 * WI * wave + 8 * i + (lane >> 3);
    row = row < M ? row : M - 1;                             // rows past M: valid reads, never stored
    ga[i] = (const bf16*)a.A + (size_t)row * a.lda + piece * 8;
  }
  const bf16* gw[WJ / 2];
#pragma unroll
  for (int i = 0; i < WJ / 2; ++i) {
    int nb = nt * 2 * WJ + (WJ / 2) * wave + i;
    nb = nb < nblocks ? nb : nblocks - 1;                    // columns past N: valid reads, never stored
    gw[i] = (const bf16*)a.W + (size_t)nb * kb16 * 512 + lane * 8;
  }
  // part q (of WJ) of this wave's loads of stage t
  auto load = [&](char* buf, int t, int q) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 2 * WI / WJ * q; i < 2 * WI / WJ * (q + 1); ++i)
      __builtin_amdgcn_global_load_lds((gptr)(ga[i] + (size_t)t * TBK), (lptr)(buf + (2 * WI * wave + i) * 1024), 16, 0, 0);
#pragma unroll
    for (int i = 2 * q; i < 2 * q + 2; ++i)
      __builtin_amdgcn_global_load_lds((gptr)(gw[i >> 2] + (size_t)(t * 4 + (i & 3)) * 512),
                                       (lptr)(buf + ABYTES + (2 * WJ * wave + i) * 1024), 16, 0, 0);
  };

  f32x16 acc[WI][WJ];
  // LDS offsets of this lane's fragments: activation row 32 WI wm + 32 i + lane % 32, piece 2 ks + lane / 32 (XOR-ed)
  const int arow = (32 * WI * wm + (lane & 31)) * 128, ax = lane & 7, ah = lane >> 5;
  const int woff = ABYTES + wn * (WJ * 4096) + lane * 16;
  bf16x8 fa[2][WI], fw[2][WJ];
  // fragment n of k-step ks in reading order: W 0, A 0 .. WI - 1, W 1 ..
  auto frag = [&](const char* buf, int ks, int set, int n) __attribute__((always_inline)) {
    if (n >= 1 && n <= WI) fa[set][n - 1] = *(const bf16x8*)(buf + arow + (n - 1) * 4096 + ((2 * ks + ah) ^ ax) * 16);
    else fw[set][n == 0 ? 0 : n - WI] = *(const bf16x8*)(buf + woff + (n == 0 ? 0 : n - WI) * 4096 + ks * 1024);
  };
  // the MFMAs of a k-step (fragments `set`), with the fragment reads of k-step ks of `buf` and the loads of stage t into
  // `lbuf` (t < 0: none) between them
  auto step = [&](const char* buf, int ks, int set, char* lbuf, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WJ; ++j) {
#pragma unroll
      for (int n = 3 * j; n < 3 * j + 3; ++n)
        if (n < WI + WJ) frag(buf, ks, set ^ 1, n);
      if (lbuf != nullptr) load(lbuf, t, j);
#pragma unroll
      for (int i = 0; i < WI; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i], fw[set][j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr int LPS = 2 * WI + 2 * WJ;                       // loads of a stage and wave
  // all of this wave's loads are there but those of its last `later` stages, and so are, behind the barrier, the others'
#define TILE_SYNC(later)                                  \
  do {                                                    \
    __builtin_amdgcn_sched_barrier(0);                    \
    __builtin_amdgcn_s_waitcnt(wait_vm((later) * LPS));   \
    __builtin_amdgcn_s_barrier();                         \
    asm volatile("" ::: "memory");                        \
    __builtin_amdgcn_sched_barrier(0);                    \
  } while (0)
  // one stage: `cur` holds it (its first fragments are in set 0), `nxt` receives the next; then `cur` is refilled
#define TILE_STAGE(cur, nxt, lbuf, t, later) \
  do {                                       \
    step(cur, 1, 0, nullptr, 0);             \
    step(cur, 2, 1, nullptr, 0);             \
    step(cur, 3, 0, nullptr, 0);             \
    TILE_SYNC(later);                        \
    step(nxt, 0, 1, lbuf, t);                \
  } while (0)

#pragma unroll
  for (int q = 0; q < WJ; ++q) load(s0, 0, q);
#pragma unroll
  for (int q = 0; q < WJ; ++q) load(s1, 1, q);
  if constexpr (NS > 2) {
#pragma unroll
    for (int q = 0; q < WJ; ++q) load(s2, 2, q);
#pragma unroll
    for (int q = 0; q < WJ; ++q) load(s3, 3, q);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < WI; ++i)
#pragma unroll
    for (int j = 0; j < WJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  TILE_SYNC(NS - 1);                                         // stage 0 is there, the others in flight
#pragma unroll
  for (int n = 0; n < WI + WJ; ++n) frag(s0, 0, 0, n);
  // n_stages is a multiple of NS.  The last NS stages are peeled, so that no load of the loop stands under a condition (the
  // compiler's count of the loads in flight would become a guess, and its waits early).
  for (int t = 0; t < n_stages - NS; t += NS) {
    TILE_STAGE(s0, s1, s0, t + NS, NS - 2);
    if constexpr (NS > 2) {
      TILE_STAGE(s1, s2, s1, t + NS + 1, NS - 2);
      TILE_STAGE(s2, s3, s2, t + NS + 2, NS - 2);
      TILE_STAGE(s3, s0, s3, t + NS + 3, NS - 2);
    } else {
      TILE_STAGE(s1, s0, s1, t + NS + 1, NS - 2);
    }
  }
  if constexpr (NS > 2) {
    TILE_STAGE(s0, s1, nullptr, 0, 2);
    TILE_STAGE(s1, s2, nullptr, 0, 1);
    TILE_STAGE(s2, s3, nullptr, 0, 0);
    TILE_STAGE(s3, s0, nullptr, 0, 0);
  } else {
    TILE_STAGE(s0, s1, nullptr, 0, 0);
    TILE_STAGE(s1, s0, nullptr, 0, 0);
  }
#undef TILE_STAGE

  // ---- the tile leaves: all waves are past their LDS reads behind the barrier
  TILE_SYNC(0);
#undef TILE_SYNC
  float* half = (float*)((wave < 2 ? s0 : s1) + (wave & 1) * (STAGE / 2));
  const int mb = m0 + 32 * WI * wm;
  if (mb >= M) return;
#define TILE_PART(J, I0)                                                                              \
  _Pragma("unroll") for (int i = 0; i < OB; ++i) _Pragma("unroll") for (int e = 0; e < 16; ++e) {     \
    d0[(32 * i + 8 * (e >> 2) + (e & 3)) * 64] = acc[(I0) + i][J][e];                                 \
    d1[(32 * i + 8 * (e >> 2) + (e & 3)) * 64] = acc[(I0) + i][(J) + 1][e];                           \
  }
  float* d0 = half + 4 * ah * 64 + ((lane & 31) ^ (ah << 5));
  float* d1 = half + 4 * ah * 64 + (((lane & 31) + 32) ^ (ah << 5));
  constexpr int PARTS = (WJ / 2) * (WI / OB);
#pragma unroll 1
  for (int p = 0; p < PARTS; ++p) {
    const int jj = p / (WI / OB), ip = p % (WI / OB);
    const int n0 = nt * TBN + 32 * WJ * wn + 64 * jj;
    if (n0 >= a.N) return;
    if (p == 0) { TILE_PART(0, 0) }
    if constexpr (PARTS > 1) if (p == 1) { TILE_PART(WI / OB > 1 ? 0 : 2, WI / OB > 1 ? OB : 0) }
    if constexpr (PARTS > 2) if (p == 2) { TILE_PART(0, 2 * OB) }
    half_out<KIND, 32 * OB>(a, half, mb + 32 * OB * ip, M, n0, lane);
  }
#undef TILE_PART
}

// ---- which tile, if any
// Both kernels are priced in microseconds and the cheapest is taken.  The prices were fitted to 2215 products timed on every
// tile and on the streaming kernel (100 pairs of 512 to 58368 columns and a K of 1024 to 13824, 256 to 8192 rows, every epilogue;
// beyond those sizes they are extrapolated): a tile's price is within 4 % of the measured time for half of them and within
// 12 % for 95 %.  Over all of them what is chosen takes 0.7 % more than the fastest choice would; it is more than 3 % behind
// the streaming kernel at 10, by up to 13 % (485 x 2752 x 8320 with SwiGLU), and the streaming kernel alone would take 18 % more.
//
// Compute units run whole tiles, and the tiles are dealt to the XCDs in fixed groups, so that a launch takes as many rounds as
// the fullest XCD's share has multiples of its 32 compute units: 255 tiles of 256 x 256 (4128 x 3840 x 1280) are two rounds, since
// one XCD gets 36 of them.  Tiles whose LDS lets two workgroups share a compute unit take `pair` for two rounds and `one` for an
// odd one; a launch that leaves compute units idle finds more of the L2 and of the clock.  Measured with all compute units busy:
//   tile       stages  microseconds for n stages of 64 k: one, pair
//   256 x 256  2       1.64 n + 12
//   192 x 128  2       0.85 n + 4.2    1.4 n + 4.9
//   128 x 128  2       0.745 n + 2.2   0.98 n + 3.3
//   192 x 128  4       0.74 n + 6
//   128 x 128  4       0.6 n + 3.5
// Four stages are for a tile that has its compute unit to itself: with two, 64 k are multiplied faster than the next 64
// arrive.  The epilogue's own work, per 64 x 64 outputs, weighs most where no second workgroup's MFMAs cover it.
struct TileVariant {
  int wi, wj, ns;
  double one_n, one_0, pair_n, pair_0;                       // pair_n 0: one workgroup per compute unit
  double gelu, silu, resid, f32;                             // epilogue, per 64 x 64 outputs
};
constexpr TileVariant VARIANTS[] = {
    {4, 4, 2, 1.64, 12.0, 0.0, 0.0, 0.9, 0.55, 0.4, 0.2},   {3, 2, 2, 0.85, 4.2, 1.4, 4.9, 0.65, 0.45, 0.45, 0.4},
    {2, 2, 2, 0.745, 2.2, 0.98, 3.3, 0.65, 0.45, 0.45, 0.4}, {3, 2, 4, 0.74, 6.0, 0.0, 0.0, 0.8, 0.45, 0.4, 0.3},
    {2, 2, 4, 0.6, 3.5, 0.0, 0.0, 0.8, 0.45, 0.4, 0.3},
};
constexpr int N_VARIANTS = (int)(sizeof(VARIANTS) / sizeof(VARIANTS[0]));

inline int up(int a, int b) { return (a + b - 1) / b; }
inline bool is_resid(const GemmArgs& a) { return a.epi == EPI_RESID || a.epi == EPI_GATE_RESID; }

double tile_us(const GemmArgs& a, const TileVariant& t) {
  const int m_tiles = up(a.M, 64 * t.wi), n_tiles = up(a.N, 64 * t.wj), xm = xcd_groups_along_m(a, m_tiles);
  const long k = (up(m_tiles, xm) * (long)up(n_tiles, 8 / xm) + 31) / 32;
  const double n = a.K / TBK, one = t.one_n * n + t.one_0;
  double us = t.pair_n > 0.0 ? (k / 2) * (t.pair_n * n + t.pair_0) + (k % 2) * one : k * one;
  // (few rows: the weights come from memory, and idle compute units help less)
  const double busy = std::min(1.0, (double)m_tiles * n_tiles / (256.0 * k));
  us *= 1.0 - (a.M > 640 ? 0.33 : 0.2) * (1.0 - busy);
  const double epi = a.act == ACT_GELU ? t.gelu : a.act == ACT_SILU ? t.silu : is_resid(a) ? t.resid : a.epi == EPI_STORE_F32 ? t.f32 : 0.0;
  return us + k * t.wi * t.wj * epi + 1.5;
}

// The streaming kernel (launch_wm's choice of tile and K splits).  It is only ahead where it has what the tiles lack: 32-row tiles,
// K splits, or few rows; everywhere else it was never more than 3 % faster than the best tile, and takes no part (infinite).
double streaming_us(const GemmArgs& a) {
  const double n = a.K / 64.0;
  const bool resid = is_resid(a);
  auto t = [&](int bm, int bn) { return (double)up(a.M, bm) * up(a.N, bn); };
  // rounds of w workgroups per compute unit: a share x of a last round's missing workgroups costs nothing
  auto rounds = [](double w, double x) { return w <= 1.0 ? 1.0 : x * w + (1.0 - x) * std::ceil(w); };
  constexpr double NEVER = 1e9;
  if (a.epi == EPI_SWIGLU) {
    if (a.M <= 640 && a.K % 256 == 0 && t(64, 128) <= 288) return 5.0 + rounds(t(64, 128) / 256, 0.5) * (0.31 * n + 1.0);
    if (t(t(128, 256) >= 900 ? 128 : 96, 256) >= 512) return a.M > 640 ? NEVER : 5.0 + rounds(t(96, 256) / 256, 0.5) * (0.8 * n + 4.0);
    return 4.0 + std::ceil(t(96, 64) / 256) * (0.31 * n + 7.0);
  }
  if (!resid && a.M <= 640) {
    const double w = t(64, 128) / 256;
    return 5.5 + rounds(w, 0.7) * (0.34 * n + 0.3) + (a.act == ACT_GELU ? 1.5 * w : a.epi == EPI_STORE_F32 ? 1.2 * w : 0.0);
  }
  if (t(96, 128) < 128 && t(32, 128) >= 64) {
    const double sp = resid ? std::min(std::max(std::ceil(256 / t(32, 128)), 1.0), std::min((double)up(a.K, 256), 4.0)) : 1.0;
    const double w = t(32, 128) * sp / 256;
    return (resid ? 4.5 : 3.0) + rounds(w, 0.6) * (0.25 * n / sp + (resid ? 0.8 : 0.5)) + (a.epi == EPI_GATE_RESID ? w : 0.0);
  }
  if (a.M > 640 && t(128, 128) > (a.K % 256 ? 320 : 192)) return NEVER;
  const double gate = a.epi == EPI_GATE_RESID ? 1.0 : 0.0;
  if (resid && !(t(64, 128) >= 512 || (t(64, 128) >= 256 && a.K <= 2048))) {
    const double t96 = t(96, 128), sp = t96 < 256 ? std::ceil(256 / t96) : 1.0;
    return 5.0 * gate + (sp == 1.0 ? 10.0 + rounds(t96 / 256, 0.5) * 0.46 * n : 20.0 + rounds(t96 * sp / 256, 0.5) * 0.3 * n / sp);
  }
  const double w = t(64, 128) / 256;
  return 5.5 + std::max(rounds(w, 0.5), 1.5) * (0.29 * n + (resid ? 3.2 : 1.5) + 3.0 * gate) + (a.act == ACT_GELU ? 0.7 * w : 0.0);
}

template <int WI, int WJ, int NS>
hipError_t launch_tile(hipStream_t s, const GemmArgs& a) {
  const int n_tiles = (a.N + 64 * WJ - 1) / (64 * WJ), m_tiles = (a.M + 64 * WI - 1) / (64 * WI);
  const int xm = xcd_groups_along_m(a, m_tiles);
  const int xn = 8 / xm;
  const int grid = 8 * ((m_tiles + xm - 1) / xm) * ((n_tiles + xn - 1) / xn);
  switch (a.epi) {
    case EPI_STORE: gemm_tile_kernel<EPI_STORE, WI, WJ, NS><<<grid, 256, 0, s>>>(a, n_tiles, m_tiles, xm); break;
    case EPI_STORE_F32: gemm_tile_kernel<EPI_STORE_F32, WI, WJ, NS><<<grid, 256, 0, s>>>(a, n_tiles, m_tiles, xm); break;
    case EPI_RESID: gemm_tile_kernel<EPI_RESID, WI, WJ, NS><<<grid, 256, 0, s>>>(a, n_tiles, m_tiles, xm); break;
    case EPI_GATE_RESID: gemm_tile_kernel<EPI_GATE_RESID, WI, WJ, NS><<<grid, 256, 0, s>>>(a, n_tiles, m_tiles, xm); break;
    case EPI_SWIGLU: gemm_tile_kernel<EPI_SWIGLU, WI, WJ, NS><<<grid, 256, 0, s>>>(a, n_tiles, m_tiles, xm); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// Index into VARIANTS, -1 where the streaming kernel stays.  Examples, streaming -> chosen (us): 3366 x 1024 x 4096 61 -> 38, 3366 x
// 1024 x 1024 24 -> 16, 4128 x 3840 x 1280 67 -> 50, 2304 x 1280 x 1280 27 -> 17, 1100 x 27648 x 5120 SwiGLU 326 -> 328, 1700 x 5120 x
// 5120 136 -> 111; it keeps 1500 x 1024 x 4096 (34 against 34), 1100 x 1280 x 5120 (39 against 42) and 576 x 5120 x 13824 (104 against 134).
int gemm_tile_variant(const GemmArgs& a) {
  if (a.epi > EPI_SWIGLU || a.M < 256 || a.K < 1024 || a.K % (2 * TBK) != 0 || a.N % 32 != 0) return -1;
  if (a.lda % 8 != 0 || a.ldo % 8 != 0 || (a.epi == EPI_GATE_RESID && a.ldg % 4 != 0) || (a.epi == EPI_SWIGLU && a.N % 64 != 0))
    return -1;
  // sixteen bytes a lane, in and out
  if ((((uintptr_t)a.A | (uintptr_t)a.W | (uintptr_t)a.out | (uintptr_t)a.bias | (uintptr_t)a.gate) & 15) != 0) return -1;
  double best = streaming_us(a);
  int choice = -1;
  for (int v = 0; v < N_VARIANTS; ++v) {
    if (a.K % (VARIANTS[v].ns * TBK) != 0) continue;
    const double us = tile_us(a, VARIANTS[v]);
    if (us < best) { best = us; choice = v; }
  }
  return choice;
}

hipError_t launch_gemm_tile(hipStream_t s, const GemmArgs& a, int variant) {
  switch (variant) {
    case 0: return launch_tile<4, 4, 2>(s, a);
    case 1: return launch_tile<3, 2, 2>(s, a);
    case 2: return launch_tile<2, 2, 2>(s, a);
    case 3: return launch_tile<3, 2, 4>(s, a);
    case 4: return launch_tile<2, 2, 4>(s, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fard
