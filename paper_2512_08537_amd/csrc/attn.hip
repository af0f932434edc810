// KV-cached causal attention for the few query rows of a speculative block.
//
// bf16 path.  One workgroup of 4 waves per (sample, kv head); the waves take the 32-position
// blocks of the cache round-robin and merge their partial results through LDS at the end.
// The products are computed transposed so that nothing but Q passes through a layout change:
//   S^T = K Q^T    A operand = one K block (keys as rows) read as contiguous 1 KiB fragments,
//                  B operand = Q^T held in registers for the whole kernel;
//   O^T = V^T P^T  A operand = one V block (dims as rows, keys along k), B operand = P^T taken
//                  directly from the S^T accumulators (the cache stores V with its keys permuted
//                  to the accumulator order, see rowops.hip), so probabilities never leave registers.
// Every output column of both products is one query row, i.e. one lane pair (lane, lane+32):
// the running softmax triple (m, l, a) with a = sum e^{s-m}(s-m) lives in those lanes; the row
// entropy ln l - a/l of the attention distribution (Eq. 1 / S2.1 indicator) falls out for free.
// With grouped KV heads the G query heads of a KV head are packed into the columns (G*n_q <= 64).
//
// With learned positions (no RoPE) the kernel also appends the new rows' K and V to the cache, so a layer
// needs no separate append launch.
//
// fp32 path, for the small fp32 configuration: a workgroup per (row, head) for head dims 32, 64 and 128 and caches of up to 7936
// positions, which also appends; one wave per (row, head) otherwise; scores in LDS.
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace fard {

namespace {

#ifndef ATTN_OCC
#define ATTN_OCC 4
#endif
#define ATTN_MIN_WG(DH, NQB) (((DH) == 64 && (NQB) == 1) ? ATTN_OCC : 1)

constexpr float LN2 = 0.6931471805599453f, LOG2E = 1.4426950408889634f;
// exponents below this are zero and stay finite times zero: the logarithm in a term p ln p and the distance of two references
// are held to it (an invisible or infinitely low score is -inf).  Never an exponent itself: the maximum would turn a NaN score into
// probability 0.
constexpr float T_MIN = -16384.f;

// An exponent is one fused s sc2 - m sc2 whose second product is rounded on its own: all exponents of a row are off by the same
// half of its last place, which cancels in the division by their sum.  For products beyond 2^24 it would be whole powers of
// two, up to an overflow: there the scores are subtracted first.  With x for m in one case and y for m sc2 in the other, the rest
// zero, an exponent is (s - x) sc2 - y.
struct Ref { float x, y; };
__device__ __forceinline__ Ref reference(float m, float sc2) {
#pragma clang fp contract(off)
  const float y = m * sc2;
  const bool big = fabsf(y) > 16777216.f;
  return Ref{big ? m : 0.f, big ? 0.f : y};
}
// the distance of two references
__device__ __forceinline__ float ref_distance(Ref a, Ref b, float sc2) { return fmaf(a.x - b.x, sc2, a.y - b.y); }

// c / nq for column indexes (c < 64)
__device__ __forceinline__ int col_head(int c, float inv_nq) { return (int)(((float)c + 0.5f) * inv_nq); }

// Short contexts are bound by the launch's chain of dependent reads (lengths -> rows -> keys -> store and re-read of the new
// rows -> merge; 8 us for 16 workgroups at 129 keys), long ones by the K / V stream.  So the wave's first block is requested
// before the lengths are there; the new rows (APPEND) go into an LDS image of the tail blocks together with the cached
// positions around them and from there into both the products and, whole 16-byte pieces, the cache; a block's K is requested
// again as soon as its scores are out, its V as soon as they are summed.  The running maximum is that of the raw
// scores, exponents and the accumulator a are in base 2.
template <int DH, int NQB, bool APPEND, bool SPLIT, bool ENT>
__global__ __launch_bounds__(256, ATTN_MIN_WG(DH, NQB)) void attn_bf16_kernel(const int* __restrict__ cache_len,
                                                        const int* __restrict__ row_start, const int* __restrict__ row_cnt,
                                                        const bf16* __restrict__ qkv, void* kcache, void* vcache, int ctx_pad,
                                                        int Hk, int ld, int n_heads,
                                                        bf16* __restrict__ out, int ldo, float* __restrict__ ent_heads,
                                                        int pass_stride, AttnSplit sp, int out_tiled) {
  constexpr int DC = DH / 16;      // k16 chunks of the head dim (QK^T)
  constexpr int DB = DH / 32;      // 32-dim row blocks of O^T
  constexpr int NCOL = 32 * NQB;
  constexpr int PK = 4 * DH;       // 16-byte pieces of a 32-key block
  // merge area: one slab of partial O^T per wave (4 DH (NCOL + 1) floats of dynamic LDS: 17-133 KB), so that the
  // four waves meet behind one barrier; with one shared accumulator and a read-modify-write round per wave the merge was
  // 5.3 us of a 15.8 us launch at DH = 128 with 64 columns.  Before the merge it holds the tail blocks.
  constexpr int OLD = NCOL + 1;                            // padded row: conflict-free column-major reads
  __shared__ float s_m[4][NCOL], s_l[4][NCOL], s_a[ENT ? 4 : 1][NCOL];
  extern __shared__ __attribute__((aligned(16))) float s_o[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cl = lane & 31, g = lane >> 5;
  const unsigned b = blockIdx.x / (unsigned)Hk, hk = blockIdx.x - b * (unsigned)Hk;
  const int G = n_heads / Hk;
  // several passes in one launch (blockIdx.y; the longest, i.e. last, pass is dispatched first): the per-sample
  // arrays of pass p start p * pass_stride entries in
  const int at = ((int)gridDim.y - 1 - (int)blockIdx.y) * pass_stride + (int)b;
  const int p0 = cache_len[at], r0 = row_start[at];
  const int nq = row_cnt ? row_cnt[at] : row_start[at + 1] - r0;   // (row_cnt: a pass over part of the sample's rows)

  const size_t head_elems = (size_t)ctx_pad * DH;
  bf16* Kb = (bf16*)kcache + ((size_t)b * Hk + hk) * head_elems;
  bf16* Vb = (bf16*)vcache + ((size_t)b * Hk + hk) * head_elems;
  bf16x8 kf[DC], vf[DB][2];
  auto load_k = [&](int kb) {
    const bf16x8* p = (const bf16x8*)(Kb + (size_t)kb * 32 * DH);
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) kf[dc] = p[dc * 64 + lane];
  };
  auto load_v = [&](int kb) {
    const bf16x8* p = (const bf16x8*)(Vb + (size_t)kb * 32 * DH);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) vf[db][hf] = p[(db * 2 + hf) * 64 + lane];
  };
  if constexpr (!SPLIT) {
    const int kb = min(wave, (ctx_pad >> 5) - 1);
    load_k(kb);
    load_v(kb);
  }
  if (nq <= 0) return;
  const int ncols = nq * G;                       // column c <-> (query head hk*G + c / nq, row c % nq)
  const float inv_nq = 1.0f / (float)nq;

  // Q^T fragments: lane supplies column cl (+32*qb), dims 16*dc + 8*g .. +7 (columns past the last repeat the first; they
  // are computed and not written)
  bf16x8 qf[DC][NQB];
  int lim[NQB];                                   // last visible position of the column
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int c = cl + 32 * qb < ncols ? cl + 32 * qb : 0;
    const int gq = G == 1 ? 0 : col_head(c, inv_nq);
    const int j = c - gq * nq;
    lim[qb] = p0 + j;
    const bf16* qp = qkv + (size_t)(r0 + j) * ld + (size_t)(hk * G + gq) * DH + 8 * g;
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) qf[dc][qb] = *(const bf16x8*)(qp + 16 * dc);
  }

  const int n_keys = p0 + nq;
  const int n_blocks = (n_keys + 31) >> 5;
  // APPEND: blocks [0, p0 / 32) hold only cached positions, visible to every row; the workgroup owns this sample's kv head,
  // assembles the blocks after them in LDS and stores the new rows' pieces of them to the cache
  const int tail0 = APPEND ? (p0 >> 5) : n_blocks;
  if constexpr (APPEND) {
    const bf16* ksrc = qkv + (size_t)r0 * ld + (size_t)(n_heads + hk) * DH;
    const bf16* vsrc = ksrc + (size_t)Hk * DH;
    for (int kb = tail0; kb < n_blocks; ++kb) {
      bf16x8* lk = (bf16x8*)s_o + (size_t)(kb - tail0) * 2 * PK;
      bf16x8* kblk = (bf16x8*)(Kb + (size_t)kb * 32 * DH);
      bf16x8* vblk = (bf16x8*)(Vb + (size_t)kb * 32 * DH);
#pragma unroll
      for (int i = 0; i < (PK + 255) / 256; ++i) {
        const int pc = tid + 256 * i;
        if (PK % 256 != 0 && pc >= PK) break;
        const int ln = pc & 63;
        // K: 8 dims of one key
        const int jk = kb * 32 + (ln & 31) - p0;
        const bool newk = (unsigned)jk < (unsigned)nq;
        const bf16x8* kp = newk ? (const bf16x8*)(ksrc + (size_t)jk * ld + (pc >> 6) * 16 + (ln >> 5) * 8) : kblk + pc;
        const bf16x8 kv8 = *kp;
        // V: 8 keys of one dim, in the order of the score accumulators
        bf16x8 vv = vblk[pc];
        const int dim = (pc >> 7) * 32 + (ln & 31), key0 = kb * 32 + ((pc >> 6) & 1) * 16 + (ln >> 5) * 4 - p0;
        bf16 ve[8];
        bool newv = false;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = key0 + ((e >> 2) << 3) + (e & 3);
          ve[e] = vsrc[(size_t)min(max(j, 0), nq - 1) * ld + dim];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = key0 + ((e >> 2) << 3) + (e & 3);
          const bool in = (unsigned)j < (unsigned)nq;
          newv = newv || in;
          vv[e] = in ? ve[e] : vv[e];
        }
        lk[pc] = kv8;
        lk[PK + pc] = vv;
        if (newk) kblk[pc] = kv8;
        if (newv) vblk[pc] = vv;
      }
    }
  }

  float m_run[NQB], l_run[NQB], a_run[NQB];
  f32x16 o[DB][NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    m_run[qb] = -INFINITY;
    l_run[qb] = 0.f;
    a_run[qb] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[db][qb][e] = 0.f;
  }
  const float sc2 = rsqrtf((float)DH) * LOG2E;
  // scores of one block, running triple, probabilities as the next product's operand
  auto softmax = [&](int kb, int qb, f32x16 s, bf16x8 (&pf)[2], auto masked) {
    constexpr bool MASK = decltype(masked)::value;
    // register e holds key 32*kb + 8*(e/4) + 4*g + e%4 for query column cl
    float bmax = -INFINITY;
    if constexpr (MASK) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = kb * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
        s[e] = (key <= lim[qb]) ? s[e] : -INFINITY;
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) bmax = fmaxf(bmax, s[e]);
    bmax = xor32_max(bmax);
    const float m_new = fmaxf(m_run[qb], bmax);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // (no key with a score above -inf so far)
    const Ref ref = reference(m_ref, sc2);
    float psum = 0.f, asum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float t = fmaf(s[e] - ref.x, sc2, -ref.y);
      const float p = __builtin_amdgcn_exp2f(t);
      psum += p;
      if constexpr (ENT) asum = fmaf(p, fmaxf(t, T_MIN), asum);
      pf[e >> 3][e & 7] = (bf16)p;
    }
    psum = xor32_sum(psum);
    const float dl = fmaxf(ref_distance(reference(m_run[qb], sc2), ref, sc2), T_MIN), corr = __builtin_amdgcn_exp2f(dl);
    if constexpr (ENT) a_run[qb] = fmaf(corr, fmaf(dl, l_run[qb], a_run[qb]), xor32_sum(asum));
    l_run[qb] = fmaf(corr, l_run[qb], psum);
    m_run[qb] = m_new;
    if (__any(corr != 1.f)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][qb][e] *= corr;
    }
  };
  auto score = [&](int qb) {
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int dc = 0; dc < DC; ++dc) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[dc], qf[dc][qb], s, 0, 0, 0);
    return s;
  };
  auto product = [&](int qb, const bf16x8 (&pf)[2]) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
        o[db][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][hf], pf[hf], o[db][qb], 0, 0, 0);
  };

  int kb_lo = 0, kb_hi = tail0;
  if constexpr (SPLIT) {                                   // this workgroup's share of the key blocks
    kb_lo = (int)(((unsigned)n_blocks * blockIdx.z) / (unsigned)sp.n);
    kb_hi = (int)(((unsigned)n_blocks * (blockIdx.z + 1)) / (unsigned)sp.n);
    if (kb_lo + wave < kb_hi) {
      load_k(kb_lo + wave);
      load_v(kb_lo + wave);
    }
  }
  // first the blocks of which every row sees every key, then the masked ones: with both softmaxes in one loop behind a branch
  // the next block's K and V did not fit beside them (36-168 bytes of scratch a lane).  Forward of 256 rows at 768 keys, 8 rotary
  // layers of 16 heads of 64: 2.84 -> 1.65 ms; prefill of 8 x 768 rows, 40 layers of 40 heads of 128: 136.3 -> 133.9 ms.
  auto block = [&](int kb, auto masked) {
    const bool more = kb + 4 < kb_hi;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      const f32x16 s = score(qb);
      if (qb == NQB - 1 && more) load_k(kb + 4);
      bf16x8 pf[2];
      softmax(kb, qb, s, pf, masked);
      product(qb, pf);
    }
    if (more) load_v(kb + 4);
  };
  const int kb_whole = APPEND ? kb_hi : min(kb_hi, (p0 + 1) >> 5);
  int kb = kb_lo + wave;
  for (; kb < kb_whole; kb += 4) block(kb, std::false_type{});
  if constexpr (!APPEND) {
    for (; kb < kb_hi; kb += 4) block(kb, std::true_type{});
  }
  if constexpr (APPEND) {
    __syncthreads();
    for (int kb = tail0 + ((wave - tail0) & 3); kb < n_blocks; kb += 4) {
      const bf16x8* lk = (const bf16x8*)s_o + (size_t)(kb - tail0) * 2 * PK;
#pragma unroll
      for (int dc = 0; dc < DC; ++dc) kf[dc] = lk[dc * 64 + lane];
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) vf[db][hf] = lk[PK + (db * 2 + hf) * 64 + lane];
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const f32x16 s = score(qb);
        bf16x8 pf[2];
        softmax(kb, qb, s, pf, std::integral_constant<bool, true>{});
        product(qb, pf);
      }
    }
  }

  // ---- merge the four waves
  if (g == 0) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      s_m[wave][cl + 32 * qb] = m_run[qb];
      s_l[wave][cl + 32 * qb] = l_run[qb];
      if constexpr (ENT) s_a[wave][cl + 32 * qb] = a_run[qb];
    }
  }
  __syncthreads();
  auto top = [&](int c) {                                  // largest reference of the column (0: no visible key at all)
    const float m = fmaxf(fmaxf(s_m[0][c], s_m[1][c]), fmaxf(s_m[2][c], s_m[3][c]));
    return m == -INFINITY ? 0.f : m;
  };
  float f_me[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) f_me[qb] = __builtin_amdgcn_exp2f(fmaxf(ref_distance(reference(m_run[qb], sc2), reference(top(cl + 32 * qb), sc2), sc2), T_MIN));
  // every wave lays its rescaled partial O^T down in its own slab: one barrier, no read-modify-write rounds
  float* slab = s_o + (size_t)wave * DH * OLD;
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int dim = 32 * db + 8 * (e >> 2) + 4 * g + (e & 3);   // O^T row
        slab[dim * OLD + cl + 32 * qb] = o[db][qb][e] * f_me[qb];
      }
  __syncthreads();
  // ---- normalise and write: thread -> (column, 8 consecutive dims)
  constexpr int D8 = DH / 8;
  for (int idx = tid; idx < NCOL * D8; idx += 256) {
    const int c = idx / D8, d8 = idx - c * D8;
    if (c >= ncols) continue;
    const float mstar = top(c);
    float lstar = 0.f, astar = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float dl = fmaxf(ref_distance(reference(s_m[w][c], sc2), reference(mstar, sc2), sc2), T_MIN), f = __builtin_amdgcn_exp2f(dl);
      lstar = fmaf(f, s_l[w][c], lstar);
      if constexpr (ENT) astar = fmaf(f, fmaf(dl, s_l[w][c], s_a[w][c]), astar);
    }
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = s_o[(d8 * 8 + i) * OLD + c];
#pragma unroll
      for (int w = 1; w < 4; ++w) acc[i] += s_o[((size_t)w * DH + d8 * 8 + i) * OLD + c];
    }
    const int gq = G == 1 ? 0 : col_head(c, inv_nq), j = c - gq * nq;
    const int head = hk * G + gq;
    if constexpr (SPLIT) {
      // keys split over workgroups: this one's running triple and unnormalised O row (relative to its own maximum)
      // go to the planes that attn_merge_kernel folds
      const size_t slot = ((size_t)blockIdx.z * sp.rows + (r0 + j)) * n_heads + head;
      *(f32x4*)(sp.o + slot * DH + d8 * 8) = f32x4{acc[0], acc[1], acc[2], acc[3]};
      *(f32x4*)(sp.o + slot * DH + d8 * 8 + 4) = f32x4{acc[4], acc[5], acc[6], acc[7]};
      if (d8 == 0) *(f32x4*)(sp.mla + slot * 4) = f32x4{mstar, lstar, astar, 0.f};
    } else {
      const float inv = 1.0f / lstar;
      bf16x8 v;
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (bf16)(acc[i] * inv);
      // (out_tiled: the rows in the tile order the output projection's narrow-tile GEMM reads; 8 dims are one piece)
      *(bf16x8*)(out + (out_tiled ? tile_offset(r0 + j, head * DH + d8 * 8, ldo) : (size_t)(r0 + j) * ldo + (size_t)head * DH + d8 * 8)) = v;
      if constexpr (ENT) {
        if (d8 == 0) ent_heads[(size_t)(r0 + j) * n_heads + head] = logf(lstar) - LN2 * astar * inv;
      }
    }
  }
}

// Folds the per-split results of attn_bf16_kernel: thread -> (row, head, 8 dims).
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnSplit sp, int n_heads, int dh, int M, const int* __restrict__ m_dev,
                                                         bf16* __restrict__ out, int ldo, float* __restrict__ ent_heads,
                                                         int out_tiled) {
  const int Me = eff_rows(M, m_dev);
  const int d8n = dh >> 3;
  const float sc2 = rsqrtf((float)dh) * LOG2E;
  const long total = (long)Me * n_heads * d8n;
  for (long idx = (long)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (long)gridDim.x * 256) {
    const int d8 = (int)(idx % d8n);
    const long rh = idx / d8n;                             // row * n_heads + head
    // every split's triple and output piece are requested before the first is used (split by split the kernel waited
    // for memory once per split)
    constexpr int NS = 8;                                  // sp.n <= 8 (checked at launch)
    f32x4 t[NS], lo[NS], hi[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const size_t slot = (size_t)(s < sp.n ? s : 0) * sp.rows * n_heads + rh;
      t[s] = *(const f32x4*)(sp.mla + slot * 4);
      lo[s] = *(const f32x4*)(sp.o + slot * dh + d8 * 8);
      hi[s] = *(const f32x4*)(sp.o + slot * dh + d8 * 8 + 4);
    }
    // (a split that saw no visible key has sum 0 and whatever reference: its maximum does not count; a NaN sum does)
    float mstar = -INFINITY;
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s < sp.n && t[s][1] != 0.f) mstar = fmaxf(mstar, t[s][0]);
    float lstar = 0.f, astar = 0.f;
    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (s >= sp.n || t[s][1] == 0.f) continue;
      const float dl = fmaxf(ref_distance(reference(t[s][0], sc2), reference(mstar, sc2), sc2), T_MIN), f = __builtin_amdgcn_exp2f(dl);
      lstar += f * t[s][1];
      astar += f * (t[s][2] + dl * t[s][1]);
#pragma unroll
      for (int i = 0; i < 4; ++i) { acc[i] += f * lo[s][i]; acc[4 + i] += f * hi[s][i]; }
    }
    const float inv = 1.0f / lstar;
    const int row = (int)(rh / n_heads), head = (int)(rh - (long)row * n_heads);
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (bf16)(acc[i] * inv);
    *(bf16x8*)(out + (out_tiled ? tile_offset(row, head * dh + d8 * 8, ldo) : (size_t)row * ldo + (size_t)head * dh + d8 * 8)) = v;
    if (ent_heads != nullptr && d8 == 0) ent_heads[rh] = logf(lstar) - LN2 * astar * inv;
  }
}

// fp32 path, head dims 32 / 64 / 128: one workgroup per (head, row, sample).  Every score is one chain of fused multiply-adds
// over the dims, every output one over the keys, and the sums of the exponentials go by lanes of one wave, all as in the
// kernel for any head dim below: the same bits.  A thread has a key for the scores (all its loads at once), the values go
// through LDS a tile of keys at a time, the first tile asked for before the scores.  append: the new rows' keys and values
// are read from qkv and stored to the cache by the first query head of their kv head.  (One wave, a key a lane and the
// values one after the other from memory: 16-17 us at 69 keys.)
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_wide_kernel(const int* __restrict__ cache_len, const int* __restrict__ row_start,
                                                            const int* __restrict__ row_cnt, const float* __restrict__ qkv, int ld,
                                                            int n_heads, KvGeom kv, int B, float* __restrict__ out, int ldo,
                                                            float* __restrict__ ent_heads, int pass_stride, int append) {
  extern __shared__ __attribute__((aligned(16))) float s_p[];   // [ctx_pad] scores / probabilities
  __shared__ float s_la[2];
  constexpr int TV = DH / 4, KT = 8192 / DH, NV = KT * TV / 256;   // threads a key of a tile, keys of a tile (32 KB), pieces a thread
  __shared__ __attribute__((aligned(16))) float s_v[KT * DH];
  const int head = blockIdx.x, j = blockIdx.y, z = blockIdx.z;
  const int b = z % B, pass_off = (z / B) * pass_stride;   // passes of one launch: blockIdx.z = pass * B + b
  const int p0 = cache_len[pass_off + b], r0 = row_start[pass_off + b];
  const int nq = row_cnt ? row_cnt[pass_off + b] : row_start[pass_off + b + 1] - r0;
  if (j >= nq) return;
  const int Hk = kv.n_kv_heads, G = n_heads / Hk, hk = head / G;
  const int tid = threadIdx.x;
  const int vis = p0 + j + 1, n_old = append ? p0 : vis;
  const float* q = qkv + (size_t)(r0 + j) * ld + (size_t)head * DH;
  const float* kn = qkv + (size_t)r0 * ld + (size_t)(n_heads + hk) * DH;   // new rows' keys; their values Hk heads on
  const float* vn = kn + (size_t)Hk * DH;
  float* Kc = (float*)kv.k + ((size_t)b * Hk + hk) * (size_t)kv.ctx_pad * DH;
  float* Vc = (float*)kv.v + ((size_t)b * Hk + hk) * (size_t)kv.ctx_pad * DH;
  f32x4 vv[NV];
  auto load_v = [&](int c0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int e = tid + 256 * i, c = min(c0 + e / TV, vis - 1), d = (e % TV) * 4;
      vv[i] = *(const f32x4*)((c < n_old ? Vc + (size_t)c * DH : vn + (size_t)(c - p0) * ld) + d);
    }
  };
  load_v(0);
  if (append && head == hk * G && tid < DH) {
    Kc[(size_t)(p0 + j) * DH + tid] = kn[(size_t)j * ld + tid];
    Vc[(size_t)(p0 + j) * DH + tid] = vn[(size_t)j * ld + tid];
  }
  const float scale = 1.0f / sqrtf((float)DH);
  for (int c = tid; c < vis; c += 256) {
    const float* kp = c < n_old ? Kc + (size_t)c * DH : kn + (size_t)(c - p0) * ld;
    f32x4 k4[DH / 4];
#pragma unroll
    for (int i = 0; i < DH / 4; ++i) k4[i] = *(const f32x4*)(kp + 4 * i);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < DH / 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(q[4 * i + e], k4[i][e], s);
    s_p[c] = s * scale;
  }
  __syncthreads();
  if (tid < WAVE) {
    float mx = -INFINITY;
    for (int c = tid; c < vis; c += WAVE) mx = fmaxf(mx, s_p[c]);
    mx = wave_max(mx);
    float l = 0.f, a = 0.f;
    for (int c = tid; c < vis; c += WAVE) {
      const float t = s_p[c] - mx, e = expf(t);
      s_p[c] = e;
      l += e;
      a = fmaf(e, t, a);
    }
    l = wave_sum(l);
    a = wave_sum(a);
    if (tid == 0) { s_la[0] = l; s_la[1] = a; }
  }
  float acc = 0.f;
  for (int c0 = 0; c0 < vis; c0 += KT) {
    if (c0 > 0) __syncthreads();                           // the previous tile is read
#pragma unroll
    for (int i = 0; i < NV; ++i) *(f32x4*)&s_v[(tid + 256 * i) * 4] = vv[i];
    __syncthreads();
    if (c0 + KT < vis) load_v(c0 + KT);
    if (tid < DH) {
      const int n = min(KT, vis - c0);
#pragma unroll 8
      for (int c = 0; c < n; ++c) acc = fmaf(s_p[c0 + c], s_v[c * DH + tid], acc);
    }
  }
  const float l = s_la[0], inv = 1.0f / l;
  if (tid < DH) out[(size_t)(r0 + j) * ldo + (size_t)head * DH + tid] = acc * inv;
  if (ent_heads != nullptr && tid == 0) ent_heads[(size_t)(r0 + j) * n_heads + head] = logf(l) - s_la[1] * inv;
}

// fp32 path, any head dim: one wave per (row, head).
__global__ __launch_bounds__(64) void attn_f32_kernel(const float* __restrict__ qkv, int ld, int n_heads, KvGeom kv,
                                                      const int* __restrict__ cache_len,
                                                      const int* __restrict__ row_start, const int* __restrict__ row_cnt,
                                                      int B, float* __restrict__ out,
                                                      int ldo, float* __restrict__ ent_heads, int max_keys, int pass_stride) {
  extern __shared__ float s_p[];                 // [max_keys] scores / probabilities
  const int head = blockIdx.x, b = blockIdx.z % B, j = blockIdx.y;
  const int pass_off = ((int)blockIdx.z / B) * pass_stride;       // passes of one launch: blockIdx.z = pass * B + b
  cache_len += pass_off;
  row_start += pass_off;
  if (row_cnt) row_cnt += pass_off;
  const int r0 = row_start[b];
  const int nq = row_cnt ? row_cnt[b] : row_start[b + 1] - r0;
  if (j >= nq) return;
  const int Hk = kv.n_kv_heads, dh = kv.d_head;
  const int hk = (head * Hk) / n_heads;
  const int lane = threadIdx.x;
  const int vis = cache_len[b] + j + 1;
  const float* q = qkv + (size_t)(r0 + j) * ld + (size_t)head * dh;
  const float* Kc = (const float*)kv.k + ((size_t)b * Hk + hk) * (size_t)kv.ctx_pad * dh;
  const float* Vc = (const float*)kv.v + ((size_t)b * Hk + hk) * (size_t)kv.ctx_pad * dh;
  const float scale = 1.0f / sqrtf((float)dh);
  float mx = -INFINITY;
  for (int c = lane; c < vis; c += WAVE) {
    float s = 0.f;
    for (int d = 0; d < dh; ++d) s += q[d] * Kc[(size_t)c * dh + d];
    s *= scale;
    s_p[c] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  float l = 0.f, a = 0.f;
  for (int c = lane; c < vis; c += WAVE) {
    const float t = s_p[c] - mx, e = expf(t);
    s_p[c] = e;
    l += e;
    a += e * t;
  }
  l = wave_sum(l);
  a = wave_sum(a);
  __syncthreads();
  const float inv = 1.0f / l;
  for (int d = lane; d < dh; d += WAVE) {
    float acc = 0.f;
    for (int c = 0; c < vis; ++c) acc += s_p[c] * Vc[(size_t)c * dh + d];
    out[(size_t)(r0 + j) * ldo + (size_t)head * dh + d] = acc * inv;
  }
  if (ent_heads != nullptr && lane == 0) ent_heads[(size_t)(r0 + j) * n_heads + head] = logf(l) - a * inv;
}

}  // namespace

bool attn_f32_wide(const KvGeom& kv, int n_heads, int ld) {
  const int dh = kv.d_head;
  return !kv.is_bf16 && (dh == 32 || dh == 64 || dh == 128) && ld % 4 == 0 && kv.n_kv_heads > 0 && n_heads % kv.n_kv_heads == 0 &&
         kv.ctx_pad <= 7936;                               // (scores and a tile of values in 64 KB of LDS)
}

hipError_t launch_attention(hipStream_t s, const void* qkv, int ld, int n_heads, KvGeom kv, const int* cache_len,
                            const int* row_start, int B, int nq_max, void* out, int ldo, float* ent_heads, int append,
                            const int* row_cnt, int n_pass, const AttnSplit* split, int M, const int* m_dev, int out_tiled) {
  if (B <= 0 || nq_max <= 0 || n_pass <= 0) return hipSuccess;
  // several passes at once read rows that an earlier pass of the same launch would have had to store
  if (n_pass > 1 && (append || row_cnt == nullptr || n_pass > 65535 || (long)B * n_pass > 65535)) return hipErrorInvalidValue;
  if (out_tiled && (!kv.is_bf16 || ldo % 32 != 0)) return hipErrorInvalidValue;
  if (!kv.is_bf16) {
    dim3 grid(n_heads, nq_max, B * n_pass);
    if (attn_f32_wide(kv, n_heads, ld)) {
      const size_t smem = (size_t)kv.ctx_pad * sizeof(float);
      auto go = [&](auto dh) {
        attn_f32_wide_kernel<decltype(dh)::value><<<grid, 256, smem, s>>>(cache_len, row_start, row_cnt, (const float*)qkv, ld, n_heads,
                                                                         kv, B, (float*)out, ldo, ent_heads, B, append);
      };
      if (kv.d_head == 32) go(std::integral_constant<int, 32>{});
      else if (kv.d_head == 64) go(std::integral_constant<int, 64>{});
      else go(std::integral_constant<int, 128>{});
      return hipGetLastError();
    }
    if (append) return hipErrorInvalidValue;
    const size_t smem = (size_t)kv.ctx_pad * sizeof(float);
    if (smem > 64 * 1024) return hipErrorInvalidValue;
    attn_f32_kernel<<<grid, 64, smem, s>>>((const float*)qkv, ld, n_heads, kv, cache_len, row_start, row_cnt, B, (float*)out,
                                           ldo, ent_heads, kv.ctx_pad, B);
    return hipGetLastError();
  }
  const int G = n_heads / kv.n_kv_heads;
  const int cols = G * nq_max;
  if (cols > 64 || n_heads % kv.n_kv_heads != 0) return hipErrorInvalidValue;
  AttnSplit sp{};
  sp.n = 1;
  if (split != nullptr && split->n > 1) {
    if (append || n_pass != 1 || split->o == nullptr || split->mla == nullptr || M > split->rows || M < 1 || split->n > 8)
      return hipErrorInvalidValue;                          // (the merge kernel holds at most 8 splits in registers)
    sp = *split;
  }
  const dim3 grid(B * kv.n_kv_heads, n_pass, sp.n);
  const int ps = B;
  const bf16* q = (const bf16*)qkv;
  bf16* o = (bf16*)out;
  const bool want_a = ent_heads != nullptr;                // (with split keys the merge writes the entropies)
#define FARD_ATT_L(DHV, NQBV, APPV, SPLV, ENTV)                                                                      \
  do {                                                                                                               \
    constexpr int slabs = 4 * DHV * (32 * NQBV + 1) * 4;   /* the four waves' slabs of partial O^T */                 \
    constexpr int tails = APPV ? 3 * 8 * DHV * 16 : 0;     /* or up to three tail blocks of K and V */                \
    constexpr int lds = slabs > tails ? slabs : tails;                                                               \
    if constexpr (lds > 64 * 1024) {                                                                                 \
      static bool attr_set = false;                                                                                  \
      if (!attr_set) {                                                                                               \
        hipError_t e = hipFuncSetAttribute((const void*)attn_bf16_kernel<DHV, NQBV, APPV, SPLV, ENTV>,               \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);                         \
        if (e != hipSuccess) return e;                                                                               \
        attr_set = true;                                                                                             \
      }                                                                                                              \
    }                                                                                                                \
    attn_bf16_kernel<DHV, NQBV, APPV, SPLV, ENTV><<<grid, 256, lds, s>>>(cache_len, row_start, row_cnt, q, kv.k, kv.v, kv.ctx_pad, \
                                                                         kv.n_kv_heads, ld, n_heads, o, ldo, ent_heads, ps, sp, out_tiled); \
  } while (0)
#define FARD_ATT_M(DHV, NQBV, ENTV)                                 \
  do {                                                              \
    if (sp.n > 1) FARD_ATT_L(DHV, NQBV, false, true, ENTV);         \
    else if (append) FARD_ATT_L(DHV, NQBV, true, false, ENTV);      \
    else FARD_ATT_L(DHV, NQBV, false, false, ENTV);                 \
  } while (0)
#define FARD_ATT(DHV, NQBV)                                                                    \
  do {                                                                                         \
    if (want_a) FARD_ATT_M(DHV, NQBV, true); else FARD_ATT_M(DHV, NQBV, false);                \
  } while (0)
  if (kv.d_head == 64) {
    if (cols <= 32) FARD_ATT(64, 1); else FARD_ATT(64, 2);
  } else if (kv.d_head == 128) {
    if (cols <= 32) FARD_ATT(128, 1); else FARD_ATT(128, 2);
  } else if (kv.d_head == 32) {
    if (cols <= 32) FARD_ATT(32, 1); else FARD_ATT(32, 2);
  } else {
    return hipErrorInvalidValue;
  }
#undef FARD_ATT
#undef FARD_ATT_M
#undef FARD_ATT_L
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || sp.n <= 1) return e;
  const long total = (long)M * n_heads * (kv.d_head / 8);
  const unsigned blocks = (unsigned)std::min<long>((total + 255) / 256, 2048);
  attn_merge_kernel<<<blocks, 256, 0, s>>>(sp, n_heads, kv.d_head, M, m_dev, o, ldo, ent_heads, out_tiled);
  return hipGetLastError();
}

}  // namespace fard
