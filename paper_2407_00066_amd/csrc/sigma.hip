// The per-token core product z'_t = Sigma_{i(t)} z_t (App. D, middle step;
// Sec. 3.1: Sigma_i is the only per-LoRA matrix), and the split-K reduction
// of the fused GEMM.
//
// Core product.  Tokens arrive sorted by (cluster, adapter), so tokens of one
// LoRA are contiguous.  The sort cuts the sorted positions into items: runs
// of one adapter, at most kSigmaChunk long.  A workgroup takes one item,
// stages that adapter's Sigma_i in LDS once (fp32, rows padded to r+1 words
// so that lanes reading one column hit distinct banks) and produces every
// output of the item's tokens with a fixed ascending-order fp32 dot product.
// z_t is first summed over the shrink's k-splits in fixed order.  No atomics:
// the result is bitwise reproducible.  With Sigma == null (uncompressed path)
// the stage only sums and converts.
#include "cts.h"
#include "cts_internal.h"
#include "ldsdma.h"

namespace cts {
namespace {

constexpr int kSigThreads = 256;
// MAXR: the largest rank a kernel instance takes (64 or 128).  LDS rows are
// MAXR + 4 floats: 16-byte aligned, and lanes reading one column of 16 rows
// (4 consecutive k each) land on distinct banks.

template <typename TI> struct Vec16;
template <> struct Vec16<float> {          // 4 floats per 16 bytes
  static constexpr int N = 4;
  __device__ static __forceinline__ void widen(const uint4& v, float* o) {
    o[0] = __uint_as_float(v.x); o[1] = __uint_as_float(v.y);
    o[2] = __uint_as_float(v.z); o[3] = __uint_as_float(v.w);
  }
};
template <> struct Vec16<bf16_t> {         // 8 bf16 per 16 bytes
  static constexpr int N = 8;
  __device__ static __forceinline__ void widen(const uint4& v, float* o) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = bf16_to_f32(static_cast<uint16_t>(w[i] & 0xffffu));
      o[2 * i + 1] = bf16_to_f32(static_cast<uint16_t>(w[i] >> 16));
    }
  }
};

template <typename TI> __device__ __forceinline__ void st(TI* p, int64_t i, float v);
template <> __device__ __forceinline__ void st<float>(float* p, int64_t i, float v) { p[i] = v; }
template <> __device__ __forceinline__ void st<bf16_t>(bf16_t* p, int64_t i, float v) { p[i].bits = f32_to_bf16(v); }

template <typename TI> __device__ __forceinline__ float ld(const TI* p, int64_t i);
template <> __device__ __forceinline__ float ld<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p, int64_t i) { return bf16_to_f32(p[i].bits); }

// Diagonal Sigma_i (Sec. 3.1, eq. JD-Diag; App. F: no batched product is
// needed): z'_t[c] = sigma_i[c] z_t[c], an elementwise scale.  Same items and
// the same fixed-order split sum as sigma_kernel; no LDS.
template <typename TI>
__global__ __launch_bounds__(kSigThreads) void sigma_diag_kernel(const float* __restrict__ zpart, int S,
                                                                 int T, int r,
                                                                 const int32_t* __restrict__ sorted_aid,
                                                                 int n, const int32_t* __restrict__ items,
                                                                 const int32_t* __restrict__ n_items,
                                                                 const TI* __restrict__ sigma,
                                                                 TI* __restrict__ zp,
                                                                 const int32_t* __restrict__ sorted_seg,
                                                                 const int32_t* __restrict__ seg_rank,
                                                                 int32_t* __restrict__ sorted_rank,
                                                                 const int32_t* __restrict__ split_dev,
                                                                 const int32_t* __restrict__ item_aid) {
  const int item = blockIdx.x;
  // the item's bounds and adapter are read with the item count (the grid
  // covers max_items items; the arrays hold max_items + 1 entries)
  const int n_it = n_items[0];
  const int lo = items[item], hi = items[item + 1];
  const int a_it = item_aid[item];
  // the shrink's split count (read from a valid address either way)
  const int s_dev = (split_dev ? split_dev : n_items)[0];
  // all five loads before the exit test: one round trip, not a chain
  asm volatile("" ::"s"(lo), "s"(hi), "s"(a_it), "s"(s_dev));
  if (item >= n_it) return;
  if (split_dev) S = min(s_dev, S);
  const int tid = threadIdx.x;
  const int cnt = (hi - lo) * r;
  const int rk = seg_rank ? seg_rank_of(seg_rank, sorted_seg[lo], r) : r;   // a multiple of 8
  if (sorted_rank && tid < hi - lo) sorted_rank[lo + tid] = rk;
  int a = a_it;
  a = a < 0 ? 0 : (a >= n ? n - 1 : a);
  const TI* sa = sigma + static_cast<int64_t>(a) * r;
  const int64_t split_stride = static_cast<int64_t>(T) * r;
  const float* zbase = zpart + static_cast<int64_t>(lo) * r;
  TI* out = zp + static_cast<int64_t>(lo) * r;
  for (int e4 = tid * 4; e4 < cnt; e4 += kSigThreads * 4) {
    const int c = e4 % r;                                  // r % 8 == 0: c..c+3 in one row
    const bool in_rank = c < rk;                           // and all four, or none, below rk
    float s[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = in_rank ? ld<TI>(sa, c + v) : 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int q = 0; in_rank && q < S; q += 16) {
      f32x4 w[16];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (q + u < S) w[u] = *reinterpret_cast<const f32x4*>(zbase + (q + u) * split_stride + e4);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (q + u < S) acc += w[u];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) st<TI>(out, e4 + v, s[v] * acc[v]);
  }
}

// Several modules in one launch (blockIdx.y = module m): module m's Sigma
// is sigma[m], and its z and z' are the columns [m r, m r + r) of rows ldz
// apart.
struct SigmaMods {
  const void* sigma[CTS_MAX_MODULES];
};

// ZB: split partials whose loads are in flight together per thread (the
// host picks the smallest of 8, 16 or 32 that covers the split; fewer
// registers mean more workgroups resident when there are many items)
template <typename TI, int MAXR, int ZB>
__global__ __launch_bounds__(kSigThreads) void sigma_kernel(const float* __restrict__ zpart, int S,
                                                            int T, int r,
                                                            const int32_t* __restrict__ sorted_aid,
                                                            int n, const int32_t* __restrict__ items,
                                                            const int32_t* __restrict__ n_items,
                                                            const TI* __restrict__ Sigma,
                                                            TI* __restrict__ zp,
                                                            const int32_t* __restrict__ sorted_seg,
                                                            const int32_t* __restrict__ seg_rank,
                                                            int32_t* __restrict__ sorted_rank, int ldz,
                                                            const int32_t* __restrict__ split_dev,
                                                            const SigmaMods mods, int nmod,
                                                            const int32_t* __restrict__ item_aid) {
  constexpr int kSigLd = MAXR + 4;
  __shared__ __attribute__((aligned(16))) float z[kSigmaChunk * kSigLd];
  __shared__ __attribute__((aligned(16))) float sig[MAXR * kSigLd];

  const int item = blockIdx.x;
  // the item's bounds and adapter are read with the item count (the grid
  // covers max_items items; the arrays hold max_items + 1 entries)
  const int n_it = n_items[0];
  const int lo = items[item], hi = items[item + 1];
  const int a_it = item_aid[item];
  // the shrink's split count (read from a valid address either way)
  const int s_dev = (split_dev ? split_dev : n_items)[0];
  // all five loads before the exit test: one round trip, not a chain
  asm volatile("" ::"s"(lo), "s"(hi), "s"(a_it), "s"(s_dev));
  if (item >= n_it) return;
  if (nmod > 0) {
    const int m = blockIdx.y;
    Sigma = static_cast<const TI*>(mods.sigma[m]);
    zpart += static_cast<int64_t>(m) * r;
    zp += static_cast<int64_t>(m) * r;
  }
  // pieces the shrink actually split the reduction into (at most S)
  if (split_dev) S = min(s_dev, S);
  const int tid = threadIdx.x;
  const int nt = hi - lo;                 // tokens of this item (<= kSigmaChunk), one adapter
  const int cnt = nt * r;                 // outputs of this item
  // rank of the item's segment (a multiple of 8): Sigma's entries past it and
  // z's are neither read nor used; they stage as zeros
  const int rk = seg_rank ? seg_rank_of(seg_rank, sorted_seg[lo], r) : r;
  if (sorted_rank && tid < nt) sorted_rank[lo + tid] = rk;

  // Loads first, uses after: this thread's split partials (they depend on
  // the item only) and its 16-byte pieces of Sigma_a (on the adapter) are
  // all in flight before the first is waited for.  z = sum over the
  // shrink's k-splits in fixed order; 4 consecutive values per thread and
  // round, ZB splits' loads in flight at a time.  Rows of zpart and zp are
  // ldz apart (ldz = r, or the stacked rank of several modules).
  const int64_t split_stride = static_cast<int64_t>(T) * ldz;
  const float* zbase = zpart + static_cast<int64_t>(lo) * ldz;
  constexpr int ZR = (kSigmaChunk * MAXR / 4 + kSigThreads - 1) / kSigThreads;   // rounds of 4 values
  f32x4 zacc[ZR];
  f32x4 zv[ZR][ZB];
#pragma unroll
  for (int u = 0; u < ZR; ++u) zacc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto zload = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < ZR; ++u) {
      const int e4 = (tid + u * kSigThreads) * 4;
      const bool ok = e4 < cnt && e4 % r < rk;
      const int64_t zo = static_cast<int64_t>(e4 / r) * ldz + e4 % r;
#pragma unroll
      for (int w = 0; w < ZB; ++w)
        if (ok && q + w < S) zv[u][w] = *reinterpret_cast<const f32x4*>(zbase + (q + w) * split_stride + zo);
    }
  };
  auto zsum = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < ZR; ++u) {
      const int e4 = (tid + u * kSigThreads) * 4;
      const bool ok = e4 < cnt && e4 % r < rk;
#pragma unroll
      for (int w = 0; w < ZB; ++w)
        if (ok && q + w < S) zacc[u] += zv[u][w];
    }
  };
  zload(0);

  // Sigma_a -> LDS as fp32
  if (Sigma != nullptr) {
    int a = a_it;
    a = a < 0 ? 0 : (a >= n ? n - 1 : a);
    constexpr int V = Vec16<TI>::N;
    constexpr int PER = (MAXR * MAXR / V + kSigThreads - 1) / kSigThreads;
    const uint4* sa = reinterpret_cast<const uint4*>(Sigma + static_cast<int64_t>(a) * r * r);
    const int nv = r * r / V;
    uint4 raw[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * kSigThreads;
      const int row = (e * V) / r, col = (e * V) % r;
      raw[u] = (e < nv && row < rk && col < rk) ? sa[e] : uint4{0u, 0u, 0u, 0u};
    }
    zsum(0);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + u * kSigThreads;
      if (e < nv) {
        float w[V];
        Vec16<TI>::widen(raw[u], w);
        const int row = (e * V) / r, col = (e * V) % r;     // V consecutive columns, col % V == 0
#pragma unroll
        for (int q = 0; q < V; q += 4)
          *reinterpret_cast<f32x4*>(sig + row * kSigLd + col + q) = f32x4{w[q], w[q + 1], w[q + 2], w[q + 3]};
      }
    }
  } else {
    zsum(0);
  }
  // splits past the first 16
  for (int q = ZB; q < S; q += ZB) {
    zload(q);
    zsum(q);
  }
#pragma unroll
  for (int u = 0; u < ZR; ++u) {
    const int e4 = (tid + u * kSigThreads) * 4;
    if (e4 < cnt) {
      const int i = e4 / r, c = e4 % r;
      *reinterpret_cast<f32x4*>(z + i * kSigLd + c) = zacc[u];
    }
  }
  __syncthreads();

  TI* out = zp + static_cast<int64_t>(lo) * ldz;
  if (Sigma == nullptr) {
    for (int e = tid; e < cnt; e += kSigThreads)
      st<TI>(out, static_cast<int64_t>(e / r) * ldz + e % r, z[(e / r) * kSigLd + e % r]);
    return;
  }
  // z'[i][c] = sum_q Sigma[c][q] z[i][q] on the fp32 matrix cores: one
  // 16x16x4 MFMA step multiplies the item's (up to 16) token rows by 16
  // columns of Sigma^T over 4 k; wave w takes column blocks w, w+4, ...
  // A lane reads one z value (row l%16, k l/16) and one Sigma value (row =
  // output column l%16, k l/16) per step.  Rows past the item's tokens and
  // columns past r read stale LDS and are never stored (an output depends
  // only on its own row of z and its own row of Sigma).
  const int lane = tid & 63, wave = tid >> 6;
  const int fr = lane & 15, fk = lane >> 4;
  for (int cb = wave; cb * 16 < r; cb += kSigThreads / 64) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float* zr = z + fr * kSigLd + fk;
    const float* sr = sig + (cb * 16 + fr) * kSigLd + fk;
    for (int q = 0; q < r; q += 4)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(zr[q], sr[q], acc, 0, 0, 0);
    const int c = cb * 16 + fr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * fk + v;
      if (i < nt && c < r) st<TI>(out, static_cast<int64_t>(i) * ldz + c, acc[v]);
    }
  }
}

// Small batches: the dense product's partials are summed and the
// up-projection U_k z'_t is added in one pass, y = sum_s part + U_k z'.
//
// Latency is the bound (a few MB in all), so a wave takes the smallest matrix-
// core tile, 16 rows by 16 sorted positions, and no barrier: its partials, its
// tokens' z' and the U rows of four cluster runs at a time are all in flight
// together.  A wave visits only the runs among its own 16 positions (as k-tiles
// of a whole token tile, 48 runs of one adapter each ran one after the other).
// 64 tokens, 4096 x 4096: 3.3 us at rank 64 with one cluster, 4.4 us with 48
// rank-16 LoRAs (with the partial sum it replaces, 13 us of the fused GEMM).
// FOLD: there is no full core, so z' is formed here from the shrink's pieces
// (one launch less: 19.9 -> 18.1 us a call at 64 tokens over 100 rank-16 LoRAs).
template <int KK, int FOLD>
__global__ __launch_bounds__(256) void expand_kernel(const ExpandParams p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int nrb = p.rb[p.n_mod];
  int rb = blockIdx.x % nrb;
  const int j0 = (blockIdx.x / nrb) * 16;
  int q = 0;
#pragma unroll
  for (int u = 1; u < kMaxGemmModules; ++u) q += (u < p.n_mod && rb >= p.rb[u]) ? 1 : 0;
  rb -= p.rb[q];
  const int M = p.M[q], m0 = rb * 64 + wave * 16;
  if (m0 >= M) return;
  const int jn = min(16, p.T - j0);
  const int jc = lane & 15, g = lane >> 4;
  const int j = j0 + min(jc, jn - 1);                  // (columns past the last repeat it; never stored)
  const int tok = p.perm[j], seg = p.sorted_seg[j];
  int rk = p.r;
  u32x4 z[KK];                                         // z' of column jc, k = 32 i + 8 g ..
  if constexpr (!FOLD) {
    if (p.sorted_rank) rk = p.sorted_rank[j];
    const __amdgpu_buffer_rsrc_t rZ = make_rsrc(p.zp, p.zp_bytes);
#pragma unroll
    for (int i = 0; i < KK; ++i) {
      const int k = 32 * i + 8 * g;
      z[i] = load16(rZ, k < p.r ? static_cast<uint32_t>((j * p.ldz + p.zoff[q] + k) * 2) : kOob);
    }
    // z' past the rank is 0 z, NaN where z overflowed: it meets U's masked
    // zeros as a zero (a rank is a multiple of 8)
    if (p.sorted_rank) {
#pragma unroll
      for (int i = 0; i < KK; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) z[i][e] = 32 * i + 8 * g < rk ? z[i][e] : 0u;
    }
  } else {
    const int S = min(p.zsplit[0], p.zS);
    int a = p.sdiag ? p.sorted_aid[j] : 0;
    a = min(max(a, 0), p.n_adapters - 1);
    if (p.seg_rank) rk = seg_rank_of(p.seg_rank, seg, p.r);
    // pieces summed in order, four pieces' loads in flight; k past the rank is
    // not read (a rank is a multiple of 8)
#pragma unroll
    for (int i = 0; i < KK; ++i) {
      const int k = 32 * i + 8 * g;
      const bool in = k < rk;
      const float* src = p.zpart + static_cast<int64_t>(j) * p.ldz + (in ? k : 0);
      const int64_t step = static_cast<int64_t>(p.T) * p.ldz;
      f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
      for (int s = 0; s < S; s += 4) {
        f32x4 x[4][2];
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (s + b < S) {
            x[b][0] = *reinterpret_cast<const f32x4*>(src + (s + b) * step);
            x[b][1] = *reinterpret_cast<const f32x4*>(src + (s + b) * step + 4);
          }
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (s + b < S) { lo += x[b][0]; hi += x[b][1]; }
      }
      if (p.sdiag) {
        const uint4 v = *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(p.sdiag) +
                                                        static_cast<int64_t>(a) * p.r + (in ? k : 0));
        float w[8];
        Vec16<bf16_t>::widen(v, w);
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] *= w[e]; hi[e] *= w[4 + e]; }
      }
      z[i] = u32x4{f32_to_bf16_pair(lo[0], lo[1]), f32_to_bf16_pair(lo[2], lo[3]), f32_to_bf16_pair(hi[0], hi[1]),
                   f32_to_bf16_pair(hi[2], hi[3])};
#pragma unroll
      for (int e = 0; e < 4; ++e) z[i][e] = in ? z[i][e] : 0u;
    }
  }
  // the partials of rows m0 + 4 g .. + 3 (M is a multiple of 8: all or none of them exist)
  const int mrow = m0 + 4 * g;
  const bool live = jc < jn && mrow < M;
  f32x4 part[kExpandMaxSplit];
  {
    const float* src = p.part + static_cast<int64_t>(tok) * p.part_ld + p.col[q] + (mrow < M ? mrow : 0);
    const int64_t stride = static_cast<int64_t>(p.T) * p.part_ld;
#pragma unroll
    for (int s = 0; s < kExpandMaxSplit; ++s)
      if (s < p.S) part[s] = *reinterpret_cast<const f32x4*>(src + s * stride);
  }
  const int prev = __shfl_up(seg, 1);
  uint32_t st = static_cast<uint32_t>(__ballot(lane < jn && (lane == 0 || seg != prev))) & 0xffffu;
  const uint32_t arow = static_cast<uint32_t>((m0 + jc) * p.r + 8 * g) * 2;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int NB = 4;                                // runs whose U loads go out together
  while (st) {
    u32x4 a[NB][KK];
    int lo[NB], hi[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      lo[b] = st ? __builtin_ctz(st) : 0;
      const uint32_t rest = st & (st - 1u);
      hi[b] = st ? (rest ? __builtin_ctz(rest) : jn) : 0;
      const int s = __builtin_amdgcn_readlane(seg, lo[b]);
      const int kl = st ? __builtin_amdgcn_readlane(rk, lo[b]) : 0;
      st = st ? rest : 0u;
      const __amdgpu_buffer_rsrc_t rU =
          make_rsrc(static_cast<const char*>(p.U[q]) + static_cast<int64_t>(s) * p.u_seg_bytes[q], p.u_seg_bytes[q]);
      // (rows past M lie past the segment's end and read zeros)
#pragma unroll
      for (int i = 0; i < KK; ++i) a[b][i] = load16(rU, 32 * i + 8 * g < kl ? arow + 64u * i : kOob);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bool in = jc >= lo[b] && jc < hi[b];
#pragma unroll
      for (int i = 0; i < KK; ++i) {
        u32x4 zb = z[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) zb[e] = in ? zb[e] : 0u;
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[b][i]),
                                                      __builtin_bit_cast(bf16x8, zb), acc, 0, 0, 0);
      }
    }
  }
  f32x4 y = part[0];
#pragma unroll
  for (int s = 1; s < kExpandMaxSplit; ++s)
    if (s < p.S) y += part[s];
  y += acc;
  if (!live) return;
  const int64_t o = static_cast<int64_t>(tok) * p.ldo[q] + mrow;
  if (p.out_dtype == 1) {
    const uint2 w = {f32_to_bf16_pair(y[0], y[1]), f32_to_bf16_pair(y[2], y[3])};
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.out[q]) + o) = w;
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(p.out[q]) + o) = y;
  }
}

template <int OUT_BF16>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int S,
                                                            int N, int M,
                                                            const int32_t* __restrict__ perm,
                                                            void* __restrict__ out, int64_t ldo,
                                                            const SplitkMods mods) {
  constexpr int V = OUT_BF16 ? 8 : 4;
  const int cpr = M / V;
  const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (c >= static_cast<int64_t>(N) * cpr) return;
  const int j = static_cast<int>(c / cpr), mc = static_cast<int>(c % cpr) * V;
  // several modules: columns [col[q], col[q+1]) of the partials are module
  // q's output (each a multiple of 8 wide, so a chunk lies in one module)
  int m = mc;
  if (mods.n > 0) {
    int q = 0;
#pragma unroll
    for (int u = 1; u < kMaxGemmModules; ++u) q += (u < mods.n && mc >= mods.col[u]) ? 1 : 0;
    out = mods.out[q];
    ldo = mods.ldo[q];
    m = mc - mods.col[q];
  }
  const int64_t row = perm ? perm[j] : j;     // read with the partials
  float acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.f;
  // the partials are summed in piece order; four pieces' loads go out before
  // their sums, so a launch waits for one round trip per four pieces (not one
  // per piece)
  const float* src0 = part + static_cast<int64_t>(j) * M + mc;
  const int64_t pstride = static_cast<int64_t>(N) * M;
  int s = 0;
  for (; s + 4 <= S; s += 4) {
    f32x4 x[4][V / 4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < V / 4; ++v)
        x[u][v] = *reinterpret_cast<const f32x4*>(src0 + (s + u) * pstride + 4 * v);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < V / 4; ++v) {
        acc[4 * v] += x[u][v][0]; acc[4 * v + 1] += x[u][v][1];
        acc[4 * v + 2] += x[u][v][2]; acc[4 * v + 3] += x[u][v][3];
      }
  }
  for (; s < S; ++s) {
#pragma unroll
    for (int v = 0; v < V / 4; ++v) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(src0 + s * pstride + 4 * v);
      acc[4 * v] += x[0]; acc[4 * v + 1] += x[1]; acc[4 * v + 2] += x[2]; acc[4 * v + 3] += x[3];
    }
  }
  if (OUT_BF16) {
    uint4 w;
    w.x = f32_to_bf16_pair(acc[0], acc[1]);
    w.y = f32_to_bf16_pair(acc[2], acc[3]);
    w.z = f32_to_bf16_pair(acc[4 % V], acc[5 % V]);
    w.w = f32_to_bf16_pair(acc[6 % V], acc[7 % V]);
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(out) + row * ldo + m) = w;
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(out) + row * ldo + m) =
        f32x4{acc[0], acc[1], acc[2], acc[3]};
  }
}

}  // namespace

hipError_t launch_sigma(const float* zpart, int S, int T, int r, const int32_t* sorted_aid, int n,
                        const int32_t* items, const int32_t* n_items, int max_items,
                        const void* Sigma, void* zp, int in_dtype, hipStream_t stream,
                        bool diag, const int32_t* sorted_seg, const int32_t* seg_rank,
                        int32_t* sorted_rank, int ldz, const int32_t* split_dev,
                        const void* const* sigmas, int nmod, const int32_t* item_aid) {
  if (seg_rank && !sorted_seg) return hipErrorInvalidValue;
  if (!item_aid) return hipErrorInvalidValue;
  if (sorted_rank && !seg_rank) return hipErrorInvalidValue;
  if (ldz <= 0) ldz = r;
  if (ldz != r && (diag || ldz < r || ldz % 4)) return hipErrorInvalidValue;
  if (nmod < 0 || nmod > CTS_MAX_MODULES || (nmod > 0 && (!sigmas || diag || ldz < nmod * r)))
    return hipErrorInvalidValue;
  SigmaMods mods{};
  for (int m = 0; m < nmod; ++m) mods.sigma[m] = sigmas[m];
  dim3 grid(max_items, nmod > 0 ? nmod : 1);
  if (diag && Sigma) {
    if (in_dtype == 0)
      hipLaunchKernelGGL(sigma_diag_kernel<float>, grid, dim3(kSigThreads), 0, stream, zpart, S, T, r,
                         sorted_aid, n, items, n_items, static_cast<const float*>(Sigma),
                         static_cast<float*>(zp), sorted_seg, seg_rank, sorted_rank, split_dev, item_aid);
    else
      hipLaunchKernelGGL(sigma_diag_kernel<bf16_t>, grid, dim3(kSigThreads), 0, stream, zpart, S, T, r,
                         sorted_aid, n, items, n_items, static_cast<const bf16_t*>(Sigma),
                         static_cast<bf16_t*>(zp), sorted_seg, seg_rank, sorted_rank, split_dev, item_aid);
    return hipGetLastError();
  }
  if (r > 128) return hipErrorInvalidValue;
  // S: the most pieces the shrink may have split into (the device-chosen
  // split is at most S)
  const int zb = S <= 8 ? 8 : (S <= 16 || r > 64) ? 16 : 32;
#define CTS_SIGMA_LAUNCH(TI_, MAXR_, ZB_)                                                              \
  hipLaunchKernelGGL((sigma_kernel<TI_, MAXR_, ZB_>), grid, dim3(kSigThreads), 0, stream, zpart, S, T, r, \
                     sorted_aid, n, items, n_items, static_cast<const TI_*>(Sigma), static_cast<TI_*>(zp), \
                     sorted_seg, seg_rank, sorted_rank, ldz, split_dev, mods, nmod, item_aid)
  if (in_dtype == 0 && r <= 64) {
    if (zb == 8) CTS_SIGMA_LAUNCH(float, 64, 8);
    else if (zb == 16) CTS_SIGMA_LAUNCH(float, 64, 16);
    else CTS_SIGMA_LAUNCH(float, 64, 32);
  } else if (in_dtype == 0) {
    if (zb == 8) CTS_SIGMA_LAUNCH(float, 128, 8);
    else CTS_SIGMA_LAUNCH(float, 128, 16);
  } else if (r <= 64) {
    if (zb == 8) CTS_SIGMA_LAUNCH(bf16_t, 64, 8);
    else if (zb == 16) CTS_SIGMA_LAUNCH(bf16_t, 64, 16);
    else CTS_SIGMA_LAUNCH(bf16_t, 64, 32);
  } else {
    if (zb == 8) CTS_SIGMA_LAUNCH(bf16_t, 128, 8);
    else CTS_SIGMA_LAUNCH(bf16_t, 128, 16);
  }
#undef CTS_SIGMA_LAUNCH
  return hipGetLastError();
}

hipError_t launch_expand(const ExpandParams& p, hipStream_t stream) {
  if (p.n_mod < 1 || p.n_mod > kMaxGemmModules || p.S < 1 || p.S > kExpandMaxSplit || p.r < 8 || p.r > 128 ||
      p.T < 1 || p.rb[0] != 0)
    return hipErrorInvalidValue;
  for (int q = 0; q < p.n_mod; ++q)
    if (p.M[q] % 8 || p.rb[q + 1] - p.rb[q] != (p.M[q] + 63) / 64) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(p.rb[p.n_mod]) * static_cast<unsigned>((p.T + 15) / 16));
  if (p.zpart && (!p.zsplit || p.zS < 1 || p.n_mod != 1 || p.zoff[0] != 0 || (p.sdiag && !p.sorted_aid)))
    return hipErrorInvalidValue;
#define CTS_EXPAND_LAUNCH(KK_)                                                                 \
  if (p.zpart) hipLaunchKernelGGL((expand_kernel<KK_, 1>), grid, dim3(256), 0, stream, p);     \
  else hipLaunchKernelGGL((expand_kernel<KK_, 0>), grid, dim3(256), 0, stream, p)
  switch ((p.r + 31) / 32) {
    case 1: CTS_EXPAND_LAUNCH(1); break;
    case 2: CTS_EXPAND_LAUNCH(2); break;
    case 3: CTS_EXPAND_LAUNCH(3); break;
    default: CTS_EXPAND_LAUNCH(4); break;
  }
#undef CTS_EXPAND_LAUNCH
  return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float* part, int S, int N, int M, const int32_t* perm,
                                void* out, int64_t ldo, int out_dtype, hipStream_t stream,
                                const SplitkMods* mods) {
  const int V = out_dtype == 1 ? 8 : 4;
  SplitkMods md{};
  if (mods) {
    if (mods->n < 1 || mods->n > kMaxGemmModules || mods->col[0] != 0 || mods->col[mods->n] != M)
      return hipErrorInvalidValue;
    for (int q = 0; q < mods->n; ++q)
      if (mods->col[q + 1] <= mods->col[q] || mods->col[q] % 8) return hipErrorInvalidValue;
    md = *mods;
  }
  const int64_t chunks = static_cast<int64_t>(N) * (M / V);
  dim3 grid(static_cast<unsigned>((chunks + 255) / 256));
  if (out_dtype == 1)
    hipLaunchKernelGGL(splitk_reduce_kernel<1>, grid, dim3(256), 0, stream, part, S, N, M, perm, out, ldo, md);
  else
    hipLaunchKernelGGL(splitk_reduce_kernel<0>, grid, dim3(256), 0, stream, part, S, N, M, perm, out, ldo, md);
  return hipGetLastError();
}

}  // namespace cts
