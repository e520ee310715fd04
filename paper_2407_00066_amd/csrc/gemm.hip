// Segmented MFMA GEMM used for both contractions of the layer that touch the
// weights:
//   * shrink   Z = V_k^T X       per cluster segment   (App. D, first step)
//   * fused    Y = W X + U_k Z'  base GEMM with the up-projection of every
//                                cluster segment accumulated into the same
//                                fp32 accumulators   (App. D: base term once
//                                for the batch, adapter term per token)
// The operand with rows m is a weight (W, V_k^T, U_k: k-contiguous); the
// operand with rows j is an activation in cluster-sorted order (x rows
// gathered through perm, or Z' rows).  A workgroup owns a BM x BN output tile
// and walks a flat list of BK-wide k-tiles: first the dense W tiles of its
// k-split, then, for every cluster segment that intersects its token columns,
// the k-tiles of that segment's basis with the other columns masked to zero.
//
// Global loads are raw buffer loads of 16 bytes straight into LDS: a row or k
// chunk outside the operand gets an out-of-range offset and reads as zero, so
// the loads carry no branches.
//
// Matrix cores: v_mfma_f32_16x16x32_bf16 (bf16 in, fp32 accumulate),
// v_mfma_f32_16x16x4_f32 for fp32 inputs.  Both
// operands of a product use the same per-lane k assignment, so the hardware's
// internal k order does not matter; only the accumulator layout (acc_row) is
// fixed by the instruction.
#include "cts_internal.h"
#include "ldsdma.h"

namespace cts {
namespace {

// MFMA shapes.  MB x MB output block per step of KS k; each lane holds the KG
// consecutive k of one 16-byte chunk of one row (A) or column (B): lane l ->
// row/column l % MB, chunk l / MB.
template <typename TI, int MB> struct MfmaTraits;
template <> struct MfmaTraits<bf16_t, 16> {      // v_mfma_f32_16x16x32_bf16
  static constexpr int KS = 32, KG = 8, NACC = 4, NI = 1;
  typedef f32x4 accv;
  __device__ static __forceinline__ accv mma(bf16x8 a, bf16x8 b, accv c, int = 0) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct MfmaTraits<float, 16> {       // 4 x v_mfma_f32_16x16x4_f32
  // NI instructions a step; number e takes every lane's e-th value of its chunk
  static constexpr int KS = 16, KG = 4, NACC = 4, NI = 4;
  typedef f32x4 accv;
  __device__ static __forceinline__ accv mma(bf16x8 a, bf16x8 b, accv c, int e) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4, a)[e], __builtin_bit_cast(f32x4, b)[e], c, 0,
                                                0, 0);
  }
};

// Row of accumulator element v of lane l inside a 16 x 16 block (the column is
// l % 16).
__device__ __forceinline__ int acc_row(int lane, int v) { return 4 * (lane >> 4) + v; }

__device__ __forceinline__ int split_lo(int n, int ks, int S) { return (int)((int64_t)n * ks / S); }

// XCD-aware tile order.  The dispatcher hands workgroup b to XCD b % 8, and
// each XCD has its own L2.  The linear block id is remapped so that XCD x
// owns one contiguous range of a grouped tile order (GROUP m-tiles by all
// n-tiles, column by column), i.e. a compact block of tiles whose weight rows
// and token columns stay in that XCD's L2.  The map is a bijection for any
// grid size.
constexpr int kXcds = 8;
constexpr int kGroupM = 8;
// group_m: m-tiles per group (0: kGroupM).
// b of nb: this workgroup among those that share the order.
__device__ __forceinline__ void tile_of_block(int gm, int gn, int* mt, int* nt, int* ks, int b, int nb,
                                              int group_m = 0) {
  const int nb_mn = gm * gn;
  const int G = group_m > 0 ? group_m : kGroupM;
  const int q = nb / kXcds, rem = nb % kXcds;
  const int x = b % kXcds, i = b / kXcds;
  const int L = x * q + min(x, rem) + i;
  *ks = L / nb_mn;
  const int l = L % nb_mn;
  const int per_group = G * gn;
  const int g = l / per_group;
  const int gsz = min(G, gm - g * G);               // m-tiles in this group
  const int r = l % per_group;
  *mt = g * G + r % gsz;
  *nt = r / gsz;
}

// The group size for a grid of gm x gn tiles split S ways: kGroupM when each
// XCD's share of the grid is a whole number of groups or of group columns;
// otherwise, when that share is a whole number of m-tiles with all their
// n-tiles, the share itself (one group per XCD), so that no weight row tile
// is fetched into two XCDs' L2s (e.g. 56 x 4 tiles: 7 m-tiles per XCD, not
// groups of 8 that straddle two XCDs).
int xcd_group_m(int gm, int gn, int S) {
  const int64_t nb = static_cast<int64_t>(gm) * gn * S;
  if (nb % kXcds) return kGroupM;
  const int64_t c = nb / kXcds, pg = static_cast<int64_t>(kGroupM) * gn, nmn = static_cast<int64_t>(gm) * gn;
  if (pg % c == 0 || c % pg == 0) return kGroupM;
  if (c % gn == 0 && nmn % c == 0) return static_cast<int>(c / gn);
  return kGroupM;
}

// ---------------------------------------------------------------------------
// The segmented GEMM on a ring of LDS stages (every shape but the prefill's).
//
// Each 16-byte buffer load writes its lane's chunk directly into LDS
// (buffer_load_dwordx4 ... lds): one wave instruction fills 1 KB, i.e. 8 tile
// rows of BK = 64 bf16 or 16 rows of BK = 32.  P LDS stages form a ring;
// k-tile t+P-1 is loaded while k-tile t is multiplied, so P-1 k-tiles of
// loads are in flight and no register holds staging data.  A lane stores
// chunk c of its row in slot c ^ key(row) (XOR swizzle; key = row % 16 for
// 256-byte rows, (row / 2) % 8 for 128-byte rows, (row / 4) % 4 for 64-byte
// rows).  The LDS serves a
// 16-byte read for 16 lanes (256 bytes, all 64 banks) per cycle, and a
// fragment read covers 16 consecutive rows at one logical chunk: with this
// key those 16 requests fall on 16 distinct bank groups.  An
// out-of-range lane (outside the operand, or a token column outside the
// current cluster segment) writes zeros.
//
// The completion of the loads and of the fragment reads is waited for
// explicitly (s_waitcnt with the exact count of loads still allowed in
// flight), and the fragment reads are issued as ds_read_b128 in inline
// assembly, so the compiler's blanket wait for LDS-writing loads before any
// LDS read does not apply.
template <typename TI, int BM, int BN, int BK, int WM, int WN, int MB, int P>
struct DmaCfg {
  static constexpr int NT = WM * WN * 64, NW = WM * WN;
  static constexpr int ELT = sizeof(TI), EPC = 16 / ELT;  // elements per 16-byte chunk
  static constexpr int ROWB = BK * ELT;                   // bytes per tile row
  static constexpr int CH = ROWB / 16;                    // 16-byte chunks per row
  static constexpr int RPI = 1024 / ROWB;                 // rows per 1 KB load
  static constexpr int SB = (BM + BN) * ROWB;             // bytes per stage
  static constexpr int QA = BM / RPI / NW, QB = BN / RPI / NW; // 1 KB loads per wave per k-tile
  static constexpr int LPT = QA + QB;                     // loads per thread per k-tile
  static constexpr int WTM = BM / WM, WTN = BN / WN;
  static constexpr int FM = WTM / MB, FN = WTN / MB;
  static constexpr int KS = MfmaTraits<TI, MB>::KS;       // k per multiply step
  static constexpr int NKS = BK / KS;
  static constexpr int SMEM = P * SB;
  static constexpr int MAXE = (128 + BK - 1) / BK;        // adapter k-tiles per run: rank <= 128
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "load split");
  static_assert(WTM % MB == 0 && WTN % MB == 0 && BK % KS == 0, "wave tile");
  static_assert(ROWB == 64 || ROWB == 128 || ROWB == 256, "row width");
  static_assert((P - 2) * LPT < 64, "vmcnt range");
};

// The epilogue writes straight from the accumulators (4 consecutive output
// features of one token per lane).
// MODS: the launch may hold several modules (p.n_mod > 0).
// DENSE: a shrink launch whose last p.d_blocks workgroups compute W x.
// Both roles read their operands at once and neither waits for the other: at
// 64 tokens, 4096 x 4096, 8.2 us for what took a shrink of 4.3 and a fused GEMM
// of 9.3 us and the gap between them.  Four stages: at six and eight the longer
// prologue costs more than the deeper ring gives (8.9 and 9.7 us).
template <typename TI, int BM, int BN, int BK, int WM, int WN, int MB, int P, int FSORT = 0, int MODS = 0,
          int DENSE = 0>
__global__ __launch_bounds__(WM * WN * 64, 1) void seg_gemm_dma_kernel(const GemmParams p) {
  using C = DmaCfg<TI, BM, BN, BK, WM, WN, MB, P>;
  using MT = MfmaTraits<TI, MB>;
  typedef typename MT::accv accv;
  constexpr uint32_t ELT = C::ELT;
  constexpr int KEYW = C::ROWB / 2;                        // the swizzle's row width

  __shared__ __attribute__((aligned(1024))) char smem[C::SMEM];
  __shared__ int32_t t_perm[BN];
  // adapter k-tiles closed by an entry of rank 0, and their number
  __shared__ __attribute__((aligned(8))) uint64_t sched[C::MAXE * BN + 1];
  __shared__ uint32_t n_sched_s;
  constexpr int FS = FSORT ? kFuseSortMaxT : 1;
  __shared__ uint64_t fs_raw[FS];                          // (key << 8) | token, in token order
  __shared__ uint32_t fs_key[FS];                          // keys, sorted
  __shared__ int32_t fs_perm[FS], fs_tile[FS + 1];
  __shared__ int32_t fs_cnt[2];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the workgroup's role, and its number among those of its role
  const int d_blocks = DENSE ? p.d_blocks : 0;
  const int nblk = static_cast<int>(gridDim.x) - d_blocks;     // the shrink's
  const bool dense_role = DENSE && static_cast<int>(blockIdx.x) >= nblk;
  const int blk = static_cast<int>(blockIdx.x) - (dense_role ? nblk : 0);
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // FSORT: bucketing of the (at most kFuseSortMaxT) tokens in LDS.  The key
  // is cluster << bits_n | adapter (the adapter alone without a cluster
  // map); the rank of token t is the number of smaller keys plus equal keys
  // of earlier tokens, the stable order of the separate sort.
  const int fs_cshift = p.fs_cluster ? p.fs_bits_n : 0;
  if (FSORT && !dense_role) {
    static_assert(!FSORT || (C::NT >= kFuseSortMaxT && BN >= 64), "one token per thread; 64-token tiles");
    const int T = p.N;
    // A cluster map that fits the ring's LDS (unused until the k loop) is
    // staged there: its loads go out with the adapter ids', one round trip
    // instead of a second, dependent one.
    const bool map_lds = p.fs_cluster && p.fs_n <= static_cast<int>(C::SMEM / 4);
    int32_t* const cmap = reinterpret_cast<int32_t*>(smem);
    int a = 0;
    if (tid < T) {
      a = p.fs_adapter[tid];
      a = a < 0 ? 0 : (a >= p.fs_n ? p.fs_n - 1 : a);
    }
    if (map_lds) {
      for (int i = tid; i < p.fs_n; i += C::NT) cmap[i] = p.fs_cluster[i];
      __syncthreads();
    }
    if (tid < T) {
      uint32_t key = static_cast<uint32_t>(a);
      if (p.fs_cluster) {
        int c = map_lds ? cmap[a] : p.fs_cluster[a];
        c = c < 0 ? 0 : (c >= p.fs_K ? p.fs_K - 1 : c);
        key |= static_cast<uint32_t>(c) << p.fs_bits_n;
      }
      fs_raw[tid] = (static_cast<uint64_t>(key) << 8) | static_cast<uint32_t>(tid);
    }
    __syncthreads();
    if (tid < T) {
      // the token index makes every composite distinct: the rank is the
      // number of smaller composites
      const uint64_t c = fs_raw[tid];
      int rank = 0;
      for (int j = 0; j < T; ++j) rank += fs_raw[j] < c ? 1 : 0;
      fs_perm[rank] = tid;
      fs_key[rank] = static_cast<uint32_t>(c >> 8);
    }
    __syncthreads();
    // wave 0: tile starts (a multiple of kSegTile or a new cluster) and, for
    // workgroup 0, core-product item starts (a multiple of kSigmaChunk or a
    // new key)
    if (wave == 0) {
      int nt_ = 0, ni_ = 0;
      for (int base = 0; base < T; base += 64) {
        const int j = base + lane;
        const bool valid = j < T;
        const uint32_t k = valid ? fs_key[j] : 0u;
        const uint32_t kp = (valid && j > 0) ? fs_key[j - 1] : 0u;
        const bool st = valid && (j % kSegTile == 0 || (k >> fs_cshift) != (kp >> fs_cshift));
        const bool si = valid && (j % kSigmaChunk == 0 || k != kp);
        const uint64_t bt = __ballot(st), bi = __ballot(si);
        if (st) fs_tile[nt_ + __popcll(bt & lt_mask)] = j;
        if (si && blk == 0) {
          p.fs_items[ni_ + __popcll(bi & lt_mask)] = j;
          if (p.fs_item_aid)
            p.fs_item_aid[ni_ + __popcll(bi & lt_mask)] = static_cast<int32_t>(k & ((1u << p.fs_bits_n) - 1u));
        }
        nt_ += __popcll(bt);
        ni_ += __popcll(bi);
      }
      if (lane == 0) {
        fs_tile[nt_] = T;
        fs_cnt[0] = nt_;
        if (blk == 0) { p.fs_items[ni_] = T; p.fs_nitems[0] = ni_; }
      }
    }
    if (blk == 0 && tid < T) {
      const uint32_t k = fs_key[tid];
      p.fs_perm[tid] = fs_perm[tid];
      p.fs_seg[tid] = static_cast<int32_t>(k >> fs_cshift);
      p.fs_aid[tid] = static_cast<int32_t>(k & ((1u << p.fs_bits_n) - 1u));
    }
    __syncthreads();
  }
  // Token-tile mode (explicit tiles, each inside one segment): the tile's
  // segment operand becomes the dense operand (A = A1 of that segment, B = B1),
  // so the whole k loop takes the dense load path and there is no second phase.
  const bool tlist = !dense_role && (FSORT || p.tile_start != nullptr);
  int mt, nt, ks;
  int s_pieces = p.ksplit;
  // the split along k follows the tile count only in the shrink's tile shape
  // (64 x 64, 128-byte rows); the other shapes keep the straight mapping
  constexpr bool kAdaptive = BM == 64 && BN == 64 && C::ROWB == 128;
  if (kAdaptive && tlist && p.split_target > 0) {
    // workgroups [0, gm n S) take the (row tile, tile, piece) triples, the
    // rest exit (whole workgroup, after every barrier above)
    const int gm = (p.M + BM - 1) / BM;
    const int ntl = FSORT ? fs_cnt[0] : p.n_tiles[0];
    const int per = max(gm * ntl, 1);
    s_pieces = min(max((p.split_target + per - 1) / per, 1), p.ksplit);
    if (blk == 0 && tid == 0 && p.split_out) p.split_out[0] = s_pieces;
    const int used = gm * ntl * s_pieces;
    if (blk >= used) return;
    tile_of_block(gm, ntl, &mt, &nt, &ks, blk, used);
  } else {
    const int rows = dense_role ? p.d_M : p.M;
    const int gm_all = ((MODS || DENSE) && !tlist && p.n_mod > 0) ? p.mod_rt[p.n_mod] : (rows + BM - 1) / BM;
    const int gn_all = tlist ? p.max_tiles : (p.N + BN - 1) / BN;
    if (dense_role) s_pieces = p.d_split;
    tile_of_block(gm_all, gn_all, &mt, &nt, &ks, blk, dense_role ? d_blocks : nblk, tlist ? 0 : p.group_m);
  }
  // the operands of this workgroup's module: with several modules in the
  // launch, row tiles [mod_rt[m], mod_rt[m+1]) are module m's
  int Mv = p.M;
  const void* A0v = p.A0;
  const void* A1v = p.A1;
  const void* B1v = p.B1;
  void* outv = p.out;
  float* partv = p.part;
  int64_t ldov = p.ldo;
  uint32_t a0v_bytes = p.a0_bytes, a1_seg_bytes = p.a1_seg_bytes, b1v_bytes = p.b1_bytes;
  if (dense_role) {
    Mv = p.d_M;
    A0v = p.d_A0; a0v_bytes = p.d_a0_bytes;
    partv = p.d_part;
  }
  if ((MODS || DENSE) && !tlist && p.n_mod > 0) {
    int mod = 0;
#pragma unroll
    for (int q = 1; q < kMaxGemmModules; ++q) mod += (q < p.n_mod && mt >= p.mod_rt[q]) ? 1 : 0;
    mod = __builtin_amdgcn_readfirstlane(mod);
    mt -= p.mod_rt[mod];
    Mv = p.mod_M[mod];
    A0v = p.mod_A0[mod]; a0v_bytes = p.mod_a0_bytes[mod];
    if (!dense_role) {
      A1v = p.mod_A1[mod]; a1_seg_bytes = p.mod_a1_seg_bytes[mod];
      B1v = p.mod_B1[mod]; b1v_bytes = p.mod_b1_bytes[mod];
      outv = p.mod_out[mod]; ldov = p.mod_ldo[mod];
    }
    if (partv) partv += p.mod_col[mod];
  }
  // row stride of the split partials (the modules' total width with several)
  const int64_t part_ld = ((MODS || DENSE) && !tlist && p.part_ld > 0) ? p.part_ld : Mv;
  const int S = s_pieces;
  int j0, jn;
  if (tlist) {
    // whole workgroup, after every barrier above
    if (nt >= (FSORT ? fs_cnt[0] : p.n_tiles[0])) return;
    j0 = FSORT ? fs_tile[nt] : p.tile_start[nt];
    jn = (FSORT ? fs_tile[nt + 1] : p.tile_start[nt + 1]) - j0;
  } else {
    j0 = nt * BN;
    jn = min(BN, p.N - j0);
  }
  const void* A0 = A0v;
  const void* B0 = p.B0;
  uint32_t a0_bytes = a0v_bytes, b0_bytes = p.b0_bytes;
  int64_t lda0 = p.lda0, ldb0 = p.ldb0;
  int K0 = p.K0, K1 = p.K1;
  bool b0_gather = true;
  if (tlist) {
    const int seg = FSORT ? static_cast<int>(fs_key[j0] >> fs_cshift) : p.tile_seg[nt];
    A0 = static_cast<const char*>(A1v) + static_cast<int64_t>(seg) * a1_seg_bytes;
    a0_bytes = a1_seg_bytes; lda0 = p.lda1; K0 = p.K1;
    B0 = B1v; b0_bytes = b1v_bytes; ldb0 = p.ldb1; b0_gather = p.b1_gather != 0;
    K1 = 0;
  } else if (dense_role) {
    lda0 = p.lda1; K0 = p.K1;
    B0 = B1v; b0_bytes = b1v_bytes; ldb0 = p.ldb1; b0_gather = false;
    K1 = 0;
  }
  const int m0 = mt * BM;
  static_assert(BN <= C::NT, "one token column per thread");

  // ---- load mapping: this lane's row and chunk in each 1 KB load ------------
  // load j of wave w covers tile rows [RPI*(w + NW*j), +RPI) of A (j < QA) or
  // B; lane l takes row +l/CH and global chunk (l%CH) ^ key(row), stored at
  // slot l%CH.
  const int lrow = lane / C::CH;
  // the key depends on the tile row modulo 16 only, and every wave's rows
  // start at a multiple of 16 plus RPI * wave
  static_assert((C::RPI * C::NW) % 16 == 0, "swizzle period");
  const int lchunk = (lane % C::CH) ^ swz_key<KEYW>(C::RPI * wave + lrow);
  const uint32_t cbytes = static_cast<uint32_t>(lchunk * 16);
  const uint32_t celem = static_cast<uint32_t>(lchunk * C::EPC);
  // Per-lane byte offsets of this lane's chunk at k = 0, for the dense (0)
  // and adapter (1) operands; kOob marks a row outside the operand (and, for
  // the dense token operand, a column outside the tile).  A k-tile adds its
  // uniform k byte offset: in the dense phase as the load's scalar offset, so
  // a full dense k-tile needs no per-lane arithmetic at all.
  uint32_t a0_v[C::QA], a1_v[C::QA], b0_v[C::QB], b1_v[C::QB];
  int b_jl[C::QB];
#pragma unroll
  for (int j = 0; j < C::QA; ++j) {
    const int m = m0 + C::RPI * (wave + C::NW * j) + lrow;
    const bool ok = m < Mv;
    a0_v[j] = ok ? static_cast<uint32_t>(m) * static_cast<uint32_t>(lda0) * ELT + cbytes : kOob;
    a1_v[j] = ok ? static_cast<uint32_t>(m) * static_cast<uint32_t>(p.lda1) * ELT + cbytes : kOob;
  }
  const __amdgpu_buffer_rsrc_t rA0 = make_rsrc(A0, a0_bytes);
  char* const smem_a = smem + wave * 1024;                  // + stage*SB + j*NW*1024
  char* const smem_b = smem + BM * C::ROWB + wave * 1024;

  // ---- dense k range of this split ----------------------------------------
  // Split ks takes its share of the dense k-tiles and the cluster runs ks, ks + S,
  // ks + 2S, ... (all of each run's k-tiles), so the adapter phase is spread over
  // the splits.
  const int nk0 = (K0 + BK - 1) / BK, nk1 = (K1 + BK - 1) / BK;
  const int d_lo = split_lo(nk0, ks, S), d_hi = split_lo(nk0, ks + 1, S);
  const int nd = d_hi - d_lo;
  // dense k-tiles that cover a whole BK slice: d_lo .. d_lo + nd_full - 1
  const int nd_full = nd - ((nd > 0 && d_hi * BK > K0) ? 1 : 0);
  auto dk = [&](int i) __attribute__((always_inline)) { return d_lo + i; };   // dense k-tile at position i

  // ---- the tokens of this lane's B rows, this thread's column for the
  // epilogue and, for wave 0, the clusters and ranks of columns lane + 64 q
  // (indices past the tile repeat its last column: no branch around the loads,
  // and each waits for the loads before it only)
  constexpr int NQ = (BN + 63) / 64;
  uint32_t tok[C::QB];
#pragma unroll
  for (int j = 0; j < C::QB; ++j) {
    const int jc = j0 + min(C::RPI * (wave + C::NW * j) + lrow, jn - 1);
    tok[j] = static_cast<uint32_t>(dense_role ? jc : FSORT ? fs_perm[jc] : p.perm[jc]);
  }
  const bool adapters = !tlist && p.sorted_seg && K1 > 0;
  int v_perm = 0, v_seg[NQ], v_rank[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) { v_seg[q] = 0; v_rank[q] = K1; }
  if (!tlist && !dense_role) v_perm = p.perm[j0 + min(tid, jn - 1)];
  if (wave == 0 && adapters) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) v_seg[q] = p.sorted_seg[j0 + min(lane + 64 * q, jn - 1)];
    if (p.seg_rank)
#pragma unroll
      for (int q = 0; q < NQ; ++q) v_rank[q] = p.sorted_rank[j0 + min(lane + 64 * q, jn - 1)];
  }

  // The weight rows do not depend on the token order: the first P - 1 dense
  // k-tiles' weight loads go out now, their token loads as soon as the lane's
  // tokens are known, and the cluster runs are listed while both are on their
  // way.  (A k-tile past the dense ones is loaded below, once the list is
  // there; its loads here are masked.)  With four stages the first k-tile's
  // wait in the loop is adjusted for this order.
  auto edge = [&](int st) __attribute__((always_inline)) {
    return st < nd_full ? 0u : (st < nd && static_cast<uint32_t>(dk(st) * BK) + celem < static_cast<uint32_t>(K0) ? 0u : kOob);
  };
#pragma unroll
  for (int st = 0; st < P - 1; ++st) {
    const uint32_t m = edge(st);
#pragma unroll
    for (int j = 0; j < C::QA; ++j)
      load16_lds(rA0, smem_a + st * C::SB + j * C::NW * 1024, a0_v[j] | m,
                 static_cast<uint32_t>(dk(st) * BK) * ELT);
  }
  // ---- token operand rows -------------------------------------------------
#pragma unroll
  for (int j = 0; j < C::QB; ++j) {
    const int jl = C::RPI * (wave + C::NW * j) + lrow;
    const uint32_t r1 = p.b1_gather ? tok[j] : static_cast<uint32_t>(j0 + jl);
    b_jl[j] = jl;
    const uint32_t r0 = b0_gather ? tok[j] : static_cast<uint32_t>(j0 + jl);
    b0_v[j] = (jl < jn) ? r0 * static_cast<uint32_t>(ldb0) * ELT + cbytes : kOob;
    b1_v[j] = r1 * static_cast<uint32_t>(p.ldb1) * ELT + cbytes;
  }
  const __amdgpu_buffer_rsrc_t rB0 = make_rsrc(B0, b0_bytes);
  const __amdgpu_buffer_rsrc_t rB1 = make_rsrc(B1v, b1v_bytes);
#pragma unroll
  for (int st = 0; st < P - 1; ++st) {
    const uint32_t m = edge(st);
#pragma unroll
    for (int j = 0; j < C::QB; ++j)
      load16_lds(rB0, smem_b + st * C::SB + j * C::NW * 1024, b0_v[j] | m,
                 static_cast<uint32_t>(dk(st) * BK) * ELT);
  }

  // ---- k-tile schedule: the dense tiles, then each cluster run's tiles ------
  // Wave 0 finds this split's runs (ks, ks + S, ...) from its
  // registers and lists their adapter k-tiles of this split below the run's
  // rank: low word = first column | columns << 9 | k-tile << 18, high word =
  // segment | rank << 16.
  const uint32_t sched_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(sched));
  const uint32_t count_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&n_sched_s));
  if (!tlist && tid < BN) lds_write4(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(t_perm)) + 4u * tid, v_perm);
  if (wave == 0) {
    uint32_t tot = 0;
    if (adapters) {
      uint64_t start[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        int prev = __shfl_up(v_seg[q], 1);
        if (q > 0 && lane == 0) prev = __builtin_amdgcn_readlane(v_seg[q > 0 ? q - 1 : 0], 63);
        const int col = lane + 64 * q;
        start[q] = __ballot(col < jn && (col == 0 || v_seg[q] != prev));
      }
      int run0 = 0;                                         // runs that start before column 64 q
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int lo = lane + 64 * q;
        int hi = jn;                                        // the next run's first column
#pragma unroll
        for (int q2 = NQ - 1; q2 > q; --q2)
          if (start[q2]) hi = 64 * q2 + __builtin_ctzll(start[q2]);
        const uint64_t above = start[q] & ~(lt_mask | (1ull << lane));
        if (above) hi = 64 * q + __builtin_ctzll(above);
        const int run = run0 + __popcll(start[q] & lt_mask);
        const bool mine = ((start[q] >> lane) & 1ull) && run >= ks && (S == 1 || (run - ks) % S == 0);
        const int kl = min(max(v_rank[q], 0), K1);
        const int c = mine ? min(nk1, (kl + BK - 1) / BK) : 0;   // at most MAXE <= 4
        const uint64_t b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4);
        const uint32_t at =
            tot + __popcll(b0 & lt_mask) + 2 * __popcll(b1 & lt_mask) + 4 * __popcll(b2 & lt_mask);
        const uint32_t ex = static_cast<uint32_t>(lo) | (static_cast<uint32_t>(hi - lo) << 9);
        const uint64_t ey =
            static_cast<uint64_t>(static_cast<uint32_t>(v_seg[q]) | (static_cast<uint32_t>(kl) << 16)) << 32;
#pragma unroll
        for (int i = 0; i < C::MAXE; ++i)
          if (i < c) lds_write8(sched_addr + 8u * (at + i), ey | (ex | (static_cast<uint32_t>(i) << 18)));
        tot += __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
        run0 += __popcll(start[q]);
      }
    }
    if (lane == 0) {
      lds_write8(sched_addr + 8u * tot, 0ull);              // rank 0: every load masked
      lds_write4(count_addr, tot);
    }
  }
  lds_barrier();
  uint32_t n_sched_v;
  lds_read4(n_sched_v, count_addr);
  wait_lgkmcnt<0>();
  pin(n_sched_v);
  const int n_sched = __builtin_amdgcn_readfirstlane(n_sched_v);
  const int ntiles = nd + n_sched;

  int lt = 0;

  // Per-k-tile load state, prepared once per k-tile (the loads themselves may
  // be issued in several groups between the multiply steps).
  struct TileLoad {
    __amdgpu_buffer_rsrc_t rA, rB;
    uint32_t kk, kmask, span, dsel;   // kk: uniform k byte offset of the k-tile
    int lo;
  };
  // the list's entry of the next k-tile to load (issued; the reader waits)
  auto read_entry = [&](uint64_t& e) __attribute__((always_inline)) {
    lds_read8(e, sched_addr + 8u * static_cast<uint32_t>(min(max(lt - nd, 0), n_sched)));
  };
  auto prep_next = [&](uint64_t entry) __attribute__((always_inline)) {
    TileLoad L;
    const bool valid = lt < ntiles;
    uint32_t k0, klim;
    if (lt < nd) {
      // dense phase (W X)
      L.lo = 0;
      L.span = static_cast<uint32_t>(jn);
      L.rA = rA0;
      L.rB = rB0;
      L.dsel = 0xffffffffu;
      k0 = static_cast<uint32_t>(dk(lt) * BK);
      klim = static_cast<uint32_t>(K0);
    } else {
      // adapter phase (U_k Z'): the entry of one k-tile of one cluster run
      // (past the end the closing entry, whose rank 0 masks every load)
      const uint32_t ex = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(entry));
      const uint32_t ey = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(entry >> 32));
      L.lo = static_cast<int>(ex & 511u);
      L.span = (ex >> 9) & 511u;
      const int seg = static_cast<int>(ey & 0xffffu);
      L.rA = make_rsrc(static_cast<const char*>(A1v) + static_cast<int64_t>(seg) * a1_seg_bytes,
                       a1_seg_bytes);
      L.rB = rB1;
      // phase select by mask arithmetic (a conditional pick between the two
      // offset arrays would make the compiler keep them in scratch memory)
      L.dsel = 0u;
      k0 = (ex >> 18) * BK;
      klim = ey >> 16;
    }
    L.kmask = (valid && k0 + celem < klim) ? 0u : kOob;
    L.kk = k0 * ELT;
    ++lt;
    return L;
  };
  // issue loads [g0, g1) of the k-tile (A loads first, then B) into stage st;
  // general form: any phase, per-lane k and column masks
  auto issue = [&](const TileLoad L, int st, int g0, int g1) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < C::QA; ++j)
      if (j >= g0 && j < g1)
        load16_lds(L.rA, smem_a + st * C::SB + j * C::NW * 1024,
                   ((a1_v[j] ^ ((a0_v[j] ^ a1_v[j]) & L.dsel)) + L.kk) | L.kmask);
#pragma unroll
    for (int j = 0; j < C::QB; ++j) {
      if (j + C::QA >= g0 && j + C::QA < g1) {
        const uint32_t jmask = (static_cast<uint32_t>(b_jl[j] - L.lo) < L.span) ? 0u : kOob;
        load16_lds(L.rB, smem_b + st * C::SB + j * C::NW * 1024,
                   ((b1_v[j] ^ ((b0_v[j] ^ b1_v[j]) & L.dsel)) + L.kk) | L.kmask | jmask);
      }
    }
  };
  // fast form: dense phase, whole k-tile; an out-of-range row stays at kOob
  // (plus a k offset below 2^31, still past the end of the operand)
  auto issue_fast = [&](const TileLoad L, int st, int g0, int g1) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < C::QA; ++j)
      if (j >= g0 && j < g1) load16_lds(rA0, smem_a + st * C::SB + j * C::NW * 1024, a0_v[j], L.kk);
#pragma unroll
    for (int j = 0; j < C::QB; ++j)
      if (j + C::QA >= g0 && j + C::QA < g1)
        load16_lds(rB0, smem_b + st * C::SB + j * C::NW * 1024, b0_v[j], L.kk);
  };
  // ---- fragment addresses ---------------------------------------------------
  const int wm = wave / WN, wn = wave % WN;
  const int fr = lane % MB, fg = lane / MB;                 // row in block, k group
  const uint32_t smem_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t a_row_addr = smem_base + static_cast<uint32_t>((wm * C::WTM + fr) * C::ROWB);
  const uint32_t b_row_addr = smem_base + static_cast<uint32_t>(BM * C::ROWB + (wn * C::WTN + fr) * C::ROWB);
  uint32_t slot[C::NKS];                                    // swizzled chunk slot per k-step
#pragma unroll
  for (int s2 = 0; s2 < C::NKS; ++s2) {
    const int chunk = s2 * (C::KS / C::EPC) + fg * (MT::KG / C::EPC);
    slot[s2] = static_cast<uint32_t>(((chunk ^ swz_key<KEYW>(fr)) * 16));
  }

  accv acc[C::FM][C::FN];
#pragma unroll
  for (int i = 0; i < C::FM; ++i)
#pragma unroll
    for (int j = 0; j < C::FN; ++j)
#pragma unroll
      for (int v = 0; v < MT::NACC; ++v) acc[i][j][v] = 0.f;

  // ---- main loop --------------------------------------------------------------
  // Per k-tile t (LDS stage cur), multiply step s uses fragment buffer s % 2:
  //  * steps before the last: the MFMAs of step s are interleaved one by one
  //    with the fragment reads of step s+1 and, in the first half of the
  //    k-tile, with the loads of k-tile t+P-1;
  //  * last step: half of its MFMAs, then the wait for this lane's loads of
  //    k-tile t+1 and the workgroup barrier (after it every wave's loads of
  //    t+1 are in LDS and every wave has finished reading k-tile t-1's stage,
  //    which the next iteration overwrites), then the fragment reads of
  //    k-tile t+1's first step interleaved with the remaining MFMAs.
  // So no multiply step waits on fragment-read latency, and the barrier sits
  // behind MFMAs already issued.
  static_assert(C::NKS % 2 == 0, "fragment buffers alternate across k-tiles");
  constexpr int NBL = C::FM * C::FN;                         // blocks of the wave
  constexpr int NM = NBL * MT::NI;                           // MFMAs per step, all blocks' first ones first
  constexpr int NR = C::FM + C::FN;                          // fragment reads per step
  constexpr int NLG = C::NKS > 2 ? C::NKS / 2 : 1;           // steps that issue loads
  constexpr int GPS = (C::LPT + NLG - 1) / NLG;              // loads per such step
  // issue slots per multiply step: one per MFMA or fragment read, or one per
  // load where a step has more loads than both (load-heavy, narrow tiles)
  constexpr int NSL0 = NM > NR ? NM : NR;
  constexpr int NSL = NSL0 > GPS ? NSL0 : GPS;
  bf16x8 fa[2][C::FM], fb[2][C::FN];
  auto read_frag = [&](int buf, int r, uint32_t sa, uint32_t sb, uint32_t sl) __attribute__((always_inline)) {
    if (r < C::FM) lds_read16(fa[buf][r], sa + sl + r * MB * C::ROWB);
    else lds_read16(fb[buf][r - C::FM], sb + sl + (r - C::FM) * MB * C::ROWB);
  };
  auto mma = [&](int buf, int m) __attribute__((always_inline)) {
    const int i = m % NBL / C::FN, j = m % C::FN;
    acc[i][j] = MT::mma(fa[buf][i], fb[buf][j], acc[i][j], m / NBL);
  };

  lt = P - 1;
  if (nd < P - 1) {
    // k-tiles of the prologue that belong to the adapter phase: after the
    // masked loads into their stages
    wait_vmcnt<0>();
    for (int st = nd; st < P - 1; ++st) {
      lt = st;
      uint64_t e;
      read_entry(e);
      wait_lgkmcnt<0>();
      pin(e);
      issue(prep_next(e), st, 0, C::LPT);
    }
    wait_vmcnt<0>();
  }
  wait_vmcnt<(P - 2) * C::QB>();         // k-tile 0's token loads, and all weight loads
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int r = 0; r < NR; ++r) read_frag(0, r, a_row_addr, b_row_addr, slot[0]);

  // Dense k-tiles that cover a whole BK slice are a prefix of the schedule;
  // while the k-tile being loaded is one of them the loop runs the fast load
  // form (uniform k offset only), then the general form to the end.
  const int nfast = max(0, min(ntiles, nd_full - (P - 1)));
  int cur = 0;   // LDS stage of k-tile t
  int t = 0;
  auto ktile = [&](const bool fast) __attribute__((always_inline)) {
    TileLoad L;
    uint64_t entry = 0;
    if (!fast) read_entry(entry);                          // waited for with the fragments
    int nst = cur + P - 1; if (nst >= P) nst -= P;         // stage of k-tile t+P-1
    int ncur = cur + 1; if (ncur >= P) ncur -= P;          // stage of k-tile t+1
    const uint32_t sa = a_row_addr + cur * C::SB, sb = b_row_addr + cur * C::SB;
    const uint32_t na = a_row_addr + ncur * C::SB, nb = b_row_addr + ncur * C::SB;
    auto iss = [&](int g0, int g1) __attribute__((always_inline)) {
      if (fast) issue_fast(L, nst, g0, g1);
      else issue(L, nst, g0, g1);
    };
#pragma unroll
    for (int s2 = 0; s2 < C::NKS; ++s2) {
      const int b = s2 & 1;
      wait_lgkmcnt<0>();                                   // step s2's fragments are in
#pragma unroll
      for (int i = 0; i < C::FM; ++i) pin(fa[b][i]);
#pragma unroll
      for (int j = 0; j < C::FN; ++j) pin(fb[b][j]);
      if (s2 == 0) {
        if (fast) {                                        // dense k-tile lt, whole
          L.kk = static_cast<uint32_t>(dk(lt) * BK) * ELT;
          ++lt;
        } else {
          pin(entry);
          L = prep_next(entry);
        }
      }
      if (s2 + 1 < C::NKS) {
#pragma unroll
        for (int m = 0; m < NSL; ++m) {
          if (m < NM) mma(b, m);
          if (m < NR) read_frag(b ^ 1, m, sa, sb, slot[s2 + 1]);
          if (s2 < NLG && m < GPS) iss(s2 * GPS + m, s2 * GPS + m + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int m = 0; m < NM / 2; ++m) {
          mma(b, m);
          __builtin_amdgcn_sched_barrier(0);
        }
        // this lane's loads of k-tile t+1.  In the prologue's order (the weight
        // loads of k-tiles 0 .. P-2, then their token loads) the token loads of
        // k-tile t+1 <= P-2 are followed by those of k-tiles t+2 .. P-2 and by
        // the t+1 k-tiles loaded since; t = 0's count serves them all.
        if (P >= 4 && t < P - 3) wait_vmcnt<(P >= 4 ? (P - 3) * C::QB + C::LPT : 0)>();
        else wait_vmcnt<(P - 2) * C::LPT>();
        __builtin_amdgcn_s_barrier();                      // ... and every wave's
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < (NM - NM / 2 > NR ? NM - NM / 2 : NR); ++m) {
          if (NM / 2 + m < NM) mma(b, NM / 2 + m);
          if (m < NR) read_frag(b ^ 1, m, na, nb, slot[0]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    cur = ncur;
  };
  for (; t < nfast; ++t) ktile(true);
  for (; t < ntiles; ++t) ktile(false);
  // (the fragments read ahead for a k-tile that does not follow keep their
  // registers until they are there)
  wait_lgkmcnt<0>();
#pragma unroll
  for (int i = 0; i < C::FM; ++i) pin(fa[0][i]);
#pragma unroll
  for (int j = 0; j < C::FN; ++j) pin(fb[0][j]);
  wait_vmcnt<0>();
  __syncthreads();

  // ---- epilogue from registers: lane holds rows acc_row(v..v+3) of column l%MB
#pragma unroll
  for (int j = 0; j < C::FN; ++j) {
    const int jl = wn * C::WTN + j * MB + lane % MB;
    const bool jok = jl < jn;
    const int64_t orow = p.out_perm ? t_perm[jl] : static_cast<int64_t>(j0 + jl);
#pragma unroll
    for (int i = 0; i < C::FM; ++i)
#pragma unroll
      for (int v = 0; v < MT::NACC; v += 4) {
        const int m = m0 + wm * C::WTM + i * MB + acc_row(lane, v);
        if (!jok || m >= Mv) continue;
        const f32x4 val = f32x4{acc[i][j][v], acc[i][j][v + 1], acc[i][j][v + 2], acc[i][j][v + 3]};
        if (partv) {
          *reinterpret_cast<f32x4*>(partv + (static_cast<int64_t>(ks) * p.N + j0 + jl) * part_ld + m) = val;
        } else if (p.out_dtype == 1) {
          uint2 w;
          w.x = f32_to_bf16_pair(val[0], val[1]);
          w.y = f32_to_bf16_pair(val[2], val[3]);
          *reinterpret_cast<uint2*>(static_cast<uint16_t*>(outv) + orow * ldov + m) = w;
        } else {
          *reinterpret_cast<f32x4*>(static_cast<float*>(outv) + orow * ldov + m) = val;
        }
      }
  }
}

// ---------------------------------------------------------------------------
// Prefill tile: 256 x 256 outputs per workgroup of eight waves (64 x 128 each),
// bf16 in, 16x16x32 MFMA.
//
// A tile of this size needs 64 B of operands per matrix-core cycle pair from
// L2, and what bounds it is how long a load may take: with the whole LDS as
// two 64-deep stages a load had three quarters of a k-tile to arrive.  Here
// the reduction is walked in 32-deep units through a ring of four, and a unit's
// slot is refilled as soon as its last fragment has been read, so a load has
// three units (one and a half of those k-tiles) to arrive:
//   first part   12 of 32 MFMAs; under them the reads of the wave's second 64
//                columns
//   wait         those reads (after which this wave is done with the unit's
//                slot) and this wave's loads of unit u + 1; then the barrier
//   second part  the other 20; under them the fragment reads of unit u + 1
// Fragments take 64 registers (a unit's rows and half its columns, twice) beside
// the 128 accumulators, so nothing spills.
// The adapter phase is a list of (run, unit) entries in LDS, uniform or mixed
// ranks alike: one 8-byte read per unit, a unit ahead of its loads.
// The setup before the loop holds no wait for the weights in flight and one
// round trip for the tokens, and the output leaves as whole rows.
// T = 4096, 4096 x 4096, 25 clusters of rank 64, against the two-stage 64-deep ring
// it replaces: 116 -> 111 us a launch with the weights in the last-level cache,
// 119 -> 118 from HBM.  PAIR (rows that start between multiples of 64 bytes):
// launch_prefill says why.
struct PrefillCfg {
  static constexpr int BM = 256, BN = 256, BK = 32, NT = 512, P = 4;   // eight waves, 4 x 2
  static constexpr int ROWB = BK * 2, SB = (BM + BN) * ROWB;
  static constexpr int WTM = 64, WTN = 128;
  static constexpr int ST_ROWB = BM * 2 + 16;         // staged bf16 output row (bytes)
  static constexpr int SMEM = P * SB > BN * ST_ROWB ? P * SB : BN * ST_ROWB;
  static constexpr int MAXU = 4;                      // adapter units per run: rank <= 128
};

template <bool PAIR>
__global__ __launch_bounds__(512, 1) void prefill_gemm_kernel(const GemmParams p) {
  using C = PrefillCfg;
  using MT = MfmaTraits<bf16_t, 16>;
  __shared__ __attribute__((aligned(1024))) char smem[C::SMEM];
  // the adapter units' list, closed by an entry of rank 0, and its length
  __shared__ __attribute__((aligned(8))) uint64_t sched[C::MAXU * C::BN + 1];
  __shared__ uint32_t n_sched_s;
  using std::integral_constant;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int mt, nt, ks;
  const int gm_all = p.n_mod > 0 ? p.mod_rt[p.n_mod] : (p.M + C::BM - 1) / C::BM;
  tile_of_block(gm_all, (p.N + C::BN - 1) / C::BN, &mt, &nt, &ks, blockIdx.x, gridDim.x, p.group_m);
  int Mv = p.M;
  const void* A0v = p.A0;
  const void* A1v = p.A1;
  const void* B1v = p.B1;
  void* outv = p.out;
  int64_t ldov = p.ldo;
  uint32_t a0_bytes = p.a0_bytes, a1_seg_bytes = p.a1_seg_bytes, b1_bytes = p.b1_bytes;
  if (p.n_mod > 0) {                                  // the module that owns this row tile
    int mod = 0;
#pragma unroll
    for (int q = 1; q < kMaxGemmModules; ++q) mod += (q < p.n_mod && mt >= p.mod_rt[q]) ? 1 : 0;
    mod = __builtin_amdgcn_readfirstlane(mod);
    mt -= p.mod_rt[mod];
    Mv = p.mod_M[mod];
    A0v = p.mod_A0[mod]; a0_bytes = p.mod_a0_bytes[mod];
    A1v = p.mod_A1[mod]; a1_seg_bytes = p.mod_a1_seg_bytes[mod];
    B1v = p.mod_B1[mod]; b1_bytes = p.mod_b1_bytes[mod];
    outv = p.mod_out[mod]; ldov = p.mod_ldo[mod];
  }
  const int m0 = mt * C::BM, j0 = nt * C::BN, jn = min(C::BN, p.N - j0);
  const int K0 = p.K0, K1 = p.sorted_seg ? p.K1 : 0;

  // ---- load mapping: wave w's loads cover rows 16 w + {0, 128} .. + 16 of each
  // operand; lane l takes row l / 4 and stores chunk (l % 4) ^ key there
  const int lrow = 16 * wave + (lane >> 2);
  const int lchunk = (lane & 3) ^ swz_key<32>(lane >> 2);
  const uint32_t cbytes = static_cast<uint32_t>(lchunk * 16);
  uint32_t a0_v[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = m0 + lrow + 128 * j;
    a0_v[j] = m < Mv ? static_cast<uint32_t>(m) * static_cast<uint32_t>(p.lda0) * 2 + cbytes : kOob;
  }
  const __amdgpu_buffer_rsrc_t rA0 = make_rsrc(A0v, a0_bytes);
  const __amdgpu_buffer_rsrc_t rB0 = make_rsrc(p.B0, p.b0_bytes);
  const __amdgpu_buffer_rsrc_t rB1 = make_rsrc(B1v, b1_bytes);
  char* const smem_a = smem + wave * 1024;
  char* const smem_b = smem + C::BM * C::ROWB + wave * 1024;

  // ---- the tokens whose rows this lane loads; for wave 0, which lists the
  // cluster runs, the clusters and ranks of columns lane + 64 q (indices past
  // the tile repeat its last column: no branch around the loads)
  uint32_t b0_v[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) b0_v[j] = static_cast<uint32_t>(p.perm[j0 + min(lrow + 128 * j, jn - 1)]);
  int v_seg[4] = {0, 0, 0, 0}, v_rank[4] = {K1, K1, K1, K1};
  if (wave == 0 && K1 > 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v_seg[q] = p.sorted_seg[j0 + min(lane + 64 * q, jn - 1)];
    if (p.seg_rank)
#pragma unroll
      for (int q = 0; q < 4; ++q) v_rank[q] = p.sorted_rank[j0 + min(lane + 64 * q, jn - 1)];
  }

  // The weight rows do not wait for the token order: the first units' go out
  // now, the token rows' as soon as this lane's two tokens are known, and the
  // adapter units are listed while both are on their way.
  const int nd = (K0 + C::BK - 1) / C::BK, nd_full = K0 / C::BK;   // nd_full >= P
#pragma unroll
  for (int u = 0; u < C::P; ++u)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      load16_lds(rA0, smem_a + u * C::SB + j * 8192, a0_v[j], static_cast<uint32_t>(u * C::ROWB));
#pragma unroll
  for (int j = 0; j < 2; ++j)
    b0_v[j] = lrow + 128 * j < jn ? b0_v[j] * static_cast<uint32_t>(p.ldb0) * 2 + cbytes : kOob;
#pragma unroll
  for (int u = 0; u < (PAIR ? C::P : C::P - 1); ++u)  // (one by one, unit 3's go out in unit 0)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      load16_lds(rB0, smem_b + u * C::SB + j * 8192, b0_v[j], static_cast<uint32_t>(u * C::ROWB));

  // ---- the adapter phase's list: run by run, unit by unit.  Low word = first
  // column | columns << 9 | unit << 18, high word = segment | rank << 16.
  const uint32_t sched_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(sched));
  const uint32_t count_addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(&n_sched_s));
  if (wave == 0) {
    const uint64_t lt = (1ull << lane) - 1ull;
    uint64_t start[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int prev = __shfl_up(v_seg[q], 1);
      if (q > 0 && lane == 0) prev = __builtin_amdgcn_readlane(v_seg[q > 0 ? q - 1 : 0], 63);
      const int col = lane + 64 * q;
      start[q] = __ballot(K1 > 0 && col < jn && (col == 0 || v_seg[q] != prev));
    }
    uint32_t tot = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool st = (start[q] >> lane) & 1ull;
      const int lo = lane + 64 * q;
      int hi = jn;                                    // the next run's first column
#pragma unroll
      for (int q2 = 3; q2 > q; --q2)
        if (start[q2]) hi = 64 * q2 + __builtin_ctzll(start[q2]);
      const uint64_t above = start[q] & ~(lt | (1ull << lane));
      if (above) hi = 64 * q + __builtin_ctzll(above);
      const int kl = min(max(v_rank[q], 0), K1);
      const int c = st ? (kl + C::BK - 1) / C::BK : 0;
      const uint64_t b0 = __ballot(c & 1), b1 = __ballot(c & 2), b2 = __ballot(c & 4);
      const uint32_t at = tot + __popcll(b0 & lt) + 2 * __popcll(b1 & lt) + 4 * __popcll(b2 & lt);
      tot += __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2);
      const uint32_t ex = static_cast<uint32_t>(lo) | (static_cast<uint32_t>(hi - lo) << 9);
      const uint64_t ey = static_cast<uint64_t>(static_cast<uint32_t>(v_seg[q]) | (static_cast<uint32_t>(kl) << 16)) << 32;
#pragma unroll
      for (int i = 0; i < C::MAXU; ++i)
        if (i < c) lds_write8(sched_addr + 8u * (at + i), ey | (ex | (static_cast<uint32_t>(i) << 18)));
    }
    if (lane == 0) {
      lds_write8(sched_addr + 8u * tot, 0ull);        // rank 0: every load masked
      lds_write4(count_addr, tot);
    }
    wait_lgkmcnt<0>();
  }

  // loads of a whole dense unit: loop-invariant lane offsets, uniform k offset
  auto issue_fast = [&](int u, int slot, int j) __attribute__((always_inline)) {
    const uint32_t k = static_cast<uint32_t>(u * C::ROWB);
    if (j < 2) load16_lds(rA0, smem_a + slot * C::SB + j * 8192, a0_v[j], k);
    else load16_lds(rB0, smem_b + slot * C::SB + (j - 2) * 8192, b0_v[j - 2], k);
  };
  // loads of any unit: the ragged dense tail, an adapter unit, or (past the
  // end) nothing, every load masked
  struct UnitLoad {
    __amdgpu_buffer_rsrc_t rA, rB;
    uint32_t av[2], bv[2];
    uint32_t halves;                                  // the halves of this wave's columns that the unit has
  };
  int n_sched = 0;                                    // read after the first barrier
  auto read_entry = [&](int u, uint64_t& e) __attribute__((always_inline)) {
    lds_read8(e, sched_addr + 8u * static_cast<uint32_t>(min(max(u - nd, 0), n_sched)));
  };
  // entry: the list's entry of unit u (read_entry, waited for)
  auto prep = [&](int u, uint64_t entry) __attribute__((always_inline)) {
    UnitLoad L;
    if (u < nd) {
      L.rA = rA0; L.rB = rB0;
      L.halves = 3u;
      const uint32_t k = static_cast<uint32_t>(u * C::BK);
      const uint32_t mask = k + lchunk * 8 < static_cast<uint32_t>(K0) ? 0u : kOob;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        L.av[j] = (a0_v[j] + 2 * k) | mask;
        L.bv[j] = (b0_v[j] + 2 * k) | mask;
      }
    } else {
      const uint32_t ex = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(entry));
      const uint32_t ey = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(entry >> 32));
      const int lo = static_cast<int>(ex & 511u);
      const uint32_t span = (ex >> 9) & 511u, k = (ex >> 18) * C::BK;
      const int64_t seg = static_cast<int64_t>(ey & 0xffffu);
      const uint32_t mask = k + lchunk * 8 < (ey >> 16) ? 0u : kOob;
      L.rA = make_rsrc(static_cast<const char*>(A1v) + seg * a1_seg_bytes, a1_seg_bytes);
      L.rB = rB1;
      const int c0 = (wave & 1) * C::WTN, hi = lo + static_cast<int>(span);
      L.halves = (lo < c0 + 64 && hi > c0 ? 1u : 0u) | (lo < c0 + 128 && hi > c0 + 64 ? 2u : 0u);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int m = m0 + lrow + 128 * j, jl = lrow + 128 * j;
        L.av[j] = (static_cast<uint32_t>(m) * static_cast<uint32_t>(p.lda1) * 2 + cbytes + 2 * k) | mask |
                  (m < Mv ? 0u : kOob);
        L.bv[j] = (static_cast<uint32_t>(j0 + jl) * static_cast<uint32_t>(p.ldb1) * 2 + cbytes + 2 * k) | mask |
                  (static_cast<uint32_t>(jl - lo) < span ? 0u : kOob);
      }
    }
    return L;
  };
  auto issue = [&](const UnitLoad& L, int slot, int j) __attribute__((always_inline)) {
    if (j < 2) load16_lds(L.rA, smem_a + slot * C::SB + j * 8192, L.av[j]);
    else load16_lds(L.rB, smem_b + slot * C::SB + (j - 2) * 8192, L.bv[j - 2]);
  };

  // ---- fragments ----------------------------------------------------------------
  const int wm = wave >> 1, wn = wave & 1;
  const int fr = lane & 15, fg = lane >> 4;
  const uint32_t smem_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
  const uint32_t sl = static_cast<uint32_t>((fg ^ swz_key<32>(fr)) * 16);
  // slots 0 and 1 lie within an instruction offset of one address, slots 2 and
  // 3 of another
  static_assert(2 * C::SB == 65536, "slots per address");
  uint32_t a_addr[2], b_addr[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    a_addr[h] = smem_base + 2 * h * C::SB + static_cast<uint32_t>((wm * C::WTM + fr) * C::ROWB) + sl;
    b_addr[h] = smem_base + 2 * h * C::SB + static_cast<uint32_t>((C::BM + wn * C::WTN + fr) * C::ROWB) + sl;
  }
  bf16x8 fa[2][4], fb[2][4];
  f32x4 acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // fragment i of the rows, or of half of the columns, of the unit in a slot
  auto rd_a = [&](auto slot_c, int buf, auto i_c) __attribute__((always_inline)) {
    constexpr int S = decltype(slot_c)::value, I = decltype(i_c)::value;
    lds_read16_at<(S & 1) * C::SB + I * 16 * C::ROWB>(fa[buf][I], a_addr[S >> 1]);
  };
  auto rd_b = [&](auto slot_c, auto half_c, auto i_c) __attribute__((always_inline)) {
    constexpr int S = decltype(slot_c)::value, H = decltype(half_c)::value, I = decltype(i_c)::value;
    lds_read16_at<(S & 1) * C::SB + (4 * H + I) * 16 * C::ROWB>(fb[H][I], b_addr[S >> 1]);
  };

  // ---- prologue: units 0 .. 2 and the weights (PAIR: all) of unit 3 in flight,
  // unit 0's first fragments
  wait_vmcnt<PAIR ? 6 : 4>();                         // the token loads of units 1 and 2 (and 3)
  __builtin_amdgcn_s_barrier();
  uint32_t n_sched_v;
  lds_read4(n_sched_v, count_addr);
  unrolled<4>([&](auto i) __attribute__((always_inline)) {
    rd_a(integral_constant<int, 0>{}, 0, i);
    rd_b(integral_constant<int, 0>{}, integral_constant<int, 0>{}, i);
  });
  wait_lgkmcnt<0>();
  pin(n_sched_v);
  n_sched = __builtin_amdgcn_readfirstlane(n_sched_v);
  const int ntot = nd + n_sched;
  UnitLoad L;
  uint32_t ring_halves = 0xffu;                       // two bits for each unit in the ring, the next one lowest

  // unit u in slot S (= u % 4).  Its first half issues the token loads of unit
  // u + 3 (whose weight loads went out in the unit before), its second half
  // the weight loads of unit u + 4 into the slot just freed: the loads are
  // spread over the unit, since eight waves issuing theirs at once fill the
  // load queue and hold up the MFMAs behind it.
  // PAIR: the second half of an odd unit issues every load of units u + 3 and
  // u + 4, into the slots of u - 1 and of u, a row's two pieces one after the
  // other (tokens first: weights first took 1 to 5 us longer).
  auto unit = [&](auto slot_c, auto fast_c, int u) __attribute__((always_inline)) {
    constexpr int S = decltype(slot_c)::value;
    constexpr bool FAST = decltype(fast_c)::value, ODD = S & 1;
    constexpr int SN = (S + 1) & 3, SP = (S + 3) & 3, PA = S & 1;
    uint64_t entry = 0, entry2 = 0;
    UnitLoad L2;                                      // (of unit u + 4; L of u + 3 while they are issued)
    auto load = [&](int uu, int slot, int j) __attribute__((always_inline)) {
      if (FAST) issue_fast(uu, slot, j);
      else issue(L, slot, j);
    };
    auto load_pair = [&](int h, int j) __attribute__((always_inline)) {
      if (FAST) issue_fast(u + C::P - 1 + h, h ? S : SP, j);
      else if (h) issue(L2, S, j);
      else issue(L, SP, j);
    };
    wait_lgkmcnt<0>();
#pragma unroll
    for (int i = 0; i < 4; ++i) { pin(fa[PA][i]); pin(fb[0][i]); }
    unrolled<12>([&](auto m_c) __attribute__((always_inline)) {
      constexpr int m = decltype(m_c)::value;
      acc[m >> 2][m & 3] = MT::mma(fa[PA][m >> 2], fb[0][m & 3], acc[m >> 2][m & 3]);
      if constexpr (m < 4) rd_b(slot_c, integral_constant<int, 1>{}, m_c);
      if (!FAST && m == 4 && (!PAIR || ODD)) read_entry(u + C::P, PAIR ? entry2 : entry);
      if (!FAST && m == 5 && PAIR && ODD) read_entry(u + C::P - 1, entry);
      if (!PAIR && m == 5) load(u + C::P - 1, SP, 2);
      if (!PAIR && m == 9) load(u + C::P - 1, SP, 3);
      __builtin_amdgcn_sched_barrier(0);
    });
    wait_lgkmcnt<0>();
#pragma unroll
    for (int i = 0; i < 4; ++i) pin(fb[1][i]);
    if (!FAST) ring_halves >>= 2;
    if (!FAST && !PAIR) {
      pin(entry);
      L = prep(u + C::P, entry);
      ring_halves |= L.halves << 6;
    }
    if (!FAST && PAIR && ODD) {
      pin(entry);
      pin(entry2);
      L = prep(u + C::P - 1, entry);
      L2 = prep(u + C::P, entry2);
      ring_halves |= (L.halves << 4) | (L2.halves << 6);
    }
    // this wave's loads of unit u + 1; u = 0 and 1 follow the prologue's order:
    // weights, then tokens.  (PAIR: of an even unit all but the last load of its
    // pair's, of an odd one all but the next pair's.)
    if (PAIR && ODD) wait_vmcnt<1>();
    else if (S == 0 && u == 0) wait_vmcnt<4>();
    else if (!PAIR && S == 1 && u == 1) wait_vmcnt<6>();
    else wait_vmcnt<8>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    unrolled<20>([&](auto k_c) __attribute__((always_inline)) {
      constexpr int k = decltype(k_c)::value;
      constexpr int m = k < 4 ? 12 + k : k - 4, h = k < 4 ? 0 : 1;
      acc[m >> 2][4 * h + (m & 3)] = MT::mma(fa[PA][m >> 2], fb[h][m & 3], acc[m >> 2][4 * h + (m & 3)]);
      // (fb[0]'s last use is k = 3)
      if constexpr (k < 4) rd_a(integral_constant<int, SN>{}, PA ^ 1, k_c);
      else if constexpr (k < 8) rd_b(integral_constant<int, SN>{}, integral_constant<int, 0>{}, integral_constant<int, k - 4>{});
      if (!PAIR && k == 10) load(u + C::P, S, 0);
      if (!PAIR && k == 15) load(u + C::P, S, 1);
      if constexpr (PAIR && ODD && k < 8) load_pair(k & 1, (k >> 1) ^ 2);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  typedef std::integral_constant<bool, true> FastT;
  typedef std::integral_constant<bool, false> AnyT;
  int u = 0;
  for (; u + 2 * C::P <= nd_full; u += 4) {           // units u .. u + 3 load whole dense units
    unit(integral_constant<int, 0>{}, FastT{}, u);
    unit(integral_constant<int, 1>{}, FastT{}, u + 1);
    unit(integral_constant<int, 2>{}, FastT{}, u + 2);
    unit(integral_constant<int, 3>{}, FastT{}, u + 3);
  }
  if (!PAIR) L = prep(u + C::P - 1, 0);               // a whole dense unit, as all four in the ring
  // Few adapter units are long runs (a prefill's requests): interleaved like the
  // dense ones.  Many are short runs: the loop below.  Over 21 shapes a line
  // anywhere up to 32 units changes a launch by 1% at most (8192 tokens of 25
  // clusters, 4096 -> 14336: 763 us at 16, 769 at 0); with every unit interleaved
  // tiles of many runs take up to 3% longer (2777 tokens over 500 LoRAs, 3000 ->
  // 5000: 133 and 138).
  // (PAIR: up to a whole pair; a unit past the end is masked)
  const int n_inter = n_sched <= 16 ? ntot : PAIR ? (nd + 1) & ~1 : nd;
  for (;;) {                                          // (four dense units at least are left)
    unit(integral_constant<int, 0>{}, AnyT{}, u);
    if (++u >= n_inter && !PAIR) break;
    unit(integral_constant<int, 1>{}, AnyT{}, u);
    if (++u >= n_inter) break;
    unit(integral_constant<int, 2>{}, AnyT{}, u);
    if (++u >= n_inter && !PAIR) break;
    unit(integral_constant<int, 3>{}, AnyT{}, u);
    if (++u >= n_inter) break;
  }
  // the fragments read ahead for a unit that does not follow: waited for before
  // their registers can be given to anything else
  wait_lgkmcnt<0>();
#pragma unroll
  for (int i = 0; i < 4; ++i) { pin(fa[0][i]); pin(fa[1][i]); pin(fb[0][i]); }
  // Adapter units.  A run has few of the tile's columns, so a wave multiplies
  // only the halves of its columns that the unit's run touches and most waves
  // only load and read: the fragments are read a unit at a time (the first ones
  // again), and nothing is interleaved.
  if (PAIR && u < ntot) {                             // (unit u + 3's tokens go out a second time)
    uint64_t entry = 0;
    read_entry(u + C::P - 1, entry);
    wait_lgkmcnt<0>();
    pin(entry);
    L = prep(u + C::P - 1, entry);
  }
  for (const int first = u; u < ntot; ++u) {
    const uint32_t so = static_cast<uint32_t>((u & 1) * C::SB);
    const uint32_t aa = a_addr[0] + static_cast<uint32_t>((u & 2) * C::SB) + so;
    const uint32_t ba = b_addr[0] + static_cast<uint32_t>((u & 2) * C::SB) + so;
    const int slot = u & 3, prev = (u + 3) & 3;
    uint64_t entry = 0;
    read_entry(u + C::P, entry);
    unrolled<4>([&](auto i_c) __attribute__((always_inline)) {
      constexpr int I = decltype(i_c)::value;
      lds_read16_at<I * 16 * C::ROWB>(fa[0][I], aa);
      lds_read16_at<I * 16 * C::ROWB>(fb[0][I], ba);
      lds_read16_at<(4 + I) * 16 * C::ROWB>(fb[1][I], ba);
    });
    issue(L, prev, 2);
    issue(L, prev, 3);
    wait_lgkmcnt<0>();
    pin(entry);
#pragma unroll
    for (int i = 0; i < 4; ++i) { pin(fa[0][i]); pin(fb[0][i]); pin(fb[1][i]); }
    const uint32_t halves = ring_halves;
    L = prep(u + C::P, entry);
    ring_halves = (ring_halves >> 2) | (L.halves << 6);
    if (PAIR && u == first + 1) wait_vmcnt<7>();      // a unit loaded with its pair: all but that one's last
    else wait_vmcnt<8>();
    __builtin_amdgcn_s_barrier();
    issue(L, slot, 0);
    issue(L, slot, 1);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (halves & (1u << h))
#pragma unroll
        for (int m = 0; m < 16; ++m)
          acc[m >> 2][4 * h + (m & 3)] = MT::mma(fa[0][m >> 2], fb[h][m & 3], acc[m >> 2][4 * h + (m & 3)]);
  }
  wait_vmcnt<0>();
  __syncthreads();

  if (p.out_dtype == 1) {
    // ---- bf16 epilogue: the tile as [token][row] in LDS, then 512 contiguous
    // bytes of a token per half wave
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 v = acc[i][j];
        uint2 w;
        w.x = f32_to_bf16_pair(v[0], v[1]);
        w.y = f32_to_bf16_pair(v[2], v[3]);
        const int col = wn * C::WTN + j * 16 + fr, row = wm * C::WTM + i * 16 + 4 * fg;
        *reinterpret_cast<uint2*>(smem + col * C::ST_ROWB + row * 2) = w;
      }
    __syncthreads();
    const int mc = (tid & 31) * 8;
    if (m0 + mc < Mv)
      for (int jl = tid >> 5; jl < jn; jl += C::NT / 32) {
        const uint4 v = *reinterpret_cast<const uint4*>(smem + jl * C::ST_ROWB + mc * 2);
        const int64_t orow = p.out_perm ? p.perm[j0 + jl] : static_cast<int64_t>(j0 + jl);
        *reinterpret_cast<uint4*>(static_cast<uint16_t*>(outv) + orow * ldov + m0 + mc) = v;
      }
    return;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int jl = wn * C::WTN + j * 16 + fr;
    const int64_t orow = p.out_perm ? p.perm[j0 + min(jl, jn - 1)] : static_cast<int64_t>(j0 + jl);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + wm * C::WTM + i * 16 + 4 * fg;
      if (jl < jn && m < Mv) *reinterpret_cast<f32x4*>(static_cast<float*>(outv) + orow * ldov + m) = acc[i][j];
    }
  }
}

hipError_t launch_prefill(const GemmParams& p, hipStream_t stream) {
  using C = PrefillCfg;
  if (p.tile_start || p.fs_adapter || p.ksplit != 1 || p.part || p.K0 <= 0 || p.b1_gather || p.K1 > C::MAXU * C::BK ||
      p.K0 < C::P * C::BK)
    return hipErrorInvalidValue;
  if (p.seg_rank && !p.sorted_rank) return hipErrorInvalidValue;
  int gm = (p.M + C::BM - 1) / C::BM;
  if (p.n_mod > 0) {
    if (p.n_mod > kMaxGemmModules || p.mod_rt[0] != 0) return hipErrorInvalidValue;
    for (int m = 0; m < p.n_mod; ++m)
      if (p.mod_rt[m + 1] - p.mod_rt[m] != (p.mod_M[m] + C::BM - 1) / C::BM) return hipErrorInvalidValue;
    gm = p.mod_rt[p.n_mod];
  }
  const int gn = (p.N + C::BN - 1) / C::BN;
  GemmParams q = p;
  q.group_m = xcd_group_m(gm, gn, 1);
  // A unit takes 64 bytes of a row.  In rows that do not start at a multiple of
  // 64 bytes these pieces straddle cache lines: 1.4 requests each, which weights
  // read from HBM feel (from the last-level cache they do not).  A pair's two
  // pieces together are two lines, but go out later: 2777 tokens, 3000 -> 5000,
  // cold 121 us a launch one by one and 107 in pairs, 2560 tokens, 4104 -> 5120
  // 153 and 131, 4096 tokens, 3000 -> 8192 211 and 191 (the two-stage 64-deep ring
  // before this one: 108, 128 and 202); aligned rows one by one, since 700
  // tokens, 4096 -> 14336 take 96 us from the last-level cache and 105 in pairs.
  if (p.K0 % 32) hipLaunchKernelGGL(prefill_gemm_kernel<true>, dim3(gm * gn), dim3(C::NT), 0, stream, q);
  else hipLaunchKernelGGL(prefill_gemm_kernel<false>, dim3(gm * gn), dim3(C::NT), 0, stream, q);
  return hipGetLastError();
}

template <typename TI, int BM, int BN, int BK, int WM, int WN, int MB, int P, int FSORT = 0, int MODS = 0,
          int DENSE = 0>
hipError_t launch_dma1(const GemmParams& p, hipStream_t stream) {
  const int gn = (p.tile_start || FSORT) ? p.max_tiles : (p.N + BN - 1) / BN;
  // row tiles: the modules' together when the launch holds several
  const bool mods = MODS && !(p.tile_start || FSORT) && p.n_mod > 0;
  if (!MODS && !DENSE && p.n_mod > 0) return hipErrorInvalidValue;
  if (!DENSE != !(p.d_blocks > 0)) return hipErrorInvalidValue;
  // every workgroup has a dense reduction (a token tile's is its segment's)
  if ((p.tile_start || FSORT ? p.K1 : p.K0) <= 0 || (p.tile_start && !p.tile_seg)) return hipErrorInvalidValue;
  if (mods) {
    if (p.n_mod > kMaxGemmModules || p.mod_rt[0] != 0) return hipErrorInvalidValue;
    for (int m = 0; m < p.n_mod; ++m)
      if (p.mod_rt[m + 1] - p.mod_rt[m] != (p.mod_M[m] + BM - 1) / BM) return hipErrorInvalidValue;
  }
  const int gm = mods ? p.mod_rt[p.n_mod] : (p.M + BM - 1) / BM;
  dim3 grid(gm * gn * p.ksplit);
  if ((p.tile_start || FSORT) && p.split_target > 0) {
    if (!(BM == 64 && BN == 64 && BK * sizeof(TI) == 128)) return hipErrorInvalidValue;   // no adaptive split here
    // gm n S workgroups are used: fewer than gm max_tiles + split_target, and
    // at most gm max_tiles ksplit
    const int64_t gmt = (p.M + BM - 1) / BM;
    grid = dim3(static_cast<unsigned>(std::min<int64_t>(gmt * gn + p.split_target, gmt * gn * p.ksplit)));
  }
  GemmParams q = p;
  q.group_m = (p.tile_start || FSORT) ? 0 : xcd_group_m(gm, (p.N + BN - 1) / BN, p.ksplit);
  if (DENSE) {
    if (!p.d_part || p.d_split < 1 || p.n_mod > kMaxGemmModules) return hipErrorInvalidValue;
    int dgm = (p.d_M + BM - 1) / BM;
    if (p.n_mod > 0) {
      if (p.mod_rt[0] != 0) return hipErrorInvalidValue;
      for (int m = 0; m < p.n_mod; ++m)
        if (p.mod_rt[m + 1] - p.mod_rt[m] != (p.mod_M[m] + BM - 1) / BM) return hipErrorInvalidValue;
      dgm = p.mod_rt[p.n_mod];
    }
    const int dgn = (p.N + BN - 1) / BN;
    q.d_blocks = dgm * dgn * p.d_split;
    q.group_m = xcd_group_m(dgm, dgn, p.d_split);
    grid.x += q.d_blocks;
  }
  hipLaunchKernelGGL((seg_gemm_dma_kernel<TI, BM, BN, BK, WM, WN, MB, P, FSORT, MODS, DENSE>),
                     grid, dim3(WM * WN * 64), 0, stream, q);
  return hipGetLastError();
}

template <typename TI, int BM, int BN, int BK, int WM, int WN, int MB, int P, int FSORT = 0>
hipError_t launch_dma(const GemmParams& p, hipStream_t stream) {
  // the list of adapter k-tiles has room for ranks of at most 128
  if (!(p.tile_start || FSORT) && p.K1 > 128) return hipErrorInvalidValue;
  // (token tiles keep no output row numbers: they write partials only)
  if ((p.tile_start || FSORT) && !p.part) return hipErrorInvalidValue;
  if (p.seg_rank && !p.sorted_rank && !(p.tile_start || FSORT)) return hipErrorInvalidValue;
  if (p.n_mod > 0) {
    if (p.seg_rank || p.tile_start || FSORT) return hipErrorInvalidValue;
    if constexpr (FSORT == 0 && sizeof(TI) == 2)
      return launch_dma1<TI, BM, BN, BK, WM, WN, MB, P, 0, 1>(p, stream);
    return hipErrorInvalidValue;
  }
  return launch_dma1<TI, BM, BN, BK, WM, WN, MB, P, FSORT>(p, stream);
}

}  // namespace

// Tile shapes (BM x BN x BK: d_out rows x tokens x k).  The bf16 tiles use
// 16x16x32 MFMA; for T > 64 the plan takes the one whose rounds over the
// compute units it estimates shortest:
//   Large   256 x 256 x  32, 8 waves, 4-unit ring (prefill kernel)
//   Wide    256 x 128 x  64, 8 waves, 3 stages
//   Mid     128 x 128 x  64, 8 waves, 4 stages
//   Narrow  128 x  64 x 128, 4 waves, 3 stages
//   Decode   64 x  64 x 128, 4 waves, 4 stages     T <= 64
//   Shrink   64 x  64 x  64, 4 waves, 3 stages     the V_k^T X products
//   F32      64 x  64 x  32, 4 waves, 3 stages     fp32 inputs: every product
void tile_dims(Tile tile, int* BM, int* BN, int* BK) {
  switch (tile) {
    case Tile::Large: *BM = 256; *BN = 256; *BK = 32; return;
    case Tile::Wide: *BM = 256; *BN = 128; *BK = 64; return;
    case Tile::Narrow: *BM = 128; *BN = 64; *BK = 128; return;
    case Tile::Decode: *BM = 64; *BN = 64; *BK = 128; return;
    case Tile::Shrink: *BM = 64; *BN = 64; *BK = 64; return;
    case Tile::Mid: *BM = 128; *BN = 128; *BK = 64; return;
    case Tile::F32: *BM = 64; *BN = 64; *BK = 32; return;
  }
}

hipError_t launch_seg_gemm(const GemmParams& p, int in_dtype, Tile tile, hipStream_t stream) {
  // several modules in one launch: the LDS-ring tiles only, without token
  // tiles (but those of a shrink that holds the modules' dense product)
  if (p.n_mod > 0 && (in_dtype == 0 || ((p.tile_start || p.fs_adapter) && !p.d_blocks)))
    return hipErrorInvalidValue;
  // the dense product rides with the bf16 shrink's token tiles only
  if (p.d_blocks > 0 && (in_dtype == 0 || tile != Tile::Shrink || !(p.tile_start || p.fs_adapter) || !p.part))
    return hipErrorInvalidValue;
  // explicit token tiles (at most kSegTile columns) only with the 64-wide tiles
  if (p.tile_start &&
      !(tile == Tile::Decode || tile == Tile::Shrink || tile == Tile::F32))
    return hipErrorInvalidValue;
  // the split chosen on the device exists in the shrinks' tiles only
  if (p.split_target > 0 && tile != Tile::Shrink && tile != Tile::F32) return hipErrorInvalidValue;
  // in-kernel bucketing exists in the bf16 shrink tile only
  if (p.fs_adapter && (in_dtype == 0 || tile != Tile::Shrink || p.N > kFuseSortMaxT || p.tile_start))
    return hipErrorInvalidValue;
  if ((in_dtype == 0) != (tile == Tile::F32)) return hipErrorInvalidValue;
  switch (tile) {
    case Tile::Large: return launch_prefill(p, stream);
    case Tile::Wide: return launch_dma<bf16_t, 256, 128, 64, 4, 2, 16, 3>(p, stream);
    case Tile::Narrow: return launch_dma<bf16_t, 128, 64, 128, 4, 1, 16, 3>(p, stream);
    case Tile::Decode: return launch_dma<bf16_t, 64, 64, 128, 2, 2, 16, 4>(p, stream);
    case Tile::Shrink:
      if (p.d_blocks > 0)
        return p.fs_adapter ? launch_dma1<bf16_t, 64, 64, 64, 2, 2, 16, 4, 1, 0, 1>(p, stream)
                            : launch_dma1<bf16_t, 64, 64, 64, 2, 2, 16, 4, 0, 0, 1>(p, stream);
      if (p.fs_adapter) return launch_dma<bf16_t, 64, 64, 64, 2, 2, 16, 3, 1>(p, stream);
      return launch_dma<bf16_t, 64, 64, 64, 2, 2, 16, 3>(p, stream);
    case Tile::Mid: return launch_dma<bf16_t, 128, 128, 64, 4, 2, 16, 4>(p, stream);
    case Tile::F32: return launch_dma<float, 64, 64, 32, 2, 2, 16, 3>(p, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace cts
