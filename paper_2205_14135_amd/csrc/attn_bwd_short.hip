// Backward pass of short sequences at d <= 64 (dense, N <= 512): one workgroup takes a whole head, and one launch
// does all five tile products.
//
// Arithmetic: Algorithm 4 of the paper; up to 256 tokens (bwd_short_kernel) with a single key block,
//     S = Q K^T, P = exp(S - L), dV = (P o Z)^T dO, dP = (dO V^T) o Z, dS = P o (dP - D), dK = tau dS^T Q, dQ = tau dS K,
// D = rowsum(dO o O).  The longer sequences take two launches (attn_bwd.hip), because a key block's share of dQ
// would have to be added up in memory; here the only key block is the whole sequence, so dQ needs no other workgroup's share.  S, P,
// dP and the dropout draw are done once instead of twice, Q, K, V and dO are read once, and nothing goes
// through the scratch vectors.  (Two key blocks: bwd_blocks_kernel below.)
// A wavefront owns 32 keys (layout "lane = key", as in attn_bwd_dkv_fr.hip) for dK and dV, and then 32 queries for dQ: dS
// changes owner through LDS, [key][query] rows written four queries at a time and read with the transposing read, so
// that dQ^T = K^T dS^T takes both operands from LDS in the layout the other kernels read V^T and K^T in.
// What bounds it: at N = 128 memory (2048 heads, d = 64: 268 MB in 67 to 72 us, 3.7 to 4.0 TB/s; the two launches move 403 MB in 83);
// with few heads the latency of one head (96 heads of 128: 13.2 -> 8.6 us); at N > 128 a compute unit holds one workgroup, and
// nothing covers its loads and stores from the second head on (256 heads of 197 27.0 -> 22.3 us, 1024 of 256 102 -> 107, not taken).
// Vector registers spilled: 5 with dropout at d = 64 and N > 128, none elsewhere.
#include "attn_common.h"
#include "attn_tiles.h"

namespace attn {
namespace {

constexpr int TILE = 64;

// KW wavefronts: heads of up to 32 KW tokens (KW = 4 or 8)
template <typename T, int D, bool CAUSAL, bool DROPOUT, int KW>
__global__ __launch_bounds__(64 * KW, 2) void bwd_short_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  typedef typename Vec<T>::x4 T4;
  constexpr int KK = D / 16, DB = D / 32;
  // One LDS block.  Two Q tiles and two dO tiles of 64 queries (Q, dO, Q, dO; KW = 4: all there are, KW = 8: a double buffer), the
  // K rows, dS of two tiles ([32 KW keys][64 queries], swizzled like a tile; KW = 8: one is read while the next is written), the
  // row vectors, and (KW = 8) room for dQ rows on their way out.  KW = 4 at d = 64: dS of the second tile takes the place
  // of the first tile's Q and dO, so that two workgroups fit on a compute unit.
  constexpr int kQ = TILE * D, kS = 32 * KW * 64;   // elements
  constexpr bool OVERLAY = KW == 4 && 2 * kQ >= kS;
  constexpr int kElems = 4 * kQ + 32 * KW * D + (OVERLAY ? kS : 2 * kS) + (KW == 8 ? KW * 32 * 32 : 0);
  __shared__ __attribute__((aligned(16))) unsigned char smem[kElems * sizeof(T) + 2 * 32 * KW * sizeof(float)];
  T* const Q0 = (T*)smem;
  T* const Kl = Q0 + 4 * kQ;
  T* const S0 = Kl + 32 * KW * D;
  T* const S1 = OVERLAY ? Q0 : S0 + kS;
  float* const Lv = (float*)(smem + kElems * sizeof(T));   // base-2 row statistic
  float* const Dv = Lv + 32 * KW;                          // -D_i
  // dropout flags in this layout: see KeepLK in attn_common.h
  __shared__ __attribute__((aligned(16))) uint32_t keep_table[DROPOUT ? KeepLK::kTable : 4];
  KeepLK keep;
  if constexpr (DROPOUT) keep.init(keep_table, a.drop_thr);

  const int item = xcd_item(a.n_items, a.chunk);
  if (item < 0) return;
  const int bh = dealt_head(a, item);
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  const int w0 = wave * 32;            // the wavefront's first key, and its first query
  const int row = w0 + r;
  const bool row_ok = row < a.N;
  const int64_t row_off = head_off + (int64_t)min(row, a.N - 1) * a.sn;
  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  const int n_tiles = (len + TILE - 1) / TILE;   // query tiles with a row that sees anything
  const int dvalid = D == 32 ? a.dvalid : D;

  TileAsync<T, D, 4> dma;   // four wavefronts copy a tile; of eight, the second four copy another one
  const int half = KW == 8 ? wave >> 2 : 0;
  dma.init(a.sn, wave & 3, dvalid);
  if (D == 32 && a.dvalid < D) {   // the copies leave columns >= 16 of the tiles untouched
    zero_tiles(Q0, 4 * kQ + 32 * KW * D);
    __syncthreads();
  }
  const T* const Qg = (const T*)a.Q + head_off;
  const T* const Gg = (const T*)a.dO + head_off;
  const T* const Kg = (const T*)a.K + head_off;
  auto fetch_tile = [&](int t, T* Qt) __attribute__((always_inline)) {
    if (KW == 4 || half == 0) dma.copy_rows(Qg, a.sn, t * TILE, a.N, Qt);
    if (KW == 4 || half == 1) dma.copy_rows(Gg, a.sn, t * TILE, a.N, Qt + kQ);
  };
  if (len > 0) fetch_tile(0, Q0);
  if (KW == 4 && len > TILE) fetch_tile(1, Q0 + 2 * kQ);
#pragma unroll
  for (int t = 0; t < KW / 2; ++t)
    if (t * TILE < len && (KW == 4 || half == (t & 1))) dma.copy_rows(Kg, a.sn, t * TILE, a.N, Kl + t * kQ);
  // this lane's key (K and V fragments, B operands) and this lane's query (row statistic, -D from half of the row)
  T8 kf[KK], vf[KK];
  float d_part = 0.f;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int64_t off = row_off + 16 * kk + 8 * g;
    if (D == 32 && 16 * kk + 8 * g >= a.dvalid) {   // head dimension 16: the upper columns are zeros
#pragma unroll
      for (int e = 0; e < 8; ++e) { kf[kk][e] = (T)0.f; vf[kk][e] = (T)0.f; }
      continue;
    }
    kf[kk] = *(const T8*)((const T*)a.K + off);
    vf[kk] = *(const T8*)((const T*)a.V + off);
    const T8 go = *(const T8*)((const T*)a.dO + off);
    if (a.o_fp32) {
      const f32x4 o0 = *(const f32x4*)((const float*)a.O + off);
      const f32x4 o1 = *(const f32x4*)((const float*)a.O + off + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) d_part += (float)go[e] * o0[e] + (float)go[4 + e] * o1[e];
    } else {
      const T8 o = *(const T8*)((const T*)a.O + off);
#pragma unroll
      for (int e = 0; e < 8; ++e) d_part += (float)go[e] * (float)o[e];
    }
  }
  const float lse = a.LSE[(int64_t)bh * a.N + min(row, a.N - 1)];
  // a row that saw no key (or lies beyond a ragged end) has P = 0 everywhere
  const float l2 = (lse == -INFINITY || !row_ok) ? INFINITY : lse * 1.4426950408889634f;
  const float neg_d = row_ok ? -(d_part + xchg32(d_part)) : 0.f;
  if (g == 0) {
    Lv[row] = l2;
    Dv[row] = neg_d;
  }

  f32x16 dv[DB], dk[DB];   // dV^T, dK^T (rows d, column = this lane's key)
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dv[db][i] = 0.f; dk[db][i] = 0.f; }
  TrOffsets<D> tro;
  tro.init();
  const float c = a.scale_log2;
  wait_async_copies();
  __syncthreads();

  // LDS operand reads run PF fragments ahead of the MFMA that consumes them
  constexpr int PF = 4;
  // out[qb] = Tile[32 qb .. +31][:] . frags, starting from out
  auto row_product = [&](const T* tile, const T8 (&bfrag)[KK], f32x16 (&out)[2]) {
    auto frag = [&](int f) { return *(const T8*)(tile + lds_off<D>(32 * (f & 1) + r, 2 * (f >> 1) + g)); };  // f = 2 kk + qb
    T8 ring[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) ring[f] = frag(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < 2 * KK; ++f) {
      const T8 cur = ring[f % PF];
      out[f & 1] = mfma32(cur, bfrag[f >> 1], out[f & 1]);
      if (f + PF < 2 * KK) ring[f % PF] = frag(f + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // acc^T += Tile^T . frag   (contraction over the 64 queries of the tile)
  auto col_product = [&](const T* tile, const T8 (&bfrag)[4], f32x16 (&acc)[DB]) {
    auto frag = [&](int f) {   // f = DB cc + db: consecutive MFMAs hit different accumulators
      const T* base = tile + 16 * (f / DB) * D;
      return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
    };
    T8 ring[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) ring[f] = frag(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < 4 * DB; ++f) {
      const T8 cur = ring[f % PF];
      acc[f % DB] = mfma32(cur, bfrag[f / DB], acc[f % DB]);
      if (f + PF < 4 * DB) ring[f % PF] = frag(f + PF);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto tile_step = [&](const int i0, const T* const Qt, T* const St) __attribute__((always_inline)) {
    const T* const Gt = Qt + kQ;
    // hidden from the whole tile: keys beyond the length, or beyond the tile's last query
    if (w0 >= len || (CAUSAL && i0 + TILE - 1 < w0)) return;
    f32x16 s[2], dp[2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[qb][i] = 0.f;
    row_product(Qt, kf, s);                // S = Q K^T
    uint32_t kept = 0;   // the keep flags of this lane's key for the tile's 64 queries it holds
    if constexpr (DROPOUT) kept = keep.draw<2>(i0, w0, bh, a.offset_lo, a.seed_lo, a.seed_hi);
    // hidden entries get the logit -inf, hence P = 0: above the causal diagonal, or padded keys
    if ((CAUSAL && i0 < w0 + 31) || w0 + 32 > len) {
      const int first_query = row < len ? (CAUSAL ? row : 0) : 0x7fffffff;   // that sees this lane's key
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (i0 + 32 * qb + 8 * (i >> 2) + 4 * g + (i & 3) < first_query) s[qb][i] = -INFINITY;
    }
    T8 pf[4];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        const f32x4 l4 = *(const f32x4*)(Lv + i0 + 32 * qb + 8 * i4 + 4 * g);
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};   // without dropout dP starts from -D
        if constexpr (!DROPOUT) d4 = *(const f32x4*)(Dv + i0 + 32 * qb + 8 * i4 + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qb][i], c, -l4[e]));
          s[qb][i] = p;
          dp[qb][i] = d4[e];
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          pf[cc][tt] = DROPOUT ? (T)keep_or_zero(p, KeepLK::mask(kept, qb, i4, e)) : (T)p;
        }
      }
    col_product(Gt, pf, dv);               // dV^T += dO^T P_dropped
    row_product(Gt, vf, dp);               // dP = dO V^T
    T8 dsf[4];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DROPOUT) d4 = *(const f32x4*)(Dv + i0 + 32 * qb + 8 * i4 + 4 * g);   // -D_i
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          float dpv = dp[qb][i];
          if constexpr (DROPOUT) dpv = dropped_dp_minus_d(dpv, a.keep_scale, KeepLK::mask(kept, qb, i4, e), d4[e]);
          dsf[cc][tt] = (T)(s[qb][i] * dpv);
        }
      }
    // dS for the wavefronts that own the queries: four queries 8 i4 + 4 g .. of this lane's key at a time
#pragma unroll
    for (int cc = 0; cc < 4; ++cc)
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        T4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = dsf[cc][4 * hb + e];
        *(T4*)(St + lds_off<64>(row, 2 * cc + hb) + 4 * g) = v;
      }
    col_product(Qt, dsf, dk);              // dK^T += Q^T dS
  };
  TrOffsets<64> trs;
  trs.init();
  // dq[db] = (K^T dS^T)[d block DB0 + db] of the 32 queries from q0 on, block qb of the tile whose dS is St, over the
  // 16-key chunks that any of them sees
  auto dq_product = [&](const int q0, const int qb, const T* const St, const int db0, auto& dq) __attribute__((always_inline)) {
    constexpr int NB = sizeof(dq) / sizeof(f32x16);
#pragma unroll
    for (int db = 0; db < NB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;
    const int n_keys = q0 < n_tiles * TILE ? (CAUSAL ? min(len, q0 + 32) : len) : 0;
    const int s_lo = qb ? trs.off[1][0] : trs.off[0][0], s_hi = qb ? trs.off[1][1] : trs.off[0][1];
#pragma unroll
    for (int cc = 0; cc < 2 * KW; ++cc) {
      if (16 * cc >= n_keys) break;
      const T8 ds = tr_frag<T8>(St + 16 * cc * 64 + s_lo, St + 16 * cc * 64 + s_hi);
      const T* const base = Kl + 16 * cc * D;
#pragma unroll
      for (int db = 0; db < NB; ++db) {
        const int k_lo = NB == DB || db0 == 0 ? tro.off[db][0] : tro.off[DB - 1][0], k_hi = NB == DB || db0 == 0 ? tro.off[db][1] : tro.off[DB - 1][1];
        dq[db] = mfma32(tr_frag<T8>(base + k_lo, base + k_hi), ds, dq[db]);
      }
    }
  };
  const int64_t out_row0 = head_off + (int64_t)w0 * a.sn;
  if constexpr (KW == 4) {
    if (n_tiles > 0) tile_step(0, Q0, S0);
    __syncthreads();   // everyone is done with the first Q and dO
    if (n_tiles > 1) tile_step(TILE, Q0 + 2 * kQ, S1);
    __syncthreads();   // dS is complete, the second Q and dO are free: they stage the output rows
  } else {
    // dQ of tile j - 1 beside tile j: a tile's 2 DB blocks of 32 x 32 are the work of as many wavefronts, which take turns
    constexpr int TURNS = KW / (2 * DB);
    const int turn = wave / (2 * DB), qb = wave & 1, db = DB == 2 ? (wave >> 1) & 1 : 0;
    T* const stage = S1 + kS + wave * 32 * 32;
    for (int j = 0; j <= n_tiles; ++j) {
      if (j + 1 < n_tiles) fetch_tile(j + 1, Q0 + 2 * ((j + 1) & 1) * kQ);
      if (j < n_tiles) tile_step(j * TILE, Q0 + 2 * (j & 1) * kQ, j & 1 ? S1 : S0);
      if (j > 0 && turn == (j - 1) % TURNS) {
        const int q0 = (j - 1) * TILE + 32 * qb;
        f32x16 dq[1];
        dq_product(q0, qb, j & 1 ? S0 : S1, db, dq);
        store_rows_coalesced<T, 32>(stage, (T*)a.dQ + head_off + (int64_t)q0 * a.sn + 32 * db, a.sn, dq, a.tau, a.N - q0, dvalid);
      }
      wait_async_copies();
      __syncthreads();
    }
  }
  T* const stage = KW == 4 ? Q0 + 2 * kQ + wave * 32 * D : Q0 + wave * 32 * D;
  store_rows_coalesced<T, D>(stage, (T*)a.dV + out_row0, a.sn, dv, DROPOUT ? a.keep_scale : 1.f, a.N - w0, dvalid);
  __builtin_amdgcn_wave_barrier();
  store_rows_coalesced<T, D>(stage, (T*)a.dK + out_row0, a.sn, dk, a.tau, a.N - w0, dvalid);
  __builtin_amdgcn_wave_barrier();
  if (KW == 4 || w0 >= n_tiles * TILE) {   // KW = 8: rows of tiles that see nothing
    f32x16 dq[DB];
    dq_product(w0, wave & 1, wave < 2 ? S0 : S1, 0, dq);
    store_rows_coalesced<T, D>(stage, (T*)a.dQ + out_row0, a.sn, dq, a.tau, a.N - w0, dvalid);
  }
}

// Heads of 257 to 512 tokens: a workgroup of eight wavefronts takes two blocks of 256 keys in turn, each against all query tiles.
// dQ of a tile is added up one tile later, beside the next tile's products, by all eight wavefronts (16 x 16 pieces, each over the block's 256 keys).  Between
// the blocks it rests in float32 in the workspace, written and read back by the same lanes (64 KB to 128 KB a head, which the L2 holds).
// What bounds it (256 heads of 512, d = 64, no dropout: 66 us on a card where the two launches take 74; clocks of a wavefront, of 145 k): everything that a
// workgroup reads before its first tile, 27 k, since all compute units ask at once and each has one workgroup; then LDS, which 12 products of
// 64 x 256 keep busy for three quarters of a tile (dQ 2.0 k a tile, dV, dP and the vector work between their MFMAs 2.1 k, S and dK 0.9 k, barrier
// 0.75 k); with dropout the vector ALU (93 | 85 us).  D of a tile when the tile comes instead of all rows first: 79 -> 81 us (18 registers spilled, and a
// wait for O waits for the copies in flight); the row vectors spread over the accumulators by a product with ones, instead of 16 LDS reads: no gain.
// Vector registers spilled at d = 64: 10, causal 9, with dropout 7 and 6.
template <typename T, int D, bool CAUSAL, bool DROPOUT>
__global__ __launch_bounds__(512, 2) void bwd_blocks_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  typedef typename Vec<T>::x4 T4;
  constexpr int KK = D / 16, DB = D / 32;
  constexpr int KEYS = 256, MAX_ROWS = 512;
  constexpr int kQ = TILE * D, kS = KEYS * TILE;   // elements
  // One LDS block: two buffers of a Q and a dO tile, the K rows, two buffers of dS ([256 keys][64 queries], swizzled like a tile), the row vectors
  constexpr int kElems = 4 * kQ + KEYS * D + 2 * kS;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kElems * sizeof(T) + 2 * MAX_ROWS * sizeof(float)];
  T* const Q0 = (T*)smem;
  T* const Kl = Q0 + 4 * kQ;
  T* const S0 = Kl + KEYS * D;
  float* const Lv = (float*)(smem + kElems * sizeof(T));   // base-2 row statistic
  float* const Dv = Lv + MAX_ROWS;                         // -D_i
  // dropout flags in this layout: see KeepLK in attn_common.h
  __shared__ __attribute__((aligned(16))) uint32_t keep_table[DROPOUT ? KeepLK::kTable : 4];
  KeepLK keep;
  if constexpr (DROPOUT) keep.init(keep_table, a.drop_thr);

  const int item = xcd_item(a.n_items, a.chunk);
  if (item < 0) return;
  const int bh = dealt_head(a, item);
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, g = lane >> 5;
  const int w0 = wave * 32;            // the wavefront's first key of a block
  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  const int n_tiles = (len + TILE - 1) / TILE;   // query tiles with a row that sees anything
  const int dvalid = D == 32 ? a.dvalid : D;
  const T* const Qg = (const T*)a.Q + head_off;
  const T* const Gg = (const T*)a.dO + head_off;
  const T* const Kg = (const T*)a.K + head_off;

  TileAsync<T, D, 4> dma;   // four wavefronts copy a tile, the other four another one
  const int half = wave >> 2;
  dma.init(a.sn, wave & 3, dvalid);
  if (D == 32 && a.dvalid < D) {   // the copies leave columns >= 16 of the tiles untouched
    zero_tiles(Q0, 4 * kQ + KEYS * D);
    __syncthreads();
  }
  auto fetch_tile = [&](int t, T* Qt) __attribute__((always_inline)) {
    dma.copy_rows(half == 0 ? Qg : Gg, a.sn, t * TILE, a.N, half == 0 ? Qt : Qt + kQ);
  };
  T8 kf[KK], vf[KK];   // K and V fragments (B operands) of this lane's key
  auto fetch_keys = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < KEYS / TILE; ++t)
      if (k0 + t * TILE < len && half == (t & 1)) dma.copy_rows(Kg, a.sn, k0 + t * TILE, a.N, Kl + t * kQ);
    const int64_t row_off = head_off + (int64_t)min(k0 + w0 + r, a.N - 1) * a.sn;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (D == 32 && 16 * kk + 8 * g >= a.dvalid) {   // head dimension 16: the upper columns are zeros
#pragma unroll
        for (int e = 0; e < 8; ++e) { kf[kk][e] = (T)0.f; vf[kk][e] = (T)0.f; }
        continue;
      }
      kf[kk] = *(const T8*)((const T*)a.K + row_off + 16 * kk + 8 * g);
      vf[kk] = *(const T8*)((const T*)a.V + row_off + 16 * kk + 8 * g);
    }
  };
  if (len > 0) fetch_tile(0, Q0);
  fetch_keys(0);
  // row statistic and -D of all rows, half a row per lane
  for (int row0 = 0; row0 < a.N; row0 += KEYS) {
    const int row = row0 + w0 + r, qi = min(row, a.N - 1);
    float d_part = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (D == 32 && 16 * kk + 8 * g >= a.dvalid) continue;
      const int64_t off = head_off + (int64_t)qi * a.sn + 16 * kk + 8 * g;
      const T8 go = *(const T8*)((const T*)a.dO + off);
      if (a.o_fp32) {
        const f32x4 o0 = *(const f32x4*)((const float*)a.O + off);
        const f32x4 o1 = *(const f32x4*)((const float*)a.O + off + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) d_part += (float)go[e] * o0[e] + (float)go[4 + e] * o1[e];
      } else {
        const T8 o = *(const T8*)((const T*)a.O + off);
#pragma unroll
        for (int e = 0; e < 8; ++e) d_part += (float)go[e] * (float)o[e];
      }
    }
    const float lse = a.LSE[(int64_t)bh * a.N + qi];
    const float neg_d = -(d_part + xchg32(d_part));
    if (g == 0) {
      // a row that saw no key (or lies beyond a ragged end) has P = 0 everywhere
      Lv[row] = (lse == -INFINITY || row >= a.N) ? INFINITY : lse * 1.4426950408889634f;
      Dv[row] = row < a.N ? neg_d : 0.f;
    }
  }
  TrOffsets<D> tro;
  tro.init();
  const float c = a.scale_log2;

  // LDS operand reads run PF fragments ahead of the MFMA that consumes them; between(f) comes after MFMA f
  constexpr int PF = 4;
  auto row_product = [&](const T* tile, const T8 (&bfrag)[KK], f32x16 (&out)[2], auto between) __attribute__((always_inline)) {
    auto frag = [&](int f) { return *(const T8*)(tile + lds_off<D>(32 * (f & 1) + r, 2 * (f >> 1) + g)); };  // f = 2 kk + qb
    T8 ring[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) ring[f] = frag(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < 2 * KK; ++f) {
      const T8 cur = ring[f % PF];
      out[f & 1] = mfma32(cur, bfrag[f >> 1], out[f & 1]);
      if (f + PF < 2 * KK) ring[f % PF] = frag(f + PF);
      between(f);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto col_product = [&](const T* tile, const T8 (&bfrag)[4], f32x16 (&acc)[DB], auto between) __attribute__((always_inline)) {
    auto frag = [&](int f) {   // f = DB cc + db: consecutive MFMAs hit different accumulators
      const T* base = tile + 16 * (f / DB) * D;
      return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
    };
    T8 ring[PF];
#pragma unroll
    for (int f = 0; f < PF; ++f) ring[f] = frag(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < 4 * DB; ++f) {
      const T8 cur = ring[f % PF];
      acc[f % DB] = mfma32(cur, bfrag[f / DB], acc[f % DB]);
      if (f + PF < 4 * DB) ring[f % PF] = frag(f + PF);
      between(f);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto nothing = [](int) {};

  // dQ of a tile: this wavefront's piece is 16 columns (d16) of 16 QH queries (from qp on).  16x16x32 products over 32 keys; lane group lane / 16 has keys
  // {0, 8, 4, 12}[lane / 16] + 0..3 and 16 more (rows that the transposing reads find in different banks).
  constexpr int QH = D == 64 ? 2 : 1;
  const int qp = D == 64 ? 32 * (wave & 1) : 16 * (wave & 3), d16 = D == 64 ? wave >> 1 : wave >> 2;
  const int i16 = lane & 15, q16 = lane >> 4;
  const int tr_row = 8 * (q16 & 1) + 4 * (q16 >> 1) + (i16 >> 2);
  const int k_off = lds_off<D>(tr_row, 2 * d16 + ((i16 & 3) >> 1)) + 4 * (i16 & 1);   // (16 rows further the swizzle is the same)
  int s_off[QH];
#pragma unroll
  for (int x = 0; x < QH; ++x) s_off[x] = lds_off<TILE>(tr_row, (qp >> 3) + 2 * x + ((i16 & 3) >> 1)) + 4 * (i16 & 1);
  float* const part = a.dQpart + ((int64_t)bh * ((a.N + TILE - 1) / TILE) * 8 + wave) * (QH * 256) + 4 * lane;

  for (int k0 = 0; k0 < a.N; k0 += KEYS) {
    const bool last_block = k0 + KEYS >= a.N;
    const int kw0 = k0 + w0, key = kw0 + r;
    const int first = CAUSAL ? k0 / TILE : 0;
    f32x16 dv[DB], dk[DB];   // dV^T, dK^T (rows d, column = this lane's key)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) { dv[db][i] = 0.f; dk[db][i] = 0.f; }
    wait_async_copies();
    __syncthreads();   // K rows, the first tile, the row vectors
    auto tile_step = [&](const int i0, const T* const Qt, T* const St) __attribute__((always_inline)) {
      const T* const Gt = Qt + kQ;
      // hidden from the whole tile: keys beyond the length, or beyond the tile's last query
      if (kw0 >= len || (CAUSAL && i0 + TILE - 1 < kw0)) return;
      f32x16 s[2], dp[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[qb][i] = 0.f;
      row_product(Qt, kf, s, nothing);       // S = Q K^T
      uint32_t kept = 0;   // the keep flags of this lane's key for the tile's 64 queries it holds
      if constexpr (DROPOUT) kept = keep.draw<2>(i0, kw0, bh, a.offset_lo, a.seed_lo, a.seed_hi);
      // hidden entries get the logit -inf, hence P = 0: above the causal diagonal, or padded keys
      if ((CAUSAL && i0 < kw0 + 31) || kw0 + 32 > len) {
        const int first_query = key < len ? (CAUSAL ? key : 0) : 0x7fffffff;   // that sees this lane's key
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (i0 + 32 * qb + 8 * (i >> 2) + 4 * g + (i & 3) < first_query) s[qb][i] = -INFINITY;
      }
      T8 pf[4], dsf[4];
      auto p_group = [&](int j) __attribute__((always_inline)) {   // four elements: j = 2 i4 + qb
        const int i4 = j >> 1, qb = j & 1;
        if constexpr (DROPOUT)   // (keeps the bit extracts where they are used)
          if (qb == 0) asm volatile("" : "+v"(kept));
        const f32x4 l4 = *(const f32x4*)(Lv + i0 + 32 * qb + 8 * i4 + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qb][i], c, -l4[e]));
          s[qb][i] = p;
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          pf[cc][tt] = DROPOUT ? (T)keep_or_zero(p, KeepLK::mask(kept, qb, i4, e)) : (T)p;
        }
      };
      auto start_dp = [&]() __attribute__((always_inline)) {   // without dropout dP starts from -D
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
            if constexpr (!DROPOUT) d4 = *(const f32x4*)(Dv + i0 + 32 * qb + 8 * i4 + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) dp[qb][4 * i4 + e] = d4[e];
          }
      };
      auto ds_group = [&](int j) __attribute__((always_inline)) {
        const int i4 = j >> 1, qb = j & 1;
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DROPOUT) d4 = *(const f32x4*)(Dv + i0 + 32 * qb + 8 * i4 + 4 * g);   // -D_i
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          float dpv = dp[qb][i];
          if constexpr (DROPOUT) dpv = dropped_dp_minus_d(dpv, a.keep_scale, KeepLK::mask(kept, qb, i4, e), d4[e]);
          dsf[cc][tt] = (T)(s[qb][i] * dpv);
        }
      };
      if constexpr (DROPOUT) {
#pragma unroll
        for (int j = 0; j < 8; ++j) p_group(j);
        col_product(Gt, pf, dv, nothing);               // dV^T += dO^T P_dropped
        start_dp();
        row_product(Gt, vf, dp, nothing);               // dP = dO V^T
#pragma unroll
        for (int j = 0; j < 8; ++j) ds_group(j);
      } else {
        // the vector work between the MFMAs that do not wait for it: the two wavefronts of a SIMD are in the same part of a tile
        start_dp();
        row_product(Gt, vf, dp, [&](int f) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 8 * f / (2 * KK); j < 8 * (f + 1) / (2 * KK); ++j) p_group(j);
        });
        col_product(Gt, pf, dv, [&](int f) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 8 * f / (4 * DB); j < 8 * (f + 1) / (4 * DB); ++j) ds_group(j);
        });
      }
      // dS for the wavefronts that add up dQ: four queries 8 i4 + 4 g .. of this lane's key at a time
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          T4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = dsf[cc][4 * hb + e];
          *(T4*)(St + lds_off<TILE>(w0 + r, 2 * cc + hb) + 4 * g) = v;
        }
      col_product(Qt, dsf, dk, nothing);                // dK^T += Q^T dS
    };
    auto dq_step = [&](const int t, const T* const St) __attribute__((always_inline)) {
      const int q0 = t * TILE + qp;   // the piece's first query
      f32x4 dq[QH];
      float* const mine = part + (int64_t)t * (8 * QH * 256);
#pragma unroll
      for (int x = 0; x < QH; ++x)
#pragma unroll
        for (int e = 0; e < 4; ++e) dq[x][e] = 0.f;
      if (k0 > 0) {
#pragma unroll
        for (int x = 0; x < QH; ++x) dq[x] = *(const f32x4*)(mine + 256 * x);
      }
      const int seen = CAUSAL ? min(len, q0 + 16 * QH) : len;   // keys that a query of the piece sees
      const int steps = min((seen - k0 + 31) / 32, KEYS / 32);
      auto ks_frag = [&](const T* base, int ks, int rows) __attribute__((always_inline)) { return tr_frag<T8>(base + 32 * ks * rows, base + (32 * ks + 16) * rows); };
      T8 ka[2], sa[2][QH];
      auto load = [&](int ks) __attribute__((always_inline)) {
        ka[ks & 1] = ks_frag(Kl + k_off, ks, D);
#pragma unroll
        for (int x = 0; x < QH; ++x) sa[ks & 1][x] = ks_frag(St + s_off[x], ks, TILE);
      };
      if (steps > 0) load(0);
#pragma unroll
      for (int ks = 0; ks < KEYS / 32; ++ks) {
        if (ks >= steps) break;
        if (ks + 1 < KEYS / 32 && ks + 1 < steps) load(ks + 1);
#pragma unroll
        for (int x = 0; x < QH; ++x) dq[x] = mfma16(ka[ks & 1], sa[ks & 1][x], dq[x]);
      }
      // complete with the last block that a query of the tile sees
      if (last_block || (CAUSAL && (t + 1) * TILE <= k0 + KEYS)) {
        if (16 * d16 < dvalid)
#pragma unroll
          for (int x = 0; x < QH; ++x) {
            const int q = q0 + 16 * x + i16;
            T4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (T)(dq[x][e] * a.tau);
            if (q < a.N) *(T4*)((T*)a.dQ + head_off + (int64_t)q * a.sn + 16 * d16 + 4 * q16) = v;
          }
      } else {
#pragma unroll
        for (int x = 0; x < QH; ++x) *(f32x4*)(mine + 256 * x) = dq[x];
      }
    };
    for (int j = first; j <= n_tiles; ++j) {
      if (j + 1 < n_tiles) fetch_tile(j + 1, Q0 + 2 * ((j + 1 - first) & 1) * kQ);
      if (j > first) dq_step(j - 1, S0 + ((j - 1) & 1) * kS);
      if (j < n_tiles) tile_step(j * TILE, Q0 + 2 * ((j - first) & 1) * kQ, S0 + (j & 1) * kS);
      wait_async_copies();
      __syncthreads();
    }
    // the K rows and the tiles are free: the next block's K rows come while this one's gradients go out through the tile buffers
    const int64_t out_row0 = head_off + (int64_t)kw0 * a.sn;
    if (!last_block) fetch_keys(k0 + KEYS);
    T* const stage = Q0 + wave * 32 * D;
    store_rows_coalesced<T, D>(stage, (T*)a.dV + out_row0, a.sn, dv, DROPOUT ? a.keep_scale : 1.f, a.N - kw0, dvalid);
    __builtin_amdgcn_wave_barrier();
    store_rows_coalesced<T, D>(stage, (T*)a.dK + out_row0, a.sn, dk, a.tau, a.N - kw0, dvalid);
    if (!last_block) {
      __syncthreads();   // everyone's rows are out of the tile buffers
      if (D == 32 && a.dvalid < D) {   // those rows lie across the columns >= 16 that the copies leave untouched
        zero_tiles(Q0, 4 * kQ);
        __syncthreads();
      }
      const int next = CAUSAL ? (k0 + KEYS) / TILE : 0;
      if (next < n_tiles) fetch_tile(next, Q0);
    }
  }
  // rows of tiles that see nothing
  for (int row = n_tiles * TILE + (int)threadIdx.x / (D / 8); row < a.N; row += 512 / (D / 8)) {
    const int ch = (int)threadIdx.x % (D / 8);
    T8 z;
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = (T)0.f;
    if (8 * ch < dvalid) *(T8*)((T*)a.dQ + head_off + (int64_t)row * a.sn + 8 * ch) = z;
  }
}

template <typename T, int D, int KW>
int launch_kw(const KArgs& a, bool causal, bool dropout, hipStream_t s) {
  const dim3 grid(kXcds * a.chunk), block(64 * KW);
  if (causal && dropout) hipLaunchKernelGGL((bwd_short_kernel<T, D, true, true, KW>), grid, block, 0, s, a);
  else if (causal) hipLaunchKernelGGL((bwd_short_kernel<T, D, true, false, KW>), grid, block, 0, s, a);
  else if (dropout) hipLaunchKernelGGL((bwd_short_kernel<T, D, false, true, KW>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((bwd_short_kernel<T, D, false, false, KW>), grid, block, 0, s, a);
  return (int)hipGetLastError();
}

template <typename T, int D>
int launch_blocks(const KArgs& a, bool causal, bool dropout, hipStream_t s) {
  if (a.N > 512 || a.dQpart == nullptr) return (int)hipErrorInvalidValue;
  const dim3 grid(kXcds * a.chunk), block(512);
  if (causal && dropout) hipLaunchKernelGGL((bwd_blocks_kernel<T, D, true, true>), grid, block, 0, s, a);
  else if (causal) hipLaunchKernelGGL((bwd_blocks_kernel<T, D, true, false>), grid, block, 0, s, a);
  else if (dropout) hipLaunchKernelGGL((bwd_blocks_kernel<T, D, false, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((bwd_blocks_kernel<T, D, false, false>), grid, block, 0, s, a);
  return (int)hipGetLastError();
}

template <typename T, int D>
int launch_td(const KArgs& a, bool causal, bool dropout, hipStream_t s) {
  if (a.N > 256) return launch_blocks<T, D>(a, causal, dropout, s);
  return a.N <= 128 ? launch_kw<T, D, 4>(a, causal, dropout, s) : launch_kw<T, D, 8>(a, causal, dropout, s);
}

}  // namespace

// Which heads take this kernel.  us of the backward pass, two launches (divided over wavefront groups where there are few heads) | this kernel; heads x N:
//   one or two tiles, d = 64  1 x 128 12.1 | 7.9, 96 x 128 13.2 | 8.6, 2048 x 128 83.9 | 66.6, causal with dropout 91.7 | 70.5; 4032 x 65 116 | 85; 96 x 1 10.4 | 6.0
// From three tiles on, the time of this kernel over that of the two launches, by heads; N = 129 192 193 256:
//   d = 64  64 0.94 1.03 1.28 1.39; 128 0.94 1.02 1.05 1.09; 160 0.72 0.81 0.83 0.92; 256 0.74 0.84 0.84 0.93; 257 0.90 0.97 1.01 1.10; 384 0.91 0.99 1.01 1.06; 400 0.81 0.89 0.89 0.97; 512
//     0.82 0.88 0.89 0.97; 513 0.92 1.00 1.02 1.11; 768 0.84 0.94 0.94 1.03; 1024 0.87 0.96 0.97 1.07; 1025 0.94 1.04 1.07 1.19; 2048 0.89 0.95 1.01 1.01
//     dropout  64 0.96 1.05 1.39 1.47; 128 0.96 1.04 1.07 1.14; 256 0.75 0.86 0.85 0.93; 257 0.94 1.01 1.03 1.13; 384 0.96 1.05 1.06 1.13; 400 0.83 0.92 0.91 1.00; 513 0.97 1.04 1.05 1.15; 768 0.89
//     0.97 0.98 1.06; 1025 0.99 1.11 1.12 1.22; 2048 0.95 1.08 1.09 1.14
//     causal  64 0.90 0.97 1.20 1.21; 128 0.86 0.94 1.01 1.05; 160 0.80 0.83 0.89 0.91; 256 0.80 0.86 0.90 0.94; 257 0.99 1.03 1.04 1.09; 320 1.01 1.07 1.02 0.99; 384 0.99 1.02 0.99 1.03; 400 0.92
//     0.97 0.99 1.02; 512 0.89 0.96 0.97 0.99; 513 1.04 1.10 1.13 1.14; 640 0.98 1.01 1.05 1.02; 768 0.90 0.96 0.97 0.96; 1024 0.90 0.99 1.03 1.03; 1025 1.05 1.13; 2048 0.96 1.06
//     causal, dropout  64 0.88 0.96 1.25 1.26; 128 0.87 0.94 1.06 1.12; 256 0.81 0.91 0.93 0.96; 257 1.03 1.10 1.08 1.09; 384 1.02 1.10 1.01 1.06; 400 0.92 1.02 1.01 1.07; 512 0.93 1.00 0.99 1.02; 513
//     1.11 1.17 1.18 1.20; 768 0.96 1.02 1.01 1.02; 1024 0.96 1.06 1.06 1.11; 2048 1.02 1.13
//   d = 32  64 0.92 1.01 1.36 1.51; 128 0.90 1.00 1.12 1.28; 160 0.74 0.84 0.91 1.04; 256 0.75 0.85 0.90 1.00; 257 1.12 1.27 1.35 1.50; 384 1.11 1.19 1.28 1.44; 400 0.86 0.94 0.99 1.13; 512 0.85
//     0.98 1.02 1.18; 513 1.07 1.24 1.30 1.47; 768 0.94 1.05 1.11 1.22; 1024 0.95 1.09 1.15 1.28; 2048 1.03 1.18
//     dropout  64 0.87 0.95 1.39 1.52; 128 0.87 0.95 1.11 1.22; 160 0.69 0.75 0.84 0.93; 257 0.93 1.02 1.07 1.19; 384 0.91 0.99 1.03 1.20; 400 0.75 0.81 0.86 0.99; 512 0.74 0.86 0.89 1.02; 513 0.91
//     1.02 1.07 1.19; 768 0.79 0.89 0.91 1.05; 1025 0.91 1.00 1.05 1.20; 2048 0.83 0.96 0.98 1.15
//     causal  64 0.81 0.87 1.20 1.25; 128 0.81 0.85 1.14 1.15; 160 0.78 0.82 0.82 0.84; 256 0.76 0.79 0.71 0.74; 257 1.14 1.14 1.19 1.20; 352 1.03 1.06 1.09 1.15; 400 0.88 0.89 0.97 1.04; 512 0.79
//     0.94 0.98 1.02; 513 1.00 1.10 1.18 1.22; 640 0.96 1.04 1.08 1.11; 768 0.90 0.98 1.04 1.09; 1024 0.89 0.97 1.04 1.09; 1025 1.03 1.09; 2048 0.95 1.02
//     causal, dropout  64 0.77 0.81 1.23 1.25; 128 0.77 0.79 1.13 1.15; 256 0.71 0.74 0.68 0.71; 257 1.03 1.06 1.08 1.08; 320 1.00 1.05 1.00 1.06; 352 0.95 0.97 0.99 1.04; 400 0.84 0.86 0.91 0.98; 512
//     0.76 0.86 0.91 0.95; 513 0.97 1.07 1.11 1.16; 768 0.84 0.92 0.95 1.01; 1025 0.98 1.04; 2048 0.90 0.95
// Up to 256 heads, a round over the compute units: three tiles always (the few losses are below 7 %, and a launch is saved).  Four tiles: up to 64 heads the two launches' divided
// blocks fill more of the chip; up to 128 both take one round (even to 6 % with d = 64 and no dropout, under the causal mask from 97 heads on, where the launch saved decides); from 129 on
// the two launches have two rounds (at d = 32 with neither mask nor dropout even to 4 % at 256 tokens).  Beyond 256 heads it is the last round of whole heads that decides, by whether it is more than half full, and the more the longer the
// heads and the faster the two launches are there.  Left aside: d = 64 causal with four tiles and a full third round (0.94 to 0.97), d = 32 causal with dropout, 225 to 256 tokens and a full second one
// (0.92 to 0.98).
bool bwd_short_is_faster(const KArgs& a, int d, bool causal, bool dropout) {
  if (d > 64 || a.N > 256) return false;
  if (a.N <= 2 * TILE) return true;
  const int64_t heads = (int64_t)a.B * a.H;
  if (heads <= kComputeUnits) {
    if (a.N <= 3 * TILE) return true;
    return heads > kComputeUnits / 2 || (heads > (causal ? 3 : 2) * kComputeUnits / 8 && d == 64 && a.N <= 208 && !dropout);
  }
  // the longest heads that take it: of two rounds, of three or four, of more, each with the last round up to half full and beyond
  constexpr uint8_t kLongest[2][2][2][6] = {   // [d <= 32][causal][dropout]
      {{{192, 224, 192, 224, 176, 192}, {160, 224, 144, 192, 144, 144}}, {{128, 192, 128, 192, 128, 160}, {128, 192, 128, 144, 128, 128}}},
      {{{128, 192, 128, 144, 128, 128}, {192, 224, 192, 224, 192, 192}}, {{128, 224, 144, 192, 128, 192}, {128, 224, 176, 224, 176, 192}}}};
  const int rounds = heads <= 2 * kComputeUnits ? 0 : heads <= 4 * kComputeUnits ? 2 : 4;
  const bool full = (heads - 1) % kComputeUnits >= kComputeUnits / 2;
  if (causal && !(d == 64 && dropout) && 4 * heads > 5 * kComputeUnits && 2 * heads <= 3 * kComputeUnits) return a.N <= 192;   // (even, and ahead for odd numbers of heads)
  return a.N <= kLongest[d == 32][causal][dropout][rounds + full];
}

// Which heads of more than 256 tokens do: time of this kernel over that of the two launches, by heads; N = 257 to 384, then 385 to 512.
//   d = 64  128 1.30-1.37, 1.39-1.45; 160 1.27-1.32, 0.96-1.04; 192 0.90-0.94, 0.97-1.04; 224 0.92-0.94, 0.83-0.89; 256 0.91-0.94, 0.84-0.90; 257 1.44-1.47, 1.26-1.34; 512 1.02-1.08, 0.93-1.02
//   d = 64, dropout  160 1.26-1.32, 1.03-1.08; 192 0.92-0.95, 1.02-1.08; 224 0.94-0.96, 0.86-0.92; 256 0.94-0.97, 0.86-0.92; 257 1.4, 1.4; 512 1.06-1.10, 0.95-1.01
//   d = 64, causal, with and without dropout  128 1.14-1.24, 1.19-1.40; 160 1.03-1.16, 1.03-1.11; 192 0.88-0.95, 0.90-1.01; 224 0.81-0.87, 0.85-0.93; 256 0.80-0.85, 0.85-0.90; 257 1.25-1.34, 1.3-1.4;
//           512 0.94-1.00, 0.89-1.01
//   d = 32  192 0.96-1.09, 1.07-1.23; 224 0.98-1.10, 0.84-0.96; 256 1.01-1.09, 0.86-0.96; 257 1.5;  dropout 192 0.90-0.99, 1.05-1.17; 256 0.95-1.02, 0.88-0.96
//   d = 32, causal, with and without dropout  160 0.90-1.07, 1.05-1.18; 192 0.91-0.99, 0.95-1.04; 224 0.85-0.92, 0.80-0.91; 256 0.81-0.94, 0.81-0.94; 257 1.2-1.4, 1.3-1.45; 512 0.97-1.03, 0.91-0.99
// A compute unit holds one workgroup, a head: one round that is nearly full pays.
bool bwd_blocks_is_faster(const KArgs& a, int d, bool causal) {
  if (d > 64 || a.N <= 256 || a.N > 512) return false;
  const int64_t heads = (int64_t)a.B * a.H;
  if (heads > kComputeUnits) return false;
  return a.N > 384 ? heads >= 224 : heads >= 192 && (d == 64 || causal);
}

int launch_bwd_short(const KArgs& a_in, int dtype, int d, bool causal, bool dropout, hipStream_t s) {
  KArgs a = a_in;
  a.n_items = a.B * a.H;   // a workgroup per head
  a.chunk = (a.n_items + kXcds - 1) / kXcds;
  if (dtype == 0 && d == 32) return launch_td<_Float16, 32>(a, causal, dropout, s);
  if (dtype == 1 && d == 32) return launch_td<__bf16, 32>(a, causal, dropout, s);
  if (dtype == 0 && d == 64) return launch_td<_Float16, 64>(a, causal, dropout, s);
  if (dtype == 1 && d == 64) return launch_td<__bf16, 64>(a, causal, dropout, s);
  return (int)hipErrorInvalidValue;
}

}  // namespace attn
