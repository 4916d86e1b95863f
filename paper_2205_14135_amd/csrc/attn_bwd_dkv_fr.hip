// dK / dV kernel for head dimensions up to 64 (dense and block-sparse): one wavefront does all
// four tile products of its 32 keys.
//
// Arithmetic: Algorithm 4 of the paper for one block of 128 keys, swept over 64-query tiles:
//     S = Q K^T, P = exp(S - L), dV += (P o Z)^T dO, dP = (dO V^T) o Z, dS = P o (dP - D), dK += tau dS^T Q.
// At d <= 64 both accumulators (dK^T, dV^T), both operand fragment sets (K, V) and the S / dP tiles
// of a wavefront fit in 256 registers, so the work of a key block need not be split over two
// wavefronts of a SIMD as in attn_bwd_dkv.hip: no probabilities travel through LDS, there is one
// workgroup barrier per tile (for the tile buffers only), and a workgroup is 4 wavefronts, so two
// or more independent workgroups share a compute unit and fill each other's stalls.  The vector
// ALU work per tile is the same at every head dimension while the matrix work shrinks with it;
// at d <= 64 that free-running arrangement is faster than the role split (at d = 128 the one-wavefront
// arrangement is attn_bwd_dkv_fr128.hip, and the role split is left large block masks: choose_dkv).
// Vector registers spilled: none.
// Register layout "lane = key" (S = Q K^T: accumulator rows = queries of the tile, column = the
// lane's key), as in attn_bwd_dkv.hip.
#include "attn_common.h"
#include "attn_sparse.h"
#include "attn_tiles.h"

namespace attn {
namespace {

constexpr int TILE = 64;

// RW wavefronts of 32 keys, times KG groups of them that each take every KG-th query tile, into buffers of their own; the groups'
// gradients are summed through LDS at the end.  (Block-sparse work is assigned by columns of 128 keys: RW = 4.)
template <typename T, int D, bool CAUSAL, bool DROPOUT, bool SPARSE, int RW, int KG>
__global__ __launch_bounds__(64 * RW * KG, 2) void dkv_fr_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  constexpr int KK = D / 16, DB = D / 32;
  static_assert(D <= 64, "the accumulators of both gradients must fit one wavefront");
  // Tile buffers, double buffered: Q tiles Qs0 + buf TILE D, dO tiles Gs0 + buf TILE D, base-2 row
  // statistic Ls0 + buf TILE, -D_i Ds0 + buf TILE.  The plain dense kernel (no mask, no dropout)
  // unrolls its tile loop by two, so that the buffer index is a constant, and keeps all of them in
  // one LDS block (row vectors first): every LDS address is then a per-lane register plus an
  // immediate.  The other forms have no registers for two copies of the loop body and keep the
  // separate arrays (the form their register allocation is tuned to).
  constexpr int UNROLL = (!CAUSAL && !DROPOUT && !SPARSE) ? 2 : 1;
  static_assert(!SPARSE || RW == 4, "mask columns are 128 keys wide");
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / RW;
  constexpr int kGroupBytes = 4 * TILE * sizeof(float) + 4 * TILE * D * sizeof(T);
  T *Qs0, *Gs0;
  float *Ls0, *Ds0;
  unsigned char* all = nullptr;   // the LDS of all groups (KG > 1)
  if constexpr (UNROLL == 2 || KG > 1) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[KG * kGroupBytes];
    all = smem;
    Ls0 = (float*)(smem + group * kGroupBytes);
    Ds0 = Ls0 + 2 * TILE;
    Qs0 = (T*)(Ls0 + 4 * TILE);
    Gs0 = Qs0 + 2 * TILE * D;
  } else {
    __shared__ __attribute__((aligned(16))) T Qs[2 * TILE * D];
    __shared__ __attribute__((aligned(16))) T Gs[2 * TILE * D];
    __shared__ __attribute__((aligned(16))) float Ls[2 * TILE];
    __shared__ __attribute__((aligned(16))) float Ds[2 * TILE];
    Qs0 = Qs; Gs0 = Gs; Ls0 = Ls; Ds0 = Ds;
  }
  // dropout flags in this layout: see KeepLK in attn_common.h
  __shared__ __attribute__((aligned(16))) uint32_t keep_table[DROPOUT ? KeepLK::kTable : 4];
  KeepLK keep;
  if constexpr (DROPOUT) keep.init(keep_table, a.drop_thr);

  constexpr int BR = 32 * RW;
  const int n_kt = RW == 4 ? a.T : (a.N + BR - 1) / BR;   // the last key block may be ragged
  // Work assignment.  Dense: one key block per workgroup (under the causal mask key block k is
  // visited by N/64 - 2k query tiles, and the early ones come first: causal_block).  Block-sparse (as in attn_bwd_dkv.hip): the first 8 * chunk workgroups take one mask
  // column each and leave the heavy ones alone; those are cut into segments (attn_sparse.h),
  // which the remaining workgroups walk.
  const int n_col_groups = kXcds * a.chunk;
  // (the list workgroups come first in the grid, a multiple of the XCD count of them, so that the
  // long segments start with the launch instead of queueing behind every column)
  const int n_list = SPARSE ? (int)gridDim.x - n_col_groups : 0;
  const bool list_mode = SPARSE && (int)blockIdx.x < n_list;
  constexpr bool DEALT = CAUSAL && !SPARSE;
  for (int round = 0;; ++round) {
  int item, slot = 0, skip_blocks = 0, take_blocks = 0x7fffffff;
  bool heavy = false;
  if (!list_mode) {
    item = DEALT ? causal_item(a) : xcd_item(a.n_items, a.chunk, (int)blockIdx.x - n_list);
    if (item < 0) return;
    if constexpr (SPARSE) {
      if (n_list > 0 && a.col_segs[item] > 0) return;   // heavy
    }
  } else {
    if (!sparse_segment((int)blockIdx.x + round * n_list, item, slot, skip_blocks, take_blocks)) return;
    heavy = true;
  }
  int bh = item / n_kt, kt = item % n_kt;
  if constexpr (DEALT)
    if (!causal_block(a, item, n_kt, bh, kt)) return;
  if (!SPARSE && !(DEALT && a.group <= 0)) bh = dealt_head(a, bh);
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const T* __restrict__ Qg = (const T*)a.Q + head_off;
  const T* __restrict__ Gg = (const T*)a.dO + head_off;
  // padded to a multiple of 128 rows per head: +inf / 0 beyond a ragged end, so those query rows
  // (whose Q and dO tile rows are copies of the last real row) contribute P = 0 and dS = 0
  const float* __restrict__ Lg = a.L2vec + (int64_t)bh * a.Nr;
  const float* __restrict__ Dg = a.Dvec + (int64_t)bh * a.Nr;

  const int lane = threadIdx.x & 63;
  // The wavefront number in a scalar register, so that addresses and branches on it are scalar: 1-4 % faster at
  // d = 64 (B H = 128, N = 2048 266 -> 260 us, block-sparse N = 16384 122 -> 117); causal with dropout (GPT-2 shape 64.2 -> 65.9)
  // and d = 32 (B H = 128, N = 700 36.4 -> 37.3) lose 2.5 % that way.
  constexpr bool SCALAR_WAVE = KG > 1 || (D == 64 && !(CAUSAL && DROPOUT));
  const int wave = SCALAR_WAVE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - RW * group : (int)threadIdx.x >> 6;
  const int r = lane & 31, g = lane >> 5;
  const int kw0 = kt * BR + wave * 32;
  const int kj = kw0 + r;  // this lane's key (>= N beyond a ragged end: masked like a padded key, never stored)

  // loop-invariant B operands: the K and V fragments of this lane's key
  T8 kf[KK], vf[KK];
  {
    const int64_t row_off = head_off + (int64_t)min(kj, a.N - 1) * a.sn;
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
  }
  // The fragments must have arrived before the tile loop: a wait for them inside the loop would
  // also wait for the asynchronous tile copies in flight there.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
  f32x16 dv[DB], dk[DB];   // dV^T, dK^T (rows d, column = this lane's key)
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dv[db][i] = 0.f; dk[db][i] = 0.f; }

  // key-padding mask: key blocks and query tiles at or beyond the batch's length are not visited
  // (rows >= len inside the last tile have LSE = -inf, hence P = 0); masked keys get P = 0
  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  TileIter<SPARSE> it;
  if constexpr (SPARSE)
    it.init(a.mask + (int64_t)h * a.mask_sh + kt, a.T, CAUSAL ? kt : 0,
            kt * 128 >= len ? 0 : min(a.T, (len + 127) / 128), skip_blocks, take_blocks);
  else
    it.init(nullptr, 0, CAUSAL ? kt * BR / TILE : 0, kt * BR >= len ? 0 : (len + TILE - 1) / TILE);   // len <= N

  TrOffsets<D> tro;
  tro.init();
  TileAsync<T, D, RW> dma;
  dma.init(a.sn, wave, D == 32 ? a.dvalid : D);
  if (D == 32 && a.dvalid < D) {   // the copies leave columns >= 16 of the tile buffers untouched
    // (again in every round: the buffers staged output rows)
    if constexpr (KG > 1) {
      zero_tiles((T*)all, KG * kGroupBytes / (int)sizeof(T));
    } else {
      zero_tiles(Qs0, 2 * TILE * D);
      zero_tiles(Gs0, 2 * TILE * D);
    }
    __syncthreads();
  }
  auto fetch_tile = [&](int t, int buf) {
    dma.copy_rows(Qg, a.sn, t * TILE, a.N, Qs0 + buf * TILE * D);
    dma.copy_rows(Gg, a.sn, t * TILE, a.N, Gs0 + buf * TILE * D);
    // (addresses from the arrays themselves: from a pointer into them the compiler tests for null, with an instruction that it
    // then finds to be illegal in the block-sparse forms)
    const uint32_t at = (uint32_t)(buf * TILE * sizeof(float));
    const uint32_t l_at = KG > 1 ? lds_addr(all) + (uint32_t)(group * kGroupBytes) : lds_addr(Ls0);
    const uint32_t d_at = KG > 1 ? l_at + (uint32_t)(2 * TILE * sizeof(float)) : lds_addr(Ds0);
    if (wave == RW / 2 - 1) async_copy_b32(Lg + t * TILE + lane, __builtin_amdgcn_readfirstlane(l_at + at));
    if (wave == RW / 2) async_copy_b32(Dg + t * TILE + lane, __builtin_amdgcn_readfirstlane(d_at + at));
  };
  const float c = a.scale_log2;

  // LDS operand reads run PF fragments ahead of the MFMA that consumes them
  constexpr int PF = 4;
  // out[qb] = Tile[32 qb .. +31][:] . frags; between(f) comes after MFMA f of 2 KK
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
  // acc^T += Tile^T . frag   (contraction over the 64 queries of the tile); between(f) comes after MFMA f of 4 DB
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
  // The vector work of P and dS in between the MFMAs of the products that do not wait for it (below).  us of this kernel, before | after: d = 32, where a product is
  // four MFMAs and latency binds, B H = 128, N = 700 34.7 | 28.9, 64 x 1500 72.7 | 57.1; d = 64 causal 128 x 1024 49.3 | 47.6, 64 x 2000 82.9 | 80.3, block-sparse N =
  // 16384 1 %; without a mask nothing (128 x 2048 294 | 290, 60 x 900 38.0 | 38.9), nor d = 32 causal (60 x 1000 21.6 | 22.1); with dropout it spills or is slower (d = 64, 256 x 512 56.4 | 61.3, d = 32, 96 x 1000
  // 63.4 | 70.9).
  constexpr bool BETWEEN = !DROPOUT && (D == 32 ? !CAUSAL : CAUSAL || SPARSE);
  // ---- pipeline over the query tiles of this key block: tile t + 1 streams in while t is used
  int buf_rt = 0;
  // t: this group's tile, -1 if there is none; more: some group (then the first) has one
  int t;
  bool more = it.template next_of<KG>(group, t);
  if (t >= 0) fetch_tile(t, 0);
  wait_async_copies();
  __syncthreads();
  while (KG == 1 ? t >= 0 : more) {
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int buf = UNROLL == 2 ? u : buf_rt;
    int t_next;
    const bool more_next = it.template next_of<KG>(group, t_next);
    if (t_next >= 0) fetch_tile(t_next, buf ^ 1);
    const int i0 = t * TILE;
    if ((KG == 1 || t >= 0) && (!CAUSAL || i0 + TILE - 1 >= kw0)) {
      f32x16 s[2], dp[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[qb][i] = 0.f;
      row_product(Qs0 + buf * TILE * D, kf, s, nothing);                       // S = Q K^T
      uint32_t kept = 0;   // the keep flags of this lane's key for the tile's 64 queries it holds
      if constexpr (DROPOUT) kept = keep.draw<2>(i0, kw0, bh, a.offset_lo, a.seed_lo, a.seed_hi);
      // hidden entries get the logit -inf, hence P = 0: above the causal diagonal (tiles that cross it
      // only: a comparison and a select per element on every tile were a third of the vector instructions;
      // B H = 128, N = 2048: 173 -> 158 us) or padded keys
      if ((CAUSAL && i0 < kw0 + 31) || kw0 + 32 > len) {
        const int first_query = kj < len ? (CAUSAL ? kj : 0) : 0x7fffffff;   // that sees this lane's key
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (i0 + 32 * qb + 8 * (i >> 2) + 4 * g + (i & 3) < first_query) s[qb][i] = -INFINITY;
      }
      // P = exp(S - L), kept in fp32 in s[] for dS; the 16-bit (dropped) copy feeds dV.  Four elements: j = 2 i4 + qb
      T8 pf[4], dsf[4];
      auto p_group = [&](int j) __attribute__((always_inline)) {
        const int i4 = j >> 1, qb = j & 1;
        // (keeps the bit extracts where they are used: hoisted, they make the forms short of registers spill; the
        // plain form is faster without)
        if constexpr (DROPOUT && (CAUSAL || SPARSE))
          if (qb == 0) asm volatile("" : "+v"(kept));
        const f32x4 l4 = *(const f32x4*)(Ls0 + buf * TILE + 32 * qb + 8 * i4 + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[qb][i], c, -l4[e]));
          s[qb][i] = p;
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          pf[cc][tt] = DROPOUT ? (T)keep_or_zero(p, KeepLK::mask(kept, qb, i4, e)) : (T)p;
        }
      };
      auto start_dp = [&]() __attribute__((always_inline)) {   // without dropout dP starts from -D, so that the result is dP - D
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
            if constexpr (!DROPOUT) d4 = *(const f32x4*)(Ds0 + buf * TILE + 32 * qb + 8 * i4 + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) dp[qb][4 * i4 + e] = d4[e];
          }
      };
      auto ds_group = [&](int j) __attribute__((always_inline)) {
        const int i4 = j >> 1, qb = j & 1;
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DROPOUT) d4 = *(const f32x4*)(Ds0 + buf * TILE + 32 * qb + 8 * i4 + 4 * g);   // -D_i
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const int cc = 2 * qb + (i4 >> 1), tt = 4 * (i4 & 1) + e;
          float dpv = dp[qb][i];
          if constexpr (DROPOUT) dpv = dropped_dp_minus_d(dpv, a.keep_scale, KeepLK::mask(kept, qb, i4, e), d4[e]);
          dsf[cc][tt] = (T)(s[qb][i] * dpv);
        }
      };
      if constexpr (!BETWEEN) {
#pragma unroll
        for (int j = 0; j < 8; ++j) p_group(j);
        col_product(Gs0 + buf * TILE * D, pf, dv, nothing);               // dV^T += dO^T P_dropped
        start_dp();
        row_product(Gs0 + buf * TILE * D, vf, dp, nothing);               // dP = dO V^T
#pragma unroll
        for (int j = 0; j < 8; ++j) ds_group(j);
      } else {
        // P comes between the MFMAs of dP and dS between those of dV: the matrix pipe and the vector ALU work at once within a wavefront, not only
        // where two wavefronts happen to be in different parts of a tile
        start_dp();
        row_product(Gs0 + buf * TILE * D, vf, dp, [&](int f) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 8 * f / (2 * KK); j < 8 * (f + 1) / (2 * KK); ++j) p_group(j);
        });
        col_product(Gs0 + buf * TILE * D, pf, dv, [&](int f) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 8 * f / (4 * DB); j < 8 * (f + 1) / (4 * DB); ++j) ds_group(j);
        });
      }
      col_product(Qs0 + buf * TILE * D, dsf, dk, nothing);                // dK^T += Q^T dS
    }
    wait_async_copies();
    __syncthreads();   // the next tile has landed, and everyone is done with this buffer
    buf_rt ^= 1;
    t = t_next;
    more = more_next;
    if (KG == 1 ? t < 0 : !more) break;
  }
  }

  if constexpr (KG > 1) {
    // the loop ended on a barrier (or never touched LDS): the groups but the first leave their gradients in the tile buffers
    constexpr int kLanes = 64 * RW;
    static_assert((KG - 1) * 2 * DB * 16 * kLanes * 4 <= KG * kGroupBytes, "LDS holds the groups' gradients");
    f32x4* const part = (f32x4*)all + wave * 64 + (SPARSE ? lane_id_here() : lane);
    if (group > 0) {
#pragma unroll
      for (int f = 0; f < 8 * DB; ++f) {   // dV^T, then dK^T
        const f32x16& x = f < 4 * DB ? dv[f / 4 % DB] : dk[f / 4 % DB];
        const int i = 4 * (f % 4);
        const f32x4 v = {x[i], x[i + 1], x[i + 2], x[i + 3]};
        part[((group - 1) * 8 * DB + f) * kLanes] = v;
      }
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int k = 0; k < KG - 1; ++k)
#pragma unroll
        for (int f = 0; f < 8 * DB; ++f) {
          f32x16& x = f < 4 * DB ? dv[f / 4 % DB] : dk[f / 4 % DB];
          const f32x4 v = part[(k * 8 * DB + f) * kLanes];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[4 * (f % 4) + e] += v[e];
        }
    }
    __syncthreads();   // the buffers stage the output rows
  }
  if (KG > 1 && group > 0) {
    // (merged)
  } else if (SPARSE && heavy) {
    // one of several segments of this column: sum in fp32; the last of them converts.  The loop
    // ended on a barrier: the two Q buffers stage the rows of wavefronts 0 and 1, the two dO buffers
    // those of wavefronts 2 and 3 (32 x D floats each), first for dV, then for dK
    float* stage = (float*)(wave < 2 ? Qs0 : Gs0) + (wave & 1) * 32 * D;
    const int64_t acc_row0 = ((int64_t)slot * 128 + (kw0 - kt * 128)) * D;
    atomic_add_rows_coalesced<D>(stage, a.dVacc + acc_row0, dv, DROPOUT ? a.keep_scale : 1.f, D == 32 ? a.dvalid : D);
    atomic_add_rows_coalesced<D>(stage, a.dKacc + acc_row0, dk, a.tau, D == 32 ? a.dvalid : D);
  } else {
    // the loop ends on a barrier (or never touched LDS): the tile buffers stage the output rows
    T* stage_v = Qs0 + wave * 32 * D;   // 4 wavefronts x 32 rows = the two Q buffers
    T* stage_k = Gs0 + wave * 32 * D;
    const int out_lane = SPARSE ? lane_id_here() : lane;
    store_rows_coalesced<T, D>(stage_v, (T*)a.dV + head_off + (int64_t)kw0 * a.sn, a.sn, dv,
                               DROPOUT ? a.keep_scale : 1.f, a.N - kw0, D == 32 ? a.dvalid : D, out_lane);
    store_rows_coalesced<T, D>(stage_k, (T*)a.dK + head_off + (int64_t)kw0 * a.sn, a.sn, dk, a.tau, a.N - kw0,
                               D == 32 ? a.dvalid : D, out_lane);
  }
  if constexpr (SPARSE)
    if (heavy) sparse_finish<T, D>(item);
  if (!list_mode) return;
  __syncthreads();   // LDS is reused by the next segment
  }  // for round
}

template <typename T, int D, int RW, int KG>
int launch_groups(KArgs a, bool causal, bool dropout, bool sparse, int extra_groups, hipStream_t s) {
  const int blocks = RW == 4 ? a.T : (a.N + 32 * RW - 1) / (32 * RW);
  a.n_items = a.B * a.H * blocks;
  a.chunk = (a.n_items + kXcds - 1) / kXcds;
  a.group = causal_group(a, D, sparse, false, 2 * (int64_t)a.N * D * (int64_t)sizeof(T));   // Q and dO
  if (causal && !sparse) whole_levels(a, D, false, blocks);
  const dim3 grid(kXcds * a.chunk + (sparse ? extra_groups : 0)), block(64 * RW * KG);
#define ATTN_DKV_FR_CASE(C, P, S)                                                           \
  if constexpr (!S || RW == 4)                                                              \
    if (causal == C && dropout == P && sparse == S) {                                       \
      hipLaunchKernelGGL((dkv_fr_kernel<T, D, C, P, S, RW, KG>), grid, block, 0, s, a);     \
      return (int)hipGetLastError();                                                        \
    }
  ATTN_DKV_FR_CASE(false, false, false)
  ATTN_DKV_FR_CASE(true, false, false)
  ATTN_DKV_FR_CASE(false, true, false)
  ATTN_DKV_FR_CASE(true, true, false)
  ATTN_DKV_FR_CASE(false, false, true)
  ATTN_DKV_FR_CASE(true, false, true)
  ATTN_DKV_FR_CASE(false, true, true)
  ATTN_DKV_FR_CASE(true, true, true)
#undef ATTN_DKV_FR_CASE
  return (int)hipErrorInvalidValue;
}

}  // namespace

// us of the backward pass with {4, 1}, and the difference with {4, 2} | {2, 2} | {2, 4} (wavefronts of keys, groups) in this kernel
// alone; heads x N:
//   d = 64   1 x 128 12.3 +1.0 -0.3 +1.4; 16 x 197 17.7 -0.4 -2.1 -0.9; 4 x 512 25.0 -1.3 -3.8 -3.4; 16 x 1024 41.0 -4.2 -7.5 -8.1; 8 x 2048 72.2 -10.2 -15.6 -18.5;
//            1 x 8192 263 -47 -68 -89; 60 x 300 20.6 -0.2 +0.1 +7.0; 24 x 1024 42.0 -4.2 -3.2 +3.2; 8 x 4096 140 -16.6 -10.8 -5.6;
//            10 x 4096 186 +9.3 -4.4 -0.2, dropout 271 +14.7 -19.0 -9.5; 24 x 2001 110 +2.6 -4.2 +3.1; 40 x 1024 57.1 +5.4 +0.4 +8.2; 32 x 2048 116 +2.3 +6.0 +19.2
//   d = 64 causal (the other kernel as its rule has it)  16 x 1024 36.0 -3.5 -8.1 -8.8; 8 x 4096 116 -17.5 -27.3 -34.0; 13 x 2382 79.7 -9.7 -14.8 -14.4; 40 x 1024 44.1 -3.6 -4.7 +3.9;
//            10 x 4096 126 -17.9 -25.8 -15.8; 32 x 2048 84.4 -4.6 -2.2 +9.6; 128 x 512 33.6 +4.4 +3.7 +16.6; 90 x 408 29.0 +2.9 +1.6 +9.7; 46 x 661 34.5 -1.6 -3.2 +1.9; 74 x 656 38.8 +3.1 +2.7 +14.9;
//            61 x 575 32.2 -1.2 -0.9 +9.9; 25 x 1470 with dropout 78.5 -9.9 -15.2 -5.0; 15 x 2832 with dropout 141 -20.9 -34.1 -18.5; 85 x 705 42.8 +4.5 +4.5 -, dropout 55.1 +4.4 +1.8 -;
//            63 x 715 39.3 +0.1 +1.3 -, dropout 52.6 -3.0 -0.9 -; 60 x 900 46.2 +1.4 +1.1 -, dropout 62.5 0 -1.1 -; 64 x 800 with dropout 54.5 -2.1 -1.6 -
//   d = 32   1 x 128 10.0 -0.3 -0.4 -0.1; 16 x 640 22.6 -2.2 -3.7 -4.5; 8 x 2048 56.2 -8.9 -12.2 -16.4; 60 x 512 20.1 -1.6 -1.5 +1.6;
//            8 x 4096 107 -18.5 -16.4 -11.7; 10 x 4096 138 +6.0 -5.7 -4.1; 64 x 1024 43.1 +2.9 +3.1 +10.6
//   d = 32 causal (the other kernel as its rule has it)  16 x 197 13.1 -0.9 -2.2 -2.2; 8 x 4096 97.4 -24.5 -33.8 -39.7; 10 x 4096 101 -23.1 -31.2 -25.2; 128 x 512 24.9 +1.3 +0.7 +7.9;
//            32 x 2048 62.6 -8.1 -7.8 +0.3; 60 x 1000 38.5 -1.5 -1.5 +5.6
//   block-sparse (butterfly mask of T x T blocks, heads x T), {4, 2} only  d = 64  4 x 8 48.1 +0.2; 8 x 16 69.8 -5.7; 4 x 32 65.8 -4.7; 8 x 32 69.6 +6.9,
//            causal 68.4 -3.8; 4 x 64 75.5 +9.2 (the workgroups of the segment list take whole compute units then)
WaveGroups dkv_fr_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide) {
  if (!divide) return {4, 1};
  const bool halves = causal && !sparse;
  const WorkItems w(a, sparse, halves);
  if (sparse) return w.of128 <= kComputeUnits / 2 ? WaveGroups{4, 2} : WaveGroups{4, 1};
  if (w.of64 <= kComputeUnits && w.tiles >= 4) return w.tiles >= (d == 64 ? 24 : 12) ? WaveGroups{2, 4} : WaveGroups{2, 2};
  if (d == 64 && halves && w.of64 <= 11 * kComputeUnits / 8 && w.tiles >= 11) return {2, 2};
  if (d == 64 && halves) return w.of128 <= (w.tiles >= 13 ? 4 : 3) * kComputeUnits / 4 && w.tiles >= 9 ? WaveGroups{4, 2} : WaveGroups{4, 1};
  if (d == 64 && w.of128 <= kComputeUnits && w.tiles >= 4) return {4, 2};
  // (causal, few tiles, {4, 1} | {2, 2}: 100 x 324 17.7 17.2, 117 x 324 19.2 20.7, 120 x 310 16.2 17.0, 152 x 310 17.9 19.4, with dropout 23.6 23.8, 150 x 205 15.6 17.7; 88 x 450 20.7 19.8, 95 x 450 23.5 24.5,
  // 112 x 512 24.5 24.8; 84 x 576 23.0 22.3, 100 x 576 26.5 26.5)
  const int eighths = !halves || w.tiles >= 9 ? 16 : w.tiles >= 7 ? 11 : 10;
  if (d == 32 && w.of64 <= eighths * kComputeUnits / 8 && w.tiles >= 4) return {2, 2};
  if (!halves && w.of64 > 2 * kComputeUnits && w.of64 <= 3 * kComputeUnits && w.tiles >= 24) return {2, 2};
  return {4, 1};
}

namespace {

template <typename T, int D>
int launch_td(const KArgs& a, bool causal, bool dropout, bool sparse, int extra_groups, bool divide, hipStream_t s) {
  const WaveGroups w = dkv_fr_groups(a, D, causal, sparse, divide);
  if (w.waves == 2 && w.groups == 4) return launch_groups<T, D, 2, 4>(a, causal, dropout, sparse, extra_groups, s);
  if (w.waves == 2) return launch_groups<T, D, 2, 2>(a, causal, dropout, sparse, extra_groups, s);
  if (w.groups == 2) return launch_groups<T, D, 4, 2>(a, causal, dropout, sparse, extra_groups, s);
  return launch_groups<T, D, 4, 1>(a, causal, dropout, sparse, extra_groups, s);
}

}  // namespace

// sparse: extra_groups workgroups walk the segments of heavy columns.
int launch_dkv_fr(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, int extra_groups, bool divide,
                  hipStream_t s) {
  if (dtype == 0 && d == 32) return launch_td<_Float16, 32>(a, causal, dropout, sparse, extra_groups, divide, s);
  if (dtype == 1 && d == 32) return launch_td<__bf16, 32>(a, causal, dropout, sparse, extra_groups, divide, s);
  if (dtype == 0 && d == 64) return launch_td<_Float16, 64>(a, causal, dropout, sparse, extra_groups, divide, s);
  if (dtype == 1 && d == 64) return launch_td<__bf16, 64>(a, causal, dropout, sparse, extra_groups, divide, s);
  return (int)hipErrorInvalidValue;
}

}  // namespace attn
