// dK / dV kernel for head dimension 128, dense problems and the block-sparse ones
// of fewer than 2048 mask columns, in which one wavefront does all four tile
// products of its 32 keys (the arrangement of attn_bwd_dkv_fr.hip carried to d = 128).
//
// Arithmetic: Algorithm 4 of the paper for one block of 128 keys, swept over 32-query tiles:
//     S = Q K^T, P = exp(S - L), dV += P^T dO, dP = dO V^T, dS = P o (dP - D), dK += tau dS^T Q.
// At d = 128 the two accumulators (dK^T, dV^T: 128 registers) and the K fragments (32) leave no
// room for the V fragments and for 64-query S / dP tiles, so here the V rows of the workgroup's 128
// keys stay in LDS (the dP product reads both operands from LDS) and the query tiles are 32 rows:
// Q/dO double buffers 4 x 8 KB + V 32 KB = 64 KB per workgroup, two free-running workgroups of four
// wavefronts per compute unit.  S and dP, and then dV and dK, are issued as alternating MFMA
// streams, so that consecutive instructions write different accumulators.  Measured 6 % faster
// than the role-split kernel of attn_bwd_dkv.hip at N = 4096 and 10 % at N = 1024.  Under the causal
// mask a workgroup takes one key block (not a pair: the loop over a pair costs registers this
// kernel does not have) and the blocks are dealt out heaviest first.  Dropout: a call of the
// generator decides 16 consecutive keys of a query, i.e. the 16 lanes of one row of the wavefront,
// which need the draws of the tile's 16 queries 8 i4 + 4 g + e: every lane draws one of them and the
// row transposes the flags (KeepLK in attn_common.h, here with 32-query tiles: one call per lane and tile).
#include <type_traits>

#include "attn_common.h"
#include "attn_sparse.h"
#include "attn_tiles.h"

namespace attn {
namespace {

constexpr int QT = 32;    // queries per streamed tile
constexpr int D = 128;

// RW wavefronts of 32 keys, times KG groups of them that each take every KG-th query tile, into buffers of their own (the V rows are
// shared); the groups' gradients are summed through LDS at the end.
template <typename T, bool CAUSAL, bool DROPOUT, bool SPARSE, int RW, int KG>
__global__ __launch_bounds__(64 * RW * KG, 2) void dkv_fr128_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  constexpr int KK = D / 16, DB = D / 32;
  // One LDS block, so that every address is a per-lane register plus a 16-bit immediate: the row
  // vectors first (1 KB), then the Q tiles, the dO tiles and the V rows of this key block.
  constexpr int BR = 32 * RW;
  constexpr int kVecBytes = 4 * 64 * 4, kGroupBytes = kVecBytes + 4 * QT * D * (int)sizeof(T);
  __shared__ __attribute__((aligned(16))) unsigned char all[KG * kGroupBytes + BR * D * sizeof(T)];
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / RW;
  unsigned char* const smem = all + group * kGroupBytes;
  float* const Ls0 = (float*)smem;                 // base-2 row statistic: Ls0 + 64 buf (first QT entries used:
  float* const Ds0 = Ls0 + 2 * 64;                 // -D_i:                 Ds0 + 64 buf  a copy moves 64 floats)
  T* const Qs0 = (T*)(smem + kVecBytes);           // Q tiles:  Qs0 + buf QT D
  T* const Gs0 = Qs0 + 2 * QT * D;                 // dO tiles: Gs0 + buf QT D
  T* const Vb = (T*)(all + KG * kGroupBytes);      // V rows of this key block

  // dropout flags in this layout: see KeepLK in attn_common.h
  __shared__ __attribute__((aligned(16))) uint32_t keep_table[DROPOUT ? KeepLK::kTable : 4];
  KeepLK keep;
  if constexpr (DROPOUT) keep.init(keep_table, a.drop_thr);

  const int n_kt = RW == 4 ? a.T : (a.N + BR - 1) / BR;   // the last key block may be ragged
  // Block-sparse: one workgroup per mask column, heavy ones in segments that the first workgroups walk (as in dkv_fr_kernel)
  const int n_list = SPARSE ? (int)gridDim.x - kXcds * a.chunk : 0;
  const bool list_mode = SPARSE && (int)blockIdx.x < n_list;
  for (int round = 0;; ++round) {
  int item, slot = 0, skip_blocks = 0, take_blocks = 0x7fffffff;
  if (!list_mode) {
    item = CAUSAL && !SPARSE ? causal_item(a) : xcd_item(a.n_items, a.chunk, (int)blockIdx.x - n_list);
    if (item < 0) return;
    if constexpr (SPARSE) {
      if (n_list > 0 && a.col_segs[item] > 0) return;   // heavy
    }
  } else {
    if (!sparse_segment((int)blockIdx.x + round * n_list, item, slot, skip_blocks, take_blocks)) return;
  }
  int bh = item / n_kt;
  int kt = item % n_kt;
  if constexpr (CAUSAL && !SPARSE)
    if (!causal_block(a, item, n_kt, bh, kt)) return;   // (key block k is visited by the query tiles from the diagonal on)
  if (!SPARSE && !(CAUSAL && a.group <= 0)) bh = dealt_head(a, bh);
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const T* __restrict__ Qg = (const T*)a.Q + head_off;
  const T* __restrict__ Gg = (const T*)a.dO + head_off;
  const T* __restrict__ Vg = (const T*)a.V + head_off;
  const float* __restrict__ Lg = a.L2vec + (int64_t)bh * a.Nr;
  const float* __restrict__ Dg = a.Dvec + (int64_t)bh * a.Nr;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - RW * group;   // in a scalar register: addresses and branches on it are scalar
  const int r = lane & 31, g = lane >> 5;
  const int kw0 = kt * BR + wave * 32;
  const int kj = kw0 + r;

  T8 kf[KK];
  {
    const int64_t row_off = head_off + (int64_t)min(kj, a.N - 1) * a.sn;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = *(const T8*)((const T*)a.K + row_off + 16 * kk + 8 * g);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): before any asynchronous copy is in flight
  f32x16 dv[DB], dk[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) { dv[db][i] = 0.f; dk[db][i] = 0.f; }

  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  const int first = CAUSAL ? kt * (BR / QT) : 0;   // causal: the tiles above the diagonal see none of these keys
  const int limit = kt * BR >= len ? 0 : (len + QT - 1) / QT;

  TrOffsets<D> tro;
  tro.init();
  TileAsync<T, D, RW, QT> dma;     // 32-row tiles: 8 / RW copy instructions per wavefront
  dma.init(a.sn, wave);
  TileAsync<T, D, RW, 64> dma64;   // the V block: 64-row pieces, copied by the first group
  dma64.init(a.sn, wave);
  auto fetch_tile = [&](int t, int buf) {
    dma.copy_rows(Qg, a.sn, t * QT, a.N, Qs0 + buf * QT * D);
    dma.copy_rows(Gg, a.sn, t * QT, a.N, Gs0 + buf * QT * D);
    const int row = min(t * QT + lane, a.Nr - 1);   // whole-wavefront copies: 64 floats, clamped to the head
    if (wave == RW / 2 - 1) async_copy_b32(Lg + row, __builtin_amdgcn_readfirstlane(lds_addr(Ls0 + 64 * buf)));
    if (wave == RW / 2) async_copy_b32(Dg + row, __builtin_amdgcn_readfirstlane(lds_addr(Ds0 + 64 * buf)));
  };
  const float c = a.scale_log2;
  constexpr int PF = 4;

  // V rows of this key block (rows >= N repeat the last one; their keys are masked)
  if (KG == 1 || group == 0) {
    if (kt * BR < a.N) dma64.copy_rows(Vg, a.sn, kt * BR, a.N, Vb);
    if (RW == 4) {
      if (kt * BR + 64 < a.N) dma64.copy_rows(Vg, a.sn, kt * BR + 64, a.N, Vb + 64 * D);
      else if (kt * BR < a.N) dma64.copy_rows(Vg, a.sn, kt * BR, a.N, Vb + 64 * D);   // all of these keys are masked
    }
  }
  // this group's first tile; block-sparse: a 64-row tile of the iterator is two of this kernel's
  TileIter<SPARSE> it;
  int mine = first + group;
  bool more = false;
  if constexpr (SPARSE) {
    it.init(a.mask + (int64_t)h * a.mask_sh + kt, a.T, CAUSAL ? kt : 0, kt * 128 >= len ? 0 : min(a.T, (len + 127) / 128), skip_blocks, take_blocks);
    more = it.template next_of<KG>(group, mine);
    if (mine >= 0) fetch_tile(2 * mine, 0);
  } else {
    if (mine < limit) fetch_tile(mine, 0);
  }
  wait_async_copies();
  __syncthreads();
  // One query tile.  The buffer index is a compile-time constant (the loop below is unrolled by
  // two), so that every LDS address is a per-lane register plus an immediate offset.
  auto tile_step = [&](int t, bool has_tile, int t_next, bool has_next, auto buf_c) __attribute__((always_inline)) {
    constexpr int buf = decltype(buf_c)::value;
    if (has_next) fetch_tile(t_next, buf ^ 1);
    // causal: of the four tiles on the diagonal of the key block, wavefront w joins from the w-th
    // on, and masks inside that one
    const int i0 = t * QT;
    if (has_tile && (!CAUSAL || i0 >= kw0)) {
      const T* Qt = Qs0 + buf * QT * D;
      const T* Gt = Gs0 + buf * QT * D;
      // ---- S = Q K^T and dP = dO V^T (32 queries x 32 keys each) as one stream of alternating
      // MFMAs: consecutive instructions write different accumulators.  dP starts from -D; its
      // second operand (the V fragments) comes from LDS too.
      f32x16 s, dp;
      {
        auto qfrag = [&](int kk) { return *(const T8*)(Qt + lds_off<D>(r, 2 * kk + g)); };
        auto gfrag = [&](int kk) { return *(const T8*)(Gt + lds_off<D>(r, 2 * kk + g)); };
        auto vfrag = [&](int kk) { return *(const T8*)(Vb + lds_off<D>(wave * 32 + r, 2 * kk + g)); };
        constexpr int PF2 = 2;
        T8 rq[PF2], rg[PF2], rv[PF2];
#pragma unroll
        for (int f = 0; f < PF2; ++f) { rq[f] = qfrag(f); rg[f] = gfrag(f); rv[f] = vfrag(f); }
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          // (with dropout -D joins after the mask: the product starts from zero)
          f32x4 c4 = {0.f, 0.f, 0.f, 0.f};
          if constexpr (!DROPOUT) c4 = *(const f32x4*)(Ds0 + 64 * buf + 8 * i4 + 4 * g);
#pragma unroll
          for (int e = 0; e < 4; ++e) { dp[4 * i4 + e] = c4[e]; s[4 * i4 + e] = 0.f; }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < KK; ++f) {
          const T8 cq = rq[f % PF2], cg = rg[f % PF2], cv = rv[f % PF2];
          s = mfma32(cq, kf[f], s);
          dp = mfma32(cg, cv, dp);
          if (f + PF2 < KK) { rq[f % PF2] = qfrag(f + PF2); rg[f % PF2] = gfrag(f + PF2); rv[f % PF2] = vfrag(f + PF2); }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // hidden entries get the logit -inf, hence P = 0: above the diagonal (one tile per wavefront) or padded keys
      if ((CAUSAL && i0 == kw0) || kw0 + 32 > len) {
        const int first_query = kj < len ? (CAUSAL ? kj : 0) : 0x7fffffff;   // that sees this lane's key
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (i0 + 8 * (i >> 2) + 4 * g + (i & 3) < first_query) s[i] = -INFINITY;
      }
      uint32_t kept = 0;   // dropout: the keep flags of this lane's key for the tile's queries it holds
      if constexpr (DROPOUT) kept = keep.draw<1>(i0, kw0, bh, a.offset_lo, a.seed_lo, a.seed_hi);
      T8 pf[2], dsf[2];
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const f32x4 l4 = *(const f32x4*)(Ls0 + 64 * buf + 8 * i4 + 4 * g);
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DROPOUT) {
          d4 = *(const f32x4*)(Ds0 + 64 * buf + 8 * i4 + 4 * g);   // -D_i
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = 4 * i4 + e;
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], c, -l4[e]));
          if constexpr (DROPOUT) {
            const uint32_t mask = KeepLK::mask(kept, 1, i4, e);
            pf[i4 >> 1][4 * (i4 & 1) + e] = (T)keep_or_zero(p, mask);
            dsf[i4 >> 1][4 * (i4 & 1) + e] = (T)(p * dropped_dp_minus_d(dp[i], a.keep_scale, mask, d4[e]));
          } else {
            pf[i4 >> 1][4 * (i4 & 1) + e] = (T)p;
            dsf[i4 >> 1][4 * (i4 & 1) + e] = (T)(p * dp[i]);
          }
        }
      }
      // ---- dV^T += dO^T P and dK^T += Q^T dS (contractions over the 32 queries), alternating
      {
        auto gtr = [&](int f) {   // f = DB cc + db
          const T* base = Gt + 16 * (f / DB) * D;
          return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
        };
        auto qtr = [&](int f) {
          const T* base = Qt + 16 * (f / DB) * D;
          return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
        };
        constexpr int PF2 = 2;
        T8 rg[PF2], rq[PF2];
#pragma unroll
        for (int f = 0; f < PF2; ++f) { rg[f] = gtr(f); rq[f] = qtr(f); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 2 * DB; ++f) {
          const T8 cg = rg[f % PF2], cq = rq[f % PF2];
          dv[f % DB] = mfma32(cg, pf[f / DB], dv[f % DB]);
          dk[f % DB] = mfma32(cq, dsf[f / DB], dk[f % DB]);
          if (f + PF2 < 2 * DB) { rg[f % PF2] = gtr(f + PF2); rq[f % PF2] = qtr(f + PF2); }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    wait_async_copies();
    __syncthreads();
  };
  const std::integral_constant<int, 0> buf0;
  const std::integral_constant<int, 1> buf1;
  if constexpr (SPARSE) {
    while (more) {
      const int t = 2 * mine;
      const bool has = KG == 1 || mine >= 0;
      tile_step(t, has, t + 1, has, buf0);
      more = it.template next_of<KG>(group, mine);
      tile_step(t + 1, has, 2 * mine, mine >= 0, buf1);
    }
  } else {
    for (int t0 = first; t0 < limit; t0 += 2 * KG) {   // (the same number of steps in every group)
      const int t = t0 + group;
      tile_step(t, KG == 1 || t < limit, t + KG, t + KG < limit, buf0);
      if (t0 + KG < limit) tile_step(t + KG, KG == 1 || t + KG < limit, t + 2 * KG, t + 2 * KG < limit, buf1);
    }
  }
  if constexpr (KG > 1) {
    // the loop ended on a barrier (or never touched LDS): the groups but the first leave dV, then dK in the buffers
    constexpr int kLanes = 64 * RW;
    static_assert((KG - 1) * DB * 16 * kLanes * 4 <= (int)sizeof(all), "LDS holds one gradient of the groups");
    f32x4* const part = (f32x4*)all + wave * 64 + (SPARSE ? lane_id_here() : lane);
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      f32x16 (&x)[DB] = which == 0 ? dv : dk;
      if (which == 0) wait_async_copies();   // (the V rows, where the loop did not run)
      __syncthreads();
      if (group > 0) {
#pragma unroll
        for (int f = 0; f < 4 * DB; ++f) {
          const int i = 4 * (f % 4);
          const f32x4 v = {x[f / 4][i], x[f / 4][i + 1], x[f / 4][i + 2], x[f / 4][i + 3]};
          part[((group - 1) * 4 * DB + f) * kLanes] = v;
        }
      }
      __syncthreads();
      if (group == 0) {
#pragma unroll
        for (int k = 0; k < KG - 1; ++k)
#pragma unroll
          for (int f = 0; f < 4 * DB; ++f) {
            const f32x4 v = part[(k * 4 * DB + f) * kLanes];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[f / 4][4 * (f % 4) + e] += v[e];
          }
      }
    }
    if (!SPARSE && group > 0) return;
    if (list_mode) __syncthreads();   // the sums are staged over what the groups left
  }
  if (KG > 1 && group > 0) {
    // (merged)
  } else if (list_mode) {
    // one of several segments of this column: sum in fp32; the last of them converts.  32 x 128 floats per wavefront
    static_assert(!SPARSE || (RW == 4 && 4 * 32 * D * 4 <= (int)sizeof(all)), "LDS stages a gradient in fp32");
    float* stage = (float*)all + wave * 32 * D;
    const int64_t acc_row0 = ((int64_t)slot * 128 + (kw0 - kt * 128)) * D;
    atomic_add_rows_coalesced<D>(stage, a.dVacc + acc_row0, dv, DROPOUT ? a.keep_scale : 1.f);
    atomic_add_rows_coalesced<D>(stage, a.dKacc + acc_row0, dk, a.tau);
  } else {
    // 4 wavefronts x 32 rows x 128 = 32 KB per gradient: the V block, then the four tile buffers
    T* stage_v = Vb + wave * 32 * D;
    const int out_lane = SPARSE ? lane_id_here() : (int)(threadIdx.x & 63);
    store_rows_coalesced<T, D>(stage_v, (T*)a.dV + head_off + (int64_t)kw0 * a.sn, a.sn, dv,
                               DROPOUT ? a.keep_scale : 1.f, a.N - kw0, D, out_lane);
    __builtin_amdgcn_wave_barrier();
    store_rows_coalesced<T, D>(stage_v, (T*)a.dK + head_off + (int64_t)kw0 * a.sn, a.sn, dk, a.tau, a.N - kw0, D, out_lane);
  }
  if (!list_mode) return;
  if constexpr (SPARSE) sparse_finish<T, D>(item);
  __syncthreads();   // LDS is reused by the next segment
  }  // for round
}

template <typename T, int RW, int KG>
int launch_t(const KArgs& a_in, bool causal, bool dropout, bool sparse, int extra_groups, hipStream_t s) {
  KArgs a = a_in;
  const int blocks = RW == 4 ? a.T : (a.N + 32 * RW - 1) / (32 * RW);
  a.n_items = a.B * a.H * blocks;
  a.chunk = (a.n_items + kXcds - 1) / kXcds;
  a.group = causal_group(a, D, sparse, false, 2 * (int64_t)a.N * D * (int64_t)sizeof(T));   // Q and dO
  if (causal && !sparse) whole_levels(a, D, false, blocks);
  const dim3 grid(kXcds * a.chunk + (sparse ? extra_groups : 0)), block(64 * RW * KG);
#define ATTN_DKV_FR128_CASE(C, P, S)                                                            \
  if constexpr (!S || RW == 4)                                                                  \
    if (causal == C && dropout == P && sparse == S) {                                           \
      hipLaunchKernelGGL((dkv_fr128_kernel<T, C, P, S, RW, KG>), grid, block, 0, s, a);         \
      return (int)hipGetLastError();                                                            \
    }
  ATTN_DKV_FR128_CASE(false, false, false)
  ATTN_DKV_FR128_CASE(true, false, false)
  ATTN_DKV_FR128_CASE(false, true, false)
  ATTN_DKV_FR128_CASE(true, true, false)
  ATTN_DKV_FR128_CASE(false, false, true)
  ATTN_DKV_FR128_CASE(true, false, true)
  ATTN_DKV_FR128_CASE(false, true, true)
  ATTN_DKV_FR128_CASE(true, true, true)
#undef ATTN_DKV_FR128_CASE
  return (int)hipErrorInvalidValue;
}

template <typename T>
int launch_groups(const KArgs& a, const WaveGroups& w, bool causal, bool dropout, bool sparse, int extra_groups, hipStream_t s) {
  if (w.waves == 2 && w.groups == 4) return launch_t<T, 2, 4>(a, causal, dropout, sparse, extra_groups, s);
  if (w.waves == 2) return launch_t<T, 2, 2>(a, causal, dropout, sparse, extra_groups, s);
  if (w.groups == 2) return launch_t<T, 4, 2>(a, causal, dropout, sparse, extra_groups, s);
  return launch_t<T, 4, 1>(a, causal, dropout, sparse, extra_groups, s);
}

}  // namespace

// us of the backward pass with {4, 1}, and the difference with {4, 2} | {2, 2} | {2, 4} (wavefronts of keys, groups) in this kernel
// alone; heads x N:
//   no mask  1 x 128 17.4 +1.1 +0.3 +3.2; 16 x 197 23.8 +0.3 -1.0 +1.5; 4 x 512 36.5 -2.4 -4.8 -3.7; 16 x 1024 60.8 -5.4 -9.6 -7.4; 8 x 2048 109 -14 -23 -23;
//            1 x 8192 399 -72 -101 -136; 96 x 197 26.0 +0.4 +7.6 +17.1; 60 x 300 30.2 -0.7 +7.7 +15.9; 24 x 1024 62.5 -4.5 +10.2 +13.1; 8 x 4096 220 -15 +20 +9;
//            40 x 1024 93.6 +7.3 +16.3 +21.6
//   causal   16 x 1024 62.4 -5.5 -9.1 -7.6; 8 x 2048 110 -15 -21 -22; 8 x 4096 213 -23 +6 -9; 40 x 1024 78.3 -2.8 +11.3 +19.4; 10 x 4096 254 +8 +42 +16
//   dropout  8 x 2048 137 -19 -31 -35; 8 x 4096 272 -30 +16 -5; 60 x 512 48.2 -2.7 +8.2 +16.5; 10 x 4096 372 +23 +46 +5
// Vector registers spilled (bytes of scratch per lane): {2, 4} 56 (228), with dropout 69 (280), whose wavefronts hold the copy offsets of twice as many
// rows each; block-sparse {4, 1} 9 to 13 (40 to 56), {4, 2} 18 (76), with dropout 27 (112); the others none.  The figures above include them.
static WaveGroups fr128_groups(const KArgs& a, bool causal, bool sparse, bool divide) {
  if (!divide) return {4, 1};
  const WorkItems w(a, sparse, false);
  if (sparse) return w.of128 <= kComputeUnits / 2 ? WaveGroups{4, 2} : WaveGroups{4, 1};
  if (w.of64 <= kComputeUnits && w.tiles >= 4) return w.tiles >= 32 ? WaveGroups{2, 4} : WaveGroups{2, 2};
  // (causal: one workgroup on a compute unit at a time takes the blocks heaviest first, and a heavy one takes half as long; {4, 1} | {4, 2}, us: 8 x 8192 510 | 463,
  // 10 x 4096 226 | 203, 30 x 2048 153 | 145, 36 x 1300 88.5 | 84.7, 48 x 900 67.9 | 65.5, 64 x 1024 with dropout 101 | 99; 128 x 512 62 | 67)
  if (causal && w.of128 <= 2 * kComputeUnits && w.tiles >= 14) return {4, 2};
  return w.of128 <= kComputeUnits && w.tiles >= 5 ? WaveGroups{4, 2} : WaveGroups{4, 1};
}

int launch_dkv_fr128(const KArgs& a, int dtype, bool causal, bool dropout, bool sparse, int extra_groups, bool divide, hipStream_t s) {
  const WaveGroups w = fr128_groups(a, causal, sparse, divide);
  return dtype == 0 ? launch_groups<_Float16>(a, w, causal, dropout, sparse, extra_groups, s)
                    : launch_groups<__bf16>(a, w, causal, dropout, sparse, extra_groups, s);
}

}  // namespace attn
