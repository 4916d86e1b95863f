// Backward pass of IO-aware exact attention for gfx950 (MI355X).
//
// The arithmetic is Algorithm 4 of the paper (Appendix B.4): S and P are recomputed tile by
// tile from Q, K, V and the saved row statistic, the dropout mask is regenerated from the
// counter-based generator, D_i = rowsum(dO_i o O_i) replaces the row reduction over P o dP
// (Eq. (4), Appendix B.2), and
//     dV = P_dropped^T dO,  dP = (dO V^T) o Z,  dS = P o (dP - D),  dQ = tau dS K,  dK = tau dS^T Q.
// The schedule differs from the paper's single K/V-outer loop with dQ read-modify-written in
// HBM: two launches, neither of which writes a partial result to HBM.
//   1. dq_kernel     : a workgroup owns 128 query rows and sweeps K/V tiles; dQ stays in
//                      registers (S^T, dP^T layout: lane = query, like the forward kernel).  It
//                      also computes D = rowsum(dO o O) of its rows and leaves -D and L in base 2
//                      in the scratch vectors for the second launch.
//   2. dK/dV kernel (attn_bwd_dkv.hip, attn_bwd_dkv_fr.hip): a workgroup owns 128 keys and
//                      sweeps Q/dO tiles; dK, dV stay in registers (S, dP layout: lane = key)
// S and dP are therefore recomputed in both launches (seven tile products per (i, j) instead of
// five) in exchange for no atomics, no fp32 dQ round trip and bit-reproducible gradients.
#include "attn_common.h"
#include "attn_sparse.h"
#include "attn_tiles.h"

#include <cstdlib>

namespace attn {
namespace {

constexpr int TILE = 64;  // keys of the streamed tile

// ---------------------------------------------------------------------------------------------
// dQ: workgroup = 128 query rows (4 wavefronts x 32), sweep over 64-key tiles.
// d <= 32, plain or block-sparse: latency binds it, and the accumulators leave room for three wavefronts per SIMD
// instead of two (168 registers, without spills with operand reads two fragments ahead instead of four).
// us, before -> after: B H = 128, N = 700 33.0 -> 30.1, B H = 64, N = 4096 253 -> 239, B H = 2048, N = 128 31.7 -> 30.4,
// d = 16, B H = 128, N = 1024 43.0 -> 39.3, block-sparse N = 16384 55.8 -> 52.2.  The causal and dropout forms have the
// three by themselves at d = 32; at d = 64 three cost more in spills or half tiles (B H = 128, N = 2048 210 -> 211, N = 128 54 -> 62).
constexpr bool three_waves(int d, bool causal, bool dropout) { return d == 32 && !causal && !dropout; }

// RW wavefronts of 32 query rows, times KG groups of them that each take every KG-th tile (as in the forward kernel): the groups'
// dQ are summed through LDS at the end.
template <typename T, int D, bool CAUSAL, bool DROPOUT, bool SPARSE, int RW, int KG>
__global__ __launch_bounds__(64 * RW * KG, KG == 1 && three_waves(D, CAUSAL, DROPOUT) ? 3 : 2) void dq_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  constexpr int KK = D / 16, DB = D / 32;
  // K and V tiles, double buffered, filled by async copies.  Without the causal mask they form one
  // LDS block (K tile of buffer b at b TILE D, V tile at (2 + b) TILE D), so that an LDS address
  // is a per-lane register plus an immediate offset once the buffer index is a compile-time
  // constant (see tile_step below); the causal kernels, which cannot afford that unrolling, keep
  // two arrays (the form that the register allocator handles without spilling).
  constexpr int BR = 32 * RW;
  T* Ks0;
  T* Vs0;
  T* all;   // the LDS of all groups, one block (KG > 1)
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / RW;
  if constexpr (!CAUSAL || KG > 1) {
    __shared__ __attribute__((aligned(16))) T smem[KG * 4 * TILE * D];
    all = smem;
    Ks0 = smem + group * 4 * TILE * D;
    Vs0 = Ks0 + 2 * TILE * D;
  } else {
    __shared__ __attribute__((aligned(16))) T Ks[2 * TILE * D];
    __shared__ __attribute__((aligned(16))) T Vs[2 * TILE * D];
    Ks0 = Ks;
    Vs0 = Vs;
    all = Ks;
  }

  if constexpr (!SPARSE) args_at_once(a);
  if constexpr (SPARSE) {
    // the first workgroups plan the dK/dV launch (a multiple of the XCD count of them)
    if ((int)blockIdx.x < a.plan_groups) {
      sparse_plan<D>(a, (int)blockIdx.x, CAUSAL, (int*)all);
      return;
    }
  }
  constexpr bool DEALT = CAUSAL && !SPARSE;   // see causal_block
  const int item = DEALT ? causal_item(a) : xcd_item(a.n_items, a.chunk, SPARSE ? (int)blockIdx.x - a.plan_groups : (int)blockIdx.x);
  if (item < 0) return;
  const int n_qt = a.T * (4 / RW);   // blocks of BR rows, to the end of the last 128-row block: the scratch vectors are written whole
  // Work item = (head, row block); under the causal mask row block q sweeps 2 (q + 1) key tiles, and the late blocks come first
  int bh = item / n_qt, q_item = item % n_qt;
  if constexpr (CAUSAL)
    if (!causal_block(a, item, n_qt, bh, q_item)) return;
  if (!SPARSE && !(DEALT && a.group <= 0)) bh = dealt_head(a, bh);
  const int qt = CAUSAL ? n_qt - 1 - q_item : q_item;
  // (one pass of a loop: the form in which the {2, 2} kernels of d = 32 stay within the 168 registers of three wavefronts per SIMD without being held to them;
  // straight on they take 182, with dropout 174, and held to 168 they spill.  dQ in us, straight | so: 100 heads of 300 13.9 | 11.3, 80 of 400 15.3 | 12.7, 8 of 5000 72.9 | 59.1,
  // with dropout 100 of 300 15.8 | 13.9)
#pragma clang loop unroll(disable)
  for (int pass = 0; pass < 1; ++pass) {
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const T* __restrict__ Kg = (const T*)a.K + head_off;
  const T* __restrict__ Vg = (const T*)a.V + head_off;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - RW * group;   // in a scalar register: addresses and branches on it are scalar
  const int r = lane & 31, g = lane >> 5;
  const int q0 = qt * BR + wave * 32;
  // lanes beyond a ragged end work on a copy of the last row with P = 0 and store nothing
  const bool row_ok = q0 + r < a.N;
  const int qi = min(q0 + r, a.N - 1);

  T8 qf[KK], gf[KK];  // Q^T and dO^T fragments (B operands) of this lane's query
  // -D_i = -sum_d dO[i][d] O[i][d] (Eq. (4), Appendix B.2), from the same 8-element pieces of the row
  // that the dO fragments hold: this lane's half of the sum, completed with the partner lane below
  float d_part = 0.f;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int64_t off = head_off + (int64_t)qi * a.sn + 16 * kk + 8 * g;
    if (D == 32 && 16 * kk + 8 * g >= a.dvalid) {   // head dimension 16: the upper columns are zeros
#pragma unroll
      for (int e = 0; e < 8; ++e) { qf[kk][e] = (T)0.f; gf[kk][e] = (T)0.f; }
      continue;
    }
    qf[kk] = *(const T8*)((const T*)a.Q + off);
    gf[kk] = *(const T8*)((const T*)a.dO + off);
    if (a.o_fp32) {
      const f32x4 o0 = *(const f32x4*)((const float*)a.O + off);
      const f32x4 o1 = *(const f32x4*)((const float*)a.O + off + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) d_part += (float)gf[kk][e] * o0[e] + (float)gf[kk][4 + e] * o1[e];
    } else {
      const T8 o = *(const T8*)((const T*)a.O + off);
#pragma unroll
      for (int e = 0; e < 8; ++e) d_part += (float)gf[kk][e] * (float)o[e];
    }
  }
  const float lse = a.LSE[(int64_t)bh * a.N + qi];
  // base-2 statistic; a row that saw no key (or lies beyond a ragged end) has P = 0 everywhere
  const float l2 = (lse == -INFINITY || !row_ok) ? INFINITY : lse * 1.4426950408889634f;
  const float neg_d = row_ok ? -(d_part + xchg32(d_part)) : 0.f;   // -D_i
  // The dK/dV kernel reads both per 64-row tile from the scratch vectors (padded to whole blocks
  // of 128 rows per head: this workgroup writes all of its block).  The tile kernels start
  // their dP accumulators from -D, so that dP - D needs no instruction of its own.
  if (g == 0 && (KG == 1 || group == 0)) {
    a.Dvec[(int64_t)bh * a.Nr + q0 + r] = neg_d;
    a.L2vec[(int64_t)bh * a.Nr + q0 + r] = l2;
  }

  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) dq[db][i] = 0.f;

  // key-padding mask: keys >= len contribute nothing (rows >= len have LSE = -inf, hence P = 0)
  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  TileIter<SPARSE> it;
  {
    int lim;
    const int mask_row = qt * BR / 128;
    if constexpr (SPARSE) lim = min(CAUSAL ? mask_row + 1 : a.T, (len + 127) / 128);
    else lim = CAUSAL ? min((qt + 1) * BR / TILE, (len + TILE - 1) / TILE) : (len + TILE - 1) / TILE;   // len <= N
    if (qt * BR >= len) lim = 0;
    it.init(SPARSE ? a.mask + (int64_t)h * a.mask_sh + (int64_t)mask_row * a.T : nullptr, 1, 0, lim);
  }
  TrOffsets<D> tro;
  tro.init();
  TileAsync<T, D, RW> dma;
  dma.init(a.sn, wave, D == 32 ? a.dvalid : D);
  if (D == 32 && a.dvalid < D) {   // the copies leave columns >= 16 of the tile buffers untouched
    if constexpr (KG > 1) {
      zero_tiles(all, KG * 4 * TILE * D);
    } else {
      zero_tiles(Ks0, 2 * TILE * D);
      zero_tiles(Vs0, 2 * TILE * D);
    }
    __syncthreads();
  }

  const float c = a.scale_log2;
  // jt: this group's tile, -1 if there is none; more: some group (then the first) has one
  int jt;
  bool more = it.template next_of<KG>(group, jt);
  if (jt >= 0) {
    dma.copy_rows(Kg, a.sn, jt * TILE, a.N, Ks0);
    dma.copy_rows(Vg, a.sn, jt * TILE, a.N, Vs0);
  }
  wait_async_copies();
  __syncthreads();   // tile 0 has landed, and so have the Q / dO fragments
  // Without the causal mask the tile loop is unrolled by two, so that the buffer index is a
  // constant in each copy of its body; the causal kernels have no registers for two copies.
  constexpr int UNROLL = CAUSAL ? 1 : 2;
  int buf_rt = 0;
  while (KG == 1 ? jt >= 0 : more) {
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int buf = UNROLL == 2 ? u : buf_rt;
    int jn;
    const bool more_next = it.template next_of<KG>(group, jn);
    if (jn >= 0) {   // next tile streams into the other buffer while this one is used
      dma.copy_rows(Kg, a.sn, jn * TILE, a.N, Ks0 + (buf ^ 1) * TILE * D);
      dma.copy_rows(Vg, a.sn, jn * TILE, a.N, Vs0 + (buf ^ 1) * TILE * D);
    }
    const T* Kt = Ks0 + buf * TILE * D;
    const T* Vt = Vs0 + buf * TILE * D;

    const int k0 = jt * TILE;
    if ((KG == 1 || jt >= 0) && (!CAUSAL || k0 <= q0 + 31)) {
      f32x16 s[2], dp[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          s[kb][i] = 0.f;
          // every accumulator element of a lane belongs to the lane's query: without dropout the
          // product starts from -D_i and ends as dP - D
          dp[kb][i] = DROPOUT ? 0.f : neg_d;
        }
      // S^T = K Q^T and dP^T = V dO^T as one stream of 4 KK MFMAs; operand reads run PF fragments
      // ahead of their MFMA (the scheduling barriers keep that distance)
      constexpr int PF = three_waves(D, CAUSAL, DROPOUT) ? 2 : 4;
      auto kv_frag = [&](int f) {   // f = 4 kk + 2 kb + (0: K, 1: V)
        const int off = lds_off<D>(32 * ((f >> 1) & 1) + r, 2 * (f >> 2) + g);
        return *(const T8*)(((f & 1) ? Vt : Kt) + off);
      };
      {
        T8 ring[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) ring[f] = kv_frag(f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 4 * KK; ++f) {
          const T8 cur = ring[f % PF];
          const int kk = f >> 2, kb = (f >> 1) & 1;
          if (f & 1) dp[kb] = mfma32(cur, gf[kk], dp[kb]);
          else s[kb] = mfma32(cur, qf[kk], s[kb]);
          if (f + PF < 4 * KK) ring[f % PF] = kv_frag(f + PF);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // hidden keys get the logit -inf, hence P = 0: beyond the causal diagonal (tiles that cross it only:
      // a comparison and a select per element on every tile were two fifths of the vector instructions;
      // B H = 64, N = 4096, d = 128: 413 -> 383 us, B H = 128, N = 2048, d = 64: 146 -> 134 us) or padded
      if ((CAUSAL && k0 + TILE - 1 > q0) || k0 + TILE > len) {
        const int last = CAUSAL ? min(qi, len - 1) : len - 1;   // last visible key of this row
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (k0 + 32 * kb + 8 * (i >> 2) + 4 * g + (i & 3) > last) s[kb][i] = -INFINITY;
      }
      // P = exp(S - L); dS = P o (dP o Z - D)
      KeepLQ kq = {};
      if constexpr (DROPOUT) kq = keep_tile_lane_query(k0, qi, bh, g, a.offset_lo, a.seed_lo, a.seed_hi);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * i4 + e;
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][i], c, -l2));
            float dpv = dp[kb][i];
            if constexpr (DROPOUT)   // Z dP - D with Z = keep_scale or 0 by the 8-bit draw of this element
              dpv = dropped(kq.w[kb][i4], e, a.drop_thr) ? neg_d : __builtin_fmaf(dpv, a.keep_scale, neg_d);
            s[kb][i] = p * dpv;
          }
        }
      T8 dsf[4];
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int t = 0; t < 8; ++t) dsf[cc][t] = (T)s[cc >> 1][8 * (cc & 1) + t];
      // dQ^T += K^T dS^T
      auto kt_frag = [&](int f) {   // f = DB cc + db: consecutive MFMAs hit different accumulators
        const T* base = Kt + 16 * (f / DB) * D;
        return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
      };
      {
        T8 ring[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) ring[f] = kt_frag(f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 4 * DB; ++f) {
          const T8 cur = ring[f % PF];
          dq[f % DB] = mfma32(cur, dsf[f / DB], dq[f % DB]);
          if (f + PF < 4 * DB) ring[f % PF] = kt_frag(f + PF);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    wait_async_copies();
    __syncthreads();   // next tile has landed, and everyone is done with this buffer
    jt = jn;
    more = more_next;
    buf_rt ^= 1;
    if (KG == 1 ? jt < 0 : !more) break;
  }
  }
  if constexpr (KG > 1) {
    // the loop ended on a barrier (or never touched LDS): the groups but the first leave their dQ in the tile buffers
    constexpr int kLanes = 64 * RW;
    static_assert((KG - 1) * DB * 16 * kLanes * 4 <= KG * 4 * TILE * D * (int)sizeof(T), "LDS holds the groups' dQ");
    f32x4* const part = (f32x4*)all + wave * 64 + lane;
    if (group > 0) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x4 v = {dq[db][4 * i4], dq[db][4 * i4 + 1], dq[db][4 * i4 + 2], dq[db][4 * i4 + 3]};
          part[((group - 1) * 4 * DB + 4 * db + i4) * kLanes] = v;
        }
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int k = 0; k < KG - 1; ++k)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4) {
            const f32x4 v = part[(k * 4 * DB + 4 * db + i4) * kLanes];
#pragma unroll
            for (int e = 0; e < 4; ++e) dq[db][4 * i4 + e] += v[e];
          }
    }
    __syncthreads();   // the buffers stage the output rows
    if (group > 0) return;
  }
  // the loop ends on a barrier (or never touched LDS): the tile buffers stage the output rows
  T* stage = (wave < 2 ? Ks0 + wave * 32 * D : Vs0 + (wave - 2) * 32 * D);
  store_rows_coalesced<T, D>(stage, (T*)a.dQ + head_off + (int64_t)q0 * a.sn, a.sn, dq, a.tau, a.N - q0,
                             D == 32 ? a.dvalid : D);
  }  // for pass
}

template <typename T, int D, int RW, int KG>
int launch_dq(KArgs a, bool causal, bool dropout, bool sparse, hipStream_t s) {
  const int blocks = a.T * (4 / RW);
  a.n_items = a.B * a.H * blocks;
  a.chunk = (a.n_items + kXcds - 1) / kXcds;
  a.group = causal_group(a, D, sparse, false, 2 * (int64_t)a.N * D * (int64_t)sizeof(T));
  if (causal && !sparse) whole_levels(a, D, false, blocks);
  if (sparse) a.plan_groups = sparse_plan_groups(a);
  const dim3 grid(kXcds * a.chunk + (sparse ? a.plan_groups : 0)), block(64 * RW * KG);
#define ATTN_DQ_CASE(C, P, S)                                                          \
  if (causal == C && dropout == P && sparse == S) {                                    \
    hipLaunchKernelGGL((dq_kernel<T, D, C, P, S, RW, KG>), grid, block, 0, s, a);      \
    return (int)hipGetLastError();                                                     \
  }
  ATTN_DQ_CASE(false, false, false)
  ATTN_DQ_CASE(true, false, false)
  ATTN_DQ_CASE(false, true, false)
  ATTN_DQ_CASE(true, true, false)
  ATTN_DQ_CASE(false, false, true)
  ATTN_DQ_CASE(true, false, true)
  ATTN_DQ_CASE(false, true, true)
  ATTN_DQ_CASE(true, true, true)
#undef ATTN_DQ_CASE
  return (int)hipErrorInvalidValue;
}

template <typename T> constexpr int kDtype = 0;
template <> constexpr int kDtype<__bf16> = 1;

}  // namespace

// us of the backward pass with {4, 1}, and the difference with {4, 2} | {2, 2} | {2, 4} (wavefronts of rows, groups) in this kernel
// alone; heads x N:
//   d = 64   1 x 128 12.3 +1.2 -0.3 +1.3; 16 x 197 17.7 +0.6 -1.3 +0.1; 4 x 512 25.0 -0.3 -2.8 -1.9; 16 x 1024 41.0 -2.0 -5.2 -5.1; 8 x 2048 72.2 -5.3 -10.2 -11.6;
//            1 x 8192 263 -28 -48 -61; 60 x 512 26.5 -0.1 +0.5 +6.2; 24 x 1024 42.0 -2.0 -1.2 +4.5; 8 x 4096 140 -8.7 -5.5 -0.8;
//            10 x 4096 186 +10.1 -1.3 +2.6, dropout 271 +9.5 -15.9 -7.3; 24 x 2001 110 +6.1 -2.1 +4.9; 40 x 1024 57.1 +5.8 +0.9 +8.1; 32 x 2048 116 +3.6 +4.8 +16.8
//   d = 64 causal (the other kernel as its rule has it)  16 x 1024 33.7 -2.1 -5.8 -5.8; 8 x 4096 105 -12.1 -17.6 -20.5; 13 x 2382 73.9 -8.0 -10.9 -8.3; 40 x 1024 42.0 -1.9 -1.1 +6.2;
//            10 x 4096 119 -13.8 -19.0 -9.0; 32 x 2048 82.2 -3.1 0 +11.3; 128 x 512 38.1 +3.1 +3.0 +15.4; 46 x 661 32.8 +0.6 -1.8 +4.2; 52 x 694 with dropout 43.5 +0.4 -2.1 +7.4; 61 x 575 30.7 +3.0
//            +1.8 +10.8; 25 x 1470 with dropout 74.7 -5.6 -8.9 +3.0; 15 x 2832 with dropout 132 -11.1 -17.8 -4.6; 60 x 1000 49.9 +1.9 +2.2 -; 51 x 1200 58.0 +2.5 +4.5 -; 50 x 1000 47.4 +1.4 +1.4 -
//   d = 32   1 x 128 10.0 -0.4 -0.4 +0.1; 16 x 640 22.6 -1.0 -2.6 -2.6; 8 x 2048 56.2 -3.8 -8.0 -10.0; 60 x 512 20.1 -0.7 -0.7 +2.1; 8 x 4096 107 -8.3 -8.1 -4.9;
//            10 x 4096 138 +8.1 -12.7 -2.7; 24 x 2001 81.7 +5.3 -5.1 +1.9; 64 x 1024 43.1 +3.1 +0.9 +8.8
//   d = 128  1 x 128 17.4 +2.5 +0.2; 16 x 640 42.5 +0.9 -2.4; 8 x 2048 130 -3.5 -9.1; 1 x 8192 474 -26 -45; 60 x 512 41.5 +2.5 +9.7;
//            16 x 2048 136 -1.5 +18.3; 8 x 4096 253 -5.1 +28.4, causal 213 -6.0 +23.5, dropout 272 -8.3 +30.0; 40 x 1024 93.6 +10.1 +18.4
//   (d = 128 without the causal mask spills one vector register in every form of 4 wavefronts of rows)
//   block-sparse (butterfly mask of T x T blocks, heads x T)  d = 64  4 x 8 48.2 -1.5 -4.2 -4.0; 4 x 32 65.7 -1.8 -4.4 -4.4; 4 x 64 76.0 -2.0 -1.4 +7.0;
//            8 x 64 112 +5.8 +6.2 +24.1; d = 128  4 x 32 89.9 -0.3 -4.4; 4 x 64 132 +0.3 +17.4
WaveGroups dq_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide) {
  if (!divide) return {4, 1};
  const bool halves = causal && !sparse && d == 64;
  const WorkItems w(a, sparse, halves);
  if (w.of64 <= kComputeUnits && w.tiles >= 4) return d <= 64 && w.tiles >= (d == 64 ? 24 : 12) && !sparse ? WaveGroups{2, 4} : WaveGroups{2, 2};
  // (causal, now | {2, 2}: d = 32 32 x 2048 58.5 54.7, 60 x 1000 with dropout
  // 50.8 48.8, 128 x 700 33.7 35.9; 8 x 4096 {2, 2} 64.8, {2, 4} 58.7, 10 x 4096 69.7, 74.9)
  if (halves && w.of64 <= 11 * kComputeUnits / 8 && w.tiles >= 11) return {2, 2};
  if (d == 32 && causal && !sparse && w.of64 <= 2 * kComputeUnits && w.tiles >= 32) return {2, 4};
  // (three workgroups fit; causal, a fourth round of light blocks, {4, 1} | {2, 2}: 9 tiles and more 100 x 576 with dropout 36.0 34.9, 53 x 1000 35.6 33.7, 27 x 2048 55.4 47.6, 32 x 2048 57.5 52.8; fewer
  // 152 x 310 20.0 19.4, 158 x 310 21.9 22.8, 204 x 310 20.9 23.1, 150 x 380 23.6 25.7, 160 x 324 with dropout 28.3 28.3, 170 x 380 with dropout 31.3 32.5, 120 x 512 23.8 25.4)
  if (d == 32) return w.of64 <= (causal && !sparse && w.tiles >= 9 ? 4 : 3) * kComputeUnits && w.tiles >= 4 ? WaveGroups{2, 2} : WaveGroups{4, 1};
  if (w.of128 <= (halves && w.tiles < 24 ? 3 : 4) * kComputeUnits / 4 && w.tiles >= (d == 64 ? 16 : 24)) return {4, 2};
  // (causal, two blocks in turn on a compute unit, heaviest first; {4, 1} | {4, 2}, us: 8 x 8192 511 | 485, 10 x 4096 226 | 214, 20 x 2000 with dropout 151 | 140;
  // 30 x 2048 151 | 152, 48 x 900 67.6 | 73.2)
  if (d == 128 && causal && !sparse && w.of128 <= (w.tiles >= 64 ? 2 : 3 / 2.) * kComputeUnits && w.tiles >= 24) return {4, 2};
  if (d == 64 && !halves && w.of64 > 2 * kComputeUnits && w.of64 <= 3 * kComputeUnits && w.tiles >= 24) return {2, 2};
  return {4, 1};
}

namespace {

template <typename T, int D>
int launch_dq_td(const KArgs& a, bool causal, bool dropout, bool sparse, bool divide, hipStream_t s) {
  const WaveGroups w = dq_groups(a, D, causal, sparse, divide);
  if constexpr (D <= 64)
    if (w.waves == 2 && w.groups == 4) return launch_dq<T, D, 2, 4>(a, causal, dropout, sparse, s);
  if (w.waves == 2) return launch_dq<T, D, 2, 2>(a, causal, dropout, sparse, s);
  if constexpr (D >= 64)
    if (w.groups == 2) return launch_dq<T, D, 4, 2>(a, causal, dropout, sparse, s);
  return launch_dq<T, D, 4, 1>(a, causal, dropout, sparse, s);
}

template <typename T, int D>
int launch_bwd_td(const KArgs& a, bool causal, bool dropout, bool sparse, const Overrides& v, hipStream_t s, hipEvent_t* ev) {
  const int choice = choose_dkv(a, D, causal, dropout, sparse, v);
  const bool divide = may_divide(v);
  if (ev) (void)hipEventRecord(ev[0], s);
  if (ev) (void)hipEventRecord(ev[1], s);   // (there is no separate preparation launch any more)
  int e;
  if (choice == kBwdShort) {
    e = launch_bwd_short(a, kDtype<T>, D, causal, dropout, s);
    if (ev) (void)hipEventRecord(ev[2], s);
    if (ev) (void)hipEventRecord(ev[3], s);
    return e;
  }
  e = launch_dq_td<T, D>(a, causal, dropout, sparse, divide, s);
  if (e != 0) return e;
  if (ev) (void)hipEventRecord(ev[2], s);
  e = launch_dkv(a, kDtype<T>, D, causal, dropout, sparse, choice, divide, s);
  if (ev) (void)hipEventRecord(ev[3], s);
  return e;
}

}  // namespace

int launch_bwd(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, const Overrides& v, hipStream_t s,
               hipEvent_t* ev) {
  if (dtype == 0 && d == 32) return launch_bwd_td<_Float16, 32>(a, causal, dropout, sparse, v, s, ev);
  if (dtype == 1 && d == 32) return launch_bwd_td<__bf16, 32>(a, causal, dropout, sparse, v, s, ev);
  if (dtype == 0 && d == 64) return launch_bwd_td<_Float16, 64>(a, causal, dropout, sparse, v, s, ev);
  if (dtype == 0 && d == 128) return launch_bwd_td<_Float16, 128>(a, causal, dropout, sparse, v, s, ev);
  if (dtype == 1 && d == 64) return launch_bwd_td<__bf16, 64>(a, causal, dropout, sparse, v, s, ev);
  if (dtype == 1 && d == 128) return launch_bwd_td<__bf16, 128>(a, causal, dropout, sparse, v, s, ev);
  return (int)hipErrorInvalidValue;
}

}  // namespace attn
