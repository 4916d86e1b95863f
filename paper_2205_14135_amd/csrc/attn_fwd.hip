// Forward pass of IO-aware exact attention for gfx950 (MI355X).
//
// What is computed is Algorithm 2 of the paper (Appendix B.3): S = tau Q K^T, mask, online
// softmax with running row max m and row sum l, dropout on the unnormalised probabilities,
// O accumulation with rescaling, and the saved statistic L = m + ln l.  The loop order is
// NOT the paper's: a workgroup owns a 128-row Q tile (4 wavefronts x 32 rows), keeps O, m, l
// in registers for the whole sweep over K/V tiles and writes O and L exactly once, so O, m, l
// never travel to HBM between tiles (the paper's K/V-outer order re-reads and re-writes them
// on every pass).  K/V tiles of 64 keys are staged in LDS.
//
// Online softmax, two departures from the printed recurrence that leave the result the same up
// to rounding.  (1) The reference m of a row is moved (and O, l rescaled) only when the sum of a
// tile's probabilities in a lane exceeds kLazySum (or, on tiles that look for it, the maximum exceeds m by kLazyRise):
// any reference gives the same softmax in exact arithmetic, and most tiles then skip both the rescaling of
// the whole O accumulator and the search for the tile's maximum.  (2) O is divided
// by the sum of the probabilities AS ROUNDED to 16 bits for the second product, not by l: O is
// then a convex combination of V rows with exactly the weights that were used, which is what
// keeps a lagging reference accurate (with the exact l a peaked row would see the rounding of its
// one large weight in full).  The saved statistic L = m + ln l uses the exact fp32 l.
//
// Register layout trick: the kernel computes S^T = K Q^T with 32x32x16 MFMA, so that a lane
// holds 16 keys of ONE query (accumulator register i of key block kb is key
// 32 kb + 8 (i/4) + 4 (lane/32) + i%4, query lane%32).  The exact row sum and, where it is looked
// for, the row maximum are then in-lane reductions plus one exchange with lane^32, the sum of the rounded
// probabilities is one small MFMA per fragment (row_sum_ones in attn_common.h), the rescale factor is a per-lane scalar, and the
// probabilities are already in the B-operand layout of the second product O^T = V^T P^T.
// V^T fragments come from the row-major V tile in LDS through the gfx950 transposing LDS read.
#include "attn_common.h"
#include "attn_tiles.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>

namespace attn {
namespace {

constexpr int BC = 64;   // keys per K/V tile

// RW wavefronts of 32 query rows each share the K/V tiles of a workgroup.  KG groups of RW wavefronts work on the same rows: group
// k takes every KG-th tile, into buffers of its own, and the groups' (m, l, O) are merged through LDS at the end.
template <typename T, int D, bool CAUSAL, bool DROPOUT, bool SPARSE, int RW, int KG>
__global__ __launch_bounds__(64 * RW * KG, KG == 1 && D <= 64 ? 3 : 2) void fwd_kernel(const KArgs a) {
  typedef typename Vec<T>::x8 T8;
  typedef typename Vec<T>::x4 T4;
  constexpr int KK = D / 16;        // MFMA k-steps over the head dimension
  constexpr int DB = D / 32;        // 32-row blocks of O^T

  // double buffered, unpadded XOR-swizzled tiles, filled by asynchronous global-to-LDS copies
  constexpr int BR = 32 * RW;       // query rows of the workgroup
  // (two arrays, the form that the register allocation of the ungrouped kernels is tuned to, or one block that the merge can use whole)
  typedef T Tile[BC * D];
  Tile *Ks, *Vs;   // buffers 2 k and 2 k + 1: key group k's
  if constexpr (KG == 1) {
    __shared__ __attribute__((aligned(16))) Tile k_bufs[2], v_bufs[2];
    Ks = k_bufs;
    Vs = v_bufs;
  } else {
    __shared__ __attribute__((aligned(16))) Tile bufs[4 * KG];
    Ks = bufs;
    Vs = bufs + 2 * KG;
  }

  args_at_once(a);
  constexpr bool DEALT = CAUSAL && !SPARSE;   // see causal_block
  const int item = DEALT ? causal_item(a) : xcd_item(a.n_items, a.chunk);
  if (item < 0) return;
  const int n_qt = RW == 4 ? a.T : (a.N + BR - 1) / BR;   // the last block may be ragged
  // Work item = (head, row block); under a causal mask the late blocks, which see most keys, first
  int bh = item / n_qt, q_item = item % n_qt;
  if constexpr (DEALT && D == 32) causal_block<false>(a, item, n_qt, bh, q_item);
  if constexpr (DEALT && D != 32)
    if (!causal_block(a, item, n_qt, bh, q_item)) return;
  if (!SPARSE && !(DEALT && (D == 32 ? a.group == 0 : a.group <= 0))) bh = dealt_head(a, bh);
  const int qt = CAUSAL ? n_qt - 1 - q_item : q_item;
  // (one pass of a loop: the form in which the compiler lays the code out with no jump between the last tile and the epilogue; one head of 128
  // tokens 4.51 -> 4.46 to 4.48 us)
#pragma clang loop unroll(disable)
  for (int pass = 0; pass < 1; ++pass) {
  const int b = bh / a.H, h = bh % a.H;
  const int64_t head_off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const T* __restrict__ Qg = (const T*)a.Q + head_off;
  const T* __restrict__ Kg = (const T*)a.K + head_off;
  const T* __restrict__ Vg = (const T*)a.V + head_off;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / RW;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - RW * group;   // in a scalar register: addresses and branches on it are scalar
  const int r = lane & 31, g = lane >> 5;
  const int q0 = qt * BR + wave * 32;  // first query row of this wavefront
  // this lane's query row; lanes beyond a ragged end work on a copy of the last row and store nothing
  const bool row_ok = q0 + r < a.N;
  const int qi = min(q0 + r, a.N - 1);

  // Q^T fragments (B operand): lane holds query qi, d = 16 kk + 8 g .. +7
  T8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    if (D == 32 && 16 * kk + 8 * g >= a.dvalid) {   // head dimension 16: the upper columns are zeros
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[kk][e] = (T)0.f;
    } else {
      qf[kk] = *(const T8*)(Qg + (int64_t)qi * a.sn + 16 * kk + 8 * g);
    }
  }

  f32x16 o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m_run = -INFINITY;  // reference of the row's probabilities, base-2 domain: lags the running
                            // maximum of the scaled logits by at most log2(kLazySum)
  float l_run = 0.f;        // this lane's share of the exact running row sum (for the saved statistic)
  f32x4 lr_run = {0.f, 0.f, 0.f, 0.f};   // the sum of the rounded probabilities (normalises O), four times the same
  int calm = kFirstTile;   // whether the next tile starts with its maximum: see softmax_tile_lane_query
  const T8 ones = row_sum_ones<T>();

  // key-padding mask: keys >= len are masked, rows >= len produce O = 0, LSE = -inf
  const int len = a.klen ? min(max(a.klen[b], 0), a.N) : a.N;
  TileIter<SPARSE> it;
  {
    int lim;
    const int mask_row = qt * BR / 128;
    if constexpr (SPARSE) lim = min(CAUSAL ? mask_row + 1 : a.T, (len + 127) / 128);
    else lim = CAUSAL ? min((qt + 1) * BR / BC, (len + BC - 1) / BC) : (len + BC - 1) / BC;   // len <= N
    if (qt * BR >= len) lim = 0;
    it.init(SPARSE ? a.mask + (int64_t)h * a.mask_sh + (int64_t)mask_row * a.T : nullptr, 1, 0, lim);
  }

  TrOffsets<D> tro;
  tro.init();
  TileAsync<T, D, RW> dma;
  dma.init(a.sn, wave, D == 32 ? a.dvalid : D);
  if (D == 32 && a.dvalid < D) {   // the copies leave columns >= 16 of the tile buffers untouched
    zero_tiles(&Ks[0][0], 2 * KG * BC * D);
    zero_tiles(&Vs[0][0], 2 * KG * BC * D);
    __syncthreads();
  }

  const float c = a.scale_log2;
  // jt: this group's tile, -1 if there is none; more: some group (then the first) has one
  int jt;
  bool more = it.template next_of<KG>(group, jt);
  int buf = 0;
  if (jt >= 0) {
    dma.copy_rows(Kg, a.sn, jt * BC, a.N, Ks[2 * group]);
    dma.copy_rows(Vg, a.sn, jt * BC, a.N, Vs[2 * group]);
  }
  wait_async_copies();
  __syncthreads();   // tile 0 has landed, and so have the Q fragments
  // the scalar loads of the kernel arguments that the loop uses have completed: one in flight makes the first
  // operand wait of the loop a wait for every LDS read issued so far (scalar loads return out of order)
  asm volatile("" :: "s"(c));
  // byte offsets of this lane's K fragments in a tile, kept whole (derived again on every tile otherwise)
  uint32_t k_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    k_off[kk] = lds_addr(&Ks[2 * group][0]) + (uint32_t)(lds_off<D>(r, 2 * kk + g) * sizeof(T));
    asm volatile("" : "+v"(k_off[kk]));
  }
  while (KG == 1 ? jt >= 0 : more) {
    int jn;
    const bool more_next = it.template next_of<KG>(group, jn);
    if (jn >= 0) {   // the next tile streams into the other buffer while this one is used
      dma.copy_rows(Kg, a.sn, jn * BC, a.N, Ks[2 * group + (buf ^ 1)]);
      dma.copy_rows(Vg, a.sn, jn * BC, a.N, Vs[2 * group + (buf ^ 1)]);
    }
    const T* Vt = Vs[2 * group + buf];

    const int k0 = jt * BC;
    const bool wave_active = (KG == 1 || jt >= 0) && (!CAUSAL || k0 <= q0 + 31);
    if (wave_active) {
      // ---- S^T = K Q^T  (64 keys x 32 queries per wavefront); operand reads run PF fragments
      // ahead of their MFMA (the scheduling barriers keep that distance)
      constexpr int PF = 4;
      f32x16 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] = 0.f;
      {
        auto k_frag = [&](int f) {   // f = 2 kk + kb
          const auto* p = (const __attribute__((address_space(3))) T8*)(k_off[f >> 1] + (uint32_t)(buf * BC * D * sizeof(T)));
          return p[32 * (f & 1) * D / 8];
        };
        T8 ring[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) ring[f] = k_frag(f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 2 * KK; ++f) {
          const T8 cur = ring[f % PF];
          s[f & 1] = mfma32(cur, qf[f >> 1], s[f & 1]);
          if (f + PF < 2 * KK) ring[f % PF] = k_frag(f + PF);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      constexpr bool PACK_LATE = D == 128 || (D == 64 && DROPOUT && !CAUSAL);
      // ---- masks, online softmax, dropout; P^T fragments (B operand) for the second product
      T8 pf[4];
      softmax_tile_lane_query<T, DB, CAUSAL, DROPOUT, PACK_LATE>(a, s, o, pf, m_run, l_run, lr_run, calm, ones, c, k0, q0, qi, len, g, bh);
      // ---- O^T += V^T P^T
      {
        auto v_frag = [&](int f) {   // f = DB cc + db: consecutive MFMAs hit different accumulators
          const T* base = Vt + 16 * (f / DB) * D;
          return tr_frag<T8>(base + tro.off[f % DB][0], base + tro.off[f % DB][1]);
        };
        T8 ring[PF];
#pragma unroll
        for (int f = 0; f < PF; ++f) ring[f] = v_frag(f);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < 4 * DB; ++f) {
          const T8 cur = ring[f % PF];
          o[f % DB] = mfma32(cur, pf[f / DB], o[f % DB]);
          if (f + PF < 4 * DB) ring[f % PF] = v_frag(f + PF);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    wait_async_copies();
    __syncthreads();   // the next tile has landed, and everyone is done with this buffer
    jt = jn;
    more = more_next;
    buf ^= 1;
  }

  if constexpr (KG > 1) {
    // The loop ended on a barrier (or never touched LDS).  The groups but the first leave O in the tile buffers from the first one
    // on; the last two take the output rows.
    constexpr int kLanes = 64 * RW;
    static_assert((KG - 1) * RW + 2 <= 4 * KG && RW <= 4 && sizeof(Tile) == 4 * D * 32, "LDS holds the groups' O and the output rows");
    __shared__ float sums[(KG - 1) * 3 * kLanes];   // references and row sums
    f32x4* const o_part = (f32x4*)Ks + (group - 1) * (4 * DB * kLanes) + wave * 64 + lane;
    float* const s_part = sums + (group - 1) * 3 * kLanes + wave * 64 + lane;
    if (group > 0) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x4 v = {o[db][4 * i4], o[db][4 * i4 + 1], o[db][4 * i4 + 2], o[db][4 * i4 + 3]};
          o_part[(4 * db + i4) * kLanes] = v;
        }
      s_part[0] = m_run;
      s_part[kLanes] = l_run;
      s_part[2 * kLanes] = lr_run[0];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int k = 1; k < KG; ++k) {
      const float* const sp = s_part + k * 3 * kLanes;
      const f32x4* const op = o_part + k * (4 * DB * kLanes);
      const float mk = sp[0], m = fmaxf(m_run, mk), ref = m == -INFINITY ? 0.f : m;
      const float w0 = __builtin_amdgcn_exp2f(m_run - ref), w1 = __builtin_amdgcn_exp2f(mk - ref);
      m_run = m;
      l_run = l_run * w0 + sp[kLanes] * w1;
      lr_run[0] = lr_run[0] * w0 + sp[2 * kLanes] * w1;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const f32x4 v = op[(4 * db + i4) * kLanes];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[db][4 * i4 + e] = o[db][4 * i4 + e] * w0 + v[e] * w1;
        }
    }
  }

  // ---- epilogue: normalise, apply the dropout scale, write O and L once
  const float l_sum = l_run + xchg32(l_run);
  const float lr_sum = lr_run[0];
  const float l_tot = qi < len ? l_sum : 0.f;   // padding rows: O = 0, LSE = -inf
  const float inv = (l_tot > 0.f && lr_sum > 0.f) ? (DROPOUT ? a.keep_scale : 1.f) / lr_sum
                                                  : (l_tot == l_tot ? 0.f : l_tot);   // (a row of NaN stays one)
  if (g == 0 && row_ok) {
    const float lse = l_tot > 0.f ? (m_run + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f : -INFINITY;
    a.LSE[(int64_t)bh * a.N + qi] = lse;
  }
  if (a.o_fp32) {
    float* Og = (float*)a.O + head_off + (int64_t)qi * a.sn;
    if (row_ok) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = o[db][4 * i4 + e] * inv;
          if (D != 32 || 8 * i4 + 4 * g < a.dvalid) *(f32x4*)(Og + 32 * db + 8 * i4 + 4 * g) = v;
        }
    }
  } else {
    // coalesced row stores through the (now idle) tile buffers: two wavefronts per buffer
    // (of several groups: two that hold nothing of the merge, which other wavefronts may still read)
    T* stage = KG > 1 ? &Vs[2 * KG - 2][0] + wave * 32 * D : (wave < 2 ? &Ks[0][0] + wave * 32 * D : &Vs[0][0] + (wave - 2) * 32 * D);
    store_rows_coalesced<T, D>(stage, (T*)a.O + head_off + (int64_t)q0 * a.sn, a.sn, o, inv, a.N - q0,
                               D == 32 ? a.dvalid : D);
  }
  }
}

template <typename T, int D, int RW, int KG>
int launch_fwd_groups(KArgs a, bool causal, bool dropout, bool sparse, hipStream_t s) {
  const int blocks = RW == 4 ? a.T : (a.N + 32 * RW - 1) / (32 * RW);
  a.n_items = a.B * a.H * blocks;
  a.chunk = (a.n_items + kXcds - 1) / kXcds;
  a.group = causal_group(a, D, sparse, true, 2 * (int64_t)a.N * D * (int64_t)sizeof(T));
  if (causal && !sparse) whole_levels(a, D, true, blocks);
  const dim3 grid(kXcds * a.chunk), block(64 * RW * KG);
#define ATTN_FWD_CASE(C, P, S)                                                              \
  if (causal == C && dropout == P && sparse == S) {                                         \
    hipLaunchKernelGGL((fwd_kernel<T, D, C, P, S, RW, KG>), grid, block, 0, s, a);          \
    return (int)hipGetLastError();                                                          \
  }
  ATTN_FWD_CASE(false, false, false)
  ATTN_FWD_CASE(true, false, false)
  ATTN_FWD_CASE(false, true, false)
  ATTN_FWD_CASE(true, true, false)
  ATTN_FWD_CASE(false, false, true)
  ATTN_FWD_CASE(true, false, true)
  ATTN_FWD_CASE(false, true, true)
  ATTN_FWD_CASE(true, true, true)
#undef ATTN_FWD_CASE
  return (int)hipErrorInvalidValue;
}

template <typename T, int D>
int launch_fwd_td(const KArgs& a, bool causal, bool dropout, bool sparse, bool divide, hipStream_t s) {
  const WaveGroups w = fwd_groups(a, D, causal, sparse, divide);
  if constexpr (D <= 64)
    if (w.waves == 2 && w.groups == 4) return launch_fwd_groups<T, D, 2, 4>(a, causal, dropout, sparse, s);
  if (w.waves == 2) return launch_fwd_groups<T, D, 2, 2>(a, causal, dropout, sparse, s);
  if (w.groups == 2) return launch_fwd_groups<T, D, 4, 2>(a, causal, dropout, sparse, s);
  return launch_fwd_groups<T, D, 4, 1>(a, causal, dropout, sparse, s);
}

// keep[bh][i][j] for the test hook: one thread per group of sixteen consecutive keys, with the generator of the product kernels and
// the test of dQ.  (The forward and the dK/dV kernels test packed fields in ways of their own; the tests read the masks
// that those apply back from their outputs.)
__global__ void dropout_mask_kernel(const KArgs a, uint8_t* keep) {
  const int64_t ngrp = ((int64_t)a.N + 15) / 16;
  const int64_t total = (int64_t)a.B * a.H * a.N * ngrp;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t g16 = (uint32_t)(idx % ngrp);
    const uint32_t i = (uint32_t)((idx / ngrp) % a.N);
    const uint32_t bh = (uint32_t)(idx / (ngrp * a.N));
    const u32x4 w = philox_draw16(g16, i, bh, a.offset_lo, a.seed_lo, a.seed_hi);
    uint32_t m = 0;   // bit f: key 16 g16 + f is kept (with a threshold of 0, where the kernels do not draw at all, every one)
#pragma unroll
    for (int f = 0; f < 16; ++f) m |= dropped(w[f >> 2], f & 3, a.drop_thr) ? 0u : 1u << f;
    uint8_t* dst = keep + ((int64_t)bh * a.N + i) * a.N + 16 * (int64_t)g16;
    const int n = min(16, a.N - 16 * (int)g16);
    if (n == 16 && a.N % 4 == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {   // four flag bytes at a time
        const uint32_t nib = (m >> (4 * q)) & 0xFu;
        *(uint32_t*)(dst + 4 * q) = (nib & 1u) | ((nib & 2u) << 7) | ((nib & 4u) << 14) | ((nib & 8u) << 21);
      }
    } else {   // rows of N bytes are not 4-byte aligned, or the last group of a row is partial
      for (int f = 0; f < n; ++f) dst[f] = (uint8_t)((m >> f) & 1u);
    }
  }
}

}  // namespace

// us, forward alone, {4, 1} | {4, 2} | {2, 2} | {2, 4} (wavefronts of rows, groups; heads x N):
//   d = 64   4 x 117 5.5 5.7 5.3 6.3; 16 x 256 6.9 7.1 6.2 6.8; 16 x 640 11.1 10.3 8.5 9.1; 16 x 1024 16.0 13.7 12.9 11.0;
//            8 x 2048 27.5 22.5 21.9 16.5; 1 x 8192 99.2 76.2 73.2 46.5; 24 x 1024 16.0 13.7 16.7 19.7; 16 x 2048 28.4 24.2 29.7 30.6;
//            8 x 4096 52.4 43.0 54.4 51.2; 60 x 512 9.9 9.6 10.7 14.7; 20 x 2048 38.5 44.2 44.9 43.9; 128 x 512 14.1 17.1 19.6 27.6
//   two tiles, {4, 1} | {2, 2}  d = 64 1 x 128 4.5 4.3, 16 x 100 5.0 4.7, 128 x 128 5.1 4.9, dropout 6.0 5.6; causal 1 x 128 5.1 7.5; d = 32 1 x 128 3.9 3.7,
//            16 x 100 4.6 4.1, 128 x 65 with dropout 5.6 4.7, causal 128 x 128 4.8 4.3; one tile d = 64 16 x 64 4.1 4.6; d = 32 16 x 64 3.7 3.9
//   d = 64 causal  64 x 129 6.0 6.2 5.7 -; 64 x 192 6.1 6.7 5.9 -, dropout 7.1 7.3 6.5 -; 60 x 400 9.4 8.8 8.1 12.0; 16 x 1024 17.2 13.8 11.2 10.6; 8 x 4096 57.0 41.7 35.3 32.4;
//            20 x 2048 30.8 23.7 20.3 28.7; 10 x 4096 57.1 42.3 36.7 44.5; 64 x 1024 18.6 18.6 19.4 29.4; 48 x 1400 24.0 25.7 24.4 38.0; 160 x 225 7.7 10.0 10.2 -; 75 x 506 11.2 11.4 13.5 -;
//            52 x 520 11.0 9.8 8.8 -; 60 x 579 12.6 11.2 12.1 -; 67 x 654 14.6 16.0 16.9 -; 82 x 648 15.1 17.9 17.7 -; 63 x 715 with dropout 19.2 17.5 19.6 25.7; 57 x 794 15.9 16.7 16.6 -;
//            85 x 705 16.7 18.8 21.7 -; 60 x 900 16.9 18.3 18.0 -; 50 x 1000 18.4 17.4 17.9 -; 51 x 985 19.6 18.8 20.4 30.7
//   d = 32   4 x 117 4.7 5.0 5.1 5.0; 16 x 640 9.7 8.9 7.1 7.1; 16 x 1024 13.5 11.6 10.3 8.4; 60 x 512 8.5 7.9 8.6 8.5; 8 x 4096 45.1 35.5 39.8 32.8;
//            10 x 4096 60.7 55.3 52.9 47.6; 32 x 2048 32.9 31.3 38.5 35.1, causal 34.0 30.0 29.2 26.9; 128 x 512 11.1 11.4 13.9 14.7
//   d = 128  4 x 117 6.6 7.8 7.2; 64 x 189 8.5 - 9.7; 40 x 359 11.7 - 11.0; 16 x 1024 22.1 19.9 18.8; 1 x 8192 140 107 107; 60 x 512 14.4 14.5 23.1; 24 x 1024 22.4 20.5 35.3;
//            8 x 4096 78.3 69.9 112, causal 75.9 58.4 62.8; 40 x 1024 32.8 39.8 51.8; causal 10 x 4096 104 71.5 116, 8 x 8192 170 141 230,
//            48 x 693 20.1 22.2 -, 24 x 2001 56.4 45.1 66.5, 40 x 1024 32.0 32.1 36.5, 48 x 1400 42.9 44.0 62.3, 64 x 1024 34.0 38.9 56.4
//   block-sparse (butterfly mask of T x T blocks, heads x T)  d = 64  4 x 16 15.5 13.1 10.8 11.0; 4 x 64 20.0 17.0 17.4 24.3; 8 x 64 27.7 31.0 31.5 46.5;
//            d = 128  4 x 16 20.4 18.3 17.4; 4 x 64 28.4 26.9 43.1; 8 x 64 43.8 51.7 85.0
WaveGroups fwd_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide) {
  if (!divide) return {4, 1};
  const WorkItems w(a, sparse, causal && !sparse && d == 64);
  // (a compute unit holds two workgroups of {2, 4} at d = 32, one otherwise.  Causal, long sweeps, {2, 2} | {2, 4}: 8 x 7975 with dropout 97.4 | 89.9, 9 x 5741 with dropout 63.2 | 57.0,
  // 4 x 10405 63.0 | 59.4, 9 x 6324 47.9 | 46.9; 15 x 4219 36.0 | 37.4, 16 x 4019 34.3 | 35.4.
  // d = 64 causal, nearly a round of half blocks, {2, 2} | {2, 4}: 21 x 1149 13.5 | 16.0, 18 x 1405 14.9 | 16.7, 20 x 1533 15.7 | 18.2, with dropout 20.1 | 22.0, 18 x 1789 17.8 | 20.7, 16 x 1917 18.5 | 19.6,
  // 13 x 2429 22.1 | 24.0, with dropout 28.6 | 29.8; fewer or longer 16 x 1149 11 % behind, 14 x 1277 14 %, with dropout 16 x 1324 13 %, 15 x 1458 11 %, 12 x 2366 6 %, 16 x 1533 even, 11 x 2301 4 %, with dropout 11 %, 10 x 3069 1 %, 9 x 3453 2 %, 5 x 6397 13 %)
  const int64_t fit24 = d == 64 ? (!causal || sparse || w.tiles >= 40 ? 32 : w.tiles >= 32 ? 29 : w.tiles >= 24 ? 26 : 23) * kComputeUnits / 32 : causal && !sparse && w.tiles >= 86 ? 4 * kComputeUnits : !causal || sparse || w.tiles >= 32 ? 5 * kComputeUnits / 2 : 2 * kComputeUnits;
  if (d <= 64 && w.of64 <= fit24 && w.tiles >= 12) return {2, 4};
  // (two tiles would gain 0.2 to 0.8 us, less than the host spends on a call; a head of up to 128 tokens keeps one form instead, and with it the same last bits in whatever
  // batch it stands)
  // (causal blocks are dealt out heaviest first: two more rounds of light ones do no harm.  {2, 2} against {4, 2} or {4, 1}: d = 64 24 x 1500 16.2 18.7, 20 x 2048 20.4 23.6,
  // 10 x 4096 36.0 41.6, 60 x 700 13.4 13.8, 12 x 5000 60.1 56.4, 32 x 2048 30.9 28.5; d = 32 40 x 1024 10.2 11.8, 60 x 700 8.6 9.8, 32 x 2048 20.7 22.2, 60 x 1000 with
  // dropout 18.0 19.8, 128 x 700 13.0 12.9; {2, 4} there 12.0, 11.1, 23.0, 20.1, 18.6, and 10 x 4096 27.4 29.9)
  const int64_t fit22 = !causal || sparse || d == 128 ? kComputeUnits : d == 64 ? (w.tiles >= 9 ? 11 : 8) * kComputeUnits / 8 : 9 * kComputeUnits / 2;
  const bool one_round = d == 64 && causal && !sparse && (int64_t)a.B * a.H * w.tiles <= 2 * kComputeUnits;   // (an odd block counts as a whole half in of64)
  if ((w.of64 <= fit22 || one_round) && w.tiles >= (d == 128 ? 6 : 3)) return {2, 2};
  if (d == 64 && causal && !sparse) return w.of128 <= (w.tiles >= 16 ? 4 : 3) * kComputeUnits / 4 && w.tiles >= 12 ? WaveGroups{4, 2} : WaveGroups{4, 1};
  if (d <= 64) return w.of128 <= (d == 32 ? 2 : 1) * kComputeUnits && w.tiles >= 10 ? WaveGroups{4, 2} : WaveGroups{4, 1};
  // d = 128: {4, 2} has one workgroup on a compute unit, {4, 1} two, which together get through a tile hardly faster than one
  // of them alone.  Estimates in us: the tiles of all items over the compute units, and under the causal mask the longest sweep.
  // (From 512 items on {4, 2} would gain for few heads of long causal sequences only, 8 x 8192 above, where the results are held to the
  // last bit to those of the two-group kernel, whose references a row's undivided sweep shares; the line stays below.)
  if (w.of128 > 3 * kComputeUnits / 2 || (w.of128 > kComputeUnits && w.tiles < 16)) return {4, 1};
  const double heads = (double)a.B * a.H, per_unit = 1.0 / kComputeUnits;
  double one, two;
  if (causal && !sparse) {
    const double tiles = heads * std::min<double>((double)a.T * (a.T + 1), (double)a.T * w.tiles);
    one = std::max(1.12 * tiles * per_unit, 1.25 * w.tiles) + 3.0;
    two = std::max(1.08 * tiles * per_unit + 4.5 * (double)w.of128 * per_unit, 0.9 * w.tiles + 4.5);
  } else {
    one = std::max(1.12 * (double)w.of128 * per_unit, 1.25) * w.tiles + 3.0;
    two = std::ceil((double)w.of128 * per_unit) * (1.08 * w.tiles + 4.5);
  }
  return two < one ? WaveGroups{4, 2} : WaveGroups{4, 1};
}

// Which dense d = 128 problems take the two-group kernel (attn_fwd_pp.hip): an estimate of either kernel's time,
// in units of one 64-key tile of the two-group kernel (256 rows on a whole compute unit, 1.78 us without
// dropout).  Per tile it is the faster one, but it has one workgroup per compute unit: its work items (pairs of row blocks
// under the causal mask) run in whole rounds over the chip, and nothing covers an item's prologue and epilogue.
// This file's kernel has two workgroups of 128 rows on a compute unit, dealt out as they finish (unpaired and
// therefore less evenly under the causal mask).  us, two-group | this file's (16384 tokens, 16 heads):
//   causal     N = 512 76 | 74, 640 111 | 70, 768 111 | 81, 1024 97 | 107, 1400 138 | 116, 2048 151 | 174, 4096 268 | 309
//   no mask    N = 512 89 | 83, 640 110 | 97, 768 115 | 111, 1024 142 | 143, 1400 205 | 184, 2048 253 | 267, 4096 485 | 517
//   causal with dropout  N = 512 85 | 84, 1024 114 | 125, 2048 182 | 206, 4096 326 | 369; 64 heads of 1024: 51 | 34
//   few heads  12 of 4096 102 | 118, 24 of 2001 55 | 62; causal with dropout, 8 of 8192 267 | 209
// The estimate is the faster kernel in all of these but for less than 1 % (no mask, 1024; causal with dropout, 512).  It is
// no better than that: for the two-group kernel it is within 4 % of the time from N = 1024 on where the rounds are full, 6-13 % short
// with dropout, and up to 36 % long where the last round is part-filled or the odd block of a head stands alone, charged
// as a pair (causal 640: 151; no mask 1400: 231); for this file's kernel within 10 %.
// Dropout without a mask is plain vector ALU work, which evens the two out in favour of this file's: N = 512
// 112 | 94, 1024 180 | 165, 2048 322 | 313, 4096 626 | 610, 8192 1215 | 1203.
static bool two_group_is_faster(const KArgs& a, bool causal, bool dropout) {
  if (dropout && !causal) return false;
  const double heads = (double)a.B * a.H;
  const double tiles = (a.N + BC - 1) / BC;              // 64-key tiles of a row without a mask
  const double tile_pp = dropout ? 1.13 : 1.0, tile_base = dropout ? 1.32 : 1.08;
  const double extra_pp = causal ? 7.2 : 4.0, extra_base = causal ? 4.1 : 1.8;   // per work item, per workgroup
  const double blocks256 = (a.N + 255) / 256, blocks128 = a.T;
  const double items = heads * (causal ? std::floor((blocks256 + 1) / 2) : blocks256);
  const double item_tiles = causal && blocks256 > 1 ? tiles + 4 : tiles;
  const double pp = std::ceil(items / kComputeUnits) * (item_tiles * tile_pp + extra_pp);
  const double groups = heads * blocks128;
  const double head_tiles = causal ? std::min(blocks128 * (blocks128 + 1), blocks128 * tiles) : blocks128 * tiles;
  // A compute unit that has only one workgroup of this file's kernel left (few workgroups, or the long ones under a
  // causal mask, whose neighbours have ended) gets through a tile in 0.65 of the time.
  const bool alone = causal || groups <= kComputeUnits;
  const double longest = tiles * (alone ? 0.65 : 1.0) * tile_base + extra_base;
  const double base = std::max((heads * head_tiles * tile_base + groups * extra_base) / (2 * kComputeUnits), longest);
  return pp < base;
}

int choose_fwd(const KArgs& a, int d, bool causal, bool dropout, bool sparse, const Overrides& v) {
  bool use_pp = d == 128 && two_group_is_faster(a, causal, dropout);
  if (v.fwd == 1) use_pp = false;
  if (v.fwd == 2 && d != 32) use_pp = true;
  return !sparse && use_pp ? kFwdTwoGroup : kFwdFreeRunning;
}

int launch_fwd(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, const Overrides& v, hipStream_t s) {
  const bool divide = may_divide(v);
  // Dense d = 128 problems: see two_group_is_faster above.
  // At d <= 64 the vector ALU work dominates and this file's kernel measured faster at every N;
  // block-sparse problems always take it.  attn_debug_set_variant overrides the choice
  // (comparisons and tests).
  if (choose_fwd(a, d, causal, dropout, sparse, v) == kFwdTwoGroup) return launch_fwd_pp(a, dtype, d, causal, dropout, s);
  if (dtype == 0 && d == 32) return launch_fwd_td<_Float16, 32>(a, causal, dropout, sparse, divide, s);
  if (dtype == 1 && d == 32) return launch_fwd_td<__bf16, 32>(a, causal, dropout, sparse, divide, s);
  if (dtype == 0 && d == 64) return launch_fwd_td<_Float16, 64>(a, causal, dropout, sparse, divide, s);
  if (dtype == 0 && d == 128) return launch_fwd_td<_Float16, 128>(a, causal, dropout, sparse, divide, s);
  if (dtype == 1 && d == 64) return launch_fwd_td<__bf16, 64>(a, causal, dropout, sparse, divide, s);
  if (dtype == 1 && d == 128) return launch_fwd_td<__bf16, 128>(a, causal, dropout, sparse, divide, s);
  return (int)hipErrorInvalidValue;
}

int launch_dropout_mask(const KArgs& a, uint8_t* keep, hipStream_t s) {
  const int64_t total = (int64_t)a.B * a.H * a.N * ((a.N + 15) / 16);
  const int blocks = (int)((total + 255) / 256 < 65536 ? (total + 255) / 256 : 65536);
  hipLaunchKernelGGL(dropout_mask_kernel, dim3(blocks), dim3(256), 0, s, a, keep);
  return (int)hipGetLastError();
}

}  // namespace attn
