// Block-sparse dK/dV load balance: which mask columns are cut into segments, who walks them, and who converts their sums.
//
// A column of the mask is the work of one workgroup, but for the heavy ones (a "global token" column): those are cut into segments,
// whose workgroups add their partial dK, dV into fp32 accumulators with atomics.  Planning needs the columns' block counts and
// nothing that dQ computes, so it runs in workgroups of its own at the head of the dQ launch, one for 16 columns
// of a head; the last segment of a column to end converts its sums.  (Three launches of 5 to 6 us each before, two between dQ and dK/dV and
// one after: backward pass of 2 heads of T = 8 blocks, d = 64, 40 us, now 31; 8 heads of 64 blocks 107, now 91; 8 x 128 181, now 167.)
#pragma once
#include "attn_common.h"
#include "attn_tiles.h"

namespace attn {

// The kernel's arguments, read again from where they were passed: the compiler keeps every argument that is named after the tile loop
// in registers (spilled ones at that) through the loop.  For kernels whose only argument is a KArgs.
typedef const __attribute__((address_space(4))) KArgs* KArgsPtr;
__device__ __forceinline__ KArgsPtr kernel_args_again() {
  KArgsPtr p = nullptr;
#if defined(__HIP_DEVICE_COMPILE__)
  p = (KArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
#endif
  return p;
}

// Planning workgroup `id` of the dQ launch (all of its threads; lds: at least 64 * wavefronts ints).  Leaves the columns' block counts and
// numbers of segments (0: not heavy), the sum of the latter, zeroed tickets, and zeroed accumulators for the heavy columns.
template <int D>
__device__ __forceinline__ void sparse_plan(const KArgs& a, int id, bool causal, int* lds) {
  const int n_cg = (a.T + kPlanCols - 1) / kPlanCols;
  if (id >= a.B * a.H * n_cg) return;
  const int bh = id / n_cg, cg = id % n_cg;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  const int len = a.klen ? min(max(a.klen[bh / a.H], 0), a.N) : a.N;
  const int c = lane % kPlanCols, col = cg * kPlanCols + c, item = bh * a.T + col;   // a wavefront reads its columns of four rows at a time
  const uint8_t* const mask = a.mask + (int64_t)(bh % a.H) * a.mask_sh + col;
  const int first = causal ? col : 0;                                             // same row range as the
  const int limit = col < a.T && col * 128 < len ? min(a.T, (len + 127) / 128) : 0;   // tile iterators of the dK/dV kernels
  int cnt = 0;
#pragma unroll 8
  for (int row = (64 / kPlanCols) * wave + lane / kPlanCols; row < a.T; row += (64 / kPlanCols) * n_waves)
    if (row >= first && row < limit) cnt += mask[(int64_t)row * a.T] != 0;
  lds[wave * 64 + lane] = cnt;
  __syncthreads();
  // every wavefront knows all totals
  cnt = 0;
  for (int i = c; i < 64 * n_waves; i += kPlanCols) cnt += lds[i];
  int total = cnt;
#pragma unroll
  for (int off = kPlanCols / 2; off > 0; off >>= 1) total += __shfl_xor(total, off, 64);
  // more than half of a compute unit's fair share, were all columns of all heads as full as these
  const int n_cols = min((int)kPlanCols, a.T - cg * kPlanCols);
  const int64_t share = (int64_t)total * a.T / n_cols * a.B * a.H / (2 * kComputeUnits);
  const bool stands_out = (int64_t)cnt * n_cols > 2 * (int64_t)total;
  const bool heavy = col < a.T && cnt > share && cnt > (stands_out ? (int)kHeavyBlocks : (int)kLongBlocks);
  const int seg_blocks = stands_out && cnt <= kShortSegLimit ? (int)kShortSegBlocks : (int)kSegBlocks;
  const uint32_t heavy_cols = (uint32_t)__ballot(heavy) & ((1u << kPlanCols) - 1);
  if (wave == 0) {
    int segs = heavy ? min((int)kMaxSegs, (cnt + seg_blocks - 1) / seg_blocks) : 0;
    if (lane < kPlanCols && col < a.T) {
      a.colcnt[item] = cnt;
      a.col_segs[item] = segs;
      a.ticket[item] = 0;
    }
#pragma unroll
    for (int off = kPlanCols / 2; off > 0; off >>= 1) segs += __shfl_xor(segs, off, 64);
    if (lane == 0) a.group_segs[id] = segs;
  }
  for (uint32_t bits = heavy_cols; bits != 0; bits &= bits - 1) {
    const int64_t off = ((int64_t)bh * a.N + (int64_t)(cg * kPlanCols + __builtin_ctz(bits)) * 128) * D;
    for (int i = threadIdx.x; i < 128 * D / 4; i += blockDim.x) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      *(f32x4*)(a.dKacc + off + 4 * i) = z;
      *(f32x4*)(a.dVacc + off + 4 * i) = z;
    }
  }
}

// Segment number idx of all heavy columns, in the order of the planning groups: its column, its first kept block, its length.  Every
// wavefront finds it by itself.  False past the end.
__device__ __forceinline__ bool sparse_segment(int idx, int& item, int& skip_blocks, int& take_blocks) {
  const auto& a = *kernel_args_again();
  const int lane = threadIdx.x & 63;
  auto inclusive = [&](int v) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int below = __shfl_up(v, off, 64);
      if (lane >= off) v += below;
    }
    return v;
  };
  const int n_cg = (a.T + kPlanCols - 1) / kPlanCols, n_groups = a.B * a.H * n_cg;
  for (int g0 = 0; g0 < n_groups; g0 += 64) {
    const int sum = inclusive(g0 + lane < n_groups ? a.group_segs[g0 + lane] : 0);
    const int total = __builtin_amdgcn_readlane(sum, 63);
    if (idx >= total) {
      idx -= total;
      continue;
    }
    const int at = __builtin_ctzll(__ballot(sum > idx));
    if (at > 0) idx -= __builtin_amdgcn_readlane(sum, at - 1);
    const int group = g0 + at, bh = group / n_cg, cg = group % n_cg;
    const int col = cg * kPlanCols + lane;
    const int segs = lane < kPlanCols && col < a.T ? a.col_segs[bh * a.T + col] : 0;
    const int csum = inclusive(segs);
    const int which = __builtin_ctzll(__ballot(csum > idx));
    // (the same in all lanes: in scalar registers)
    item = __builtin_amdgcn_readfirstlane(bh * a.T + cg * kPlanCols + which);
    const int n = __builtin_amdgcn_readlane(segs, which), seg = idx - (which > 0 ? __builtin_amdgcn_readlane(csum, which - 1) : 0);
    take_blocks = __builtin_amdgcn_readfirstlane((a.colcnt[item] + n - 1) / n);
    skip_blocks = __builtin_amdgcn_readfirstlane(seg * take_blocks);
    return true;
  }
  return false;
}

// After a segment's atomics, with all threads of its workgroup: the last of the column's segments to get here converts the sums to
// the 16-bit outputs.  Everything that changes hands is in device-scope atomics, which are carried out beyond the L2 of an XCD: a
// segment's sums are in place once its atomics have been acknowledged, which is what it waits for before it takes its ticket, and
// device-scope loads find them there.  (Fences of that scope, which write back and invalidate a whole L2 per segment, cost
// more than the launch they would save: backward of a dense mask of 4 heads x 48 blocks, d = 64, 227 -> 270 us.)
template <typename T, int D>
__device__ __forceinline__ void sparse_finish(int item) {
  const auto& a = *kernel_args_again();
  typedef typename Vec<T>::x4 T4;
  __shared__ int is_last;
  asm volatile("" ::: "memory");
  wait_async_copies();   // vmcnt(0): this wavefront's atomics
  __syncthreads();
  if (threadIdx.x == 0) is_last = __hip_atomic_fetch_add(a.ticket + item, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.col_segs[item] - 1;
  __syncthreads();
  if (!is_last) return;
  const int bh = item / a.T, kt = item % a.T;
  const int64_t head_off = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int64_t acc_off = ((int64_t)bh * a.N + (int64_t)kt * 128) * D;
  const int tid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64 + lane_id_here();
#pragma unroll 4
  for (int i = tid; i < 128 * D / 4; i += blockDim.x) {
    const int row = (4 * i) / D, colx = (4 * i) % D;
    T4 ko, vo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      ko[e] = (T)__hip_atomic_load(a.dKacc + acc_off + 4 * i + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      vo[e] = (T)__hip_atomic_load(a.dVacc + acc_off + 4 * i + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (D == 32 && colx >= a.dvalid) continue;   // head dimension 16: the tensors' rows end there
    const int64_t o = head_off + (int64_t)(kt * 128 + row) * a.sn + colx;
    *(T4*)((T*)a.dK + o) = ko;
    *(T4*)((T*)a.dV + o) = vo;
  }
}

}  // namespace attn
