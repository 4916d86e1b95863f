// Block-sparse dK/dV load balance: which mask columns are cut into segments, who walks them, and who converts their sums.
//
// A column of the mask is the work of one workgroup, but for the heavy ones (a "global token" column): those are cut into segments,
// whose workgroups add their partial dK, dV into fp32 accumulators with atomics.  Planning needs the columns' block counts and
// nothing that dQ computes, so it runs in workgroups of its own at the head of the dQ launch, one for 16 columns
// of a head; the last segment of a column to end converts its sums.  (Three launches of 5 to 6 us each before, two between dQ and dK/dV and
// one after: backward pass of 2 heads of T = 8 blocks, d = 64, 40 us, now 31; 8 heads of 64 blocks 107, now 91; 8 x 128 181, now 167.)
#pragma once
#include <type_traits>

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

// Kept blocks of the whole problem, from some rows of the masks: all of them up to 4096 bytes (a shared mask of T = 64), otherwise as many as
// make 4096 bytes (16 at least), spread over the lengths and the heads' masks in turn, and over the rows by the fractions of the
// golden ratio.  Every planning workgroup counts for itself and finds the same: a sum over the workgroups would take a launch of its own, and the
// columns that one workgroup plans say least about the others where a global-token column is among them.  us, backward, butterfly mask of heads x T,
// d = 64, heavy by a share estimated from the planned columns | from these rows (by the exact sum, in a launch of its own):
//   16 x 512 2744 | 1577 (1560); 24 x 256 1492 | 1090 (1085); 32 x 128 843 | 664 (668); 48 x 64 540 | 448 (456); 8 x 128 173 | 174 (186)
struct MaskSample {
  int lengths, masks, rows;   // different lengths, different masks, rows looked at
  __host__ __device__ explicit MaskSample(const KArgs& a) {
    lengths = a.klen ? a.B : 1;
    masks = a.mask_sh != 0 ? a.H : 1;
    const int64_t all = (int64_t)lengths * masks * a.T, some = 4096 / a.T > 16 ? 4096 / a.T : 16;
    rows = (int)(all < some ? all : some);
  }
  // this thread's part of the kept blocks in those rows
  __host__ __device__ int count(const KArgs& a, bool causal, int thread, int n_threads) const {
    const bool all = rows == (int64_t)lengths * masks * a.T;
    const int words = (a.T + 3) / 4;   // four mask bytes at a time
    int n = 0;
#pragma unroll 4
    for (int p = thread; p < rows * words; p += n_threads) {
      const int i = p / words, c = 4 * (p % words);
      const int lm = all ? i / a.T : (int)((int64_t)i * lengths * masks / rows);
      const int row = all ? i % a.T : (int)((uint64_t)((uint32_t)i * 2654435769u + 0x80000000u) * (uint32_t)a.T >> 32);
      int blocks = a.T;
      if (a.klen) blocks = (min(max(a.klen[lm / masks], 0), a.N) + kMaskBlock - 1) / kMaskBlock;
      const int end = row < blocks ? min(causal ? row + 1 : a.T, blocks) - c : 0;   // columns from c on that count
      const uint8_t* const m = a.mask + (int64_t)(lm % masks) * a.mask_sh + (int64_t)row * a.T + c;
      uint32_t w = 0;
      if (c + 4 <= a.T) __builtin_memcpy(&w, m, 4);
      else for (int e = 0; c + e < a.T; ++e) w |= (uint32_t)m[e] << 8 * e;
      uint32_t kept = (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;   // a bit per byte that is not 0
      if (end < 4) kept &= end > 0 ? (1u << 8 * end) - 1 : 0;
      n += __builtin_popcount(kept);
    }
    return n;
  }
  __host__ __device__ int64_t total(const KArgs& a, int64_t counted) const { return counted * a.B * a.H * a.T / rows; }
};

// The planning workgroups of a head look at kPlanCols columns each.  Those of the last one start early where T is no multiple, so that a
// column always has neighbours to stand out from; it leaves alone the ones that the workgroup before it plans.
__host__ __device__ inline int plan_window(int T, int cg) { return min(cg * kPlanCols, max(T - kPlanCols, 0)); }

// Segments that a column of cnt kept blocks is cut into (0: it is not heavy), by the rule at kLongBlocks; near: the kept blocks of the n_near columns looked at
// together, this one among them, total: those of the whole problem.
__host__ __device__ inline int column_segments(int cnt, int near, int n_near, int64_t total) {
  const bool stands_out = (int64_t)cnt * (n_near - 1) > 2 * (int64_t)(near - cnt);
  if (cnt <= total / (2 * kComputeUnits) || cnt <= (stands_out ? (int)kHeavyBlocks : (int)kLongBlocks)) return 0;
  const int seg_blocks = stands_out && cnt <= kShortSegLimit ? (int)kShortSegBlocks : (int)kSegBlocks;
  return min((int)kMaxSegs, (cnt + seg_blocks - 1) / seg_blocks);
}

// Columns of up to kLongBlocks blocks keep reproducible gradients.  Sums of two addends do not depend on which comes first, so two of a column's
// three segments add into its own accumulators and the third into those of a light column, which stand idle; the last one to end adds
// the two.  (Two segments where no light column is left.  Two for all: 8 x 24 at d = 64 53 -> 64 us, at d = 128 85 -> 103.)  A column's entry in col_segs is
// its number of segments, and from bit 8 on where the third one goes: the other column's number less its own plus kPlanCols, or 0.
__host__ __device__ inline int segs_of(int entry) { return entry & 255; }
// The column whose accumulators segment seg of column item adds into.
__host__ __device__ inline int slot_of(int item, int entry, int seg) { return seg == 2 && entry > 255 ? item + (entry >> 8) - kPlanCols : item; }
// The entry of column c among those looked at together, from their segments; light, three: of which columns the accumulators are idle, and which have
// three segments and must not have more than two addends (bits).
__host__ __device__ inline int column_entry(int c, int segs, uint32_t light, uint32_t three) {
  if (!(three >> c & 1)) return segs;
  for (uint32_t before = three & ((1u << c) - 1); before != 0; before &= before - 1) light &= light - 1;   // taken
  return light == 0 ? 2 : 3 | (__builtin_ctz(light) - c + kPlanCols) << 8;
}

// Planning workgroup `id` of the dQ launch (all of its threads; lds: at least 65 * wavefronts ints).  Leaves the columns' block counts and
// numbers of segments (0: not heavy), the sum of the latter, zeroed tickets, and zeroed accumulators for the heavy columns.
template <int D>
__device__ __forceinline__ void sparse_plan(const KArgs& a, int id, bool causal, int* lds) {
  const int n_cg = (a.T + kPlanCols - 1) / kPlanCols;
  if (id >= a.B * a.H * n_cg) return;
  const int bh = id / n_cg, cg = id % n_cg;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
  const int len = a.klen ? min(max(a.klen[bh / a.H], 0), a.N) : a.N;
  const int col0 = plan_window(a.T, cg);
  const int c = lane % kPlanCols, col = col0 + c, item = bh * a.T + col;   // a wavefront reads its columns of four rows at a time
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
  int near = cnt;
#pragma unroll
  for (int off = kPlanCols / 2; off > 0; off >>= 1) near += __shfl_xor(near, off, 64);
  int segs = 0;
  if (__ballot(cnt > kHeavyBlocks) != 0) {   // (the same in all wavefronts)
    const MaskSample sample(a);
    int counted = sample.count(a, causal, threadIdx.x, blockDim.x);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) counted += __shfl_xor(counted, off, 64);
    if (lane == 0) lds[64 * n_waves + wave] = counted;
    __syncthreads();
    int64_t all_counted = 0;
    for (int w = 0; w < n_waves; ++w) all_counted += lds[64 * n_waves + w];
    segs = column_segments(cnt, near, min((int)kPlanCols, a.T), sample.total(a, all_counted));
  }
  const bool mine = col >= cg * kPlanCols && col < a.T;
  if (!mine) segs = 0;
  constexpr uint32_t kCols = (1u << kPlanCols) - 1;
  const uint32_t heavy = (uint32_t)__ballot(segs > 0) & kCols, light = (uint32_t)__ballot(mine && segs == 0) & kCols;
  const uint32_t three = (uint32_t)__ballot(segs == 3 && cnt <= kLongBlocks) & kCols;
  const int entry = column_entry(c, segs, light, three);
  const uint32_t lent = (uint32_t)__ballot(entry > 255) & kCols;
  if (wave == 0) {
    if (lane < kPlanCols && mine) {
      a.colcnt[item] = cnt;
      a.col_segs[item] = entry;
      a.ticket[item] = 0;
    }
    segs = segs_of(entry);
#pragma unroll
    for (int off = kPlanCols / 2; off > 0; off >>= 1) segs += __shfl_xor(segs, off, 64);
    if (lane == 0) a.group_segs[id] = segs;
  }
  uint32_t cleared = heavy;   // and the first light ones, one for each column that adds into one
  for (uint32_t rest = light, n = __builtin_popcount(lent); n > 0; --n, rest &= rest - 1) cleared |= rest & -rest;
  for (uint32_t bits = cleared; bits != 0; bits &= bits - 1) {
    const int64_t off = ((int64_t)bh * a.N + (int64_t)(col0 + __builtin_ctz(bits)) * 128) * D;
    for (int i = threadIdx.x; i < 128 * D / 4; i += blockDim.x) {
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      *(f32x4*)(a.dKacc + off + 4 * i) = z;
      *(f32x4*)(a.dVacc + off + 4 * i) = z;
    }
  }
}

// Segment number idx of all heavy columns, in the order of the planning groups: its column, the column whose accumulators it adds into, its first kept block, its length.  Every
// wavefront finds it by itself: each lane adds up a run of the groups' sums, whose loads do not wait for one another, then the run that holds the
// segment is searched.  Backward of masks of the diagonal alone, heads x T, the sums in turns of 64 (a load and a scan each) | this: d = 32 512 x 64
// 812 | 799 us, 1024 x 32 814 | 800, 4096 x 16 1595 | 1572; d = 64 64 x 512 1573 | 1562.  False past the end.
__device__ __forceinline__ bool sparse_segment(int idx, int& item, int& slot, int& skip_blocks, int& take_blocks) {
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
  const int n_cg = (a.T + kPlanCols - 1) / kPlanCols, n_groups = a.B * a.H * n_cg, run = (n_groups + 63) / 64;
  int sum = 0;
#pragma unroll 8
  for (int k = 0; k < run; ++k) sum += lane * run + k < n_groups ? a.group_segs[lane * run + k] : 0;
  sum = inclusive(sum);
  if (idx >= __builtin_amdgcn_readlane(sum, 63)) return false;
  int at = __builtin_ctzll(__ballot(sum > idx));
  if (at > 0) idx -= __builtin_amdgcn_readlane(sum, at - 1);
  int group = at * run;
  if (run > 1) {
    for (const int end = min(group + run, n_groups);; group += 64) {
      sum = inclusive(group + lane < end ? a.group_segs[group + lane] : 0);
      const int total = __builtin_amdgcn_readlane(sum, 63);
      if (idx < total) break;
      idx -= total;
    }
    at = __builtin_ctzll(__ballot(sum > idx));
    if (at > 0) idx -= __builtin_amdgcn_readlane(sum, at - 1);
    group += at;
  }
  const int bh = group / n_cg, cg = group % n_cg, col = cg * kPlanCols + lane;
  const int entry = lane < kPlanCols && col < a.T ? a.col_segs[bh * a.T + col] : 0;
  sum = inclusive(segs_of(entry));
  at = __builtin_ctzll(__ballot(sum > idx));
  // (the same in all lanes: in scalar registers)
  item = __builtin_amdgcn_readfirstlane(bh * a.T + cg * kPlanCols + at);
  const int found = __builtin_amdgcn_readlane(entry, at), n = segs_of(found), seg = idx - (at > 0 ? __builtin_amdgcn_readlane(sum, at - 1) : 0);
  take_blocks = __builtin_amdgcn_readfirstlane((a.colcnt[item] + n - 1) / n);
  skip_blocks = __builtin_amdgcn_readfirstlane(seg * take_blocks);
  slot = __builtin_amdgcn_readfirstlane(slot_of(item, found, seg));
  return true;
}

// After a segment's atomics, with all threads of its workgroup: the last of the column's segments to get here converts the sums to
// the 16-bit outputs.  Everything that changes hands is in device-scope atomics, which are carried out beyond the L2 of an XCD: a
// segment's sums are in place once its atomics have been acknowledged, which is what it waits for before it takes its ticket, and
// device-scope loads find them there.  (Fences of that scope, which write back and invalidate a whole L2 per segment, cost
// more than the launch they would save: backward of a dense mask of 4 heads x 48 blocks, d = 64, 227 -> 270 us.)
template <typename T, int D>
__device__ __forceinline__ void sparse_finish(int item) {
  const auto& a = *kernel_args_again();
  __shared__ int is_last;
  asm volatile("" ::: "memory");
  wait_async_copies();   // vmcnt(0): this wavefront's atomics
  __syncthreads();
  if (threadIdx.x == 0) is_last = __hip_atomic_fetch_add(a.ticket + item, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == segs_of(a.col_segs[item]) - 1;
  __syncthreads();
  if (!is_last) return;
  const int bh = item / a.T, kt = item % a.T;
  const int64_t head_off = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
  const int64_t acc_off = (int64_t)item * 128 * D;
  const int64_t more = (int64_t)(slot_of(item, a.col_segs[item], 2) - item) * 128 * D;   // 0: one accumulator holds the sum
  const int tid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64 + lane_id_here();
  // Two floats a lane, so that a line is asked for once, beyond the L2 where it is; all loads of a batch before its first store, which they are
  // not moved across.  (One load at a time, four floats a lane | this, both with two accumulators: 8 x 24 at d = 64 61 | 53 us, 3 x 20 at d = 128 78 | 67.)
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef T T2 __attribute__((ext_vector_type(2)));
  constexpr int kBatch = 8;
  auto part = [](const float* p) {
    return __builtin_bit_cast(f32x2, __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  auto convert = [&](auto two) {
    for (int i0 = tid; i0 < 128 * D / 2; i0 += kBatch * (int)blockDim.x) {
      f32x2 k[kBatch], v[kBatch];
#pragma unroll
      for (int n = 0; n < kBatch; ++n) {
        const int64_t at = acc_off + 2 * min(i0 + n * (int)blockDim.x, 128 * D / 2 - 1);
        k[n] = part(a.dKacc + at);
        v[n] = part(a.dVacc + at);
        if (two) {
          const f32x2 k2 = part(a.dKacc + at + more), v2 = part(a.dVacc + at + more);
#pragma unroll
          for (int e = 0; e < 2; ++e) { k[n][e] += k2[e]; v[n][e] += v2[e]; }
        }
      }
#pragma unroll
      for (int n = 0; n < kBatch; ++n) {
        const int i = i0 + n * (int)blockDim.x, row = (2 * i) / D, colx = (2 * i) % D;
        if (i >= 128 * D / 2 || (D == 32 && colx >= a.dvalid)) continue;   // head dimension 16: the tensors' rows end there
        const int64_t o = head_off + (int64_t)(kt * 128 + row) * a.sn + colx;
        const T2 ko = {(T)k[n][0], (T)k[n][1]}, vo = {(T)v[n][0], (T)v[n][1]};
        *(T2*)((T*)a.dK + o) = ko;
        *(T2*)((T*)a.dV + o) = vo;
      }
    }
  };
  if (more != 0) convert(std::true_type());
  else convert(std::false_type());
}

}  // namespace attn
