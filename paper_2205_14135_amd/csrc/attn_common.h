// Internal declarations shared by the gfx950 attention kernels and the C-ABI front end.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace attn {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Problem description handed to every kernel (plain data, passed by value).  What every dense kernel reads first stands in the first two cache
// lines (args_at_once).
struct KArgs {
  int n_items;             // work items (B*H*tiles)
  int chunk;               // items per XCD = ceil(n_items / 8)
  int group;               // causal kernels with a block of rows per item: heads whose blocks are dealt out together, 0: all (causal_block), < 0: all, in levels of -group places (whole_levels)
  int deal;                // heads are dealt round the XCDs (dealt_head)
  int B, H, N, T;          // T = ceil(N / 128)
  const int* klen;         // key-padding lengths [B] or nullptr
  int64_t sb, sh, sn;      // element strides of the [B,H,N,d] tensors
  const void* Q; const void* K; const void* V;
  void* O;                 // fwd: out; bwd: in
  float* LSE;              // fwd: out; bwd: in        [B,H,N]
  int Nr;                  // 128 T: rows per head of the backward scratch vectors
  int dvalid;              // head dimension of the tensors: 16 with the D = 32 kernels (columns 16..31 are zeros on chip), else D
  float tau;               // softmax scale
  float scale_log2;        // tau * log2(e)
  float keep_scale;        // 1 / (1 - p_drop)
  uint32_t drop_thr;       // T: keep iff 8-bit philox field >= T (1..255 when dropout is on)
  uint32_t seed_lo, seed_hi, offset_lo;
  int o_fp32;
  const uint8_t* mask;     // block mask [T,T] (per head if mask_sh != 0) or nullptr
  int64_t mask_sh;
  const void* dO;          // bwd in
  void* dQ; void* dK; void* dV;   // bwd out
  float* Dvec;             // bwd scratch: -D_i = -rowsum(dO_i o O_i)   [B,H,Nr], 0 for rows >= N
  float* L2vec;            // bwd scratch: L_i * log2(e), +inf where L_i = -inf and for rows >= N   [B,H,Nr]
  int* colcnt;             // block-sparse bwd scratch: kept blocks per mask column   [B*H, T]
  int* col_segs;           // block-sparse bwd scratch: segments of a heavy column, 0 for the others (column_entry in attn_sparse.h)   [B*H, T]
  int* ticket;             // block-sparse bwd scratch: segments of a heavy column that have ended   [B*H, T]
  int* group_segs;         // block-sparse bwd scratch: segments of the heavy columns among kPlanCols   [B*H, ceil(T / kPlanCols)]
  float* dKacc;            // block-sparse bwd scratch: fp32 dK / dV of the columns that are
  float* dVacc;            //   split over several workgroups                         [B,H,N,d]
  float* dQpart;           // one-launch backward of heads of more than 256 tokens: fp32 dQ between the key blocks (nullptr: no room for it)
  int plan_groups;         // block-sparse bwd: planning workgroups at the head of the dQ launch (0: no column can be heavy)
};

static_assert(offsetof(KArgs, LSE) + sizeof(float*) <= 128, "the dense kernels' first arguments in two cache lines");

enum { kXcds = 8, kMaskBlock = 128 };
// Block-sparse dK/dV: a mask column is "heavy" when it keeps more than kLongBlocks blocks, or more than kHeavyBlocks and twice as
// many as its neighbours (the columns looked at with it, but itself) on average, AND more than half of a compute unit's fair share of all kept blocks (so a mask whose columns are
// all long, e.g. a dense one, is not split at all).  Heavy columns are cut into segments (at most kMaxSegs), one workgroup
// each, summed with fp32 atomics: of about kSegBlocks blocks, or kShortSegBlocks where a single column stands out from its neighbours
// and is not longer than kShortSegLimit.  us, backward with 24 and segments of 12 for all | this; heads x T, butterfly mask: d = 64
// 8 x 24 92 | 53, 3 x 20 80 | 41, 4 x 32 66 | 44, 8 x 64 106 | 91; d = 128 8 x 24 124 | 85, 16 x 16 101 | 85, 8 x 64 186 | 152 (with the planning launches and,
// at d = 128, the role-split kernel of then).  A dense mask of 4 x 48: 182 | 207 with 14 and 8 for all columns, 8 x 128 at d = 128 292 | 294 with segments of 8
// for the longest.
enum { kLongBlocks = 24, kHeavyBlocks = 14, kSegBlocks = 12, kShortSegBlocks = 8, kShortSegLimit = 64, kMaxSegs = 32, kComputeUnits = 256 };

// Kernel-choice overrides (attn_debug_set_variant; initial values from the environment, read once
// when first needed).  fwd: 0 = by measurement, 1 = free-running kernel, 2 = two-group kernel;
// dkv: 0 = by measurement, 1 = role-split kernel wherever it exists, 2 = the 64-key kernel is not used,
// 3 = the 64-key kernel wherever it exists.
// A call reads them once: another thread may set them while it is under way.
struct Overrides { int fwd, dkv; };
Overrides overrides();

// Which kernel serves a problem (the launchers use these; attn_debug_kernel_choice reports them).
enum { kFwdFreeRunning = 0, kFwdTwoGroup = 1 };
enum { kDkvRoleSplit = 0, kDkvOneWave = 1, kDkvOneWave128 = 2, kDkvOneWave64 = 3, kBwdShort = 4 };
int choose_fwd(const KArgs& a, int d, bool causal, bool dropout, bool sparse, const Overrides& v);
int choose_dkv(const KArgs& a, int d, bool causal, bool dropout, bool sparse, const Overrides& v);

// How a tile kernel divides its work: `waves` wavefronts of 32 rows (dK/dV: keys) each share the streamed tiles of a workgroup,
// and `groups` groups of that many wavefronts work on the same rows, group k on every groups-th tile; what the groups
// accumulated is added up through LDS at the end, in a fixed order.  With few work items the chip holds one wavefront per SIMD or
// fewer, and a row's sweep over the tiles is what a launch takes: half the rows make twice the items, and two or four groups
// sweep a half or a quarter of the tiles each.  With more items than fit at once neither helps, {4, 1} has least overhead.
// A dK/dV override (comparisons and tests) keeps every kernel at {4, 1}.
struct WaveGroups { int waves, groups; };
inline bool may_divide(const Overrides& v) { return v.dkv == 0; }
// The problem as these choices see it: work items with 64 and with 128 rows (halves: two blocks under a causal mask count as one, they see half the tiles),
// 64-wide tiles that a row sweeps (block-sparse: a guess, the masks are on the GPU; a row of the butterfly mask keeps 5 to 10 blocks).
struct WorkItems {
  int64_t of64, of128;
  int tiles;
  WorkItems(const KArgs& a, bool sparse, bool halves) {
    const int64_t heads = (int64_t)a.B * a.H, blocks64 = ((int64_t)a.N + 63) / 64, blocks128 = a.T;
    of64 = heads * (halves ? (blocks64 + 1) / 2 : blocks64);
    of128 = heads * (halves ? (blocks128 + 1) / 2 : blocks128);
    tiles = sparse ? 16 : (int)blocks64;
  }
};

// The division of the forward (attn_fwd.hip), of dQ (attn_bwd.hip), and of dK and dV at d <= 64 (attn_bwd_dkv_fr.hip).
WaveGroups fwd_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide);
WaveGroups dq_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide);
WaveGroups dkv_fr_groups(const KArgs& a, int d, bool causal, bool sparse, bool divide);

// Planning workgroups of a block-sparse backward: one for kPlanCols mask columns of a head (what each clears takes no longer than the
// launch it is part of), padded to whole rounds over the XCDs; none where the columns are too short for any to be heavy.
constexpr int kPlanCols = 16;
inline int sparse_plan_groups(const KArgs& a) {
  if (a.T <= kHeavyBlocks) return 0;
  return (a.B * a.H * ((a.T + kPlanCols - 1) / kPlanCols) + kXcds - 1) / kXcds * kXcds;
}

// Launchers (defined in the .hip files).  dtype: 0 fp16, 1 bf16.  Return hipError_t as int.
int launch_fwd(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, const Overrides& v, hipStream_t s);
// ev: nullptr, or four events: two recorded before the first launch, one after the dQ kernel, one after dK/dV.
int launch_bwd(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, const Overrides& v, hipStream_t s,
               hipEvent_t* ev);
int launch_dropout_mask(const KArgs& a, uint8_t* keep, hipStream_t s);
// the dK/dV kernel that `choice` names (kDkv...); divide: its work may be divided over groups of wavefronts.  The kernel with the S->P->dV
// and dP->dS->dK halves on two wavefronts of a SIMD (attn_bwd_dkv.hip) is launched by this function itself
int launch_dkv(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, int choice, bool divide, hipStream_t s);
// dK/dV kernel for d <= 64: one wavefront does all four tile products (attn_bwd_dkv_fr.hip)
int launch_dkv_fr(const KArgs& a, int dtype, int d, bool causal, bool dropout, bool sparse, int extra_groups, bool divide,
                  hipStream_t s);
// the same at d = 128 (attn_bwd_dkv_fr128.hip)
int launch_dkv_fr128(const KArgs& a, int dtype, bool causal, bool dropout, bool sparse, int extra_groups, bool divide, hipStream_t s);
// the same with 64 keys per wavefront and the accumulators in the accumulation registers (attn_bwd_dkv_w64.hip)
int launch_dkv_w64(const KArgs& a, int dtype, bool causal, hipStream_t s);
// the whole backward pass of short dense heads at d <= 64, one launch (attn_bwd_short.hip), and which heads take it
bool bwd_short_is_faster(const KArgs& a, int d, bool causal, bool dropout);    // up to 256 tokens
bool bwd_blocks_is_faster(const KArgs& a, int d, bool causal);   // more, given a.dQpart
int launch_bwd_short(const KArgs& a, int dtype, int d, bool causal, bool dropout, hipStream_t s);
// dense forward with two wavefront groups in ping-pong (attn_fwd_pp.hip); sets its own work items
int launch_fwd_pp(const KArgs& a, int dtype, int d, bool causal, bool dropout, hipStream_t s);
// MFMA-only kernel for measuring the sustained matrix rate (attn_probe.hip); *flops = FLOPs launched
int launch_mfma_rate(int dtype, int iters, int operand_sets, float* sink, hipStream_t s, double* flops);

// a.group: how many heads the causal kernels deal out together (causal_block); head_bytes: what a head's items stream; fwd: the forward kernel asks, not a
// backward one.  All of them (0), unless their K and V exceed the last-level cache, or whole runs pay (both below), or many heads of 128 columns fill every XCD evenly or nearly so: then what an XCD streams at a time stays within 8 MiB, the L2
// working set (a level of all heads streams them all).  A run of whole groups per XCD leaves some XCDs the heavy blocks of a group and others the light ones where the
// heads do not divide evenly, and one head at a time puts blocks of the same weight on a compute unit.  us, runs | all heads, heads x N:
//   d = 128, forward  64 x 1024 37.1 | 30.0, dropout 44.2 | 34.0; 48 x 900 29.7 | 24.0; 36 x 2048 63.9 | 50.8; 20 x 4096 124 | 97.5; 12 x 8192 265 | 214;
//            96 x 1024 43.8 | 37.4; 64 x 2352 125 | 102; 300 x 300 25.5 | 31.2, 250 x 512 36.9 | 39.3, 256 x 512 33.7 | 36.8
//   d = 128, backward  64 x 1024 87 | 88; 60 x 700 58.0 | 54.5; 36 x 2048 185 | 158; 10 x 8192 699 | 582; 72 x 1024 110 | 90; 136 x 1024 191 | 164; 192 x 1024
//            233 | 225 (taken as runs all the same: 64 x 1500 145 | 151, 64 x 4096 847 | 862);   128 x 1024 150 | 158, 250 x 512 110 | 119, 256 x 512 105 | 114, 1000 x 300 234 | 239
//   d = 32, forward  96 x 2048 68.3 | 45.1; 100 x 1024 24.9 | 17.3; 60 x 1000, dropout 26.1 | 19.9; 1024 x 512 48.6 | 45.2; backward 96 x 2048 156 | 143; 1024 x 512 136 | 135
// d = 64, forward without dropout, heads that are whole runs of 32 on every XCD, pairs (causal_block) | all | runs: 1024 x 450 61.6 | 65.5 | 61.6, 1024 x 512 65.2 | 69.4 | 66.6, 512 x 512 35.9 | 36.6 | 34.4, 512 x 600
// 51.4 | 48.5 | 45.6, 768 x 512 49.6 | 52.2 | 50.1, 768 x 1536 321 | 335 | 321, 512 x 1024 102.5 | 103.5 | 102.5; with dropout even (1024 x 600 128 | 112 | 114), three blocks 512 x 300 26.2 | 21.3 | 22.4; heads
// that are not whole runs: 600 x 900 124 | 118 | 124.
// More than the 256 MB of the last-level cache: a level of all heads comes from HBM again and again.  One head at a time (pairs at d = 64) | all | runs: d = 64, forward 380 x 4106 1010 | 1090 | 1070, 638 x 3671
// 1330 | 1640 | 1370, 3175 x 738 400 | 540 | 401, 2304 x 1695 1220 | 1720 | 1240, backward 289 x 5395 3930 | 4180 | 3970, 459 x 5100 5420 | 6120 | 5470, 1817 x 2149 4370 | 5020 | 4320; d = 32, forward 992 x 4725
// 2340 | 2640 | 2420, 1502 x 5199 4200 | 4950 | 4280, backward 437 x 10720 14600 | 15800 | 14000; d = 128 55 x 14029 2720 | 3020 | 2770, backward 84 x 13932 11900 | 13300 | 12400.  At 320 MB the
// two are even at d <= 64 (d = 64 forward 751 x 1664 365 | 379 | 397, 1412 x 885 263 | 252 | 242), at 400 MB and more at d = 128 (132 x 5886 1408 | 1436 | 1535)
// and in the forward with dropout, which does more work on what it reads (837 x 1862 754 | 730 | 808, 2027 x 1214 798 | 852 | 867, 282 x 11633, 840 MB, ahead in runs by 14 %).
// d = 128, no more items than compute units: nothing is left to even out, and one head after the other (1) keeps its items on one XCD, whose L2 then
// loads K and V (or Q and dO) once.  us, all heads | one: forward 13 x 993 19.2 | 18.2, 23 x 1030 21.6 | 19.6, 35 x 677 16.6 | 15.3, 63 x 474 15.0 | 13.3, 11 x 2033 34.1 | 31.4, 5 x 4273
// 61.4 | 58.5; backward 61 x 194 23.7 | 22.4, 62 x 206 with dropout 26.5 | 24.6, 31 x 444 31.5 | 29.4, 25 x 703 with dropout 52.2 | 51.5 (but 50 x 274 28.2 | 31.9).
// Heads of one block: nothing to deal out, and the backward reads consecutive heads faster on one XCD: 1414 x 111 backward 106 | 102, forward 481 x 103 11.6 | 12.2.
// Two or three blocks of which the last is short, up to two rounds (three blocks in the forward: up to three halves) over the compute units: forward, all heads | runs of 8 |
// one head 236 x 142 12.0 | - | 10.4, 238 x 151 12.4 | - | 11.2, 164 x 308 with dropout 18.7 | 17.6 | 17.7, 245 x 342 27.0 | 26.4 | 24.3, 213 x 320 22.8 | 24.0 | 21.7, 256 x 272 21.5 |
// 24.1 | 23.4; fewer heads 230 x 195 15.4 | 16.4 | 16.3, 199 x 327 22.3 | 22.8 | 23.4; backward 250 x 206 42.2 | 40.5 | 40.1, 146 x 328 with dropout 50.0 | 47.8 | 50.9, 164 x 302
// 42.6 | 40.9 | 43.0; 224 x 197 34.4 | 36.8 | 36.9.
inline int causal_group(const KArgs& a, int d, bool sparse, bool fwd, int64_t head_bytes) {
  const int64_t heads = (int64_t)a.B * a.H, levels = a.n_items / heads;
  const int64_t fit = ((int64_t)8 << 20) / head_bytes;
  const int run = (int)(fit < 1 ? 1 : (fit > 8 ? 8 : fit));
  if (sparse) return run;
  const bool beyond_cache = heads * head_bytes > (int64_t)(d < 128 && !(fwd && a.drop_thr > 0) ? 320 : 512) << 20;
  if (d < 128) {
    if (beyond_cache) return (int)(fit < 1 ? 1 : (fit > 32 ? 32 : fit));
    return fwd && d == 64 && a.drop_thr == 0 && levels >= 4 && heads % (32 * kXcds) == 0 && heads >= 512 && heads <= 1024 ? 32 : 0;
  }
  if (levels == 1) return fwd ? 0 : 1;
  if (a.n_items <= kComputeUnits) return 1;
  if (levels <= 3 && a.n_items > (levels == 2 ? 7 : 6) * kComputeUnits / 4 && a.n_items <= 2 * kComputeUnits) return fwd ? 1 : run;
  if (levels == 3 && fwd && 2 * a.n_items >= 5 * kComputeUnits && a.n_items <= 3 * kComputeUnits) return 1;
  if (a.n_items <= 2 * kComputeUnits) return 0;
  return beyond_cache || heads >= 224 || (heads % (8 * kXcds) == 0 && (heads >= 128 || !fwd)) ? run : 0;
}

// All heads together (a.group == 0), and their number no multiple of the XCDs: a level padded to whole rounds over them (a.group = -padded; the places without a head
// end at once) keeps a head's blocks on one XCD, whose L2 then loads its K and V once, as pairs of blocks in runs of items did.  Where the padding is up to 3 %, which is also how uneven the XCDs
// become; not in the forward at d = 32 (1 % slower on average, 5 % at most).  us, pairs | unpadded | padded: d = 64, forward
// 462 x 192 12.8 | 14.6 | 12.8, 373 x 512 27.3 | 29.3 | 26.9, 441 x 450 34.1 | 33.2 | 30.4, 500 x 150 12.5 | 13.7 | 12.4; over 250 random shapes with padding forward and backward take 0.87 to 1.03 of
// the time, 0.98 on average.
inline void whole_levels(KArgs& a, int d, bool fwd, int blocks) {
  const int heads = a.B * a.H, padded = (heads + kXcds - 1) / kXcds * kXcds;
  if (a.group != 0 || padded == heads || 100 * (int64_t)padded > 103 * (int64_t)heads || (d == 32 && fwd)) return;
  a.group = -padded;
  a.n_items = padded * blocks;
  a.chunk = a.n_items / kXcds;
}

#if defined(__HIPCC__)
// ---------------------------------------------------------------- device helpers
template <typename T> struct Vec;
template <> struct Vec<_Float16> { typedef f16x8 x8; typedef f16x4 x4; };
template <> struct Vec<__bf16> { typedef bf16x8 x8; typedef bf16x4 x4; };

__device__ __forceinline__ f32x16 mfma32(f16x8 a, f16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Row sums of 16-bit probabilities on the matrix cores, "lane = query" layout.  A fragment of P^T is
// the B operand of a 32x32x16 MFMA: lane (r, g) holds eight keys of query r.  Read as the B operand of
// a 16x16x32 MFMA the same registers are column lane % 16, k group lane / 16, so the two lanes of a
// query are the two k groups of one parity, that of bit 4 of r.  With A[i][k] = 1 where the parity
// of k's group equals bit 2 of i, and 0 elsewhere, row i = 4 (lane / 16) + j of the result is the
// sum over both lanes of this lane's own query, the same in all four registers.  One such MFMA
// (16 clocks of the matrix pipe) adds a 16-key fragment of 32 queries.  The vector ALU's two-element
// dot products that did it before (four per fragment) do not run beside an MFMA: 64 of them next to 16
// 32x32x16 MFMAs take 405 ns on a SIMD with two wavefronts against 235 to 250 ns for 64 adds,
// multiplies, conversions or comparisons (219 ns for the MFMAs alone).
template <typename T> __device__ __forceinline__ typename Vec<T>::x8 row_sum_ones() {
  const int lane = threadIdx.x & 63;
  const T one = (((lane >> 4) ^ (lane >> 2)) & 1) ? (T)0.f : (T)1.f;   // k group lane / 16, row lane % 16
  typename Vec<T>::x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = one;
  return v;
}

// Online softmax, when the reference of a row is moved: when a lane's sum of the 32 probabilities it holds of a new 64-key
// tile, against the reference so far, exceeds kLazySum, or where the tile's maximum is looked for first, when that
// exceeds the reference by more than kLazyRise (base-2 exponent units).  What makes a lagging reference as accurate as
// the running maximum is that O is normalised by the sum of the ROUNDED 16-bit probabilities, the very weights
// the second product used: O stays a convex combination of V rows whatever the reference is.  It still matters how far it
// lags where a few keys dominate a row: at the reference itself a probability is exactly 1, away from it the largest is rounded as well.
// Error of O against 64 bits (bf16, d = 64, N = 2048; logits of standard deviation 4 and 8, in units of e): 8.58e-4 and
// 5.06e-4 here, 8.97e-4 and 5.37e-4 with a bar of 2^10 for the sum, 9.27e-4 and 5.54e-4 with 2^15.
constexpr float kLazySum = 256.0f, kLazyRise = 8.0f;
// How many tiles after a move another one still counts as restless, and how many quiet tiles end that (see
// softmax_tile_lane_query); the state before a row's first tile.
constexpr int kRestless = 8, kFirstTile = -kRestless - 1;

// Philox-4x32-10 (Salmon et al., SC'11): counter (c0..c3), key (k0,k1) -> 4 words.
__device__ __forceinline__ u32x4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    // the two three-way exclusive ors of a round, one instruction each
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c1 = (uint32_t)p1; c3 = (uint32_t)p0; c0 = n0; c2 = n2;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  u32x4 r = {c0, c1, c2, c3};
  return r;
}

// Dropout draw (see the contract in include/attn.h): one Philox call decides the sixteen keys
// 16 g16 .. 16 g16 + 15 of query row i; key 16 g16 + f is KEPT iff byte f % 4 of word f / 4 of the
// result is >= T.
__device__ __forceinline__ u32x4 philox_draw16(uint32_t g16, uint32_t i, uint32_t bh, uint32_t offset_lo,
                                               uint32_t seed_lo, uint32_t seed_hi) {
  return philox4x32_10(g16, i, bh, offset_lo, seed_lo, seed_hi);
}
__device__ __forceinline__ float keep_or_zero(float x, uint32_t mask) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & mask);
}
// true when the 8-bit draw in byte e (a constant, 0..3) of the word is below the threshold: the element is dropped
__device__ __forceinline__ bool dropped(uint32_t w, int e, uint32_t thr8) { return ((w >> (8 * e)) & 0xFFu) < thr8; }
// Dropout on a fragment of eight packed 16-bit values (four registers; element t in half t % 2 of
// register t / 2): element t is zeroed when its 8-bit draw, byte t % 4 of word t / 4 (w_lo, w_hi), is
// below the threshold.  Sub-dword operand addressing does the field extract, the compare and the
// half-register write in two instructions per element, on the values already rounded to 16 bits.
// thr8 and zero are registers holding T and 0.  Written out by hand because the compiler has no
// half-register select; a register written through a sub-dword destination must not be read by the
// next instruction (one wait state), which the order below keeps (the two halves of a register are
// eight instructions apart), and the closing s_nop separates the last writes from whatever follows.
template <typename T8>
__device__ __forceinline__ void drop_fragment8(T8& frag, uint32_t w_lo, uint32_t w_hi, uint32_t thr8, uint32_t zero) {
  const u32x4 p = __builtin_bit_cast(u32x4, frag);
  uint32_t p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3];
#define ATTN_DROP_HALF(REG, WORD, BYTE, HALF)                                                       \
  "v_cmp_lt_u32_sdwa vcc, " WORD ", %6 src0_sel:BYTE_" #BYTE " src1_sel:DWORD\n\t"                   \
  "v_cndmask_b32_sdwa " REG ", " REG ", %7, vcc dst_sel:WORD_" #HALF                                \
  " dst_unused:UNUSED_PRESERVE src0_sel:WORD_" #HALF " src1_sel:DWORD\n\t"
  asm volatile(
      ATTN_DROP_HALF("%0", "%4", 0, 0) ATTN_DROP_HALF("%1", "%4", 2, 0)
      ATTN_DROP_HALF("%2", "%5", 0, 0) ATTN_DROP_HALF("%3", "%5", 2, 0)
      ATTN_DROP_HALF("%0", "%4", 1, 1) ATTN_DROP_HALF("%1", "%4", 3, 1)
      ATTN_DROP_HALF("%2", "%5", 1, 1) ATTN_DROP_HALF("%3", "%5", 3, 1)
      "s_nop 1"
      : "+v"(p0), "+v"(p1), "+v"(p2), "+v"(p3)
      : "v"(w_lo), "v"(w_hi), "v"(thr8), "v"(zero)
      : "vcc");
#undef ATTN_DROP_HALF
  const u32x4 q = {p0, p1, p2, p3};
  frag = __builtin_bit_cast(T8, q);
}
// value of the lane 32 positions away (wave64)
__device__ __forceinline__ float xchg32(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // r[0] = {lo half, lo half}, r[1] = {hi half, hi half}
  const uint32_t other = (threadIdx.x & 32) ? r[0] : r[1];
  return __builtin_bit_cast(float, other);
}

// Dropout words of a 64-key tile in the "lane = query" layout (forward, dQ).  A call decides 16
// consecutive keys of the lane's query: the four calls of a tile are key block kb = 0, 1 times half
// 0, 1 of its 32 keys, and word w of a call holds keys 4 w .. 4 w + 3 of that half, which belong to
// lane g' = w % 2 of the query's two lanes, row group i4 = 2 half + w / 2.  Lane g draws half g of
// both key blocks, and the pair exchanges the words that belong to the other lane (four swaps serve
// both directions).  Result: byte e of w[kb][i4] decides element (kb, i4, e) of THIS lane.
struct KeepLQ { uint32_t w[2][4]; };
__device__ __forceinline__ KeepLQ keep_tile_lane_query(int k0, int qi, int bh, int g, uint32_t offset_lo,
                                                       uint32_t seed_lo, uint32_t seed_hi) {
  KeepLQ k;
#pragma unroll
  for (int kb = 0; kb < 2; ++kb) {
    const u32x4 r = philox_draw16((uint32_t)(k0 >> 4) + 2 * kb + g, (uint32_t)qi, (uint32_t)bh, offset_lo, seed_lo, seed_hi);
    // v_permlane32_swap(x, y): the upper 32 lanes' x and the lower 32 lanes' y change places
    auto s01 = __builtin_amdgcn_permlane32_swap(r[0], r[1], false, false);
    auto s23 = __builtin_amdgcn_permlane32_swap(r[2], r[3], false, false);
    // lane 0 now holds (own word 0, lane 1's word 0, own word 2, lane 1's word 2) = row groups 0, 2, 1, 3;
    // lane 1 holds (lane 0's word 1, own word 1, lane 0's word 3, own word 3) = row groups 0, 2, 1, 3
    k.w[kb][0] = s01[0]; k.w[kb][2] = s01[1]; k.w[kb][1] = s23[0]; k.w[kb][3] = s23[1];
  }
  return k;
}

// Lane index read by an instruction the compiler will not move: address arithmetic of a rarely
// taken path that starts from it stays inside that path instead of being hoisted out of the tile
// loop, where it would occupy registers for the whole kernel.
__device__ __forceinline__ int lane_id_here() {
  int lane = 0;
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
#endif
  return lane;
}

// Dropout in the "lane = key" layout (dK / dV kernels): a wavefront holds 32 keys (lane r, twice:
// g = 0, 1) times 32 or 64 queries; lane (r, g) holds its key for the queries i0 + 32 qb + 8 i4 + 4 g + e.
// A call decides 16 consecutive keys of one query, i.e. the 16 lanes of one row of the wavefront
// (same g, same r / 16), which all need the draws of the same 16 queries per block qb.  Lane u = r % 16
// of a row draws query (i4 = u / 4, e = u % 4) of every block and packs the keep flags into one word:
//   threshold test of the four fields of a word at once, in three instructions: with H the top bit of
//     each byte, (w | H) - T (T below 128: no borrow between the bytes) has the top bit set where the
//     lower seven bits reach T; the field is kept if that bit OR its own top bit is set.  For T of 128
//     and more, T - 128 is subtracted and the two bits are ANDed; OR and AND are the majority of the two
//     and a constant.
//   the flags of word t of block qb (key 4 t + byte) end up at bit 8 byte + 4 qb + t.
// The 16 lanes of the row then transpose their 16 x 16 flags (both blocks at once): four exchanges,
// each swapping one bit of the lane number with one bit of the position in the word, by DPP moves in
// the vector ALU.  Every lane ends up with the flags of its OWN key in one word, the one of query
// (qb, i4, e) at the constant bit 8 e + 4 qb + i4, so that an element costs one bit extract in either pass.
// (Before, the packing took twelve instructions per word instead of five and the words of all sixteen lanes were
// fetched, through LDS or by row broadcasts, in both passes over a tile.  dK/dV with dropout 0.1: BERT-large shape
// 60.3 -> 57.3 us, B H = 64, N = 4096, d = 64: 720 -> 682 us, causal 400 -> 392 us.)
// The per-lane constants sit in a small LDS table (two reads per tile): in registers they made the forms
// that are short of them spill.
struct KeepLK {
  static constexpr int kTable = 64 * 8;   // words of LDS
  const uint32_t* tab;
  uint32_t sub, maj;            // threshold test (uniform)
  // table: filled by the first wavefront of the workgroup; the caller synchronises before the first draw
  __device__ __forceinline__ void init(uint32_t* table, uint32_t thr8) {
    const uint32_t lane = threadIdx.x & 63u;
    sub = (thr8 & 127u) * 0x01010101u;
    maj = thr8 < 128u ? 0xFFFFFFFFu : 0u;
    tab = table;
    if (threadIdx.x < 64u) {
      uint32_t* t = table + 8 * lane;
      t[0] = lane & 8u ? 2u : 30u;
      t[1] = lane & 8u ? 0xCCCCCCCCu : 0x33333333u;
      t[2] = lane & 4u ? 1u : 31u;
      t[3] = lane & 4u ? 0xAAAAAAAAu : 0x55555555u;
      t[4] = lane & 2u ? 0x07060302u : 0x01000504u;
      t[5] = lane & 1u ? 0x07030501u : 0x02060004u;
      t[6] = 8u * ((lane & 15u) >> 2) + 4u * (lane >> 5) + (lane & 3u);   // query of the block that the lane draws
      t[7] = (lane & 31u) >> 4;                                           // its group of 16 keys
    }
  }
  // flags of the four words of a call, appended to those of the calls before
  __device__ __forceinline__ uint32_t pack(const u32x4& w, uint32_t before) const {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t x = (w[t] | 0x80808080u) - sub;
      const uint32_t kept = __builtin_amdgcn_bitop3_b32(x, w[t], maj, 0xE8);
      before = (kept & 0x80808080u) | (before >> 1);
    }
    return before;
  }
  template <int CTRL> static __device__ __forceinline__ uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
  }
  static __device__ __forceinline__ uint32_t select(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }
  // own key's flags for BLOCKS blocks of 32 queries from i0 on, keys kw0 .. kw0 + 31 (a multiple of 16); a single
  // block takes the place of qb = 1
  template <int BLOCKS>
  __device__ __forceinline__ uint32_t draw(int i0, int kw0, int bh, uint32_t offset_lo, uint32_t seed_lo, uint32_t seed_hi) const {
    const uint32_t* const mine = tab + 8 * lane_id_here();   // (an address the compiler does not keep for the whole loop)
    const u32x4 hi = *(const u32x4*)(mine + 4);
    uint32_t x = 0;
#pragma unroll
    for (int qb = 0; qb < BLOCKS; ++qb)
      x = pack(philox_draw16((uint32_t)(kw0 >> 4) + hi[3], (uint32_t)(i0 + 32 * qb) + hi[2], (uint32_t)bh, offset_lo, seed_lo, seed_hi), x);
    const u32x4 k = *(const u32x4*)mine;
    uint32_t t = dpp<0x128>(x);                          // lane ^ 8: rotate the row by 8
    x = select(k[1], x, __builtin_amdgcn_alignbit(t, t, k[0]));
    t = dpp<0x1B>(dpp<0x141>(x));                        // lane ^ 4: mirror eight, then reverse four
    x = select(k[3], x, __builtin_amdgcn_alignbit(t, t, k[2]));
    x = __builtin_amdgcn_perm(x, dpp<0x4E>(x), hi[0]);   // lane ^ 2
    return __builtin_amdgcn_perm(x, dpp<0xB1>(x), hi[1]);   // lane ^ 1
  }
  // all ones if the lane's key is kept for query (qb, i4, e)
  static __device__ __forceinline__ uint32_t mask(uint32_t own, int qb, int i4, int e) {
    return (uint32_t)__builtin_amdgcn_sbfe((int)own, 8 * e + 4 * qb + i4, 1);
  }
};
// Z dP - D for one element: dP times keep_scale where the key was kept (mask all ones), times zero
// where it was dropped, plus -D, as one multiply-add with a masked factor
__device__ __forceinline__ float dropped_dp_minus_d(float dp, float keep_scale, uint32_t mask, float neg_d) {
  return __builtin_fmaf(dp, __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, keep_scale) & mask), neg_d);
}

// Online softmax of one 64-key tile in the "lane = query" layout of the forward kernels (Algorithm 2
// of the paper's follow-up formulation of Algorithm 1's inner loop, base 2): s holds the raw logits
// S^T (two 32-key blocks; lane (r, g) has query row q0 + r and keys 32 kb + 8 (i / 4) + 4 g + i % 4)
// (masked ones set to -inf); pf receives the unnormalised probabilities rounded to T as the four
// 16-key B-operand fragments of O^T += V^T P^T, with dropout applied.  Masks keys beyond `last`
// on tiles that cross the causal diagonal or the end of the sequence, moves the running reference
// m_run (and rescales o, l_run, lr_run) only when a lane of the wavefront outgrew it by kLazySum,
// and keeps two row sums, both before dropout: l_run, this lane's share, of the exact
// probabilities (for the saved statistic), and lr_run, complete, of the rounded ones (the normaliser of O).
// The vector ALU bounds the forward at d <= 64 (65 % of the issue slots at N = 2048): a logit costs an
// fma, an exp, an add and half a conversion, and no comparison: the maximum of a tile is only
// looked for when the sum of its probabilities asks for it (170 -> 138 vector instructions per tile;
// B H = 128, N = 2048, d = 64: 166.8 -> 154.2 us; d = 32, N = 4096: 227 -> 209 us; d = 128, N = 4096: 495 -> 487 us).
// `calm` (the same in all lanes) keeps tiles that are likely to move the reference from forming their probabilities twice.
// Above 0 it counts the tiles since the last move, and the next tile is tried as it is.  From 0 down the tile looks for its maximum
// first and moves the reference by that: the first tile, and after two moves within kRestless tiles every one until
// kRestless in a row have moved nothing (peaked rows, logits that rise along the keys).  us, with the trial on every tile | this | a maximum
// on every tile: logits that rise by 0.1 per key (in units of e), B H = 128, N = 2048, d = 64 205 | 170 | 173, d = 32, N = 700
// 27.8 | 22.2 | 21.6, B H = 64, d = 128, N = 4096 596 | 531 | 514; Gaussian logits of standard deviation 8: 178 | 172 | 173,
// 25.6 | 22.2 | 21.4, 539 | 540 | 525; standard deviation 1, N = 512 causal 38.1 | 36.1, GPT-2 shape 39.8 | 38.1 | 41.8.
// PACK_LATE: probabilities are rounded after the two passes have met, not inside each.  The exps then have more room between
// them, for 13 registers more (d = 128, B H = 64, N = 1024 causal with dropout 40.8 -> 39.4 us; BERT-large shape 34.6 -> 34.1);
// the causal d = 64 forms spill with it (N = 512 38.2 -> 46 us).
template <typename T, int DB, bool CAUSAL, bool DROPOUT, bool PACK_LATE>
__device__ __forceinline__ void softmax_tile_lane_query(const KArgs& a, f32x16 (&s)[2], f32x16 (&o)[DB],
                                                        typename Vec<T>::x8 (&pf)[4], float& m_run, float& l_run,
                                                        f32x4& lr_run, int& calm, const typename Vec<T>::x8& ones, float c, int k0, int q0, int qi, int len, int g,
                                                        int bh) {
  if ((CAUSAL && k0 + 63 > q0) || k0 + 64 > len) {   // diagonal tiles, and the padded last tile
    const int last = CAUSAL ? min(qi, len - 1) : len - 1;   // last visible key of this row
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = k0 + 32 * kb + 8 * (i >> 2) + 4 * g + (i & 3);
        if (key > last) s[kb][i] = -INFINITY;
      }
  }
  // Probabilities against the reference the row has, with no look at the tile's maximum: their sum
  // says whether the reference still serves.  (A row that has seen no key has m_run = -inf: its sum is inf or NaN.)
  float neg_m = -m_run;
  float psum;
  f32x16 pr[2];      // PACK_LATE: the probabilities
  uint32_t pw[16];   // else: the P^T fragments, in whole words, so that the two passes meet in 16 registers and not in 32
                     // halves that are packed again (5 % of the forms with dropout)
  auto probabilities = [&]() __attribute__((always_inline)) {
    typedef T T2 __attribute__((ext_vector_type(2)));
    float part[2] = {0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        T2 pair;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][i + e], c, neg_m));
          part[e] += p;
          if constexpr (PACK_LATE) pr[kb][i + e] = p;
          else pair[e] = (T)p;
        }
        if constexpr (!PACK_LATE) pw[8 * kb + i / 2] = __builtin_bit_cast(uint32_t, pair);
      }
    psum = part[0] + part[1];
  };
  bool search = calm <= 0, move = false;
  if (__builtin_expect(!search, 1)) {
    probabilities();
    search = move = __builtin_amdgcn_ballot_w64(!(psum <= kLazySum)) != 0;
    ++calm;
  }
  if (__builtin_expect(search, 0)) {
    float mx = s[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kb][i]);
    mx = fmaxf(mx, xchg32(mx)) * c;
    if (move) calm = calm <= kRestless ? -kRestless : 1;
    else if ((move = __builtin_amdgcn_ballot_w64(mx > m_run + kLazyRise) != 0)) calm = calm < -kRestless ? 1 : -kRestless;
    else ++calm;
    if (move) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.f : m_new));
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) lr_run[i] *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] *= alpha;
    }
    neg_m = m_run == -INFINITY ? 0.f : -m_run;
    probabilities();
    // A row with a logit that is not a number (an input that is not finite, or a product beyond float32) must not
    // reach the sum of row r +- 16, which shares its column of the MFMA below and is separated from it by factors 0:
    // its probabilities become zeros, and l_run, which is NaN from here on, makes its O NaN in the epilogue.
    if (__builtin_amdgcn_ballot_w64(psum != psum) != 0) {
      const bool number = psum == psum;
      if constexpr (PACK_LATE) {
#pragma unroll
        for (int i = 0; i < 32; ++i) pr[i >> 4][i & 15] = number ? pr[i >> 4][i & 15] : 0.f;
      } else {
#pragma unroll
        for (int w = 0; w < 16; ++w) pw[w] = number ? pw[w] : 0u;
      }
    }
  }
  l_run += psum;
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) {   // 16-key chunk cc
    if constexpr (PACK_LATE) {
#pragma unroll
      for (int t = 0; t < 8; ++t) pf[cc][t] = (T)pr[cc >> 1][8 * (cc & 1) + t];
    } else {
      const u32x4 chunk = {pw[4 * cc], pw[4 * cc + 1], pw[4 * cc + 2], pw[4 * cc + 3]};
      pf[cc] = __builtin_bit_cast(typename Vec<T>::x8, chunk);
    }
  }
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) lr_run = mfma16(ones, pf[cc], lr_run);
  if constexpr (DROPOUT) {   // element t of chunk cc has field t % 4 of word 2 (cc & 1) + t / 4 of its block
    const KeepLQ kq = keep_tile_lane_query(k0, qi, bh, g, a.offset_lo, a.seed_lo, a.seed_hi);
#pragma unroll
    for (int cc = 0; cc < 4; ++cc)
      drop_fragment8(pf[cc], kq.w[cc >> 1][2 * (cc & 1)], kq.w[cc >> 1][2 * (cc & 1) + 1], a.drop_thr, 0u);
  }
}

// Work-item index for this workgroup: consecutive items share an XCD (workgroups are
// dealt round-robin to the 8 XCDs, each with its own L2).  Returns -1 for padding groups.
__device__ __forceinline__ int xcd_item(int n_items, int chunk, int id = (int)blockIdx.x) {
  const int item = (id % kXcds) * chunk + id / kXcds;
  return item < n_items && (id / kXcds) < chunk ? item : -1;
}
// Asks for the arguments that a dense kernel reads before its first tile in one go: left to itself, the compiler loads what stands behind each branch of the
// prologue behind it, and a problem of few tiles waits for the scalar cache two to four times in a row, about 0.08 us each (one head of 128 tokens, d = 64:
// 4.71 us with three such waits, 4.79 with four, 4.44 so; dQ of 64 causal heads of 4096, d = 128, with the head as one value below, 374 -> 369 us).  In the forward and in dQ; no
// gain in the two-group forward (487 | 488), nor from the dropout arguments (16 heads of 8 x 1024, causal, forward 39.4 | 39.5).
__device__ __forceinline__ void args_at_once(const KArgs& a) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::"s"(a.n_items), "s"(a.chunk), "s"(a.deal), "s"(a.H), "s"(a.N), "s"(a.T), "s"(a.klen), "s"(a.sb), "s"(a.sh), "s"(a.sn), "s"(a.Q), "s"(a.K),
               "s"(a.V));
#endif
}
// The head that the dealt-out position `pos` of a dense problem stands for.  xcd_item gives each XCD a run of consecutive positions.  With a
// key-padding mask the heads of a batch entry cost what its length says, and entries of like length tend to stand together
// (batches sorted by length), so that one XCD would get the long ones: there the j-th head of XCD x is 8 j + (x + j) % 8.  (Not
// 8 j + x: heads of 64 KB that are 512 KB apart fall on the same quarter of an L2: 16 x 16 heads of 512, causal, d = 64, backward 64 us.)  Every
// XCD still has whole heads, whose K and V (or Q and dO) its L2 holds.  Without a mask all heads cost the same, and positions are heads; nor do heads of one
// block of rows gain (64 x 12 of 128, d = 64: forward 11.5 | 12.0).  us, forward + backward, lengths from N to N / 2 in falling order, runs of
// heads | dealt round: 16 x 8 of 700, d = 32 68.3 | 57.7, d = 64 101 | 86, d = 128 166 | 145; 16 x 16 of 512, dropout 127 | 109, causal 82 | 78; 5 x 12 of
// 1000 88 | 72; 16 x 16 of 1024 316 | 246; 4 x 16 of 4096, d = 128 1958 | 1338; 8 x 16 of 1024 causal with dropout, d = 128 216 | 181; 32 x 12 of 197 46.4 | 44.9.
__device__ __forceinline__ int dealt_head(const KArgs& a, int pos) {
  int head = pos;
  if (__builtin_expect(a.deal, 0)) {   // (out of the way, so that no jump stands before the first loads)
    const int n = a.B * a.H, whole = n / kXcds, rest = n % kXcds;   // XCDs below `rest` have one head more
    const int in_long = rest * (whole + 1);
    const int x = pos < in_long ? pos / (whole + 1) : rest + (pos - in_long) / (whole > 0 ? whole : 1);
    const int j = pos - x * whole - (x < rest ? x : rest);
    head = j * kXcds + (j < whole ? (x + j) % kXcds : x);
  }
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(head));   // one value from here on
#endif
  return head;
}
// The dense causal kernels of one block of rows (or keys) per work item: this workgroup's item
// (-1: none), and the item's head and block, counted from the head's heaviest, level 0.  The blocks of all heads (a.group <= 0) or of a.group consecutive heads
// (each XCD a run of items) are dealt out together, heaviest first, so that a compute unit gets blocks of different weights at the start and light ones
// last.  All heads: see causal_group.  (The order of the heads: see dealt_head.)  At d <= 64 an item was a pair of a light and a heavy block before: half as many
// workgroups, a loop over the two that cost registers, and an odd block that counted as a pair.  us, pairs | blocks: d = 64, forward 16 x 16384 619 | 600, 128 x 1024 with dropout
// 40.8 | 34.5, 128 x 2048 98 | 91, 100 x 700 with dropout 31.3 | 22.2, 16 x 700 12.1 | 9.1; backward 16 x 16384 1950 | 1860, 16 x 8192 502 | 516, with dropout 712 | 703, 16 x 4096 136 | 141, 24 x 8192 771 | 728, 128 x 1024 94 | 95, with dropout 111 | 109, 100 x 700 with dropout 79.5 |
// 59.7, 40 x 1024 48.6 | 40.3, 16 x 700 30.9 | 22.9; d = 32, backward 128 x 700 40.7 | 33.9.
__device__ __forceinline__ int causal_item(const KArgs& a) {
  if (a.group > 0) return xcd_item(a.n_items, a.chunk);
  return (int)blockIdx.x < a.n_items ? (int)blockIdx.x : -1;
}
// (false: a place without a head; PADDED: there may be some, whole_levels)
template <bool PADDED = true>
__device__ __forceinline__ bool causal_block(const KArgs& a, int item, int n_levels, int& head, int& level) {
  const int n_heads = a.B * a.H;
  if (!PADDED && a.group == 0) {
    head = item % n_heads;
    level = item / n_heads;
    const int j = head / kXcds;
    if (j < n_heads / kXcds) head = j * kXcds + (head + j) % kXcds;
  } else if (!PADDED) {   // (the form in which the compiler lays out the forward at d = 32 best: the other one costs its long sweeps 1 %, 5 % at most)
    const int grp0 = item / n_levels / a.group * a.group;
    const int gsz = min(a.group, n_heads - grp0);
    const int within = item - grp0 * n_levels;
    head = grp0 + within % gsz;
    level = within / gsz;
  } else if (a.group <= 0) {
    const int in_level = a.group < 0 ? -a.group : n_heads;
    head = item % in_level;
    level = item / in_level;
    if (head >= n_heads) return false;
    const int j = head / kXcds;
    if (j < n_heads / kXcds) head = j * kXcds + (head + j) % kXcds;
  } else {   // (one division for a.group == 1, and few in front of the first loads: 653 heads of 42 tokens, d = 128, pay 0.3 us of 10.4 for three)
    const uint32_t per = (uint32_t)(a.group * n_levels), grp = (uint32_t)item / per, within = (uint32_t)item - grp * per;
    head = (int)grp * a.group;   // first head of this group
    level = (int)within;
    if (a.group > 1) {
      const uint32_t gsz = (uint32_t)min(a.group, n_heads - head);   // heads in it (the last group may be short)
      level = (int)(within / gsz);
      head += (int)(within - (uint32_t)level * gsz);
    }
  }
  return true;
}
// XOR swizzle of the 16-byte chunk index inside an unpadded [rows][D] LDS tile.  It makes both
// access patterns used on the tiles conflict-free on a 64-bank LDS: 16 consecutive rows at one
// chunk (row-wise 16-byte operand reads) and 4 consecutive rows x 64 bytes (transposing reads).
template <int D> __device__ __forceinline__ int swz_bits(int row) {
  if constexpr (D == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
  else if constexpr (D == 64) return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
  else return (row >> 2) & 3;   // D == 32: four chunks per row, four rows per 256 bytes
}
template <int D> __device__ __forceinline__ int lds_off(int row, int chunk) {
  return row * D + ((chunk ^ swz_bits<D>(row)) << 3);
}

// Iterates, in increasing order, over the 64-wide tiles a workgroup must visit.
// Dense: first .. limit-1 (in tiles).  Sparse: the two 64-wide halves of every 128-block b in
// [first, limit) with mask[b * stride] != 0.  All state is wavefront-uniform.
// Sparse only: the first `skip` kept blocks are passed over and at most `take` are delivered.
template <bool SPARSE> struct TileIter {
  const uint8_t* mask;
  int64_t stride;
  int limit, pos, base, half, skip, take;
  uint64_t bits;
  __device__ __forceinline__ void init(const uint8_t* m, int64_t st, int first, int lim,
                                       int skip_blocks = 0, int take_blocks = 0x7fffffff) {
    mask = m; stride = st; limit = lim; pos = first; bits = 0; base = 0; half = -1;
    skip = skip_blocks; take = take_blocks;
  }
  // The next GROUPS tiles, one for each group of wavefronts; own: that of `group`, -1 past the end.  False once there is none for any.
  template <int GROUPS> __device__ __forceinline__ bool next_of(int group, int& own) {
    own = next();
    const bool any = own >= 0;
#pragma unroll
    for (int k = 1; k < GROUPS; ++k) {
      const int t = next();
      if (group == k) own = t;
    }
    return any;
  }
  __device__ __forceinline__ int next() {
    if constexpr (!SPARSE) {
      return pos < limit ? pos++ : -1;
    } else {
      if (half >= 0) { const int t = half; half = -1; return t; }
      if (take <= 0) return -1;
      while (true) {
        while (bits == 0) {
          if (pos >= limit) return -1;
          const int blk = pos + (int)(threadIdx.x & 63);
          const bool on = blk < limit && mask[(int64_t)blk * stride] != 0;
          bits = __ballot(on);
          base = pos;
          pos += 64;
          const int n = __builtin_popcountll(bits);
          if (n <= skip) { skip -= n; bits = 0; }   // the whole chunk is before this segment
        }
        const int b = __builtin_ctzll(bits);
        bits &= bits - 1;
        if (skip > 0) { --skip; continue; }
        --take;
        half = 2 * (base + b) + 1;
        return 2 * (base + b);
      }
    }
  }
};
#endif  // __HIPCC__

}  // namespace attn
