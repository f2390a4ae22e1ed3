// Optimal Variance Filtering per group (paper Sec. 4.2, Eq. 10; in-loop form in Sec. 5.1), the
// group-normalised advantages (Eq. 5, Eq. 18) and the small index kernels around a prune.
//
// Why k+1 candidates per group are enough: with the other members fixed the variance is a convex
// quadratic in one member's value, so some optimum is "j lowest and k-j highest".
// Two decompositions for groups of at most 64 members (the paper's groups, cf. the group-size
// ablation), both with the same order of fp64 additions and therefore the same bits:
//   few groups: one 64-lane wavefront owns one group: ranks by all-pairs comparison of values from LDS (equal ones
//   are told apart afterwards), fp64 prefix sums by a six-step scan, k+1 candidate scores in lanes 0..k, a butterfly
//   arg-max, a ballot for the survivor mask.  4096 groups of 64 are four waves per SIMD, whose instructions bound it:
//   9.9 us with the slot in every comparison and scans and arg-max by shuffles through LDS, 7.8 here;
//   many groups: one LANE owns one group (ovf_select_lanes_kernel below).
#include <algorithm>
#include <mutex>
#include <type_traits>
#include "ctx.hpp"
#include "operands.hpp"
#include "philox.hpp"

namespace pg {

constexpr int OVF_WAVES = 4;           // groups per workgroup
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;          // groups per lane in the offsets scan
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_ITEMS;

__device__ __forceinline__ double shfl_up_f64(double v, int delta) { return __shfl_up(v, delta, WAVE); }

// Inclusive prefix sums of four values across the wave by the doubling recurrence: after the pass with distance dd lane i holds
// the sum of lanes max(0, i-2dd+1) .. i.  The order of additions is part of the library's bit-exactness contract.  A lane
// that has no partner adds +0, which changes nothing: no sum here is -0.  Distances 1, 2 and 4 are that many shifts by one lane, 16
// and 32 exchanges of rows, without the shuffles through LDS that 8 takes.
template <class Shift>
__device__ __forceinline__ double add_shifted(double v, Shift shift) {
  const uint64_t w = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = shift((uint32_t)w), hi = shift((uint32_t)(w >> 32));
  return __dadd_rn(v, __builtin_bit_cast(double, (uint64_t)hi << 32 | lo));
}
template <int LANES> __device__ __forceinline__ uint32_t shifted(uint32_t v) {          // by 1, 2 or 4 lanes, zeros move in
#pragma unroll
  for (int i = 0; i < LANES; ++i) v = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);
  return v;
}
__device__ __forceinline__ void wave_scans(double& a, double& b, double& c, double& d) {
  const int lane = threadIdx.x & (WAVE - 1);
  auto all = [&](auto shift) { a = add_shifted(a, shift); b = add_shifted(b, shift); c = add_shifted(c, shift); d = add_shifted(d, shift); };
  all([](uint32_t v) { return shifted<1>(v); });
  all([](uint32_t v) { return shifted<2>(v); });
  all([](uint32_t v) { return shifted<4>(v); });
  const int at8 = 4 * (lane - 8);
  all([&](uint32_t v) { const uint32_t t = (uint32_t)__builtin_amdgcn_ds_bpermute(at8, (int)v); return lane >= 8 ? t : 0u; });
  all([&](uint32_t v) {                              // rows 1 and 3 get rows 0 and 2, row 2 gets row 1
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const auto q = __builtin_amdgcn_permlane32_swap(r[1], r[1], false, false);
    return lane & 16 ? (uint32_t)r[0] : lane & 32 ? (uint32_t)q[0] : 0u;
  });
  all([&](uint32_t v) { const auto q = __builtin_amdgcn_permlane32_swap(v, v, false, false); return lane & 32 ? (uint32_t)q[0] : 0u; });
}

// A group whose size or count the selection cannot take (size outside 1..limit, k outside 1..size): its mask is
// empty and the error flag is raised, but the k slots that the offsets scan reserved for it in sel_idx are still
// filled with row indices that exist (its own rows, else row 0), so that a caller who gathers before reading
// the status stays in bounds.  The scan counts a negative k as 0.
__device__ __forceinline__ int counted_k(int k) { return k > 0 ? k : 0; }
__device__ __forceinline__ void fill_bad_group(int32_t* __restrict__ sel_idx, int out0, int b, int n, int k, int lane,
                                               int lanes) {
  for (int i = lane; i < k; i += lanes) sel_idx[out0 + i] = n >= 1 ? b + (i < n ? i : n - 1) : 0;
}

// ---- where a group's survivors go: new_offsets[g] = sum of k[0..g) ----
// The selection kernels work that out themselves instead of waiting for a scan in launches of its own (three of them
// cost more than the selection: 4096 groups took 20 us, of which the selection was 6).  OFF_GIVEN: the caller knows the
// offsets (the sampling loop has them from its schedule).  OFF_DIRECT, up to OFF_DIRECT_MAX groups: a workgroup adds up all
// counts before its first group (at most 16 KB, from L2).  OFF_SUMS, above that: one launch sums blocks of SCAN_BLOCK
// counts, and a workgroup adds the sums before its block and the counts before it inside the block.
enum OffsetsFrom { OFF_GIVEN = 0, OFF_DIRECT = 1, OFF_SUMS = 2 };
constexpr int OFF_DIRECT_MAX = 4096;

// Sum over all THREADS lanes of the workgroup, the same in every lane; `part` holds one int per wave.
template <int THREADS>
__device__ __forceinline__ int block_allsum(int s, int* part) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, WAVE);
  if (THREADS == WAVE) return s;
  if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x / WAVE] = s;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int w = 0; w < THREADS / WAVE; ++w) t += part[w];
  return t;
}

// sum of k[0..first) by the whole workgroup (first < n_groups)
template <int FROM, int THREADS>
__device__ __forceinline__ int counts_before(const int32_t* __restrict__ kk, const int32_t* __restrict__ sums, int first,
                                             int* part) {
  int s = 0, from = 0;
  if (FROM == OFF_SUMS) {
    const int blk = first / SCAN_BLOCK;
    for (int i = threadIdx.x; i < blk; i += THREADS) s += sums[i];
    from = blk * SCAN_BLOCK;
  }
  int i = from + threadIdx.x;
  for (; i + 3 * THREADS < first; i += 4 * THREADS)
    s += (counted_k(kk[i]) + counted_k(kk[i + THREADS])) + (counted_k(kk[i + 2 * THREADS]) + counted_k(kk[i + 3 * THREADS]));
  for (; i < first; i += THREADS) s += counted_k(kk[i]);
  return block_allsum<THREADS>(s, part);
}

// Kernels with one wave per group: where group g's survivors start (written to new_offsets unless it is given).  Called by
// the whole workgroup; the result of a wave past the last group is not used.
template <int FROM>
__device__ __forceinline__ int place_group(const int32_t* __restrict__ kk, const int32_t* __restrict__ sums, int g, int n_groups,
                                           int32_t* new_offsets, int* part) {
  if (FROM == OFF_GIVEN) return g < n_groups ? new_offsets[g] : 0;
  const int g0 = blockIdx.x * OVF_WAVES;
  int out0 = counts_before<FROM, OVF_WAVES * WAVE>(kk, sums, g0, part);
  if (g >= n_groups) return 0;
  for (int i = g0; i < g; ++i) out0 += counted_k(kk[i]);
  if ((threadIdx.x & (WAVE - 1)) == 0) {
    new_offsets[g] = out0;
    if (g == n_groups - 1) new_offsets[n_groups] = out0 + counted_k(kk[g]);
  }
  return out0;
}

// sums[blk] = the counts of block blk, by a workgroup of SCAN_THREADS lanes
__device__ __forceinline__ void sum_block_of_counts(const int32_t* __restrict__ kk, int n, int blk, int32_t* __restrict__ sums, int* part) {
  int s = 0;
  const int base = blk * SCAN_BLOCK + threadIdx.x;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) if (base + i * SCAN_THREADS < n) s += counted_k(kk[base + i * SCAN_THREADS]);
  s = block_allsum<SCAN_THREADS>(s, part);
  if (threadIdx.x == 0) sums[blk] = s;
}
__global__ __launch_bounds__(SCAN_THREADS) void scan_block_sums_kernel(const int32_t* __restrict__ kk,
                                                                       int n, int32_t* __restrict__ sums) {
  __shared__ int part[SCAN_THREADS / WAVE];
  sum_block_of_counts(kk, n, blockIdx.x, sums, part);
}

// a group that the selection cannot take (an empty group that keeps nothing is none: its mask is simply empty)
__device__ __forceinline__ bool bad_group(int n, int k) { return (n < 1 || n > WAVE || k < 1 || k > n) && !(n == 0 && k == 0); }
// the first k slots (1 <= k <= 64)
__device__ __forceinline__ uint64_t first_slots(int k) { return k == WAVE ? ~0ull : (1ull << k) - 1ull; }

// the lane's reward of a group (anything past its end)
__device__ __forceinline__ float reward_of_lane(const float* __restrict__ rewards, int b, int n) {
  const int lane = threadIdx.x & (WAVE - 1);
  return lane < n ? rewards[b + lane] : 0.0f;
}

// the better of two candidates: the larger score, the smaller index of equal ones
__device__ __forceinline__ void keep_better(double& score, int& best, double os, int ob) {
  const bool other = os > score || (os == score && ob < best);
  score = other ? os : score;
  best = other ? ob : best;
}
__device__ __forceinline__ double from_halves(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo); }
// the best candidate of the wave, in every lane: a butterfly inside rows of 16 lanes by data-parallel primitives (see head_sum), then
// over the rows
template <int CTRL> __device__ __forceinline__ uint32_t permuted(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xF, 0xF, false);
}
template <int CTRL> __device__ __forceinline__ void best_of_permuted(double& score, int& best) {
  const uint64_t w = __builtin_bit_cast(uint64_t, score);
  keep_better(score, best, from_halves(permuted<CTRL>((uint32_t)w), permuted<CTRL>((uint32_t)(w >> 32))), (int)permuted<CTRL>((uint32_t)best));
}
template <bool HALVES> __device__ __forceinline__ void best_of_rows(double& score, int& best) {
  const uint64_t w = __builtin_bit_cast(uint64_t, score);
  auto swap = [](uint32_t v) {
    if (HALVES) return __builtin_amdgcn_permlane32_swap(v, v, false, false);
    else return __builtin_amdgcn_permlane16_swap(v, v, false, false);
  };
  const auto lo = swap((uint32_t)w), hi = swap((uint32_t)(w >> 32)), b = swap((uint32_t)best);
  score = from_halves((uint32_t)lo[0], (uint32_t)hi[0]);             // one of the two is the lane's own
  best = (int)b[0];
  keep_better(score, best, from_halves((uint32_t)lo[1], (uint32_t)hi[1]), (int)b[1]);
}
__device__ __forceinline__ void wave_best(double& score, int& best) {
  best_of_permuted<0xB1>(score, best);
  best_of_permuted<0x4E>(score, best);
  best_of_permuted<0x141>(score, best);
  best_of_permuted<0x140>(score, best);
  best_of_rows<false>(score, best);
  best_of_rows<true>(score, best);
}

// Ranks under the order (value, slot) from `rank`, the count of smaller values (-1 past the end of the group); `sorted`: 64 floats of LDS
// of this wave.  The values that several members have are gone through one by one.  Calls of 2^20 groups 64 -> 40 with 1, 2, 12 and 32
// different values take 888, 897, 999 and 1084 us; with a second round of comparisons, of slots where values are equal, 1221 whatever
// the values, with value and slot compared from the start 1170, for values without ties, too (those take 875).
__device__ __forceinline__ int ranks_by_slot(int rank, float* sorted) {
  const int lane = threadIdx.x & (WAVE - 1);
  auto settle = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  if (rank >= 0) sorted[rank] = __builtin_bit_cast(float, lane);     // one member of each value stays
  settle();
  uint64_t left = __ballot(rank >= 0 && __builtin_bit_cast(int, sorted[max(rank, 0)]) != lane);
  settle();
  while (left) {
    const int first = __builtin_amdgcn_readlane(rank, __builtin_ctzll(left));
    const uint64_t same = __ballot(rank == first);
    left &= ~same;
    const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, rank));
    if (rank == first) rank = at;
  }
  return rank;
}

// Optimal Variance Filtering of one group by one wavefront: the survivor mask, in every lane; `raw`: reward_of_lane; `vals`,
// `sorted`: 64 floats of LDS of this wave.
__device__ __forceinline__ uint64_t survivors_by_wave(float raw, int n, int k, float* vals, float* sorted, int32_t* __restrict__ status) {
  const int lane = threadIdx.x & (WAVE - 1);
  if (n < 1 || n > WAVE || k < 1 || k > n) {        // nothing to select: empty mask
    if (lane == 0 && bad_group(n, k)) atomicOr(status, 2);
    return 0ull;
  }
  const bool live = lane < n;
  const float v = live ? raw + 0.0f : 0.0f;          // -0.0 becomes +0.0
  const bool bad = live && !(__builtin_fabsf(v) <= 3.4028234663852886e38f);
  if (__ballot(bad) != 0ull || k == n) {
    // k == n keeps everything; a non-finite reward is flagged and the first k slots are kept so
    // that every index written stays valid for the kernels that follow
    if (__ballot(bad) != 0ull && lane == 0) atomicOr(status, 1);
    return first_slots(k);
  }
  // rank under the strict order (value, slot): every value is read from LDS by all lanes at once, four at a time
  vals[lane] = live ? v : __builtin_huge_valf();
  sorted[lane] = 0.0f;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  int rank = 0;
  for (int l = 0; l < n; l += 4) {
    const float4 q = *reinterpret_cast<const float4*>(vals + l);
    rank += q.x < v ? 1 : 0;
    rank += q.y < v ? 1 : 0;
    rank += q.z < v ? 1 : 0;
    rank += q.w < v ? 1 : 0;
  }
  // members with equal values have the same count of smaller ones so far, and the counts add up to less than 0 + 1 + .. + n - 1
  if ((int)wave_allsum(live ? (float)rank : 0.f) != n * (n - 1) / 2) rank = ranks_by_slot(live ? rank : -1, sorted);
  if (live) sorted[rank] = v;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const double y = (double)sorted[lane];                           // ascending, zero padded
  const double z = live ? (double)sorted[n - 1 - lane] : 0.0;      // descending, zero padded
  double s_lo = y, s_lo2 = __dmul_rn(y, y), s_hi = z, s_hi2 = __dmul_rn(z, z);
  wave_scans(s_lo, s_lo2, s_hi, s_hi2);
  // candidate j (lane j, 0 <= j <= k <= 63): j lowest + (k - j) highest
  const int j = lane;
  const int m = k - j;                                              // taken from the top
  double lo = shfl_up_f64(s_lo, 1), lo2 = shfl_up_f64(s_lo2, 1);
  if (j == 0) { lo = 0.0; lo2 = 0.0; }
  const int srcl = (m >= 1) ? (m - 1) : 0;
  double hi = __shfl(s_hi, srcl, WAVE), hi2 = __shfl(s_hi2, srcl, WAVE);
  if (m < 1) { hi = 0.0; hi2 = 0.0; }
  const double s1 = __dadd_rn(lo, hi);
  const double s2 = __dadd_rn(lo2, hi2);
  double score = __dsub_rn(__dmul_rn((double)k, s2), __dmul_rn(s1, s1));
  int best = j;
  if (j > k) score = -__builtin_huge_val();
  wave_best(score, best);                            // arg-max, ties to the smaller j
  return __ballot(live && (rank < best || rank >= n - (k - best)));
}

template <int FROM>
__global__ __launch_bounds__(OVF_WAVES * WAVE) void ovf_select_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, const int32_t* __restrict__ kk,
    int n_groups, const int32_t* __restrict__ sums, int32_t* new_offsets, uint64_t* __restrict__ masks,
    int32_t* __restrict__ sel_idx, int32_t* __restrict__ status) {
  __shared__ __align__(16) float vals[OVF_WAVES][WAVE];
  __shared__ float sorted[OVF_WAVES][WAVE];
  __shared__ int part[OVF_WAVES];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), lane = threadIdx.x & (WAVE - 1);
  const int g = blockIdx.x * OVF_WAVES + wv;
  const bool have = g < n_groups;                   // the same in the whole wave
  const int b = have ? offsets[g] : 0, n = have ? offsets[g + 1] - b : 0, k = have ? kk[g] : 0;
  const float v = reward_of_lane(rewards, b, n);
  const int out0 = place_group<FROM>(kk, sums, g, n_groups, new_offsets, part);
  if (!have) return;                                // whole wave leaves together
  const uint64_t mask = survivors_by_wave(v, n, k, vals[wv], sorted[wv], status);
  if (lane == 0) masks[g] = mask;
  if (bad_group(n, k)) fill_bad_group(sel_idx, out0, b, n, k, lane, WAVE);
  else if ((mask >> lane) & 1ull) sel_idx[out0 + __popcll(mask & ((1ull << lane) - 1ull))] = b + lane;
}

// ---- many groups: one lane per group ----
// The wave-per-group form needs about 400 wave instructions per group, most of them cross-lane traffic (an all-pairs rank and
// four fp64 scans by shuffles): 2^20 groups of 64 -> 16 took 1.53 ms, here 0.14 (64 groups in 2812 vector, 162 LDS and 29 load
// instructions; with two waves per SIMD the vector ALU issues in 0.53 of the cycles, some instruction is active in 0.71, and a wave
// waits for memory and LDS for 0.40 of its time: instructions and exposed latency bound it together).  The kernel has 256
// registers; up to 16 of a group take 231 of them, more than 16 spill 100.  What
// took it from 0.21 ms (4462, 358 and 141 instructions): values stay floats in the sort, they stay in registers for the
// thresholds instead of being staged a second time, and whole chunks are staged by direct loads.  Here a lane
// sorts its own group in registers by a compare-exchange network (Batcher's odd-even merge sort: 543 compare-exchanges for 64
// slots, two instructions each, for 64 groups at once) and runs the scans of the same doubling recurrence on registers.
// Only the values are sorted; members are picked afterwards by comparing them with the two threshold values, with
// ties at a threshold resolved by slot.  What a lane has to index by its own n and k (the descending order, the prefix
// sums from the top) goes through LDS as [index][lane], so that every access is conflict free.
// A lane takes counts k <= 32 by that route, and everything that needs no sorting: k = n, an empty group, a group with a reward
// that is not finite, a bad count.  Groups with 32 < k < n are the wave-per-group code's, in the launch that sums the counts
// (counts_and_rest_kernel), which leaves their masks for the lanes to place; so are all 64 groups of a wave when one has a size
// outside 0..64, because the wave's rewards are then no run that fits its LDS.
constexpr int LANE_K = 32;                         // largest count of the register scans
constexpr int LANE_ROW = WAVE * WAVE + 2 * WAVE;   // staged rewards of 64 groups: one float of padding per 64, and a margin
constexpr int LANE_WAVES = 2;                      // waves per workgroup (33 KB of LDS)

// Batcher's odd-even merge sort (Knuth, vol. 3, algorithm 5.2.2M) of N registers: P the length of the sorted runs, Q the
// distance of the compare-exchanges.  Recursive templates, so that every index is a constant.
template <int N, int P, int Q>
__device__ __forceinline__ void sort_registers(float (&v)[N]) {
  if constexpr (P < N) {
#pragma unroll
    for (int i = 0; i + Q < N; ++i)
      if (i >= Q % P && (i - Q % P) % (2 * Q) < Q && i / (2 * P) == (i + Q) / (2 * P)) {
        const float lo = fminf(v[i], v[i + Q]), hi = fmaxf(v[i], v[i + Q]);
        v[i] = lo;
        v[i + Q] = hi;
      }
    if constexpr (Q > 1) sort_registers<N, P, Q / 2>(v);
    else sort_registers<N, 2 * P, 2 * P>(v);
  }
}

// inclusive prefix sums by the doubling recurrence (see wave_scans)
template <int K, int DD = 1>
__device__ __forceinline__ void scan_registers(double (&a)[K]) {
  if constexpr (DD < K) {
#pragma unroll
    for (int i = K - 1; i >= DD; --i) a[i] = __dadd_rn(a[i], a[i - DD]);
    scan_registers<K, 2 * DD>(a);
  }
}

__device__ __forceinline__ void lanes_sync() {     // this wave's LDS accesses, handed over between its lanes
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ int padded(int e) { return e + (e >> 6); }

// Rewards [first, first + total) of a wave's groups into its LDS row, total <= 4096; returns whether one is not finite.
__device__ __forceinline__ bool stage_rewards(const float* __restrict__ rewards, int first, int total, int lane, float* row) {
  bool bad = false;
#pragma unroll
  for (int c = 0; c < 64; c += 16) {
    if (c * 64 >= total) break;
    float t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i] = rewards[first + min((c + i) * 64 + lane, total - 1)];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      bad = bad || !(__builtin_fabsf(t[i]) <= 3.4028234663852886e38f);
      row[padded((c + i) * 64 + lane)] = t[i];
    }
  }
  return bad;
}
// The same where the wave's rewards are whole 16-byte chunks and every group starts with one (WHOLE below): by direct loads, in
// chunks whose positions are XOR-swizzled inside every sixteen, so that lanes that read the i-th chunk of their groups meet in
// different banks.
__device__ __forceinline__ int swizzled(int chunk) { return chunk ^ ((chunk >> 4) & 15); }
__device__ __forceinline__ bool stage_chunks(const float* rewards, int first, int total, int lane, float* row) {
  const float* base = rewards + __builtin_amdgcn_readfirstlane(first);
  const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)row);
  const int chunks = __builtin_amdgcn_readfirstlane(total) / 4, pieces = (chunks + WAVE - 1) / WAVE;
  for (int j = 0; j < pieces; ++j) dma16((uint32_t)min(swizzled(j * WAVE + lane), chunks - 1) * 16u, base, at + j * 1024u);
  wait_dma();
  lanes_sync();
  float zero = 0.f;                                  // becomes NaN with the first value that is not finite
  for (int j = 0; j < pieces; ++j) {
    const float4 q = *reinterpret_cast<const float4*>(row + 4 * (j * WAVE + lane));
    zero = __builtin_fmaf(q.x, 0.f, __builtin_fmaf(q.y, 0.f, __builtin_fmaf(q.z, 0.f, __builtin_fmaf(q.w, 0.f, zero))));
  }
  return zero != 0.f;
}
// where the wave's e-th reward is staged
template <bool WHOLE>
__device__ __forceinline__ int staged(int e) { return WHOLE ? 4 * swizzled(e >> 2) + (e & 3) : padded(e); }

// One group per lane, n <= N members from the wave's o-th staged reward on, 1 <= k < n, k <= K.  `sorts`: the lane's result is
// used; `full`: every such lane has n = N.  Returns the survivor mask.
template <int N, int K, bool WHOLE>
__device__ __forceinline__ uint64_t select_lane(const float* __restrict__ rewards, int first, int total, int o, int n, int k, bool sorts,
                                                bool full, int lane, float* row) {
  constexpr bool KEEP = K <= 16;                     // the members stay in registers for the thresholds (beside 32 counts they do not fit)
  float y[K], z[K], w[N];
  {
    float v[N];
    if (WHOLE) {
#pragma unroll
      for (int i = 0; i < N; i += 4) {
        const float4 q = *reinterpret_cast<const float4*>(row + 4 * swizzled((o + i) >> 2));
        w[i] = q.x + 0.0f; w[i + 1] = q.y + 0.0f; w[i + 2] = q.z + 0.0f; w[i + 3] = q.w + 0.0f;            // -0.0 becomes +0.0
      }
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) w[i] = row[padded(o + i)] + 0.0f;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = w[i];
    if (!full)
#pragma unroll
      for (int i = 0; i < N; ++i) v[i] = i < n ? v[i] : __builtin_huge_valf();
    lanes_sync();
    sort_registers<N, 1, 1>(v);
#pragma unroll
    for (int i = 0; i < K; ++i) y[i] = v[i];
    if (KEEP && full) {
#pragma unroll
      for (int i = 0; i < K; ++i) z[i] = v[N - 1 - i];
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) row[i * WAVE + lane] = v[i];
      lanes_sync();
#pragma unroll
      for (int i = 0; i < K; ++i) z[i] = row[max(n - 1 - i, 0) * WAVE + lane];
    }
    lanes_sync();
  }
  // Entries at or past n hold padding; they enter no sum that is used, because candidates take at most k < n of either end.
  double* top = reinterpret_cast<double*>(row);      // [K][64 lanes]
  double s1[K + 1], a[K];
#pragma unroll
  for (int i = 0; i < K; ++i) a[i] = (double)z[i];
  scan_registers<K>(a);
#pragma unroll
  for (int i = 0; i < K; ++i) top[i * WAVE + lane] = a[i];
  lanes_sync();
#pragma unroll
  for (int i = 0; i < K; ++i) a[i] = (double)y[i];
  scan_registers<K>(a);
#pragma unroll
  for (int j = 0; j <= K; ++j) {
    const int m = k - j;
    const double hi = m >= 1 ? top[(m - 1) * WAVE + lane] : 0.0;
    s1[j] = __dadd_rn(j ? a[j ? j - 1 : 0] : 0.0, hi);
  }
  lanes_sync();
#pragma unroll
  for (int i = 0; i < K; ++i) a[i] = __dmul_rn((double)z[i], (double)z[i]);
  scan_registers<K>(a);
#pragma unroll
  for (int i = 0; i < K; ++i) top[i * WAVE + lane] = a[i];
  lanes_sync();
#pragma unroll
  for (int i = 0; i < K; ++i) a[i] = __dmul_rn((double)y[i], (double)y[i]);
  scan_registers<K>(a);
  double score = -__builtin_huge_val();
  int best = 0;
  float tlo = -__builtin_huge_valf();                // largest value taken from the bottom
#pragma unroll
  for (int j = 0; j <= K; ++j) {
    const int m = k - j;
    const double hi2 = m >= 1 ? top[(m - 1) * WAVE + lane] : 0.0;
    const double s2 = __dadd_rn(j ? a[j ? j - 1 : 0] : 0.0, hi2);
    const double sc = __dsub_rn(__dmul_rn((double)k, s2), __dmul_rn(s1[j], s1[j]));
    if (j <= k && sc > score) {                      // ties stay with the smaller j
      score = sc;
      best = j;
      if (j) tlo = y[j ? j - 1 : 0];
    }
  }
  const int take_hi = k - best;
  float thi = __builtin_huge_valf();                 // smallest value taken from the top
  int quota_lo = 0, quota_hi = 0;                    // members equal to a threshold that are taken
#pragma unroll
  for (int i = 0; i < K; ++i) {
    if (i + 1 == take_hi) thi = z[i];
    quota_lo += (i < best && y[i] == tlo) ? 1 : 0;
  }
#pragma unroll
  for (int i = 0; i < K; ++i) quota_hi += (i < take_hi && z[i] == thi) ? 1 : 0;
  lanes_sync();
  uint64_t mask = 0ull;
  if (!KEEP) {
    stage_rewards(rewards, first, total, lane, row);
    lanes_sync();
    // the N addresses of the row are computed again instead of being carried in N registers from the top
    asm volatile("" : "+v"(o));
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = row[padded(o + i)];
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < n && (w[i] <= tlo || w[i] >= thi)) mask |= 1ull << i;
  // Somewhere members tie across a threshold: lowest / highest slots first.  A lane whose result is not used has no say: without
  // padding behind its two members its count never fits, and one group that keeps everything sent the whole wave through here
  // (2^20 groups of 64 -> 16, every 64th unpruned: 228 -> 153 us, 64 -> 32 297 -> 240, 32 -> 8 143 -> 102, 16 -> 4 105 -> 82).
  if (__ballot(sorts && __popcll(mask) != k) != 0ull) {
    if (KEEP) {
      stage_rewards(rewards, first, total, lane, row);
      lanes_sync();
    }
    mask = 0ull;
    for (int i = 0; i < n; ++i) {
      const float v = row[padded(o + i)];
      const bool eq = v == tlo && quota_lo > 0;
      if (v < tlo || eq) mask |= 1ull << i;
      quota_lo -= eq ? 1 : 0;
    }
    for (int i = n - 1; i >= 0; --i) {
      const float v = row[padded(o + i)];
      const bool eq = v == thi && quota_hi > 0;
      if (v > thi || eq) mask |= 1ull << i;
      quota_hi -= eq ? 1 : 0;
    }
  }
  lanes_sync();
  return mask;
}
// n_max, k_max: the largest n and k of the lanes that sort; `same`: all of them have n_max members
template <bool WHOLE>
__device__ __forceinline__ uint64_t select_lane_sized(const float* __restrict__ rewards, int first, int total, int n_max, int k_max, int o,
                                                      int n, int k, bool sorts, bool same, int lane, float* row) {
  if (n_max <= 16) return select_lane<16, 16, WHOLE>(rewards, first, total, o, n, k, sorts, same && n_max == 16, lane, row);
  if (n_max <= 32) {
    const bool full = same && n_max == 32;
    return k_max <= 16 ? select_lane<32, 16, WHOLE>(rewards, first, total, o, n, k, sorts, full, lane, row)
                       : select_lane<32, 32, WHOLE>(rewards, first, total, o, n, k, sorts, full, lane, row);
  }
  const bool full = same && n_max == 64;
  return k_max <= 16 ? select_lane<64, 16, WHOLE>(rewards, first, total, o, n, k, sorts, full, lane, row)
                     : select_lane<64, 32, WHOLE>(rewards, first, total, o, n, k, sorts, full, lane, row);
}

// whether the wave-per-group code computes the mask of a group (n members, k kept; `odd`: of a wave with a size outside 0..64)
__device__ __forceinline__ bool by_wave(int n, int k, bool odd) { return !bad_group(n, k) && (odd || (k > LANE_K && k < n)); }

// The launch before ovf_select_lanes_kernel: the first `sum_blocks` workgroups sum blocks of counts; in the others a wave looks
// at `per_wave` groups (a divisor of 64) and computes the masks of those that the lanes do not take.  Groups of that kind come
// in whole batches (a schedule that keeps 40 of 64) as well as one here and there, so they are spread over as many waves as the
// chip holds: in the wave that meets them, one after another, 16384 groups of 64 -> 40 took 234 us (here 33).
__global__ __launch_bounds__(OVF_WAVES * WAVE) void counts_and_rest_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, const int32_t* __restrict__ kk, int n_groups,
    int32_t* __restrict__ sums, int sum_blocks, int per_wave, uint64_t* __restrict__ masks, int32_t* __restrict__ status) {
  __shared__ __align__(16) float vals[OVF_WAVES][WAVE];
  __shared__ float sorted[OVF_WAVES][WAVE];
  __shared__ int part[SCAN_THREADS / WAVE];
  if ((int)blockIdx.x < sum_blocks) {
    sum_block_of_counts(kk, n_groups, blockIdx.x, sums, part);
    return;
  }
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int64_t first = ((int64_t)(blockIdx.x - sum_blocks) * OVF_WAVES + wv) * per_wave;
  if (first >= n_groups) return;
  const int chunk = (int)(first / WAVE) * WAVE, g = chunk + lane;     // the 64 groups of one wave of the lane kernel
  const bool have = g < n_groups;
  const int k = have ? kk[g] : 0, b = have ? offsets[g] : 0, n = have ? offsets[g + 1] - b : 0;
  const bool odd = __ballot(n < 0 || n > WAVE) != 0ull;
  const int own = (int)first - chunk;
  uint64_t left = __ballot(lane >= own && lane < own + per_wave && have && by_wave(n, k, odd));
  for (; left; left &= left - 1ull) {
    const int i = __builtin_ctzll(left);
    const int ni = __shfl(n, i, WAVE);
    const uint64_t mask = survivors_by_wave(reward_of_lane(rewards, __shfl(b, i, WAVE), ni), ni, __shfl(k, i, WAVE), vals[wv], sorted[wv],
                                            status);
    if (lane == 0) masks[chunk + i] = mask;
  }
}

__global__ __launch_bounds__(LANE_WAVES * WAVE, 2) void ovf_select_lanes_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, const int32_t* __restrict__ kk,
    int n_groups, const int32_t* __restrict__ sums, int32_t* __restrict__ new_offsets, uint64_t* masks,
    int32_t* __restrict__ sel_idx, int32_t* __restrict__ status) {
  __shared__ __align__(16) float rows[LANE_WAVES][LANE_ROW];
  __shared__ int part[LANE_WAVES], wave_total[LANE_WAVES];
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int g_wave = (blockIdx.x * LANE_WAVES + wv) * WAVE, g = g_wave + lane;
  const int before = counts_before<OFF_SUMS, LANE_WAVES * WAVE>(kk, sums, blockIdx.x * LANE_WAVES * WAVE, part);
  const bool have = g < n_groups;
  const int k = have ? kk[g] : 0;
  int incl = counted_k(k);
#pragma unroll
  for (int dd = 1; dd < WAVE; dd <<= 1) {
    const int t = __shfl_up(incl, dd, WAVE);
    if (lane >= dd) incl += t;
  }
  if (lane == WAVE - 1) wave_total[wv] = incl;
  __syncthreads();
  int out0 = before + incl - counted_k(k);
  for (int w = 0; w < wv; ++w) out0 += wave_total[w];
  if (have) {
    new_offsets[g] = out0;
    if (g == n_groups - 1) new_offsets[n_groups] = out0 + counted_k(k);
  }
  if (g_wave >= n_groups) return;                   // no barrier of the workgroup follows
  const int b = have ? offsets[g] : 0;
  const int n = have ? offsets[g + 1] - b : 0;
  float* row = rows[wv];
  const int members = min(WAVE, n_groups - g_wave);
  const int first = __shfl(b, 0, WAVE), total = __shfl(b + n, members - 1, WAVE) - first;
  const bool odd = __ballot(n < 0 || n > WAVE) != 0ull;
  const bool bad = have && bad_group(n, k), given = have && by_wave(n, k, odd);
  const bool whole = !odd && __ballot(have && ((b | n) & 3) != 0) == 0ull && (((uintptr_t)(rewards + first)) & 15) == 0 && total > 0;
  bool infinite = false;                             // the group holds a reward that is not finite
  if (!odd) {
    const bool some = __ballot(whole ? stage_chunks(rewards, first, total, lane, row) : stage_rewards(rewards, first, total, lane, row)) != 0ull;
    lanes_sync();
    if (some)
      for (int i = 0; i < n; ++i) {
        const int e = b - first + i;
        infinite = infinite || !(__builtin_fabsf(row[whole ? staged<true>(e) : staged<false>(e)]) <= 3.4028234663852886e38f);
      }
  }
  const bool sorts = !odd && have && !bad && !given && !infinite && k >= 1 && k < n;
  const bool any = __ballot(sorts) != 0ull;
  uint64_t mask = 0ull;
  if (any) {
    int n_max = sorts ? n : 0, k_max = sorts ? k : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      n_max = max(n_max, __shfl_xor(n_max, o, WAVE));
      k_max = max(k_max, __shfl_xor(k_max, o, WAVE));
    }
    // lanes with nothing to sort work on the first rewards of the wave, and the result is not used
    const int o = sorts ? b - first : 0, nn = sorts ? n : 2, kq = sorts ? k : 1;
    const bool same = __ballot(sorts && n != n_max) == 0ull;
    mask = whole ? select_lane_sized<true>(rewards, first, total, n_max, k_max, o, nn, kq, sorts, same, lane, row)
                 : select_lane_sized<false>(rewards, first, total, n_max, k_max, o, nn, kq, sorts, same, lane, row);
  }
  if (!sorts) mask = have && !bad && k >= 1 ? (given ? masks[g] : first_slots(k)) : 0ull;
  if (have) masks[g] = mask;
  const uint64_t bads = __ballot(bad);
  const bool flag_infinite = __ballot(infinite && !bad) != 0ull;
  if (lane == 0 && (bads != 0ull || flag_infinite)) atomicOr(status, (bads != 0ull ? 2 : 0) | (flag_infinite ? 1 : 0));
  lanes_sync();
  if (bads != 0ull) {
    int at = out0;
    for (uint64_t left = mask; left; left &= left - 1ull) sel_idx[at++] = b + __builtin_ctzll(left);
    for (uint64_t left = bads; left; left &= left - 1ull) {
      const int i = __builtin_ctzll(left);
      fill_bad_group(sel_idx, __shfl(out0, i, WAVE), __shfl(b, i, WAVE), __shfl(n, i, WAVE), __shfl(k, i, WAVE), lane, WAVE);
    }
    return;
  }
  // survivors of the wave are contiguous in sel_idx: packed in LDS first (at most 64 * 64), written out coalesced
  int* idx = reinterpret_cast<int*>(row);
  const int out_first = __shfl(out0, 0, WAVE), out_n = __shfl(out0 + k, members - 1, WAVE) - out_first;
  int at = out0 - out_first;
  for (uint64_t left = mask; left; left &= left - 1ull) idx[at++] = b + __builtin_ctzll(left);
  lanes_sync();
  for (int i = lane; i < out_n; i += WAVE) sel_idx[out_first + i] = idx[i];
}

// ---- the same selection for groups of up to 1024 members (beyond the paper's group sizes): one workgroup of
// THREADS lanes per group, one member per lane, THREADS the smallest of 128..1024 that the caller's mask words can
// name.  Same evaluation order as above with the prefix sums taken over S zero-padded slots, S = 64 up to 64
// members, else the next power of two.  A workgroup sized for 1024 members spent most of its time in the
// barriers of idle waves; the running sums keep two copies in LDS, so that a pass costs one barrier.
constexpr int OVF_LARGE = 1024;

template <int FROM, int THREADS>
__global__ __launch_bounds__(THREADS) void ovf_select_large_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, const int32_t* __restrict__ kk,
    int n_groups, const int32_t* __restrict__ sums, int32_t* new_offsets, int mask_words, uint64_t* __restrict__ masks,
    int32_t* __restrict__ sel_idx, int32_t* __restrict__ status) {
  __shared__ __align__(16) float val[THREADS];
  __shared__ float sorted[THREADS];
  __shared__ double sc[2][4][THREADS];             // running sums of y, y^2, z, z^2, two copies
  __shared__ double red_s[THREADS / WAVE];
  __shared__ int red_b[THREADS / WAVE];
  __shared__ int wave_cnt[THREADS / WAVE];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
  const int g = blockIdx.x;
  const int b = offsets[g];
  const int n = offsets[g + 1] - b;
  const int k = kk[g];
  const int out0 = counts_before<FROM, THREADS>(kk, sums, g, wave_cnt);
  if (tid == 0) {
    new_offsets[g] = out0;
    if (g == n_groups - 1) new_offsets[n_groups] = out0 + counted_k(k);
  }
  uint64_t* mrow = masks + (int64_t)g * mask_words;
  if (n < 1 || n > THREADS || n > 64 * mask_words || k < 1 || k > n) {
    if (tid == 0 && !(n == 0 && k == 0)) atomicOr(status, 2);
    if (tid < mask_words) mrow[tid] = 0ull;
    fill_bad_group(sel_idx, out0, b, n, k, tid, THREADS);
    return;                                          // whole workgroup leaves together
  }
  const bool live = tid < n;
  const float v = live ? rewards[b + tid] + 0.0f : 0.0f;
  const bool bad = live && !(__builtin_fabsf(v) <= 3.4028234663852886e38f);
  const int any_bad = __syncthreads_or(bad ? 1 : 0);
  bool keep;
  if (any_bad || k == n) {
    if (any_bad && tid == 0) atomicOr(status, 1);
    keep = tid < k;
  } else {
    val[tid] = live ? v : __builtin_huge_valf();
    sorted[tid] = 0.0f;
    __syncthreads();
    int rank = 0;
    if (wv * WAVE < n) {
      // slots before this wave's count when equal, slots behind it do not; its own 64 are compared by slot
      const int own = wv * WAVE, own_end = min(own + WAVE, n);
      for (int l = 0; l < own; l += 4) {
        const float4 q = *reinterpret_cast<const float4*>(val + l);
        rank += (q.x <= v ? 1 : 0) + (q.y <= v ? 1 : 0) + (q.z <= v ? 1 : 0) + (q.w <= v ? 1 : 0);
      }
      for (int l = own; l < own_end; ++l) rank += (val[l] < v || (val[l] == v && l < tid)) ? 1 : 0;
      for (int l = own + WAVE; l < n; l += 4) {      // past n: +inf, never below v
        const float4 q = *reinterpret_cast<const float4*>(val + l);
        rank += (q.x < v ? 1 : 0) + (q.y < v ? 1 : 0) + (q.z < v ? 1 : 0) + (q.w < v ? 1 : 0);
      }
    }
    if (live) sorted[rank] = v;
    __syncthreads();
    int S = WAVE;
    while (S < n) S <<= 1;
    const double y = (double)sorted[tid];
    const double z = live ? (double)sorted[n - 1 - tid] : 0.0;
    double run[4] = {y, __dmul_rn(y, y), z, __dmul_rn(z, z)};
    int cur = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) sc[0][q][tid] = run[q];
    __syncthreads();
    for (int dd = 1; dd < S; dd <<= 1) {             // all slots updated from the values of the previous pass
      if (tid >= dd && tid < S)
#pragma unroll
        for (int q = 0; q < 4; ++q) run[q] = __dadd_rn(run[q], sc[cur][q][tid - dd]);
      cur ^= 1;
#pragma unroll
      for (int q = 0; q < 4; ++q) sc[cur][q][tid] = run[q];
      __syncthreads();
    }
    // candidate j = tid (0 <= j <= k): j lowest + (k - j) highest
    const int j = tid, m = k - j;
    double score = -__builtin_huge_val();
    int best = j;
    if (j <= k) {
      const double lo = j ? sc[cur][0][j - 1] : 0.0, lo2 = j ? sc[cur][1][j - 1] : 0.0;
      const double hi = m ? sc[cur][2][m - 1] : 0.0, hi2 = m ? sc[cur][3][m - 1] : 0.0;
      const double s1 = __dadd_rn(lo, hi), s2 = __dadd_rn(lo2, hi2);
      score = __dsub_rn(__dmul_rn((double)k, s2), __dmul_rn(s1, s1));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {               // arg-max, ties to the smaller j
      const double os = __shfl_xor(score, o, WAVE);
      const int ob = __shfl_xor(best, o, WAVE);
      if (os > score || (os == score && ob < best)) { score = os; best = ob; }
    }
    if (lane == 0) { red_s[wv] = score; red_b[wv] = best; }
    __syncthreads();
    score = red_s[0]; best = red_b[0];
    for (int w = 1; w < THREADS / WAVE; ++w)
      if (red_s[w] > score || (red_s[w] == score && red_b[w] < best)) { score = red_s[w]; best = red_b[w]; }
    keep = live && (rank < best || rank >= n - (k - best));
  }
  const uint64_t ballot = __ballot(keep);
  __syncthreads();                                   // every wave has read what counts_before left in wave_cnt
  if (lane == 0) {
    wave_cnt[wv] = __popcll(ballot);
    if (wv < mask_words) mrow[wv] = ballot;
  }
  __syncthreads();
  if (keep) {
    int before = 0;
    for (int w = 0; w < wv; ++w) before += wave_cnt[w];
    sel_idx[out0 + before + __popcll(ballot & ((1ull << lane) - 1ull))] = b + tid;
  }
}

// ---- advantages: one wave per group ----
__device__ __forceinline__ double wave_allsum_f64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

__global__ __launch_bounds__(OVF_WAVES * WAVE) void group_advantages_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, int n_groups, double eps,
    float* __restrict__ adv) {
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int g = blockIdx.x * OVF_WAVES + wv;
  if (g >= n_groups) return;
  const int b = offsets[g], e = offsets[g + 1];
  const int n = e - b;
  // groups larger than a wave are walked in strides of 64 (not used by the sampling loop)
  double s = 0.0;
  for (int i = b + lane; i < e; i += WAVE) s += (double)rewards[i];
  const double mu = wave_allsum_f64(s) / (double)n;
  double q = 0.0;
  for (int i = b + lane; i < e; i += WAVE) { const double dv = (double)rewards[i] - mu; q += dv * dv; }
  const double sigma = sqrt(wave_allsum_f64(q) / (double)n);
  for (int i = b + lane; i < e; i += WAVE) adv[i] = (float)(((double)rewards[i] - mu) / (sigma + eps));
}

// ---- comparison arm of Sec. 4.1: a uniformly random k-subset per group ----
// Slot j of group g draws one 32-bit key, word 0 of the Philox-4x32-10 block with counter
// (j, draw, g, STREAM_SUBSAMPLE) under the run's seed; the k slots with the smallest (key, slot) stay.
constexpr uint32_t STREAM_SUBSAMPLE = 2u;

// A wave takes `per_wave` groups one after another (at most 16), so that a call of very many groups does not add up the counts
// before every four of them: with four to a workgroup 2^20 groups of 8 -> 4 took 400 us and 2^24 10.1 ms, here 242 us and 3.85.
template <int FROM>
__global__ __launch_bounds__(OVF_WAVES * WAVE) void uniform_select_kernel(
    const int32_t* __restrict__ offsets, const int32_t* __restrict__ kk, int n_groups, int per_wave,
    const int32_t* __restrict__ sums, int32_t* new_offsets, uint32_t k0, uint32_t k1, uint32_t draw,
    uint64_t* __restrict__ masks, int32_t* __restrict__ sel_idx, int32_t* __restrict__ status) {
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int64_t g0 = (int64_t)blockIdx.x * OVF_WAVES * per_wave, first = g0 + wv * per_wave;
  __shared__ int part[OVF_WAVES];
  int out0 = 0;
  if (FROM != OFF_GIVEN) {
    int s = lane < wv * per_wave && g0 + lane < n_groups ? counted_k(kk[g0 + lane]) : 0;   // of this workgroup's earlier waves
    out0 = counts_before<FROM, OVF_WAVES * WAVE>(kk, sums, (int)g0, part) + block_allsum<WAVE>(s, nullptr);
  }
  for (int64_t g = first; g < first + per_wave && g < n_groups; ++g) {
    const int b = offsets[g];
    const int n = offsets[g + 1] - b;
    const int k = kk[g];
    if (FROM == OFF_GIVEN) {
      out0 = new_offsets[g];
    } else if (lane == 0) {
      new_offsets[g] = out0;
      if (g == n_groups - 1) new_offsets[n_groups] = out0 + counted_k(k);
    }
    if (n < 1 || n > WAVE || k < 1 || k > n) {
      if (lane == 0) {
        if (bad_group(n, k)) atomicOr(status, 2);
        masks[g] = 0ull;
      }
      fill_bad_group(sel_idx, out0, b, n, k, lane, WAVE);
    } else {
      const uint32_t key = philox4x32_10(u32x4{(uint32_t)lane, draw, (uint32_t)g, STREAM_SUBSAMPLE}, k0, k1).x;
      int rank = 0;
      for (int l = 0; l < n; ++l) {
        const uint32_t kl = (uint32_t)__shfl((int)key, l, WAVE);
        rank += (kl < key || (kl == key && l < lane)) ? 1 : 0;
      }
      const bool keep = lane < n && rank < k;
      const uint64_t mask = __ballot(keep);
      if (keep) sel_idx[out0 + __popcll(mask & ((1ull << lane) - 1ull))] = b + lane;
      if (lane == 0) masks[g] = mask;
    }
    if (FROM != OFF_GIVEN) out0 += counted_k(k);
  }
}

// ---- the end of a checkpoint or of a run in one launch: a workgroup per group (of at most 64 members, the loop's) gets its rewards, and
// its first wave selects and packs, or forms the advantages.  A launch less is 4 to 6 us less of a prune, of which a loop of short
// trajectories has three: rewards, selection, packing. ----
// Where the rewards come from: REWARDS_READY, what the caller has; REWARDS_PARTIAL, the partial sums of preview_reward_kernel, at
// most 16 to a trajectory, a lane each, added in the order of reward_finish_kernel; REWARDS_DIRECT, the latents, four members of one
// chunk at a time, summed in the order of preview_reward_kernel.
enum RewardsFrom { REWARDS_READY, REWARDS_PARTIAL, REWARDS_DIRECT };
constexpr int PARTIALS_MAX = 16, DIRECT_GROUPS = 4;
struct GroupEnd {
  const float* x; const float* u; const float* w; int d4; float Pc, Qc;      // REWARDS_DIRECT; u NULL: not used
  const float* partials; int chunks;
  double bias;
  float* rewards;
  const int32_t* offsets;                          // of the members
  // selection: counts and offsets of the survivors, where they go
  const int32_t* k; const int32_t* new_offsets; uint64_t* masks; int32_t* sel_idx; int32_t* status;
  const int32_t* ids_in; int32_t* ids_out; int32_t* group_of; int32_t* offsets_out; int P;
  double eps; float* adv;                          // advantages
};
// sum of `chunks` <= 16 partials by one lane, as wave_sum_of adds them: neighbours 8, 4, 2 and 1 apart
__device__ __forceinline__ double sum_of_partials(const float* __restrict__ p, int chunks) {
  double v[PARTIALS_MAX];
#pragma unroll
  for (int c = 0; c < PARTIALS_MAX; ++c) v[c] = (double)p[min(c, chunks - 1)];
#pragma unroll
  for (int c = 0; c < PARTIALS_MAX; ++c) v[c] = c < chunks ? 0.0 + v[c] : 0.0;
#pragma unroll
  for (int o = PARTIALS_MAX / 2; o > 0; o >>= 1)
#pragma unroll
    for (int c = 0; c < o; ++c) v[c] = __dadd_rn(v[c], v[c + o]);
  return v[0];
}
template <int FROM, bool SELECT>
__global__ __launch_bounds__(FROM == REWARDS_DIRECT ? DIRECT_GROUPS * STREAM_THREADS : WAVE) void group_end_kernel(const GroupEnd a) {
  __shared__ __align__(16) float vals[WAVE];
  __shared__ float sorted[WAVE], reward[WAVE];
  const int g = blockIdx.x, lane = threadIdx.x & (WAVE - 1);
  const int b = a.offsets[g], n = a.offsets[g + 1] - b;
  float v = 0.f;
  if (FROM == REWARDS_DIRECT) {
    __shared__ float part[DIRECT_GROUPS][4];
    const int q = threadIdx.x / STREAM_THREADS, lane256 = threadIdx.x & (STREAM_THREADS - 1);
    for (int i0 = 0; i0 < n; i0 += DIRECT_GROUPS) {
      const int i = min(i0 + q, n - 1);
      const f32x4* xr = reinterpret_cast<const f32x4*>(a.x) + (size_t)(b + i) * a.d4;
      const f32x4* ur = reinterpret_cast<const f32x4*>(a.u) + (size_t)(b + i) * a.d4;
      float acc = 0.f;
#pragma unroll
      for (int it = 0; it < STREAM_ITERS; ++it) {
        const int e4 = it * STREAM_THREADS + lane256;
        if (e4 < a.d4) {
          const f32x4 xv = xr[e4], wv = reinterpret_cast<const f32x4*>(a.w)[e4];
          f32x4 h;
          if (a.u) {
            const f32x4 uv = ur[e4];
            h.x = a.Pc * xv.x + a.Qc * uv.x; h.y = a.Pc * xv.y + a.Qc * uv.y;
            h.z = a.Pc * xv.z + a.Qc * uv.z; h.w = a.Pc * xv.w + a.Qc * uv.w;
          } else {
            h.x = a.Pc * xv.x; h.y = a.Pc * xv.y; h.z = a.Pc * xv.z; h.w = a.Pc * xv.w;
          }
          acc += (wv.x * h.x + wv.y * h.y) + (wv.z * h.z + wv.w * h.w);
        }
      }
      acc = wave_allsum(acc);
      if (lane == 0) part[q][(threadIdx.x / WAVE) & 3] = acc;
      __syncthreads();
      if (lane256 == 0 && i0 + q < n) reward[i0 + q] = (float)(a.bias + (double)((part[q][0] + part[q][1]) + (part[q][2] + part[q][3])));
      __syncthreads();
    }
    if (threadIdx.x >= WAVE) return;
    if (lane < n) v = reward[lane];
  } else if (lane < n) {
    v = FROM == REWARDS_PARTIAL ? (float)(a.bias + sum_of_partials(a.partials + (size_t)(b + lane) * a.chunks, a.chunks)) : a.rewards[b + lane];
  }
  if (FROM != REWARDS_READY && lane < n) a.rewards[b + lane] = v;
  if (SELECT) {
    const int k = a.k[g], out0 = a.new_offsets[g];
    if (lane == 0) {
      a.offsets_out[g] = out0;
      if (g == a.P - 1) a.offsets_out[a.P] = a.new_offsets[a.P];
    }
    const uint64_t mask = survivors_by_wave(v, n, k, vals, sorted, a.status);
    if (lane == 0) a.masks[g] = mask;
    if ((mask >> lane) & 1ull) {
      const int at = out0 + __popcll(mask & ((1ull << lane) - 1ull));
      a.sel_idx[at] = b + lane;
      a.ids_out[at] = a.ids_in[b + lane];
      a.group_of[at] = g;
    }
  } else {                                           // as group_advantages_kernel
    const double mu = wave_allsum_f64(lane < n ? 0.0 + (double)v : 0.0) / (double)n;
    const double dv = (double)v - mu;
    const double sigma = sqrt(wave_allsum_f64(lane < n ? 0.0 + dv * dv : 0.0) / (double)n);
    if (lane < n) a.adv[b + lane] = (float)(dv / (sigma + a.eps));
  }
}

// ---- group diagnostics: sigma_G (population) and the share of members within delta sigma_G of the
// group mean (the clustered region of Eq. 7); one wave per group, any group size ----
__global__ __launch_bounds__(OVF_WAVES * WAVE) void group_stats_kernel(
    const float* __restrict__ rewards, const int32_t* __restrict__ offsets, int n_groups, double delta,
    float* __restrict__ sigma_out, float* __restrict__ share_out) {
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int g = blockIdx.x * OVF_WAVES + wv;
  if (g >= n_groups) return;
  const int b = offsets[g], e = offsets[g + 1];
  const int n = e - b;
  if (n <= 0) {
    if (lane == 0) { if (sigma_out) sigma_out[g] = 0.f; if (share_out) share_out[g] = 0.f; }
    return;
  }
  double s = 0.0;
  for (int i = b + lane; i < e; i += WAVE) s += (double)rewards[i];
  const double mu = wave_allsum_f64(s) / (double)n;
  double q = 0.0;
  for (int i = b + lane; i < e; i += WAVE) { const double dv = (double)rewards[i] - mu; q += dv * dv; }
  const double sigma = sqrt(wave_allsum_f64(q) / (double)n);
  int inside = 0;
  for (int i = b + lane; i < e; i += WAVE) inside += (fabs((double)rewards[i] - mu) <= delta * sigma) ? 1 : 0;
  for (int o = 32; o > 0; o >>= 1) inside += __shfl_xor(inside, o, WAVE);
  if (lane == 0) {
    if (sigma_out) sigma_out[g] = (float)sigma;
    if (share_out) share_out[g] = (float)((double)inside / (double)n);
  }
}

// ---- index bookkeeping around a prune ----
__global__ void gather_ids_kernel(const int32_t* __restrict__ ids_in, const int32_t* __restrict__ sel,
                                  int n_out, int32_t* __restrict__ ids_out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < n_out) ids_out[r] = ids_in[sel[r]];
}

// After a selection: ids, group and offsets of the packed survivors (group of a row: binary search in the new offsets)
__global__ void pack_state_kernel(const int32_t* __restrict__ ids_in, const int32_t* __restrict__ sel, int n_out,
                                  int32_t* __restrict__ ids_out, const int32_t* __restrict__ new_offsets, int P,
                                  int32_t* __restrict__ offsets, int32_t* __restrict__ group_of) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  for (int g = r; g <= P; g += gridDim.x * blockDim.x) offsets[g] = new_offsets[g];
  if (r >= n_out) return;
  ids_out[r] = ids_in[sel[r]];
  int lo = 0, hi = P - 1;                          // last group that starts at or before r
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (new_offsets[mid] <= r) lo = mid; else hi = mid - 1;
  }
  group_of[r] = lo;
}

// survivors imposed from outside: sel_idx from masks (test hook of the sampling loop)
__global__ void masks_to_sel_kernel(const uint64_t* __restrict__ masks, const int32_t* __restrict__ offsets,
                                    const int32_t* __restrict__ new_offsets, int n_groups,
                                    int32_t* __restrict__ sel_idx) {
  const int g = blockIdx.x;
  const int lane = threadIdx.x;
  if (g >= n_groups || lane >= WAVE) return;
  const uint64_t m = masks[g];
  const int n = offsets[g + 1] - offsets[g];
  if (lane < n && ((m >> lane) & 1ull))
    sel_idx[new_offsets[g] + __popcll(m & ((1ull << lane) - 1ull))] = offsets[g] + lane;
}

__global__ void fill_u32_kernel(uint32_t* __restrict__ p, uint32_t v, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

pg_status launch_fill_u32(void* p, uint32_t v, size_t n, hipStream_t s) {
  if (n == 0) return PG_OK;
  const unsigned blocks = (unsigned)((n + 1023) / 1024 > 4096 ? 4096 : (n + 1023) / 1024);
  fill_u32_kernel<<<dim3(blocks), dim3(256), 0, s>>>((uint32_t*)p, v, n);
  PG_LAUNCH_CHECK("fill_u32_kernel");
  return PG_OK;
}

pg_status launch_pack_state(const int32_t* ids_in, const int32_t* sel, int n_out, int32_t* ids_out, const int32_t* new_offsets,
                            int P, int32_t* offsets, int32_t* group_of, hipStream_t s) {
  pack_state_kernel<<<dim3((std::max(n_out, 1) + 255) / 256), dim3(256), 0, s>>>(ids_in, sel, n_out, ids_out, new_offsets, P,
                                                                                offsets, group_of);
  PG_LAUNCH_CHECK("pack_state_kernel");
  return PG_OK;
}

// Rewards of a run's groups from the latents, then the selection (k set) or the advantages.  REWARDS_DIRECT saves the preview's launch but
// takes a group's members four at a time, 0.4 us for each four (advantages) and 1.2 us (selection, which reads u too), with 1024 lanes
// to a group.  us, a preview of its own / direct, groups x members of d elements: selection 64 x 4 of 16 10.8 / 8.0, of 1024
// 10.7 / 8.4, of 4096 11.4 / 12.5, 64 x 12 of 1024 10.6 / 12.3, 64 x 64 of 16 12.2 / 26.8, 2048 x 4 of 16 14.0 / 18.7; advantages
// 64 x 4 of 16 9.6 / 6.2, of 4096 9.6 / 8.3, 64 x 24 of 256 9.6 / 7.8, 64 x 64 of 256 9.4 / 12.3, 512 x 12 of 1024 10.4 / 10.2,
// 2048 x 12 of 16 13.3 / 16.7.
static bool rewards_direct(const GroupEndArgs& a, int P, int N, int64_t d) {
  return P <= 512 && d <= STREAM_CHUNK && (a.k ? N <= 8 && N * d <= 8192 : N <= 24 && N * d <= 16384);
}
pg_status launch_group_end(GroupEndArgs& a, int P, int N, int M, int64_t d, hipStream_t s) {
  GroupEnd e{a.x, a.u, a.w, (int)(d / 4), (float)a.Pc, (float)a.Qc, a.partials, (int)chunks_per_traj(d), a.bias, a.rewards, a.offsets,
             a.k, a.new_offsets, a.masks, a.sel_idx, a.status, a.ids_in, a.ids_out, a.group_of, a.offsets_out, P, a.eps, a.adv};
  int from = REWARDS_DIRECT;
  if (!rewards_direct(a, P, N, d)) {
    bool unfinished = false;
    PG_TRY(launch_preview(a.x, a.u, a.w, a.rewards, M, d, a.Pc, a.Qc, a.bias, a.partials, e.chunks <= PARTIALS_MAX ? &unfinished : nullptr, s));
    from = unfinished ? REWARDS_PARTIAL : REWARDS_READY;
  }
  auto run = [&](auto select) {
    constexpr bool SELECT = decltype(select)::value;
    if (from == REWARDS_DIRECT) group_end_kernel<REWARDS_DIRECT, SELECT><<<dim3(P), dim3(DIRECT_GROUPS * STREAM_THREADS), 0, s>>>(e);
    else if (from == REWARDS_PARTIAL) group_end_kernel<REWARDS_PARTIAL, SELECT><<<dim3(P), dim3(WAVE), 0, s>>>(e);
    else group_end_kernel<REWARDS_READY, SELECT><<<dim3(P), dim3(WAVE), 0, s>>>(e);
  };
  const int rec = from == REWARDS_DIRECT ? prof_open(PROF_PREVIEW, (a.u ? 8.0 : 4.0) * (double)M * (double)d, s) : -1;
  if (a.k) run(std::true_type{});
  else run(std::false_type{});
  prof_close(rec, s);
  PG_LAUNCH_CHECK("group_end_kernel");
  return PG_OK;
}

pg_status launch_gather_ids(const int32_t* in, const int32_t* sel, int n_out, int32_t* out, hipStream_t s) {
  if (n_out <= 0) return PG_OK;
  gather_ids_kernel<<<dim3((n_out + 255) / 256), dim3(256), 0, s>>>(in, sel, n_out, out);
  PG_LAUNCH_CHECK("gather_ids_kernel");
  return PG_OK;
}

pg_status launch_masks_to_sel(const uint64_t* masks, const int32_t* offsets, const int32_t* new_offsets,
                              int n_groups, int32_t* sel_idx, hipStream_t s) {
  masks_to_sel_kernel<<<dim3(n_groups), dim3(64), 0, s>>>(masks, offsets, new_offsets, n_groups, sel_idx);
  PG_LAUNCH_CHECK("masks_to_sel_kernel");
  return PG_OK;
}

// With offsets already known (the sampling loop knows them from its schedule) the kernels only read them.
pg_status launch_uniform_select(const int32_t* offsets, const int32_t* k, int n_groups, const int32_t* new_offsets,
                                uint64_t seed, uint32_t draw, uint64_t* masks, int32_t* sel_idx, int32_t* status,
                                hipStream_t s) {
  uniform_select_kernel<OFF_GIVEN><<<dim3((n_groups + OVF_WAVES - 1) / OVF_WAVES), dim3(OVF_WAVES * WAVE), 0, s>>>(
      offsets, k, n_groups, 1, nullptr, const_cast<int32_t*>(new_offsets), (uint32_t)seed, (uint32_t)(seed >> 32), draw, masks,
      sel_idx, status);
  PG_LAUNCH_CHECK("uniform_select_kernel");
  return PG_OK;
}

pg_status launch_ovf(const float* rewards, const int32_t* offsets, const int32_t* k, int n_groups,
                     const int32_t* new_offsets, uint64_t* masks, int32_t* sel_idx, int32_t* status,
                     hipStream_t s) {
  ovf_select_kernel<OFF_GIVEN><<<dim3((n_groups + OVF_WAVES - 1) / OVF_WAVES), dim3(OVF_WAVES * WAVE), 0, s>>>(
      rewards, offsets, k, n_groups, nullptr, const_cast<int32_t*>(new_offsets), masks, sel_idx, status);
  PG_LAUNCH_CHECK("ovf_select_kernel");
  return PG_OK;
}

// block sums of k for the kernels that work out the offsets themselves (nothing to do below OFF_DIRECT_MAX groups)
static pg_status sum_counts(const int32_t* k, int n_groups, int32_t* sums, hipStream_t s) {
  if (n_groups <= OFF_DIRECT_MAX) return PG_OK;
  scan_block_sums_kernel<<<dim3((n_groups + SCAN_BLOCK - 1) / SCAN_BLOCK), dim3(SCAN_THREADS), 0, s>>>(k, n_groups, sums);
  PG_LAUNCH_CHECK("scan_block_sums_kernel");
  return PG_OK;
}

// The stand-alone selection of groups of up to 64 members.  One lane per group from LANE_MIN_GROUPS groups on, where enough
// waves of 64 groups exist to pay for each one's 20 us: wave per group against lane per group, us per call, at 8192 groups
// 15.5 / 21.0 (64 -> 16), 13.4 / 14.2 (24 -> 12), 13.0 / 10.9 (16 -> 4), at 16384 groups 24.4 / 21.2, 21.4 / 14.4, 20.8 / 11.2.
constexpr int LANE_MIN_GROUPS = 16384;
// Groups per wave of the rest, at least, and the waves that are enough to fill the chip where groups are many.  When all groups
// are the rest's (64 -> 40), 8 / 4 / 2 a wave take 43.6 / 32.7 / 30.1 us at 16384 groups and 54 / 49 / 46 at 32768 (one wave per
// group and no lanes: 38 and 62); when none is (16 -> 4 at 65536 groups) 13.8 / 14.3 / 14.3.
constexpr int REST_GROUPS = 4, REST_WAVES = 16384;
static pg_status select_groups(const float* rewards, const int32_t* offsets, const int32_t* k, int n_groups, int32_t* sums,
                               int32_t* new_offsets, uint64_t* masks, int32_t* sel_idx, int32_t* status, hipStream_t s) {
  if (n_groups >= LANE_MIN_GROUPS) {
    static_assert(SCAN_THREADS == OVF_WAVES * WAVE, "both parts of the first launch");
    int per_wave = REST_GROUPS;
    while (per_wave < WAVE && n_groups / per_wave > REST_WAVES) per_wave *= 2;
    const int sum_blocks = (n_groups + SCAN_BLOCK - 1) / SCAN_BLOCK, per_block = OVF_WAVES * per_wave;
    counts_and_rest_kernel<<<dim3(sum_blocks + (n_groups + per_block - 1) / per_block), dim3(SCAN_THREADS), 0, s>>>(
        rewards, offsets, k, n_groups, sums, sum_blocks, per_wave, masks, status);
    PG_LAUNCH_CHECK("counts_and_rest_kernel");
    ovf_select_lanes_kernel<<<dim3((n_groups + LANE_WAVES * WAVE - 1) / (LANE_WAVES * WAVE)), dim3(LANE_WAVES * WAVE), 0, s>>>(
        rewards, offsets, k, n_groups, sums, new_offsets, masks, sel_idx, status);
    PG_LAUNCH_CHECK("ovf_select_lanes_kernel");
    return PG_OK;
  }
  PG_TRY(sum_counts(k, n_groups, sums, s));
  const dim3 grid((n_groups + OVF_WAVES - 1) / OVF_WAVES), block(OVF_WAVES * WAVE);
  if (n_groups <= OFF_DIRECT_MAX)
    ovf_select_kernel<OFF_DIRECT><<<grid, block, 0, s>>>(rewards, offsets, k, n_groups, sums, new_offsets, masks, sel_idx, status);
  else
    ovf_select_kernel<OFF_SUMS><<<grid, block, 0, s>>>(rewards, offsets, k, n_groups, sums, new_offsets, masks, sel_idx, status);
  PG_LAUNCH_CHECK("ovf_select_kernel");
  return PG_OK;
}

template <int THREADS>
static pg_status select_large(const float* rewards, const int32_t* offsets, const int32_t* k, int n_groups, int32_t* sums,
                              int32_t* new_offsets, int mask_words, uint64_t* masks, int32_t* sel_idx, int32_t* status,
                              hipStream_t s) {
  if (n_groups <= OFF_DIRECT_MAX)
    ovf_select_large_kernel<OFF_DIRECT, THREADS><<<dim3(n_groups), dim3(THREADS), 0, s>>>(
        rewards, offsets, k, n_groups, sums, new_offsets, mask_words, masks, sel_idx, status);
  else
    ovf_select_large_kernel<OFF_SUMS, THREADS><<<dim3(n_groups), dim3(THREADS), 0, s>>>(
        rewards, offsets, k, n_groups, sums, new_offsets, mask_words, masks, sel_idx, status);
  PG_LAUNCH_CHECK("ovf_select_large_kernel");
  return PG_OK;
}

}  // namespace pg

using namespace pg;

extern "C" int64_t pg_ovf_scratch_ints(int64_t n_groups) {
  if (n_groups <= 0) return 0;
  return (n_groups + SCAN_BLOCK - 1) / SCAN_BLOCK + 1;
}

extern "C" pg_status pg_ovf_select(const float* rewards, const int32_t* group_offsets, const int32_t* k,
                                   int32_t n_groups, uint64_t* masks, int32_t* sel_idx,
                                   int32_t* new_offsets, int32_t* status, int32_t* scratch, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_ovf_select: n_groups = %d", n_groups);
  if (n_groups == 0) return PG_OK;
  if (!rewards || !group_offsets || !k || !masks || !sel_idx || !new_offsets || !status || !scratch)
    return fail(PG_EINVAL, "pg_ovf_select: null pointer");
  hipStream_t s = (hipStream_t)stream;
  return select_groups(rewards, group_offsets, k, n_groups, scratch, new_offsets, masks, sel_idx, status, s);
}

// ---- the same selection for callers that cannot allocate: the scan's block sums live in a file-scope device
// array (one copy per GPU, held until the process ends) instead of a buffer the caller brings ----
constexpr int NOALLOC_SCRATCH_INTS = PG_OVF_NOALLOC_MAX_GROUPS / SCAN_BLOCK + 1;
static __device__ __align__(256) int32_t g_ovf_scratch[NOALLOC_SCRATCH_INTS];

// On the host the array's name stands for the symbol, not for device memory: its address on a GPU is looked up
// once per device (with that device current) and kept.
constexpr int MAX_DEVICES = 64;
static int32_t* g_ovf_scratch_ptr[MAX_DEVICES] = {};
static std::mutex g_ovf_scratch_mu;

static pg_status ovf_scratch_on_current_device(hipStream_t s, int32_t** out) {
  int dev = -1;
  PG_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) return fail(PG_EHIP, "pg_ovf_select_noalloc: device index %d", dev);
  if (s) {
    int sdev = -1;
    PG_HIP(hipStreamGetDevice(s, &sdev));
    if (sdev != dev)
      return fail(PG_EINVAL, "pg_ovf_select_noalloc: the stream belongs to device %d, the current device is %d", sdev, dev);
  }
  std::lock_guard<std::mutex> lock(g_ovf_scratch_mu);
  if (!g_ovf_scratch_ptr[dev]) {
    void* p = nullptr;
    PG_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(g_ovf_scratch)));
    if (!p) return fail(PG_EHIP, "pg_ovf_select_noalloc: the scratch symbol has no address on device %d", dev);
    g_ovf_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_ovf_scratch_ptr[dev];
  return PG_OK;
}

extern "C" pg_status pg_ovf_select_noalloc(const float* rewards, const int32_t* group_offsets, const int32_t* k,
                                           int32_t n_groups, uint64_t* masks, int32_t* sel_idx,
                                           int32_t* new_offsets, int32_t* status, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_ovf_select_noalloc: n_groups = %d", n_groups);
  if (n_groups > PG_OVF_NOALLOC_MAX_GROUPS)
    return fail(PG_ESHAPE, "pg_ovf_select_noalloc: %d groups exceed the built-in scratch (at most %d); use pg_ovf_select",
                n_groups, PG_OVF_NOALLOC_MAX_GROUPS);
  if (n_groups == 0) return PG_OK;
  if (!rewards || !group_offsets || !k || !masks || !sel_idx || !new_offsets || !status)
    return fail(PG_EINVAL, "pg_ovf_select_noalloc: null pointer");
  hipStream_t s = (hipStream_t)stream;
  int32_t* sums = nullptr;
  PG_TRY(ovf_scratch_on_current_device(s, &sums));
  // every word of the scratch that the call reads back it has written itself
  return select_groups(rewards, group_offsets, k, n_groups, sums, new_offsets, masks, sel_idx, status, s);
}

extern "C" pg_status pg_group_advantages(const float* rewards, const int32_t* group_offsets,
                                         int32_t n_groups, double eps, float* adv, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_group_advantages: n_groups = %d", n_groups);
  if (!(eps >= 0.0)) return fail(PG_EINVAL, "pg_group_advantages: eps = %g", eps);
  if (n_groups == 0) return PG_OK;
  if (!rewards || !group_offsets || !adv) return fail(PG_EINVAL, "pg_group_advantages: null pointer");
  group_advantages_kernel<<<dim3((n_groups + OVF_WAVES - 1) / OVF_WAVES), dim3(OVF_WAVES * WAVE), 0,
                            (hipStream_t)stream>>>(rewards, group_offsets, n_groups, eps, adv);
  PG_LAUNCH_CHECK("group_advantages_kernel");
  return PG_OK;
}

extern "C" pg_status pg_uniform_select(const int32_t* group_offsets, const int32_t* k, int32_t n_groups,
                                       uint64_t seed, uint32_t draw, uint64_t* masks, int32_t* sel_idx,
                                       int32_t* new_offsets, int32_t* status, int32_t* scratch, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_uniform_select: n_groups = %d", n_groups);
  if (n_groups == 0) return PG_OK;
  if (!group_offsets || !k || !masks || !sel_idx || !new_offsets || !status || !scratch)
    return fail(PG_EINVAL, "pg_uniform_select: null pointer");
  hipStream_t s = (hipStream_t)stream;
  PG_TRY(sum_counts(k, n_groups, scratch, s));
  const int per_wave = std::min(16, std::max(1, n_groups / 32768)), per_block = OVF_WAVES * per_wave;   // 32768 waves fill the chip
  const dim3 grid(n_groups / per_block + (n_groups % per_block != 0)), block(OVF_WAVES * WAVE);
  if (n_groups <= OFF_DIRECT_MAX)
    uniform_select_kernel<OFF_DIRECT><<<grid, block, 0, s>>>(group_offsets, k, n_groups, per_wave, scratch, new_offsets,
                                                             (uint32_t)seed, (uint32_t)(seed >> 32), draw, masks, sel_idx, status);
  else
    uniform_select_kernel<OFF_SUMS><<<grid, block, 0, s>>>(group_offsets, k, n_groups, per_wave, scratch, new_offsets,
                                                           (uint32_t)seed, (uint32_t)(seed >> 32), draw, masks, sel_idx, status);
  PG_LAUNCH_CHECK("uniform_select_kernel");
  return PG_OK;
}

extern "C" pg_status pg_group_stats(const float* rewards, const int32_t* group_offsets, int32_t n_groups,
                                    double delta, float* sigma, float* clustered_share, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_group_stats: n_groups = %d", n_groups);
  if (!(delta >= 0.0)) return fail(PG_EINVAL, "pg_group_stats: delta = %g", delta);
  if (n_groups == 0) return PG_OK;
  if (!rewards || !group_offsets || (!sigma && !clustered_share)) return fail(PG_EINVAL, "pg_group_stats: null pointer");
  group_stats_kernel<<<dim3((n_groups + OVF_WAVES - 1) / OVF_WAVES), dim3(OVF_WAVES * WAVE), 0,
                       (hipStream_t)stream>>>(rewards, group_offsets, n_groups, delta, sigma, clustered_share);
  PG_LAUNCH_CHECK("group_stats_kernel");
  return PG_OK;
}

extern "C" pg_status pg_ovf_select_large(const float* rewards, const int32_t* group_offsets, const int32_t* k,
                                         int32_t n_groups, int32_t mask_words, uint64_t* masks, int32_t* sel_idx,
                                         int32_t* new_offsets, int32_t* status, int32_t* scratch, void* stream) {
  if (n_groups < 0) return fail(PG_EINVAL, "pg_ovf_select_large: n_groups = %d", n_groups);
  if (mask_words < 1 || mask_words > OVF_LARGE / WAVE)
    return fail(PG_EINVAL, "pg_ovf_select_large: mask_words = %d (1..%d)", mask_words, OVF_LARGE / WAVE);
  if (n_groups == 0) return PG_OK;
  if (!rewards || !group_offsets || !k || !masks || !sel_idx || !new_offsets || !status || !scratch)
    return fail(PG_EINVAL, "pg_ovf_select_large: null pointer");
  hipStream_t s = (hipStream_t)stream;
  // masks of one word: groups of at most 64 members, the same sums in the same order
  if (mask_words == 1) return select_groups(rewards, group_offsets, k, n_groups, scratch, new_offsets, masks, sel_idx, status, s);
  PG_TRY(sum_counts(k, n_groups, scratch, s));
  auto large = mask_words <= 2 ? select_large<128> : mask_words <= 4 ? select_large<256> : mask_words <= 8 ? select_large<512> : select_large<1024>;
  return large(rewards, group_offsets, k, n_groups, scratch, new_offsets, mask_words, masks, sel_idx, status, s);
}
