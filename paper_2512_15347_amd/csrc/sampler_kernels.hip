// Streaming (HBM-bound) kernels of the sampling loop: initial latents, the fused Euler-Maruyama
// update + Gaussian log-prob (paper Eq. 13 and the policy of Eq. 19), the one-step ODE preview with
// the linear reward proxy (Eq. 15-16), and the ragged survivor gather (Sec. 5.1, early termination).
//
// Work decomposition: 256 lanes (of the update in chunks mostly 1024) own one STREAM_CHUNK (4096 floats) of one trajectory and move it
// with 16-byte accesses; a chunk's sum is one partial, and a trajectory's partials are added up in a fixed
// order (fp64), so results do not depend on scheduling: by the workgroup itself where it holds all chunks
// of a short trajectory, else by a second tiny kernel.
#include <algorithm>
#include <type_traits>
#include "ctx.hpp"
#include "logprob.hpp"
#include "operands.hpp"
#include "philox.hpp"

namespace pg {

// Sum over the 256 lanes of the workgroup; valid in lane 0 of wave 0.
__device__ __forceinline__ float block_sum_256(float v) {
  __shared__ float part[STREAM_THREADS / WAVE];
  v = wave_allsum(v);
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  if (lane == 0) part[wv] = v;
  __syncthreads();
  float t = 0.f;
  if (threadIdx.x == 0) t = (part[0] + part[1]) + (part[2] + part[3]);
  return t;
}

// A workgroup per chunk of the update has a lane for every 16 bytes (lane_per_access): bound by HBM, which a sweep of many waves with
// one access of each array serves best.  The 1024 x 262144 update, 3.2 GB, takes 506 to 546 us with four accesses of each array in a lane
// of 256 (585 where the arrays lie at odd multiples of 4 KB) and 487 to 516 us so, by where the arrays lie and from box to box, 3 to 8 %
// apart in calls that follow other work; 6.2 to 6.6 TB/s, the plain copy 6.0 to 6.25.  After half a second without work the clocks
// give way under this form alone: the 4th to 25th call (2 to 12 ms on) take 520 to 605 us, then 500 again, with 256 lanes 540 from the
// second one on.  In a loop an update follows a network evaluation, and a dozen calls after a pause take 543 to 552 us against
// 540.  512 lanes with two accesses each take 511 to 519 us with and without a pause.  Two inputs and one output without arithmetic
// take 505 and 497, in waves of their own 471, but their sums would be 16 to a chunk.
// The bf16 storage keeps four waves: its Philox blocks bound it as much as memory (267 us; a lane per access 269, two chunks to a
// workgroup 279).
constexpr int CHUNK_THREADS = STREAM_CHUNK / 4;
// Sum over the lanes of such a workgroup, in the order of four accesses by each of 256 lanes (block_sum_256); valid in lane 0 of wave
// 0, the other waves are done.
__device__ __forceinline__ float chunk_sum(float v) {
  __shared__ float part[CHUNK_THREADS];
  part[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x >= WAVE) return 0.f;
  float w[STREAM_THREADS / WAVE];
#pragma unroll
  for (int i = 0; i < STREAM_THREADS / WAVE; ++i) {
    float s = 0.f;
#pragma unroll
    for (int it = 0; it < STREAM_ITERS; ++it) s += part[it * STREAM_THREADS + i * WAVE + threadIdx.x];
    w[i] = wave_allsum(s);
  }
  return (w[0] + w[1]) + (w[2] + w[3]);
}

__device__ __forceinline__ void init_chunk(float* __restrict__ x, int r, int c, uint32_t id, int d4, uint32_t k0, uint32_t k1) {
  f32x4* xr = reinterpret_cast<f32x4*>(x) + (size_t)r * d4;
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it) {
    const int e4 = c * (STREAM_CHUNK / 4) + it * STREAM_THREADS + threadIdx.x;
    if (e4 < d4) xr[e4] = philox_normal4((uint32_t)e4, 0u, id, STREAM_INIT, k0, k1);
  }
}
__global__ __launch_bounds__(STREAM_THREADS) void init_latents_kernel(
    float* __restrict__ x, const int32_t* __restrict__ orig_id, int d4, int chunks, uint32_t k0,
    uint32_t k1) {
  const int r = blockIdx.x / chunks;
  init_chunk(x, r, blockIdx.x - r * chunks, (uint32_t)orig_id[r], d4, k0, k1);
}

// ---- sums over a trajectory: one partial per chunk of STREAM_CHUNK elements (256 lanes), added up in fp64 in a fixed order ----
// Two decompositions with the same partials and the same order, hence the same bits:
//   a workgroup per chunk, whose partials a second launch adds up;
//   a workgroup per trajectory of at most four chunks, 256 lanes for each, which adds up its own partials: no second launch, whose
//   2 to 3 us a loop pays at every step.  Update, us a call: 64 x 1024 11.2 -> 9.4, 64 x 16384 11.2 -> 9.0, 384 x 16384
//   15.6 -> 14.7; from about 512 trajectories on the second launch is hidden and the larger workgroups fill the chip less
//   evenly (1024 x 16384: 36.0 -> 36.8), and a workgroup that walks more chunks is slower (256 x 65536: 36.0 -> 36.6,
//   272 x 65536: 38.0 -> 52.2).
constexpr int ROW_GROUPS = 4;
static bool row_per_workgroup(int64_t n_traj, int chunks) { return chunks == 1 || (chunks <= ROW_GROUPS && n_traj <= 512); }

// Sum of `chunks` values partial(c) by one wavefront, the same in every lane
template <class F>
__device__ __forceinline__ double wave_sum_of(int chunks, F partial) {
  double s = 0.0;
  for (int c = threadIdx.x & (WAVE - 1); c < chunks; c += WAVE) s += (double)partial(c);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, WAVE);
  return s;
}
// A workgroup of GROUPS x 256 lanes, 256 for each of `chunks` <= GROUPS chunks: `v` is the lane's share of its chunk (0 past the last
// one); finish(sum) is called by the first lane.
template <int GROUPS, class Finish>
__device__ __forceinline__ void row_sum(int chunks, float v, Finish finish) {
  __shared__ float part[GROUPS][4];
  v = wave_allsum(v);
  if ((threadIdx.x & (WAVE - 1)) == 0) part[threadIdx.x / STREAM_THREADS][(threadIdx.x / WAVE) & 3] = v;
  __syncthreads();
  if (threadIdx.x == 0) {                            // in the order of wave_sum_of (whose other lanes add zeros)
    double p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = i < GROUPS && i < chunks ? (double)((part[i][0] + part[i][1]) + (part[i][2] + part[i][3])) : 0.0;
    finish(GROUPS == 1 ? p[0] : (p[0] + p[2]) + (p[1] + p[3]));
  }
}
// launch(tag<GROUPS>) with the smallest workgroup that holds the chunks (0: a workgroup per chunk)
template <int N> struct groups_tag { static constexpr int value = N; };
template <class F>
static void with_groups(int chunks, F launch) {
  if (chunks == 0) launch(groups_tag<0>{});
  else if (chunks == 1) launch(groups_tag<1>{});
  else if (chunks == 2) launch(groups_tag<2>{});
  else launch(groups_tag<ROW_GROUPS>{});
}

// x_out[r] = A x[q] + B u[q] + C xi, q = src ? src[r] : r; sum xi^2 per trajectory.  GROUPS 0: a workgroup per chunk,
// which leaves its partial, or adds it to `arrived` (one word per row, 0 before and after), with a lane for every 16 bytes (WIDE) or
// 256 lanes, the same sums in the same order; else a workgroup of GROUPS x 256 lanes per trajectory.
constexpr int ARRIVED_SHIFT = 58, ARRIVED_UNIT = 36;   // 6 bits of count above 22 of whole and 36 of fractional sum
constexpr int step_lanes(int groups, bool wide) { return groups || !wide ? STREAM_THREADS : CHUNK_THREADS; }     // of a chunk
template <int GROUPS, bool WIDE>
__global__ __launch_bounds__((GROUPS ? GROUPS : 1) * step_lanes(GROUPS, WIDE)) void sde_step_kernel(
    const float* __restrict__ x, const float* __restrict__ u, float* __restrict__ x_out,
    const int32_t* __restrict__ src, const int32_t* __restrict__ orig_id, int d4, int chunks, float A,
    float B, float C, uint32_t k0, uint32_t k1, uint32_t step, float* __restrict__ partials,
    float* __restrict__ hist_next, const LogProb out, uint64_t* __restrict__ arrived) {
  constexpr int LANES = step_lanes(GROUPS, WIDE), ITERS = STREAM_CHUNK / 4 / LANES;
  const int r = GROUPS ? blockIdx.x : blockIdx.x / chunks, c = GROUPS ? threadIdx.x / STREAM_THREADS : blockIdx.x - r * chunks;
  const int at = GROUPS > 1 ? threadIdx.x & (STREAM_THREADS - 1) : threadIdx.x;
  const int q = src ? src[r] : r;
  const uint32_t id = (uint32_t)orig_id[r];
  f32x4* hn = hist_next ? reinterpret_cast<f32x4*>(hist_next) + (size_t)id * d4 : nullptr;
  const f32x4* xq = reinterpret_cast<const f32x4*>(x) + (size_t)q * d4;
  const f32x4* uq = reinterpret_cast<const f32x4*>(u) + (size_t)q * d4;
  f32x4* xo = reinterpret_cast<f32x4*>(x_out) + (size_t)r * d4;
  f32x4 xv[ITERS], uv[ITERS];
  int e4[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    e4[it] = c * (STREAM_CHUNK / 4) + it * LANES + at;
    if (e4[it] < d4) {
      xv[it] = __builtin_nontemporal_load(xq + e4[it]);
      uv[it] = __builtin_nontemporal_load(uq + e4[it]);
    }
  }
  float acc = 0.f;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    if (e4[it] < d4) {
      const f32x4 z = philox_normal4((uint32_t)e4[it], step, id, STREAM_STEP, k0, k1);
      f32x4 o;
      o.x = A * xv[it].x + B * uv[it].x + C * z.x;
      o.y = A * xv[it].y + B * uv[it].y + C * z.y;
      o.z = A * xv[it].z + B * uv[it].z + C * z.z;
      o.w = A * xv[it].w + B * uv[it].w + C * z.w;
      __builtin_nontemporal_store(o, xo + e4[it]);
      if (hn) __builtin_nontemporal_store(o, hn + e4[it]);      // trajectory record by original id
      acc += (z.x * z.x + z.y * z.y) + (z.z * z.z + z.w * z.w);
    }
  }
  if constexpr (GROUPS > 0) {
    row_sum<GROUPS>(chunks, acc, [&](double s) { finish_logprob(out, r, (int)id, s); });
  } else {
    float t;
    if constexpr (WIDE) t = chunk_sum(acc);
    else t = block_sum_256(acc);
    if (threadIdx.x != 0) return;
    if (!arrived) {
      partials[blockIdx.x] = t;
      return;
    }
    // The workgroup that adds its share last has the sum: no second launch, which a step paid 4 us for.  Sum and number of shares are
    // one 64-bit word, so that nothing else has to be ordered.  In units of 2^-36 a share of 2^-13 and more is exact, and the sum then
    // the one that fp64 gives, whatever the order (a share that small, of a last chunk of a few elements, is off by 2^-37 at most, which
    // is what fp64 rounds sums of 65536 and more to, too).
    constexpr double UNITS = (double)(1ull << ARRIVED_UNIT);
    const uint64_t share = (uint64_t)__double2ull_rn((double)t * UNITS);
    const uint64_t before = __hip_atomic_fetch_add(arrived + r, (1ull << ARRIVED_SHIFT) + share, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((int)(before >> ARRIVED_SHIFT) + 1 != chunks) return;
    __hip_atomic_store(arrived + r, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // for the next step
    finish_logprob(out, r, (int)id, (double)((before & ((1ull << ARRIVED_SHIFT) - 1)) + share) * (1.0 / UNITS));
  }
}

// The same update with the latents and the network output stored as bf16 (6 instead of 12 bytes per element):
// arithmetic in fp32, the result rounded to nearest-even.  A lane handles 8 elements per access (two Philox
// blocks); the noise of an element does not depend on the storage format.
typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float bf_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }
__device__ __forceinline__ uint32_t bf_pack(float a, float b) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)b) << 16);
}

template <int GROUPS>
__global__ __launch_bounds__((GROUPS ? GROUPS : 1) * STREAM_THREADS) void sde_step_bf16_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ u, uint16_t* __restrict__ x_out,
    const int32_t* __restrict__ src, const int32_t* __restrict__ orig_id, int d8, int chunks, float A, float B,
    float C, uint32_t k0, uint32_t k1, uint32_t step, float* __restrict__ partials, const LogProb out) {
  const int r = GROUPS ? blockIdx.x : blockIdx.x / chunks, c = GROUPS ? threadIdx.x / STREAM_THREADS : blockIdx.x - r * chunks;
  const int lane256 = GROUPS > 1 ? threadIdx.x & (STREAM_THREADS - 1) : threadIdx.x;
  const int q = src ? src[r] : r;
  const uint32_t id = (uint32_t)orig_id[r];
  const u32x4s* xq = reinterpret_cast<const u32x4s*>(x) + (size_t)q * d8;
  const u32x4s* uq = reinterpret_cast<const u32x4s*>(u) + (size_t)q * d8;
  u32x4s* xo = reinterpret_cast<u32x4s*>(x_out) + (size_t)r * d8;
  constexpr int ITERS = STREAM_CHUNK / 8 / STREAM_THREADS;         // 16-byte accesses per lane and chunk
  float acc = 0.f;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int e8 = c * (STREAM_CHUNK / 8) + it * STREAM_THREADS + lane256;
    if (e8 < d8) {
      const u32x4s xv = __builtin_nontemporal_load(xq + e8);
      const u32x4s uv = __builtin_nontemporal_load(uq + e8);
      const f32x4 z0 = philox_normal4((uint32_t)(2 * e8), step, id, STREAM_STEP, k0, k1);
      const f32x4 z1 = philox_normal4((uint32_t)(2 * e8 + 1), step, id, STREAM_STEP, k0, k1);
      u32x4s o;
      o.x = bf_pack(A * bf_lo(xv.x) + B * bf_lo(uv.x) + C * z0.x, A * bf_hi(xv.x) + B * bf_hi(uv.x) + C * z0.y);
      o.y = bf_pack(A * bf_lo(xv.y) + B * bf_lo(uv.y) + C * z0.z, A * bf_hi(xv.y) + B * bf_hi(uv.y) + C * z0.w);
      o.z = bf_pack(A * bf_lo(xv.z) + B * bf_lo(uv.z) + C * z1.x, A * bf_hi(xv.z) + B * bf_hi(uv.z) + C * z1.y);
      o.w = bf_pack(A * bf_lo(xv.w) + B * bf_lo(uv.w) + C * z1.z, A * bf_hi(xv.w) + B * bf_hi(uv.w) + C * z1.w);
      __builtin_nontemporal_store(o, xo + e8);
      acc += ((z0.x * z0.x + z0.y * z0.y) + (z0.z * z0.z + z0.w * z0.w)) +
             ((z1.x * z1.x + z1.y * z1.y) + (z1.z * z1.z + z1.w * z1.w));
    }
  }
  if constexpr (GROUPS > 0) {
    row_sum<GROUPS>(chunks, acc, [&](double s) { finish_logprob(out, r, (int)id, s); });
  } else {
    const float t = block_sum_256(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
  }
}

// sums[t, r] = sum xi^2 over the noise of step t for original id r, t = blockIdx.y: what a step's log-prob is made of, in the order of
// sde_step_kernel.  The noise depends on seed, step and id alone, so a loop whose updates are spread over several workgroups of a
// trajectory takes its sums from here instead of putting them together at every step (64 tokens of 4 channels, 8 trajectories,
// ten steps: one launch of 3 us).
__device__ __forceinline__ float noise_square_sum(int c, int lane256, int d4, uint32_t step, uint32_t id, uint32_t k0, uint32_t k1) {
  float acc = 0.f;
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it) {
    const int e4 = c * (STREAM_CHUNK / 4) + it * STREAM_THREADS + lane256;
    if (e4 < d4) {
      const f32x4 z = philox_normal4((uint32_t)e4, step, id, STREAM_STEP, k0, k1);
      acc += (z.x * z.x + z.y * z.y) + (z.z * z.z + z.w * z.w);
    }
  }
  return acc;
}
template <int GROUPS>
__global__ __launch_bounds__(GROUPS * STREAM_THREADS) void noise_sums_kernel(int d4, int chunks, uint32_t k0, uint32_t k1,
                                                                             double* __restrict__ sums) {
  const int r = blockIdx.x, step = blockIdx.y;
  const float acc = noise_square_sum(threadIdx.x / STREAM_THREADS, threadIdx.x & (STREAM_THREADS - 1), d4, (uint32_t)step, (uint32_t)r, k0, k1);
  row_sum<GROUPS>(chunks, acc, [&](double s) { sums[(size_t)step * gridDim.x + r] = s; });
}

// The kernels that finish a sum are pure latency, once per step: one wavefront per trajectory (a lane that walked its
// trajectory's partials one by one took 4 us for 16 of them and more for more).
__device__ __forceinline__ double wave_sum_partials(const float* __restrict__ p, int chunks, int stride) {
  return wave_sum_of(chunks, [&](int c) { return p[(size_t)c * stride]; });
}
constexpr int FINISH_ROWS = 4;                     // trajectories per workgroup of the finishing kernels

__global__ void logprob_finish_kernel(const float* __restrict__ partials, int chunks, int n_traj, const int32_t* __restrict__ orig_id,
                                      const LogProb out) {
  const int r = blockIdx.x * FINISH_ROWS + threadIdx.x / WAVE;
  if (r >= n_traj) return;
  const double s = wave_sum_partials(partials + (size_t)r * chunks, chunks, 1);
  if ((threadIdx.x & (WAVE - 1)) == 0) finish_logprob(out, r, orig_id[r], s);
}

// <w, Pc x + Qc u> per trajectory; GROUPS as above
template <bool WITH_U, int GROUPS>
__global__ __launch_bounds__((GROUPS ? GROUPS : 1) * STREAM_THREADS) void preview_reward_kernel(
    const float* __restrict__ x, const float* __restrict__ u, const float* __restrict__ w, int d4,
    int chunks, float Pc, float Qc, float* __restrict__ partials, double bias,
    float* __restrict__ rewards) {
  const int r = GROUPS ? blockIdx.x : blockIdx.x / chunks, c = GROUPS ? threadIdx.x / STREAM_THREADS : blockIdx.x - r * chunks;
  const int lane256 = GROUPS > 1 ? threadIdx.x & (STREAM_THREADS - 1) : threadIdx.x;
  const f32x4* xr = reinterpret_cast<const f32x4*>(x) + (size_t)r * d4;
  const f32x4* ur = reinterpret_cast<const f32x4*>(u) + (size_t)r * d4;
  const f32x4* w4 = reinterpret_cast<const f32x4*>(w);
  float acc = 0.f;
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it) {
    const int e4 = c * (STREAM_CHUNK / 4) + it * STREAM_THREADS + lane256;
    if (e4 < d4) {
      const f32x4 xv = __builtin_nontemporal_load(xr + e4);
      const f32x4 wv = w4[e4];
      f32x4 h;
      if (WITH_U) {
        const f32x4 uv = __builtin_nontemporal_load(ur + e4);
        h.x = Pc * xv.x + Qc * uv.x; h.y = Pc * xv.y + Qc * uv.y;
        h.z = Pc * xv.z + Qc * uv.z; h.w = Pc * xv.w + Qc * uv.w;
      } else {
        h.x = Pc * xv.x; h.y = Pc * xv.y; h.z = Pc * xv.z; h.w = Pc * xv.w;
      }
      acc += (wv.x * h.x + wv.y * h.y) + (wv.z * h.z + wv.w * h.w);
    }
  }
  if constexpr (GROUPS > 0) {
    row_sum<GROUPS>(chunks, acc, [&](double s) { rewards[r] = (float)(bias + s); });
  } else {
    const float t = block_sum_256(acc);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
  }
}

__global__ void reward_finish_kernel(const float* __restrict__ partials, int chunks, int n_traj,
                                     double bias, float* __restrict__ rewards) {
  const int r = blockIdx.x * FINISH_ROWS + threadIdx.x / WAVE;
  if (r >= n_traj) return;
  const double s = wave_sum_partials(partials + (size_t)r * chunks, chunks, 1);
  if ((threadIdx.x & (WAVE - 1)) == 0) rewards[r] = (float)(bias + s);
}

__global__ __launch_bounds__(STREAM_THREADS) void compact_gather_kernel(
    const float* __restrict__ x, float* __restrict__ out, const int32_t* __restrict__ src, int d4,
    int chunks) {
  const int r = blockIdx.x / chunks, c = blockIdx.x - r * chunks;
  const int q = src[r];
  const f32x4* xq = reinterpret_cast<const f32x4*>(x) + (size_t)q * d4;
  f32x4* xo = reinterpret_cast<f32x4*>(out) + (size_t)r * d4;
  f32x4 v[STREAM_ITERS];
  int e4[STREAM_ITERS];
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it) {
    e4[it] = c * (STREAM_CHUNK / 4) + it * STREAM_THREADS + threadIdx.x;
    if (e4[it] < d4) v[it] = __builtin_nontemporal_load(xq + e4[it]);
  }
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it)
    if (e4[it] < d4) __builtin_nontemporal_store(v[it], xo + e4[it]);
}

// Stored transition (x, x_next) of a survivor under another network output u (Eq. 19): two partials per
// workgroup, the squared residual |x_next - (A x + B u)|^2 and, with xi the noise the sampler drew for this
// element (regenerated from its counter) and w = residual / C the noise the new policy would need,
// sum (xi - w)(xi + w) = sum xi^2 - sum w^2 = 2 (log pi_new - log pi_old): the log-ratio is summed from its small
// per-element terms instead of being the difference of two large log-probs.
__global__ __launch_bounds__(STREAM_THREADS) void transition_sq_kernel(
    const float* __restrict__ x, const float* __restrict__ u, const float* __restrict__ x_next_by_id,
    const int32_t* __restrict__ orig_id, int d4, int chunks, float A, float B, float C, uint32_t k0, uint32_t k1,
    uint32_t step, float* __restrict__ partials) {
  __shared__ float part[2][STREAM_THREADS / WAVE];
  const int r = blockIdx.x / chunks, c = blockIdx.x - r * chunks;
  const uint32_t id = (uint32_t)orig_id[r];
  const f32x4* xr = reinterpret_cast<const f32x4*>(x) + (size_t)r * d4;
  const f32x4* ur = reinterpret_cast<const f32x4*>(u) + (size_t)r * d4;
  const f32x4* nr = reinterpret_cast<const f32x4*>(x_next_by_id) + (size_t)id * d4;
  float acc = 0.f, dif = 0.f;
#pragma unroll
  for (int it = 0; it < STREAM_ITERS; ++it) {
    const int e4 = c * (STREAM_CHUNK / 4) + it * STREAM_THREADS + threadIdx.x;
    if (e4 < d4) {
      const f32x4 xv = __builtin_nontemporal_load(xr + e4), uv = __builtin_nontemporal_load(ur + e4);
      const f32x4 nv = __builtin_nontemporal_load(nr + e4);
      const f32x4 z = philox_normal4((uint32_t)e4, step, id, STREAM_STEP, k0, k1);
      const float a0 = nv.x - (A * xv.x + B * uv.x), a1 = nv.y - (A * xv.y + B * uv.y);
      const float a2 = nv.z - (A * xv.z + B * uv.z), a3 = nv.w - (A * xv.w + B * uv.w);
      acc += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
      // divided by the very fp32 scale the sampler multiplied its noise with: a rounded reciprocal would bias every
      // term the same way, and the bias would add up over the d elements
      const float w0 = a0 / C, w1 = a1 / C, w2 = a2 / C, w3 = a3 / C;
      dif += ((z.x - w0) * (z.x + w0) + (z.y - w1) * (z.y + w1)) + ((z.z - w2) * (z.z + w2) + (z.w - w3) * (z.w + w3));
    }
  }
  acc = wave_allsum(acc);
  dif = wave_allsum(dif);
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  if (lane == 0) { part[0][wv] = acc; part[1][wv] = dif; }
  __syncthreads();
  if (threadIdx.x == 0) {
    partials[2 * (size_t)blockIdx.x] = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
    partials[2 * (size_t)blockIdx.x + 1] = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
  }
}

// logp[id] = -sum / (2 C^2) - d (ln C + 1/2 ln 2 pi);  log_ratio[id] = 1/2 sum (xi - w)(xi + w), kept in fp64
__global__ void transition_finish_kernel(const float* __restrict__ partials, int chunks, int n_traj, double inv_2c2,
                                         double log_norm, const int32_t* __restrict__ orig_id,
                                         float* __restrict__ logp_by_id, double* __restrict__ log_ratio_by_id) {
  const int r = blockIdx.x * FINISH_ROWS + threadIdx.x / WAVE;
  if (r >= n_traj) return;
  const float* p = partials + 2 * (size_t)r * chunks;
  const double s = wave_sum_partials(p, chunks, 2), dsum = wave_sum_partials(p + 1, chunks, 2);
  if ((threadIdx.x & (WAVE - 1)) != 0) return;
  logp_by_id[orig_id[r]] = (float)(-s * inv_2c2 - log_norm);
  log_ratio_by_id[orig_id[r]] = 0.5 * dsum;
}

// Eq. 19 and the first term of Eq. 20 per group: one wave per group, lanes over survivors
__global__ __launch_bounds__(256) void surrogate_kernel(const double* __restrict__ log_ratio,
                                                        const float* __restrict__ adv,
                                                        const int32_t* __restrict__ offsets,
                                                        const int32_t* __restrict__ orig_id, int n_groups, int T,
                                                        int M0, float lo, float hi, float* __restrict__ ratio,
                                                        float* __restrict__ J) {
  const int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
  const int g = blockIdx.x * 4 + wv;
  if (g >= n_groups) return;
  const int b = offsets[g], e = offsets[g + 1];
  double acc = 0.0;
  for (int i = b + lane; i < e; i += WAVE) {
    const int id = orig_id[i];
    const double a = (double)adv[i];
    for (int s = 0; s < T; ++s) {
      const double r = exp(log_ratio[(size_t)s * M0 + id]);
      ratio[(size_t)s * M0 + id] = (float)r;
      const double rc = fmin(fmax(r, (double)lo), (double)hi);
      acc += fmin(r * a, rc * a);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, WAVE);
  if (lane == 0) J[g] = (e > b) ? (float)(acc / ((double)(e - b) * T)) : 0.f;
}

static pg_status check_stream_shape(int64_t n_traj, int64_t d) {
  if (n_traj < 0 || d <= 0) return fail(PG_EINVAL, "n_traj = %lld, d = %lld", (long long)n_traj, (long long)d);
  if (d % 4 != 0) return fail(PG_ESHAPE, "latent size d = %lld must be a multiple of 4", (long long)d);
  // a launch takes less than 2^32 lanes; of more, HIP refuses a multiple of 2^32 and starts the remainder of any other number
  constexpr int64_t MOST = (1ll << 32) / STREAM_THREADS;
  if (d / 4 > INT32_MAX || n_traj >= MOST || n_traj * chunks_per_traj(d) >= MOST)
    return fail(PG_ESHAPE, "n_traj * ceil(d/4096) exceeds the grid limit");
  return PG_OK;
}

}  // namespace pg

using namespace pg;

extern "C" int64_t pg_step_scratch_floats(int64_t n_traj, int64_t d) {
  if (n_traj <= 0 || d <= 0) return 0;
  return n_traj * chunks_per_traj(d);
}

extern "C" pg_status pg_init_latents(float* x, const int32_t* orig_id, int64_t n_traj, int64_t d,
                                     uint64_t seed, void* stream) {
  PG_TRY(check_stream_shape(n_traj, d));
  if (n_traj == 0) return PG_OK;
  if (!x || !orig_id) return fail(PG_EINVAL, "pg_init_latents: null pointer");
  const int chunks = (int)chunks_per_traj(d);
  init_latents_kernel<<<dim3((unsigned)(n_traj * chunks)), dim3(STREAM_THREADS), 0, (hipStream_t)stream>>>(
      x, orig_id, (int)(d / 4), chunks, (uint32_t)seed, (uint32_t)(seed >> 32));
  PG_LAUNCH_CHECK("init_latents_kernel");
  return PG_OK;
}

namespace pg {
static pg_status launch_logprob_finish(const float* partials, int chunks, int64_t n_traj, const int32_t* orig_id, const LogProb& out,
                                       hipStream_t stream) {
  logprob_finish_kernel<<<dim3((unsigned)((n_traj + FINISH_ROWS - 1) / FINISH_ROWS)), dim3(FINISH_ROWS * WAVE), 0, stream>>>(
      partials, chunks, (int)n_traj, orig_id, out);
  PG_LAUNCH_CHECK("logprob_finish_kernel");
  return PG_OK;
}

// Whether the update of chunks has a lane for every 16 bytes: where a launch may have so many (HIP takes less than 2^32 of them; with 256
// a chunk four times as many trajectories, see check_stream_shape), and where few of them would have nothing to do.  A last chunk of a
// few elements costs 1024 lanes as much as a whole one, 256 lanes less: us with 256 / 1024 for trajectories of two chunks 4096 x 4100
// 49.3 / 54.9, 8192 x 5120 96.5 / 102.6, x 6144 109.4 / 111.8, x 7168 125.5 / 120.0, of three 8192 x 8448 136.9 / 141.5, x 10240 167.2 /
// 159.6, of four x 12544 209.5 / 215.2, x 13312 220.0 / 221.6, x 14336 243.2 / 231.6, of five x 16388 283.4 / 268.1, of six x 20484 385 /
// 360.
static bool lane_per_access(int64_t n_traj, int64_t d) {
  const int64_t chunks = chunks_per_traj(d);
  return n_traj * chunks < (1ll << 32) / CHUNK_THREADS && (chunks > 4 || 6 * d >= 5 * chunks * STREAM_CHUNK);
}

pg_status launch_sde_step(const float* x, const float* u, float* x_out, float* logp, float* logp_hist,
                          float* logp_sum, const int32_t* src, const int32_t* orig_id, int64_t n_traj, int64_t d,
                          double A, double B, double C, uint64_t seed, uint32_t step, float* partials,
                          float* hist_next, uint64_t* arrived, hipStream_t stream) {
  PG_TRY(check_stream_shape(n_traj, d));
  if (n_traj == 0) return PG_OK;
  if (!x || !u || !x_out || !orig_id || !partials) return fail(PG_EINVAL, "pg_sde_step_logprob: null pointer");
  if (x_out == x) return fail(PG_EINVAL, "pg_sde_step_logprob: x_out must not alias x");
  if (!(C > 0.0)) return fail(PG_EINVAL, "pg_sde_step_logprob: noise scale C = %g must be > 0", C);
  const int chunks = (int)chunks_per_traj(d);
  const LogProb out{logp, logp_hist, logp_sum, (double)d * (log(C) + 0.5 * log(2.0 * M_PI))};
  const bool row = row_per_workgroup(n_traj, chunks);
  const int rec = prof_open(PROF_SDE_STEP, 12.0 * (double)n_traj * (double)d, stream);
  with_groups(row ? chunks : 0, [&](auto groups) {
    constexpr int G = decltype(groups)::value;
    auto launch = [&](auto wide) {
      constexpr bool WIDE = decltype(wide)::value;
      sde_step_kernel<G, WIDE><<<dim3((unsigned)(G ? n_traj : n_traj * chunks)), dim3((G ? G : 1) * step_lanes(G, WIDE)), 0, stream>>>(
          x, u, x_out, src, orig_id, (int)(d / 4), chunks, (float)A, (float)B, (float)C, (uint32_t)seed, (uint32_t)(seed >> 32), step,
          partials, hist_next, out, arrived);
    };
    if (G || !lane_per_access(n_traj, d)) launch(std::false_type{});
    else if constexpr (G == 0) launch(std::true_type{});
  });
  prof_close(rec, stream);
  PG_LAUNCH_CHECK("sde_step_kernel");
  return row || arrived ? PG_OK : launch_logprob_finish(partials, chunks, n_traj, orig_id, out, stream);
}

// Whether an update of so many trajectories may be given `arrived`.  The shares of a trajectory arrive at one word one after another, so
// it pays for few chunks and small launches only.  us with a second launch / by arrival, trajectories x chunks: 384 x 5 22.7 / 20.4,
// 1024 x 5 43.6 / 42.2, 4096 x 5 147.8 / 160.9, 4096 x 4 135.2 / 141.7, 96 x 16 21.3 / 20.2, 384 x 16 56.5 / 57.6, 1024 x 16
// 134.7 / 138.3, 16 x 32 12.4 / 12.1, 96 x 32 33.5 / 33.3, 16 x 64 17.0 / 20.8, 96 x 64 56.0 / 61.0, 96 x 173 135 / 164.
bool sums_on_arrival(int64_t n_traj, int64_t d) {
  const int64_t chunks = chunks_per_traj(d);
  // a sum of d squared normals is below 23 d: a pair's is -2 ln u, u >= 2^-33
  static_assert(23 * 32 * STREAM_CHUNK < 1 << (ARRIVED_SHIFT - ARRIVED_UNIT) && 32 < 1 << (64 - ARRIVED_SHIFT), "sum and count have room");
  return chunks <= 32 && n_traj * chunks <= 5120;
}

// What a run starts from, in one launch: initial latents by chunk (ids are the rows), then, 256 lanes a workgroup, the sums of the noise
// of `steps` steps where they are asked for (latents of one chunk), then the state: offsets of the full groups, ids, group of
// every row, no log-prob yet (NaN), zero sums, clear status and counts.  (Two launches, with the noise three, of 2 to 3 us before.)
struct InitGroup {
  float* x; int d4, chunks; uint32_t k0, k1;
  double* sums; int steps;
  int P, N; int32_t* offsets; int32_t* ids; int32_t* group_of; uint32_t* logp_hist; size_t hist_n; float* logp_sum; int32_t* status;
  uint64_t* arrived;
  int latent_blocks, noise_blocks;
};
__global__ __launch_bounds__(STREAM_THREADS) void init_group_kernel(const InitGroup a) {
  int blk = blockIdx.x;
  if (blk < a.latent_blocks) {
    const int r = blk / a.chunks;
    init_chunk(a.x, r, blk - r * a.chunks, (uint32_t)r, a.d4, a.k0, a.k1);
    return;
  }
  blk -= a.latent_blocks;
  if (blk < a.noise_blocks) {
    const int M0 = a.P * a.N, step = blk / M0, r = blk - step * M0;
    const float acc = noise_square_sum(0, threadIdx.x, a.d4, (uint32_t)step, (uint32_t)r, a.k0, a.k1);
    row_sum<1>(1, acc, [&](double s) { a.sums[(size_t)step * M0 + r] = s; });
    return;
  }
  blk -= a.noise_blocks;
  const size_t i = (size_t)blk * STREAM_THREADS + threadIdx.x;
  const size_t stride = (size_t)(gridDim.x - a.latent_blocks - a.noise_blocks) * STREAM_THREADS;
  if (i < 4) a.status[i] = 0;
  for (size_t g = i; g <= (size_t)a.P; g += stride) a.offsets[g] = (int32_t)g * a.N;
  for (size_t r = i; r < (size_t)a.P * a.N; r += stride) {
    a.ids[r] = (int32_t)r;
    a.group_of[r] = (int32_t)(r / a.N);
    a.logp_sum[r] = 0.f;
    a.arrived[r] = 0;
  }
  for (size_t j = i; j < a.hist_n; j += stride) a.logp_hist[j] = 0x7FC00000u;
}

// `sums`: see launch_noise_sums, or NULL
pg_status launch_init_group(float* x, int P, int N, int64_t d, uint64_t seed, double* sums, int steps, int32_t* offsets, int32_t* ids,
                            int32_t* group_of, float* logp_hist, size_t hist_n, float* logp_sum, int32_t* status, uint64_t* arrived,
                            hipStream_t s) {
  const int64_t M0 = (int64_t)P * N;
  PG_TRY(check_stream_shape(M0, d));
  const int chunks = (int)chunks_per_traj(d);
  const bool noise_here = sums && chunks == 1 && M0 * steps <= (1 << 23);    // a launch has room for less than 2^24 workgroups
  InitGroup a{x, (int)(d / 4), chunks, (uint32_t)seed, (uint32_t)(seed >> 32), sums, steps, P, N, offsets, ids, group_of,
              (uint32_t*)logp_hist, hist_n, logp_sum, status, arrived, (int)(M0 * chunks), noise_here ? (int)(M0 * steps) : 0};
  const size_t n = std::max(hist_n, (size_t)M0) + 1;
  const int state_blocks = (int)std::min<size_t>((n + 255) / 256, 1024);
  // Very many latents get a launch of their own: a launch takes less than 2^32 lanes, and their workgroups start faster without the
  // rest of this kernel (us in one launch / in two: 65536 trajectories of 16 elements 36 / 38, 262144 131 / 127, 4194304 2008 / 1973).
  const bool apart = a.latent_blocks >= 1 << 17;
  if (apart) a.latent_blocks = 0;
  init_group_kernel<<<dim3((unsigned)(a.latent_blocks + a.noise_blocks + state_blocks)), dim3(STREAM_THREADS), 0, s>>>(a);
  PG_LAUNCH_CHECK("init_group_kernel");
  if (apart) PG_TRY(pg_init_latents(x, ids, M0, d, seed, s));
  return sums && !noise_here ? launch_noise_sums((int)M0, steps, d, seed, sums, s) : PG_OK;
}

pg_status launch_noise_sums(int M0, int steps, int64_t d, uint64_t seed, double* sums, hipStream_t stream) {
  const int chunks = (int)chunks_per_traj(d);
  if (d % 4 || chunks > ROW_GROUPS) return fail(PG_ESHAPE, "noise sums: latent size %lld", (long long)d);
  with_groups(chunks, [&](auto groups) {
    constexpr int G = decltype(groups)::value;
    if constexpr (G > 0)
      noise_sums_kernel<G><<<dim3((unsigned)M0, (unsigned)steps), dim3(G * STREAM_THREADS), 0, stream>>>(
          (int)(d / 4), chunks, (uint32_t)seed, (uint32_t)(seed >> 32), sums);
  });
  PG_LAUNCH_CHECK("noise_sums_kernel");
  return PG_OK;
}

pg_status launch_transition_logprob(const float* x, const float* u, const float* x_next_by_id,
                                    const int32_t* orig_id, int64_t n_traj, int64_t d, double A, double B, double C,
                                    uint64_t seed, uint32_t step, float* logp_by_id, double* log_ratio_by_id,
                                    float* partials, hipStream_t stream) {
  PG_TRY(check_stream_shape(n_traj, d));
  if (n_traj == 0) return PG_OK;
  const int chunks = (int)chunks_per_traj(d);
  transition_sq_kernel<<<dim3((unsigned)(n_traj * chunks)), dim3(STREAM_THREADS), 0, stream>>>(
      x, u, x_next_by_id, orig_id, (int)(d / 4), chunks, (float)A, (float)B, (float)C, (uint32_t)seed,
      (uint32_t)(seed >> 32), step, partials);
  PG_LAUNCH_CHECK("transition_sq_kernel");
  transition_finish_kernel<<<dim3((unsigned)((n_traj + FINISH_ROWS - 1) / FINISH_ROWS)), dim3(FINISH_ROWS * WAVE), 0, stream>>>(
      partials, chunks, (int)n_traj, 1.0 / (2.0 * C * C), (double)d * (log(C) + 0.5 * log(2.0 * M_PI)), orig_id,
      logp_by_id, log_ratio_by_id);
  PG_LAUNCH_CHECK("transition_finish_kernel");
  return PG_OK;
}

pg_status launch_surrogate(const double* log_ratio, const float* adv, const int32_t* offsets,
                           const int32_t* orig_id, int n_groups, int T, int M0, double clip_eps, float* ratio,
                           float* J, hipStream_t stream) {
  surrogate_kernel<<<dim3((n_groups + 3) / 4), dim3(256), 0, stream>>>(
      log_ratio, adv, offsets, orig_id, n_groups, T, M0, (float)(1.0 - clip_eps), (float)(1.0 + clip_eps),
      ratio, J);
  PG_LAUNCH_CHECK("surrogate_kernel");
  return PG_OK;
}
}  // namespace pg

extern "C" pg_status pg_sde_step_logprob(const float* x, const float* u, float* x_out, float* logp,
                                         float* logp_hist, float* logp_sum, const int32_t* src,
                                         const int32_t* orig_id, int64_t n_traj, int64_t d, double A,
                                         double B, double C, uint64_t seed, uint32_t step,
                                         float* partials, void* stream) {
  return launch_sde_step(x, u, x_out, logp, logp_hist, logp_sum, src, orig_id, n_traj, d, A, B, C, seed, step,
                         partials, nullptr, nullptr, (hipStream_t)stream);
}

extern "C" pg_status pg_sde_step_logprob_bf16(const uint16_t* x, const uint16_t* u, uint16_t* x_out, float* logp,
                                              float* logp_hist, float* logp_sum, const int32_t* src,
                                              const int32_t* orig_id, int64_t n_traj, int64_t d, double A,
                                              double B, double C, uint64_t seed, uint32_t step,
                                              float* partials, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  PG_TRY(check_stream_shape(n_traj, d));
  if (d % 8) return fail(PG_ESHAPE, "pg_sde_step_logprob_bf16: d = %lld must be a multiple of 8", (long long)d);
  if (n_traj == 0) return PG_OK;
  if (!x || !u || !x_out || !orig_id || !partials) return fail(PG_EINVAL, "pg_sde_step_logprob_bf16: null pointer");
  if (x_out == x) return fail(PG_EINVAL, "pg_sde_step_logprob_bf16: x_out must not alias x");
  if (!(C > 0.0)) return fail(PG_EINVAL, "pg_sde_step_logprob_bf16: noise scale C = %g must be > 0", C);
  const int chunks = (int)chunks_per_traj(d);
  const LogProb out{logp, logp_hist, logp_sum, (double)d * (log(C) + 0.5 * log(2.0 * M_PI))};
  const bool row = row_per_workgroup(n_traj, chunks);
  with_groups(row ? chunks : 0, [&](auto groups) {
    constexpr int G = decltype(groups)::value;
    sde_step_bf16_kernel<G><<<dim3((unsigned)(G ? n_traj : n_traj * chunks)), dim3((G ? G : 1) * STREAM_THREADS), 0, stream>>>(
        x, u, x_out, src, orig_id, (int)(d / 8), chunks, (float)A, (float)B, (float)C, (uint32_t)seed, (uint32_t)(seed >> 32), step,
        partials, out);
  });
  PG_LAUNCH_CHECK("sde_step_bf16_kernel");
  return row ? PG_OK : launch_logprob_finish(partials, chunks, n_traj, orig_id, out, stream);
}

namespace pg {
pg_status launch_preview(const float* x, const float* u, const float* w, float* rewards, int64_t n_traj, int64_t d, double Pc, double Qc,
                         double bias, float* partials, bool* unfinished, hipStream_t s) {
  PG_TRY(check_stream_shape(n_traj, d));
  if (n_traj == 0) return PG_OK;
  if (!x || !w || !rewards || !partials) return fail(PG_EINVAL, "pg_preview_reward: null pointer");
  if (!u && Qc != 0.0) return fail(PG_EINVAL, "pg_preview_reward: u is NULL but Qc = %g", Qc);
  const int chunks = (int)chunks_per_traj(d);
  const bool with_u = u && Qc != 0.0;
  const bool row = row_per_workgroup(n_traj, chunks);
  const int rec = prof_open(PROF_PREVIEW, (with_u ? 8.0 : 4.0) * (double)n_traj * (double)d, s);
  with_groups(row ? chunks : 0, [&](auto groups) {
    constexpr int G = decltype(groups)::value;
    const dim3 grid((unsigned)(G ? n_traj : n_traj * chunks)), block((G ? G : 1) * STREAM_THREADS);
    if (with_u) preview_reward_kernel<true, G><<<grid, block, 0, s>>>(x, u, w, (int)(d / 4), chunks, (float)Pc, (float)Qc, partials, bias, rewards);
    else preview_reward_kernel<false, G><<<grid, block, 0, s>>>(x, x, w, (int)(d / 4), chunks, (float)Pc, 0.f, partials, bias, rewards);
  });
  prof_close(rec, s);
  PG_LAUNCH_CHECK("preview_reward_kernel");
  if (unfinished) *unfinished = !row;
  if (row || unfinished) return PG_OK;
  reward_finish_kernel<<<dim3((unsigned)((n_traj + FINISH_ROWS - 1) / FINISH_ROWS)), dim3(FINISH_ROWS * WAVE), 0, s>>>(
      partials, chunks, (int)n_traj, bias, rewards);
  PG_LAUNCH_CHECK("reward_finish_kernel");
  return PG_OK;
}
}  // namespace pg

extern "C" pg_status pg_preview_reward(const float* x, const float* u, const float* w, float* rewards,
                                       int64_t n_traj, int64_t d, double Pc, double Qc, double bias,
                                       float* partials, void* stream) {
  return launch_preview(x, u, w, rewards, n_traj, d, Pc, Qc, bias, partials, nullptr, (hipStream_t)stream);
}

extern "C" pg_status pg_compact_gather(const float* x, float* out, const int32_t* src, int64_t n_out,
                                       int64_t d, void* stream) {
  PG_TRY(check_stream_shape(n_out, d));
  if (n_out == 0) return PG_OK;
  if (!x || !out || !src) return fail(PG_EINVAL, "pg_compact_gather: null pointer");
  if (out == x) return fail(PG_EINVAL, "pg_compact_gather: out must not alias x");
  const int chunks = (int)chunks_per_traj(d);
  compact_gather_kernel<<<dim3((unsigned)(n_out * chunks)), dim3(STREAM_THREADS), 0, (hipStream_t)stream>>>(
      x, out, src, (int)(d / 4), chunks);
  PG_LAUNCH_CHECK("compact_gather_kernel");
  return PG_OK;
}
