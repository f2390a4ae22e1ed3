// Narrow networks on short sequences (width 64 or 128, a sequence that fits one compute unit's LDS; small_net_takes): one workgroup
// evaluates the whole network for one trajectory, from the latents to u, in one launch.
//
// Layer by layer such a network is a chain of launches of 3 to 5 us that each hold less than a microsecond of work (a block of
// width 128 over 64 tokens is 27 MFLOP).  Trajectories do not depend on each other inside the network, so here nothing leaves the
// compute unit between the layers: the residual stream (fp32), the operand of the next layer, queries / keys (later the MLP's
// hidden values) and the transposed values live in LDS.  A wave reads the weights of its own output columns straight from
// global memory into registers, since no other wave of the workgroup needs the same ones.
// What bounds it is latency: a block takes 14 us (31 layer by layer), of which the queries, keys and values are 1.8, the attention
// 1.9, the output projection 0.9, each half of the MLP 3.3, a LayerNorm 1.0 (ten barriers).  A launch finds no weights in its
// L2, so every layer's are asked for one to three phases before they are used: asked for one unit of work ahead, a block took 22 us.
// The sequence length is a template parameter in steps, so that all operand reads of a phase are in flight together (16 us with
// loops over the row tiles).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include "operands.hpp"
#include "philox.hpp"
#include "small_net.hpp"

namespace pg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

namespace {
constexpr int THREADS = 512, WAVES = THREADS / WAVE;
constexpr int LDS_MAX = 160 * 1024;
constexpr int up16(int v) { return (v + 15) & ~15; }
// Row pitches: eight bf16 (four floats) more than the row, so that the 16 rows of a fragment start in different banks
constexpr int h_pitch(int D) { return D + 4; }
constexpr int a_pitch(int D) { return D + 8; }
constexpr int q_pitch(int D) { return 2 * D + 8; }
constexpr int v_pitch(int T) { return T * 16 + 8; }
// Row tiles of 16 that the kernel is built for (a multiple of two: 32 keys make one step of the value product), 0: it is not
constexpr int tiles_for(int D, int L) {
  const int t = up16(L) / 16;
  if (D == 128) return t <= 2 ? 2 : t <= 4 ? 4 : t <= 6 ? 6 : 0;
  return t <= 2 ? 2 : t <= 4 ? 4 : t <= 8 ? 8 : t <= 12 ? 12 : 0;
}
constexpr size_t lds_bytes(int D, int T) {
  return 4 * (size_t)(T * 16 * h_pitch(D) + 6 * D) + 2 * (size_t)(T * 16 * (a_pitch(D) + q_pitch(D)) + D * v_pitch(T) + 9 * D);
}

// Eight waves are WC column groups times WR row groups.  A wave owns column tiles of 16 that lie WC apart: three of q | k | v (one
// of each), one of a product that is D wide, two of one that is 2 D wide.
constexpr int col_groups(int D) { return D / 16; }
constexpr int row_groups(int D) { return WAVES / col_groups(D); }

// Weights of NC column tiles over K columns of A.  A operand / B operand of the 16x16x32 MFMA alike: lane l holds row l % 16, 8
// columns from 8 (l / 16) on.
template <int NC, int K> struct Weights { bf16x8 f[NC][K / 32]; };
template <int D, int NC, int K>
__device__ __forceinline__ void load_weights(Weights<NC, K>& r, const uint16_t* w, int64_t ld, int wc, int rows, int lane) {
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const uint16_t* p = w + (int64_t)min((wc + j * col_groups(D)) * 16 + (lane & 15), rows - 1) * ld + 8 * (lane >> 4);
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks) r.f[j][ks] = *reinterpret_cast<const bf16x8*>(p + 32 * ks);
  }
}
// [rows, K] x [cols, K]^T: out(j, column tile, row tile, n, acc) for every 16 x 16 tile of the wave, the wave's n-th row tile (a
// constant), start(j, column tile) the first value of its accumulators.  A lane holds four consecutive columns of one row; for j >= TR (transposed) four consecutive rows of
// one column.
template <int D, int NC, int K, int TR, int T, class Start, class Out>
__device__ __forceinline__ void product(const uint16_t* A, int pitch, const Weights<NC, K>& w, int wc, int wr, int lane, Start start, Out out) {
  const int lr = lane & 15, lk = lane >> 4;
  constexpr int KG = K < 128 ? K / 32 : 4;           // slabs of 32 columns whose fragments are read together
  f32x4v first[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) first[j] = start(j, wc + j * col_groups(D));
#pragma unroll
  for (int c = 0; c < T / 2; c += row_groups(D)) {
    const int rt = 2 * (c + wr);
    if (rt >= T) break;                              // wave-uniform
    const uint16_t* a0 = A + (rt * 16 + lr) * pitch + 8 * lk;
    f32x4v acc[2][NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) acc[0][j] = acc[1][j] = first[j];
#pragma unroll
    for (int kg = 0; kg < K / 32; kg += KG) {
      bf16x8 x[2][KG];
#pragma unroll
      for (int ks = 0; ks < KG; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i][ks] = *reinterpret_cast<const bf16x8*>(a0 + i * 16 * pitch + 32 * (kg + ks));
      __builtin_amdgcn_sched_barrier(0);             // all in flight before the first is waited for
#pragma unroll
      for (int ks = 0; ks < KG; ++ks)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < NC; ++j)
            acc[i][j] = j >= TR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i][ks], w.f[j][kg + ks], acc[i][j], 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.f[j][kg + ks], x[i][ks], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int i = 0; i < 2; ++i) out(j, wc + j * col_groups(D), rt + i, 2 * (c / row_groups(D)) + i, acc[i][j]);
  }
}

__device__ __forceinline__ f32x4v widen4(uint2 v) {
  return f32x4v{bf16_to_f32((uint16_t)v.x), bf16_to_f32((uint16_t)(v.x >> 16)), bf16_to_f32((uint16_t)v.y), bf16_to_f32((uint16_t)(v.y >> 16))};
}
__device__ __forceinline__ f32x4v bias4(const uint16_t* b) { return widen4(*reinterpret_cast<const uint2*>(b)); }   // 8-byte aligned
__device__ __forceinline__ void store4(uint16_t* p, f32x4v v) { *reinterpret_cast<uint2*>(p) = pack_bf16x4({v[0], v[1], v[2], v[3]}); }

// act[r, :] = bf16(LN(h[r, :]) (1 + scale) + shift), 16 lanes per row
template <int D, int ROWS>
__device__ __forceinline__ void layer_norm(const float* h, uint16_t* act, const float* shift, const float* scale) {
  constexpr int V = D / 64;
  const int j = threadIdx.x & 15;
#pragma unroll 1
  for (int r0 = 0; r0 < ROWS; r0 += THREADS / 16) {
    const int r = r0 + (threadIdx.x >> 4);
    if (ROWS % (THREADS / 16) != 0 && r >= ROWS) break;
    float4 v[V];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      v[i] = *reinterpret_cast<const float4*>(h + r * h_pitch(D) + 4 * j + 64 * i);
      s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mu = head_sum(s, true) * (1.f / D);
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      v[i].x -= mu; v[i].y -= mu; v[i].z -= mu; v[i].w -= mu;
      q += (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
    }
    const float rstd = rsqrtf(head_sum(q, true) * (1.f / D) + 1e-6f);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int n = 4 * j + 64 * i;
      const float4 a = *reinterpret_cast<const float4*>(scale + n), b = *reinterpret_cast<const float4*>(shift + n);
      store4(act + r * a_pitch(D) + n, f32x4v{v[i].x * rstd * (1.f + a.x) + b.x, v[i].y * rstd * (1.f + a.y) + b.y,
                                              v[i].z * rstd * (1.f + a.z) + b.z, v[i].w * rstd * (1.f + a.w) + b.w});
    }
  }
}

// Softmax attention inside the workgroup: a unit is 16 queries of one head, whose scores over all keys stay in registers.
// Scores are computed transposed, so a lane holds one query and, of every 16 keys, four; two such tiles are the 32-key
// operand of the value product with the keys in the order that the values are read in.
template <int D, int HD, int T>
__device__ __forceinline__ void attention(const uint16_t* qk, const uint16_t* vt, uint16_t* att, int L, int wave, int lane) {
  constexpr int KS = HD / 32, CT = HD / 16;
  const int lr = lane & 15, lk = lane >> 4;
#pragma unroll 1
  for (int u = wave; u < D / HD * T; u += WAVES) {
    const int head = u / T, qt = u - head * T;
    const uint16_t* keys = qk + lr * q_pitch(D) + D + head * HD + 8 * lk;
    const uint16_t* vals = vt + (head * HD + lr) * v_pitch(T) + 4 * lk;
    bf16x8 q[KS];
    f32x4v s[T];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      q[ks] = *reinterpret_cast<const bf16x8*>(qk + (qt * 16 + lr) * q_pitch(D) + head * HD + 32 * ks + 8 * lk);
#pragma unroll
    for (int t0 = 0; t0 < T; t0 += 4) {              // the keys of four tiles in flight
      bf16x8 k[4][KS];
#pragma unroll
      for (int t = t0; t < T && t < t0 + 4; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) k[t - t0][ks] = *reinterpret_cast<const bf16x8*>(keys + t * 16 * q_pitch(D) + 32 * ks);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int t = t0; t < T && t < t0 + 4; ++t)
          s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[t - t0][ks], q[ks], ks ? s[t] : f32x4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    if (L < 16 * T)                                  // wave-uniform
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (t * 16 + 4 * lk + e >= L) s[t][e] = -__builtin_huge_valf();
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[t][e]);
    mx = across_rows(mx, [](float x, float y) { return fmaxf(x, y); });
    f32x4v o[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) o[c] = f32x4v{0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < T; t += 2) {
      uint2 v[CT][2];
#pragma unroll
      for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) v[c][i] = *reinterpret_cast<const uint2*>(vals + c * 16 * v_pitch(T) + (t + i) * 16);
      uint32_t p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4v& x = s[t + i / 2];
        p[i] = pack_bf16x2(__builtin_amdgcn_exp2f(x[2 * (i & 1)] - mx), __builtin_amdgcn_exp2f(x[2 * (i & 1) + 1] - mx));
        // the normaliser sums the probabilities as the value product sees them (rounded to bf16)
        sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[i]), bf16x2{(__bf16)1.0f, (__bf16)1.0f}, sum, false);
      }
      const bf16x8 pf = __builtin_bit_cast(bf16x8, uint4{p[0], p[1], p[2], p[3]});
#pragma unroll
      for (int c = 0; c < CT; ++c)
        o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, uint4{v[c][0].x, v[c][0].y, v[c][1].x, v[c][1].y}), pf,
                                                       o[c], 0, 0, 0);
    }
    const float inv = 1.0f / across_rows(sum, [](float x, float y) { return x + y; });
#pragma unroll
    for (int c = 0; c < CT; ++c) store4(att + (qt * 16 + lr) * a_pitch(D) + head * HD + c * 16 + 4 * lk, o[c] * inv);
  }
}
}  // namespace

template <int D, int HD, int T>
__global__ __launch_bounds__(THREADS, 2) void small_net_kernel(const SmallNetArgs a) {
  // of a fixed size, so that no launch depends on an attribute that a process would have to set once per device
  static_assert(lds_bytes(D, T) <= LDS_MAX, "fits");
  __shared__ __align__(16) unsigned char smem[lds_bytes(D, T)];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  constexpr int L16 = T * 16, vp = v_pitch(T);
  float* h = reinterpret_cast<float*>(smem);                           // [L16][D + 4]
  float* md = h + L16 * h_pitch(D);                                    // [6 D] modulation vectors of the block
  uint16_t* act = reinterpret_cast<uint16_t*>(md + 6 * D);             // [L16][D + 8]
  uint16_t* qk = act + L16 * a_pitch(D);                               // [L16][2 D + 8]: queries | keys, then half the hidden values
  uint16_t* vt = qk + L16 * q_pitch(D);                                // [D][16 T + 8]
  uint16_t* bs = vt + D * vp;                                          // [9 D] biases of the block: qkv, out, fc1, fc2
  const int m = blockIdx.x, g = a.group_of[m], row = a.mod_of[m];
  const int Wp = a.W / 2, HW = a.H * a.W;
  const float* mod = a.mod + (int64_t)row * a.blocks * 6 * D;

  // modulation vectors and biases of a block, at most one access of either kind per thread
  static_assert(6 * D / 4 <= THREADS && 9 * D / 8 <= THREADS, "one access per thread");
  f32x4v md_next = {0.f, 0.f, 0.f, 0.f}, bs_next = md_next;
  auto fetch_vectors = [&](int b) {
    if (tid < 6 * D / 4) md_next = *reinterpret_cast<const f32x4v*>(mod + (int64_t)b * 6 * D + 4 * tid);
    if (tid < 9 * D / 8) {
      const int i = 8 * tid;
      const uint16_t* p = i < 3 * D ? a.qkv.b + i : i < 4 * D ? a.out.b + (i - 3 * D) : i < 8 * D ? a.fc1.b + (i - 4 * D) : a.fc2.b + (i - 8 * D);
      bs_next = *reinterpret_cast<const f32x4v*>(p + (int64_t)b * a.block_stride);
    }
  };
  auto put_vectors = [&] {
    if (tid < 6 * D / 4) *reinterpret_cast<f32x4v*>(md + 4 * tid) = md_next;
    if (tid < 9 * D / 8) *reinterpret_cast<f32x4v*>(bs + 8 * tid) = bs_next;
  };
  fetch_vectors(0);

  // ---- patch tokens (columns past 4 C and rows past Li are zero), context rows, padding ----
  const int wc = wave % col_groups(D), wr = wave / col_groups(D);
  Weights<1, 64> w_e;
  load_weights<D>(w_e, a.embed.w, a.embed.ld, wc, D, lane);
  Weights<3, D> w_qkv;
  load_weights<D>(w_qkv, a.qkv.w, a.qkv.ld, wc, 3 * D, lane);
  const f32x4v b_e = bias4(a.embed.b + wc * 16 + 4 * lk);
  uint2 pos[T];                                      // the wave's rows of the position table
#pragma unroll
  for (int c = 0; c < T / 2; c += row_groups(D))
#pragma unroll
    for (int i = 0; i < 2; ++i)
      pos[2 * (c / row_groups(D)) + i] = *reinterpret_cast<const uint2*>(
          a.pos + (int64_t)min((2 * (c + wr) + i) * 16 + lr, a.Li - 1) * D + wc * 16 + 4 * lk);
  const float* x = a.x + (int64_t)m * a.C * HW;
  for (int i = tid; i < L16 * 16; i += THREADS) {                      // four columns (one channel) of one token
    const int tok = i % L16, c = i / L16;
    uint2 v = {0u, 0u};
    if (c < a.C && tok < a.Li) {
      const int py = tok / Wp, px = tok - py * Wp;
      const float* src = x + (int64_t)c * HW + 2 * py * a.W + 2 * px;
      const float2 r0 = *reinterpret_cast<const float2*>(src), r1 = *reinterpret_cast<const float2*>(src + a.W);
      v = pack_bf16x4({r0.x, r0.y, r1.x, r1.y});
    }
    *reinterpret_cast<uint2*>(act + tok * a_pitch(D) + 4 * c) = v;
  }
  for (int i = tid; i < (L16 - a.Li) * (D / 4); i += THREADS) {
    const int j = i / (D / 4), k = i - j * (D / 4);
    float4 v = {0.f, 0.f, 0.f, 0.f};
    if (j < a.Lc) v = reinterpret_cast<const float4*>(a.ctx_h)[((int64_t)g * a.Lc + j) * (D / 4) + k];
    *reinterpret_cast<float4*>(h + (a.Li + j) * h_pitch(D) + 4 * k) = v;
  }
  put_vectors();
  __syncthreads();

  // ---- patch embedding + position table ----
  product<D, 1, 64, 1, T>(act, a_pitch(D), w_e, wc, wr, lane, [&](int, int) { return b_e; },
                          [&](int, int col, int rt, int n, const f32x4v& v) {
                            const int tok = rt * 16 + lr;
                            if (tok < a.Li) *reinterpret_cast<f32x4v*>(h + tok * h_pitch(D) + col * 16 + 4 * lk) = v + widen4(pos[n]);
                          });
  __syncthreads();

  // h[r, :] += gate (acc): the layers that add into the residual stream
  auto add_gated = [&](const float* gate) {
    return [=](int, int col, int rt, int, const f32x4v& v) {
      const int n = col * 16 + 4 * lk;
      f32x4v* p = reinterpret_cast<f32x4v*>(h + (rt * 16 + lr) * h_pitch(D) + n);
      *p = *p + *reinterpret_cast<const f32x4v*>(gate + n) * v;
    };
  };
  // Every layer's weights are asked for one to three phases before they are used
  Weights<1, D> w_o;
  Weights<2, D> w_1;
  Weights<1, 2 * D> w_2;
  for (int b = 0; b < a.blocks; ++b) {
    const int64_t at = (int64_t)b * a.block_stride;
    const uint16_t* fc1 = a.fc1.w + at;
    const uint16_t* fc2 = a.fc2.w + at;
    // ---- attention sub-block ----
    load_weights<D>(w_o, a.out.w + at, a.out.ld, wc, D, lane);
    layer_norm<D, L16>(h, act, md, md + D);
    __syncthreads();
    load_weights<D>(w_1, fc1, a.fc1.ld, wc, 4 * D, lane);
    product<D, 3, D, 2, T>(act, a_pitch(D), w_qkv, wc, wr, lane,
                        [&](int j, int col) {
                          if (j < 2) return bias4(bs + col * 16 + 4 * lk);
                          const float v = bf16_to_f32(bs[col * 16 + lr]);
                          return f32x4v{v, v, v, v};
                        },
                        [&](int j, int col, int rt, int, const f32x4v& v) {
                          if (j == 2) store4(vt + (col * 16 - 2 * D + lr) * vp + rt * 16 + 4 * lk, v);   // four tokens of a channel
                          else store4(qk + (rt * 16 + lr) * q_pitch(D) + col * 16 + 4 * lk, j == 0 ? v * a.scale_log2 : v);
                        });
    __syncthreads();
    load_weights<D>(w_2, fc2, a.fc2.ld, wc, D, lane);
    attention<D, HD, T>(qk, vt, act, a.L, wave, lane);
    __syncthreads();
    product<D, 1, D, 1, T>(act, a_pitch(D), w_o, wc, wr, lane, [&](int, int col) { return bias4(bs + 3 * D + col * 16 + 4 * lk); },
                        add_gated(md + 2 * D));
    __syncthreads();
    // ---- MLP sub-block, the hidden values in two halves ----
    layer_norm<D, L16>(h, act, md + 3 * D, md + 4 * D);
    const bool more = b + 1 < a.blocks;
    if (!more) {                                     // the final layer's shift and scale, and its weights where the projection's were
      if (tid < 2 * D / 4) md_next = *reinterpret_cast<const f32x4v*>(a.fmod + (int64_t)row * 2 * D + 4 * tid);
      load_weights<D>(w_o, a.fin.w, a.fin.ld, wc, 4 * a.C, lane);
    } else {
      fetch_vectors(b + 1);
      load_weights<D>(w_qkv, a.qkv.w + at + a.block_stride, a.qkv.ld, wc, 3 * D, lane);
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      product<D, 2, D, 2, T>(act, a_pitch(D), w_1, wc, wr, lane,
                          [&](int, int col) { return bias4(bs + 4 * D + half * 2 * D + col * 16 + 4 * lk); },
                          [&](int, int col, int rt, int, const f32x4v& v) {
                            store4(qk + (rt * 16 + lr) * q_pitch(D) + col * 16 + 4 * lk,
                                   f32x4v{gelu_tanh(v[0]), gelu_tanh(v[1]), gelu_tanh(v[2]), gelu_tanh(v[3])});
                          });
      if (half == 0) load_weights<D>(w_1, fc1 + (int64_t)2 * D * a.fc1.ld, a.fc1.ld, wc, 2 * D, lane);
      __syncthreads();
      product<D, 1, 2 * D, 1, T>(qk, q_pitch(D), w_2, wc, wr, lane,
                              [&](int, int col) { return half == 0 ? bias4(bs + 8 * D + col * 16 + 4 * lk) : f32x4v{0.f, 0.f, 0.f, 0.f}; },
                              add_gated(md + 5 * D));
      if (half == 0) load_weights<D>(w_2, fc2 + 2 * D, a.fc2.ld, wc, D, lane);
      __syncthreads();
    }
    put_vectors();
    __syncthreads();
  }

  // ---- final layer on the image tokens, written straight into the latent layout ----
  const int c_f = wc * 4 + lk;                       // channel of the wave's columns 4 c .. 4 c + 3: one channel's 2 x 2 patch
  f32x4v b_f = {0.f, 0.f, 0.f, 0.f};
  if (c_f < a.C) b_f = bias4(a.fin.b + 4 * c_f);
  layer_norm<D, L16>(h, act, md, md + D);
  __syncthreads();
  float* u = a.u + (int64_t)m * a.C * HW;
  if (wc * 16 >= 4 * a.C) return;                    // no barrier follows
  product<D, 1, D, 1, T>(act, a_pitch(D), w_o, wc, wr, lane, [&](int, int) { return b_f; },
                         [&](int, int, int rt, int, const f32x4v& v) {
                           const int tok = rt * 16 + lr;
                           if (tok >= a.Li || c_f >= a.C) return;
                           const int py = tok / Wp, px = tok - py * Wp;
                           float* dst = u + (int64_t)c_f * HW + 2 * py * a.W + 2 * px;
                           *reinterpret_cast<float2*>(dst) = float2{v[0], v[1]};
                           *reinterpret_cast<float2*>(dst + a.W) = float2{v[2], v[3]};
                         });
}

// ---- the same network, a workgroup per 16 rows and a launch per block ----
// With one workgroup per trajectory most compute units are idle while 8 or 36 of them take 35 us for two blocks of 64 tokens: the
// products, the GELUs and the LayerNorms of all its rows pass through one compute unit, and so do its weights, 393 KB a block of
// width 128, as fragments: loads of 16 rows x 64 bytes, of which a compute unit takes 16 bytes a cycle (12 us for these; 1 KB
// contiguous per load 4.5 us, the same straight into LDS 2.6 us, measured with 8 and with 216 workgroups alike).
// Here a workgroup has 16 rows; only attention needs other rows, their keys and values, and gets them through memory from the launch
// before.  Weights pass through LDS: a wave asks for the pieces that it alone needs (16 rows x D columns) with direct loads, SLOTS of
// them ahead, and reads each into registers when it has arrived, with no barrier.  Queries, keys and values are stored in the
// order in which attention holds them, 1 KB contiguous per load.
// A wave owns column tiles of 16 as above; every sum is formed in the order of small_net_kernel, so both give the same bits.
// A launch takes 7.9 us (width 128, 64 tokens, 16 or 32 workgroups), with the final layer, the update and the next step's first
// rows 10.5 us; what is left is latency: 2 us of launch, 2 us until keys, values and the first weights are there, 4 us for seven
// phases between barriers.  The loop of 8 trajectories and ten steps takes 250 us (461 with one workgroup per trajectory and an
// update launch per step), three groups of 12 with 90 tokens and six steps 209 us (387).
namespace {
// What a launch does: the first rows of a step, a block with the queries / keys / values of the next one, the last block and u
// (and the update), or that and the next step's first rows
enum RowsKind { ROWS_START, ROWS_BLOCK, ROWS_LAST, ROWS_LAST_START };

// Where a block's tensors lie behind its QKV weights (build_weight_layout: rows of D or 4 D, starts rounded up to 128), and the
// patch embedding's bias and the position table behind its weights (rows of 64)
constexpr int up128(int v) { return (v + 127) & ~127; }
template <int D> struct BlockLayout {
  static constexpr int qkv_b = 3 * D * D, o_w = qkv_b + up128(3 * D), o_b = o_w + D * D, fc1_w = o_b + up128(D), fc1_b = fc1_w + 4 * D * D,
                       fc2_w = fc1_b + up128(4 * D), fc2_b = fc2_w + 4 * D * D;
  static constexpr int pe_b = 64 * D, pos = pe_b + up128(D);
};

// The pieces of weights that a wave of a launch needs, in the order of use
enum Piece { PIECE_O = 0, PIECE_FC1 = 1, PIECE_FC2 = 5, PIECE_QKV = 9, PIECE_FIN = 12, PIECE_EMBED = 13, PIECE_NONE = 14 };
template <int KIND> constexpr int pieces() { return KIND == ROWS_START ? 4 : KIND == ROWS_BLOCK ? 12 : KIND == ROWS_LAST ? 10 : 14; }
template <int KIND> constexpr int piece_at(int i) {
  if (i >= pieces<KIND>()) return PIECE_NONE;
  if (KIND == ROWS_START) return i == 0 ? PIECE_EMBED : PIECE_QKV + i - 1;
  if (i < 9) return i;                               // output projection, fc1, fc2
  if (KIND == ROWS_BLOCK) return i;                  // qkv
  return i == 9 ? PIECE_FIN : i == 10 ? PIECE_EMBED : PIECE_QKV + i - 11;
}

template <int D> struct Fragments { bf16x8 f[D / 32]; };

template <int D>
struct RowsWeights {
  static constexpr int ROW = 2 * D, CPR = D / 8, RPI = 64 / CPR;        // bytes and chunks of a piece's row, rows per direct load
  static constexpr int BYTES = 16 * ROW, LOADS = BYTES / 1024, SLOTS = D == 128 ? 3 : 6;
  // position of a row's chunk: the 16 rows of a fragment put one chunk of theirs into different banks
  static __device__ __forceinline__ int turn(int row) { return D == 128 ? row & 15 : (row ^ (row >> 3)) & 7; }
  const unsigned char* ring;                         // the wave's slots
  uint32_t lds;                                      // their address
  uint32_t off[LOADS], off4[LOADS];                  // a lane's byte offsets in a piece of rows of D and of 4 D columns
  int lane, wave;
  __device__ __forceinline__ void init(unsigned char* smem, int wave_, int lane_) {
    lane = lane_; wave = wave_;
    ring = smem + wave * SLOTS * BYTES;
    lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * SLOTS * BYTES);
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
      const int row = q * RPI + lane / CPR, chunk = (lane % CPR) ^ turn(row);
      off[q] = (uint32_t)(row * D + chunk * 8) * 2;
      off4[q] = (uint32_t)(row * 4 * D + chunk * 8) * 2;
    }
  }
  static constexpr int loads(int piece) { return piece == PIECE_NONE ? 0 : piece == PIECE_EMBED ? 2 : LOADS; }
  template <int KIND, int I> __device__ __forceinline__ void request(const RowsArgs& a) const {
    constexpr int piece = piece_at<KIND>(I);
    using LO = BlockLayout<D>;
    const uint32_t to = lds + I % SLOTS * BYTES;
    if constexpr (piece == PIECE_NONE) return;
    else if constexpr (piece == PIECE_EMBED) {       // 16 rows of 64 columns
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int row = q * 8 + lane / 8;
        dma16((uint32_t)(row * 64 + ((lane & 7) ^ ((row ^ (row >> 3)) & 7)) * 8) * 2, a.embed + wave * 16 * 64, to + q * 1024);
      }
    } else if constexpr (piece == PIECE_FIN) {       // 4 C rows in all
#pragma unroll
      for (int q = 0; q < LOADS; ++q) {
        const int row = q * RPI + lane / CPR;
        dma16((uint32_t)(min(wave * 16 + row, 4 * a.C - 1) * D + ((lane % CPR) ^ turn(row)) * 8) * 2, a.fin, to + q * 1024);
      }
    } else {
      const uint16_t* base = piece == PIECE_O ? a.w + LO::o_w + wave * 16 * D
                             : piece < PIECE_FC2 ? a.w + LO::fc1_w + ((piece - PIECE_FC1) * D + wave * 16) * D
                             : piece < PIECE_QKV ? a.w + LO::fc2_w + wave * 16 * 4 * D + (piece - PIECE_FC2) * D
                                                 : a.w_next + ((piece - PIECE_QKV) * D + wave * 16) * D;
#pragma unroll
      for (int q = 0; q < LOADS; ++q) dma16(piece >= PIECE_FC2 && piece < PIECE_QKV ? off4[q] : off[q], base, to + q * 1024);
    }
  }
  // loads that were asked for behind piece I while it is waited for
  template <int KIND> static constexpr int behind(int i) {
    int n = 0;
    for (int k = i + 1; k < i + SLOTS; ++k) n += loads(piece_at<KIND>(k));
    return n;
  }
  // piece I of the launch: awaited, read, and its slot given to the piece that comes SLOTS later
  template <int KIND, int I, int K = D> __device__ __forceinline__ void take(const RowsArgs& a, Fragments<K>& w) const {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(behind<KIND>(I)) : "memory");
    const int lr = lane & 15, lk = lane >> 4;
    const unsigned char* at = ring + I % SLOTS * BYTES + lr * 2 * K;
    const int t = K == 128 ? lr : (lr ^ (lr >> 3)) & 7;
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks) w.f[ks] = *reinterpret_cast<const bf16x8*>(at + ((4 * ks + lk) ^ t) * 16);
    if constexpr (piece_at<KIND>(I + SLOTS) != PIECE_NONE) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      request<KIND, I + SLOTS>(a);
    }
  }
  template <int KIND, int I, int N> __device__ __forceinline__ void take_all(const RowsArgs& a, Fragments<D>* w) const {
    if constexpr (N > 0) {
      take<KIND, I>(a, *w);
      take_all<KIND, I + 1, N - 1>(a, w + 1);
    }
  }
  template <int KIND, int I = 0> __device__ __forceinline__ void begin(const RowsArgs& a) const {
    if constexpr (I < SLOTS) {
      request<KIND, I>(a);
      begin<KIND, I + 1>(a);
    }
  }
};

// one row tile x the 16 rows of a piece, on top of acc; TR: a lane gets four rows of one column, else four columns of one row
template <int K, bool TR>
__device__ __forceinline__ f32x4v product_rows(const uint16_t* A, int pitch, const Fragments<K>& w, int lane, f32x4v acc) {
  const uint16_t* a0 = A + (lane & 15) * pitch + 8 * (lane >> 4);
  bf16x8 x[K / 32];
#pragma unroll
  for (int ks = 0; ks < K / 32; ++ks) x[ks] = *reinterpret_cast<const bf16x8*>(a0 + 32 * ks);
#pragma unroll
  for (int ks = 0; ks < K / 32; ++ks)
    acc = TR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[ks], w.f[ks], acc, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.f[ks], x[ks], acc, 0, 0, 0);
  return acc;
}

// attention() for the 16 queries of this workgroup and one head of a wave; `tiles` of the T key tiles exist.  Queries and keys
// [tile][head][32 columns][lane][8], values [head][two tiles][16 channels][lane][4 of either tile].
template <int D, int HD, int T>
struct RowsAttention {
  static constexpr int KS = HD / 32, CT = HD / 16, HEADS = D / HD;
  typedef uint32_t four __attribute__((ext_vector_type(4)));
  bf16x8 q[KS], k[T][KS];
  four v[T / 2][CT];
  __device__ __forceinline__ void load(const uint16_t* queries, const uint16_t* keys, const uint16_t* values, int tiles, int tile, int head,
                                       int lane) {
    const int pairs = (tiles + 1) / 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) q[ks] = *reinterpret_cast<const bf16x8*>(queries + ((tile * HEADS + head) * KS + ks) * 512 + lane * 8);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        k[t][ks] = *reinterpret_cast<const bf16x8*>(keys + ((min(t, tiles - 1) * HEADS + head) * KS + ks) * 512 + lane * 8);
#pragma unroll
    for (int t = 0; t < T / 2; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c)
        v[t][c] = *reinterpret_cast<const four*>(values + ((head * pairs + min(t, pairs - 1)) * CT + c) * 512 + lane * 8);
  }
  __device__ __forceinline__ void compute(uint16_t* att, int L, int tiles, int head, int lane) {
    const int lr = lane & 15, lk = lane >> 4;
    f32x4v s[T];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int t = 0; t < T; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[t][ks], q[ks], ks ? s[t] : f32x4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    if (L < 16 * T)                                  // wave-uniform; keys of a tile that does not exist are past L, too
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (t * 16 + 4 * lk + e >= L) s[t][e] = -__builtin_huge_valf();
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[t][e]);
    mx = across_rows(mx, [](float x, float y) { return fmaxf(x, y); });
    f32x4v o[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) o[c] = f32x4v{0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < T; t += 2) {
      uint32_t p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4v& x = s[t + i / 2];
        p[i] = pack_bf16x2(__builtin_amdgcn_exp2f(x[2 * (i & 1)] - mx), __builtin_amdgcn_exp2f(x[2 * (i & 1) + 1] - mx));
        sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[i]), bf16x2{(__bf16)1.0f, (__bf16)1.0f}, sum, false);
      }
      const bf16x8 pf = __builtin_bit_cast(bf16x8, four{p[0], p[1], p[2], p[3]});
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        four w = v[t / 2][c];
        if (t + 1 >= tiles) w[2] = w[3] = 0u;        // nobody wrote the second tile of an odd last pair; pairs past the last repeat it
        o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), pf, o[c], 0, 0, 0);
      }
    }
    const float inv = 1.0f / across_rows(sum, [](float x, float y) { return x + y; });
#pragma unroll
    for (int c = 0; c < CT; ++c) store4(att + lr * a_pitch(D) + head * HD + c * 16 + 4 * lk, o[c] * inv);
  }
};
}  // namespace

template <int D, int HD, int T, int KIND>
__global__ __launch_bounds__(4 * D, D / 64) void small_rows_kernel(const RowsArgs a) {
  constexpr bool BLOCK = KIND != ROWS_START, LAST = KIND == ROWS_LAST || KIND == ROWS_LAST_START;
  constexpr bool START = KIND == ROWS_START || KIND == ROWS_LAST_START, NEXT = KIND != ROWS_LAST;
  using LO = BlockLayout<D>;
  using RW = RowsWeights<D>;
  constexpr int hp = 4 * D + 8;                      // pitch of the hidden values
  constexpr int WAVES_D = D / 16, HEADS = D / HD, KS = HD / 32, CT = HD / 16;
  __shared__ __align__(16) unsigned char ring[WAVES_D * RW::SLOTS * RW::BYTES];
  __shared__ __align__(16) float h[16 * h_pitch(D)];
  __shared__ __align__(16) float md[8 * D];          // gate, shift, scale, gate of the block | of the final layer | shift, scale of the next block
  __shared__ __align__(16) uint16_t act[16 * a_pitch(D)], hid[BLOCK ? 16 * hp : 8], pat[16 * 72], bs[9 * D];
  constexpr int MN = LAST ? 6 * D : 4 * D;           // the next block's part of md
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lk = lane >> 4, n0 = wave * 16 + 4 * lk;     // the lane's columns of a D wide product: n0 .. n0 + 3
  const int tile = blockIdx.x, m = blockIdx.y, tok0 = tile * 16;
  const int rows0 = m * a.tiles * 16, pairs0 = m * ((a.tiles + 1) & ~1) * 16;      // of the trajectory; few thousand rows
  const bool image = tok0 < a.Li;                    // some rows are image tokens
  const bool block = BLOCK && (!LAST || image);      // after the last block the context's rows are not used any more
  const int hr = tid / (D / 4), hc = 4 * (tid - hr * (D / 4));           // every thread holds four columns of one row
  const int at_row = (rows0 + tok0 + hr) * D + hc, at_lane = (rows0 + tok0 + lr) * D + n0;

  // ---- asked for at once, in the order of use ----
  RowsAttention<D, HD, T> attn;
  f32x4v h_in = {0.f, 0.f, 0.f, 0.f}, bias_in = h_in, gate = h_in, vec = h_in;
  const int row = a.mod_of[m];
  RW weights;
  weights.init(ring, wave, lane);
  if (block) {
    if (wave < HEADS) attn.load(a.qk_in + rows0 * 2 * D, a.qk_in + rows0 * 2 * D + a.tiles * 16 * D, a.vt_in + pairs0 * D, a.tiles, tile, wave, lane);
    h_in = *reinterpret_cast<const f32x4v*>(a.hs + at_row);
  }
  // biases, eight per thread: output projection, fc1, fc2 of the block, qkv of the next one
  const int bi = 8 * tid;
  if (BLOCK ? bi < 9 * D : bi < 3 * D) {
    const int of_block = bi < D ? LO::o_b + bi : bi < 5 * D ? LO::fc1_b - D + bi : LO::fc2_b - 5 * D + bi;
    const uint16_t* p = !BLOCK ? a.w_next + LO::qkv_b + bi : bi < 6 * D ? a.w + of_block : a.w_next + LO::qkv_b - 6 * D + bi;
    bias_in = *reinterpret_cast<const f32x4v*>(p);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (block) weights.template begin<KIND>(a);
  else if (START) weights.template begin<ROWS_START>(a);
  __builtin_amdgcn_sched_barrier(0);
  // modulation vectors, four floats per thread: the block's, [the final layer's,] the next block's
  {
    const float* mb = a.mod + (int64_t)row * a.mod_ld;
    const float* mn = BLOCK && !LAST ? mb + 6 * D : a.mod_next + (int64_t)row * a.mod_ld;
    const int i = 4 * tid;
    const float* p = i < 4 * D ? mb + 2 * D + i : LAST && i < 6 * D ? a.fmod + (int64_t)row * 2 * D + i - 4 * D : mn + i - MN;
    if (i >= (BLOCK ? 0 : 4 * D) && i < (NEXT ? MN + 2 * D : 6 * D)) vec = *reinterpret_cast<const f32x4v*>(p);
    if (block) gate = *reinterpret_cast<const f32x4v*>(mb + 2 * D + n0);
  }

  // ---- latents of the lane's patch: channel c, image token t ----
  const int c_p = tid >> 4, t_p = tok0 + (tid & 15);
  const int Wp = a.W / 2, HW = a.H * a.W;
  bool patch = false;
  int e_p = 0, id = 0;
  float2 x0 = {0.f, 0.f}, x1 = x0, u0 = x0, u1 = x0;
  uint2 pos = {0u, 0u}, be_in = pos;
  f32x4v ctx = {0.f, 0.f, 0.f, 0.f}, b_f = ctx;
  const int ctx_row = tok0 + hr - a.Li;              // context row of the thread's row
  if (START || LAST) {
    patch = c_p < a.C && t_p < a.Li;
    const int py = t_p / Wp, px = t_p - py * Wp;
    e_p = c_p * HW + 2 * py * a.W + 2 * px;
    if (a.update) id = a.up.orig_id[m];
    if (patch && (!BLOCK || a.update)) {
      const int q = a.update && a.up.src ? a.up.src[m] : m;
      const float* px_ = a.x + q * a.C * HW + e_p;
      x0 = *reinterpret_cast<const float2*>(px_);
      x1 = *reinterpret_cast<const float2*>(px_ + a.W);
      if (!BLOCK && a.update) {
        const float* pu = a.u + q * a.C * HW + e_p;
        u0 = *reinterpret_cast<const float2*>(pu);
        u1 = *reinterpret_cast<const float2*>(pu + a.W);
      }
    }
    if (LAST && c_p < a.C) b_f = bias4(a.fin_b + 4 * c_p);
    if (START) {
      be_in = *reinterpret_cast<const uint2*>(a.embed + LO::pe_b + n0);
      pos = *reinterpret_cast<const uint2*>(a.embed + LO::pos + min(tok0 + lr, a.Li - 1) * D + n0);
      if (ctx_row >= 0 && ctx_row < a.Lc) ctx = *reinterpret_cast<const f32x4v*>(a.ctx_h + ((int64_t)a.group_of[m] * a.Lc + ctx_row) * D + hc);
    }
  }
  // the update's noise, while the first loads are under way: two neighbours are half a block of it
  float2 z0 = {0.f, 0.f}, z1 = z0;
  if ((START || LAST) && a.update && patch) {
    auto noise = [&](int e) {
      const f32x4 z = philox_normal4((uint32_t)e >> 2, a.up.step, (uint32_t)id, STREAM_STEP, a.up.k0, a.up.k1);
      return e & 2 ? float2{z.z, z.w} : float2{z.x, z.y};
    };
    z0 = noise(e_p);
    z1 = noise(e_p + a.W);
  }
  auto put_bias = [&] { if (BLOCK ? bi < 9 * D : bi < 3 * D) *reinterpret_cast<f32x4v*>(bs + (BLOCK ? 0 : 6 * D) + bi) = bias_in; };
  auto put_vectors = [&] { if (4 * tid < (NEXT ? MN + 2 * D : 6 * D)) *reinterpret_cast<f32x4v*>(md + 4 * tid) = vec; };
  Fragments<D> w_qkv[3];
  Fragments<64> w_e;

  if (block) {
    Fragments<D> w_o, w_1[4], w_2[4];
    if (wave < HEADS) attn.compute(act, a.L, a.tiles, wave, lane);
    put_bias();
    *reinterpret_cast<f32x4v*>(h + hr * h_pitch(D) + hc) = h_in;
    weights.template take<KIND, 0>(a, w_o);
    weights.template take_all<KIND, 1, 2>(a, w_1);
    __syncthreads();
    f32x4v* hv = reinterpret_cast<f32x4v*>(h + lr * h_pitch(D) + n0);
    *hv = *hv + gate * product_rows<D, false>(act, a_pitch(D), w_o, lane, bias4(bs + n0));
    put_vectors();
    weights.template take_all<KIND, 3, 2>(a, w_1 + 2);
    __syncthreads();
    layer_norm<D, 16>(h, act, md + D, md + 2 * D);
    weights.template take_all<KIND, 5, 2>(a, w_2);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4v v = product_rows<D, false>(act, a_pitch(D), w_1[j], lane, bias4(bs + D + j * D + n0));
      store4(hid + lr * hp + j * D + n0, f32x4v{gelu_tanh(v[0]), gelu_tanh(v[1]), gelu_tanh(v[2]), gelu_tanh(v[3])});
    }
    weights.template take_all<KIND, 7, 2>(a, w_2 + 2);
    __syncthreads();
    f32x4v sum = *hv;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x4v v = half == 0 ? bias4(bs + 5 * D + n0) : f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 2 * half; i < 2 * half + 2; ++i) v = product_rows<D, false>(hid + i * D, hp, w_2[i], lane, v);
      sum = sum + *reinterpret_cast<const f32x4v*>(md + 3 * D + n0) * v;
    }
    *hv = sum;
    if (!LAST) *reinterpret_cast<f32x4v*>(a.hs + at_lane) = sum;
    if (KIND == ROWS_BLOCK) weights.template take_all<KIND, 9, 3>(a, w_qkv);
  } else {
    put_bias();
    put_vectors();
  }

  // ---- final layer: u of the lane's patch ----
  if (LAST && image) {
    Fragments<D> w_f;
    weights.template take<KIND, 9>(a, w_f);
    if (START) weights.template take<KIND, 10>(a, w_e);
    __syncthreads();
    layer_norm<D, 16>(h, act, md + 4 * D, md + 5 * D);
    __syncthreads();
    if (wave * 16 < 4 * a.C) {                       // lane (lr, lk) of this product is the patch of channel 4 wave + lk = c_p, token lr
      const f32x4v v = product_rows<D, false>(act, a_pitch(D), w_f, lane, b_f);
      u0 = float2{v[0], v[1]};
      u1 = float2{v[2], v[3]};
    }
    if (patch) {
      float* dst = a.u + m * a.C * HW + e_p;
      *reinterpret_cast<float2*>(dst) = u0;
      *reinterpret_cast<float2*>(dst + a.W) = u1;
    }
  }

  // ---- sampler update of the lane's patch (the latents that the next step starts from) ----
  if ((START || LAST) && a.update && image) {
    if (patch) {
      auto moved = [&](float2 xv, float2 uv, float2 z) {
        return float2{a.up.A * xv.x + a.up.B * uv.x + a.up.C * z.x, a.up.A * xv.y + a.up.B * uv.y + a.up.C * z.y};
      };
      x0 = moved(x0, u0, z0);
      x1 = moved(x1, u1, z1);
      auto put = [&](float* dst) {
        *reinterpret_cast<float2*>(dst + e_p) = x0;
        *reinterpret_cast<float2*>(dst + e_p + a.W) = x1;
      };
      put(a.up.x_out + m * a.C * HW);
      if (a.up.hist_next) put(a.up.hist_next + (int64_t)id * a.C * HW);
    }
    if (tile == 0 && tid == 0) finish_logprob(a.up.out, m, id, a.up.sums[id]);
  }

  // ---- a step's first rows: patch embedding + position table, context rows, zeros past the end ----
  if (START) {
    if (tid < 256) *reinterpret_cast<uint2*>(pat + (tid & 15) * 72 + 4 * c_p) = pack_bf16x4({x0.x, x0.y, x1.x, x1.y});   // zeros without a patch
    if (!block) {
      weights.template take<ROWS_START, 0>(a, w_e);
      weights.template take_all<ROWS_START, 1, 3>(a, w_qkv);
    } else {
      weights.template take_all<KIND, 11, 3>(a, w_qkv);
    }
    __syncthreads();
    if (ctx_row >= 0) {
      *reinterpret_cast<f32x4v*>(h + hr * h_pitch(D) + hc) = ctx;
      *reinterpret_cast<f32x4v*>(a.hs + at_row) = ctx;
    }
    const f32x4v v = product_rows<64, false>(pat, 72, w_e, lane, widen4(be_in));
    if (tok0 + lr < a.Li) {
      const f32x4v e = v + widen4(pos);
      *reinterpret_cast<f32x4v*>(h + lr * h_pitch(D) + n0) = e;
      *reinterpret_cast<f32x4v*>(a.hs + at_lane) = e;
    }
  }

  // ---- queries | keys and values of the next block ----
  if (NEXT) {
    __syncthreads();
    layer_norm<D, 16>(h, act, md + MN, md + MN + D);
    __syncthreads();
    const int w = n0 & (HD - 1);                     // the lane's columns in their head
    uint16_t* qk = a.qk_out + rows0 * 2 * D + ((tile * HEADS + n0 / HD) * KS + w / 32) * 512 + ((w & 31) / 8 * 16 + lr) * 8 + (w & 7);
    store4(qk, product_rows<D, false>(act, a_pitch(D), w_qkv[0], lane, bias4(bs + 6 * D + n0)) * a.scale_log2);
    store4(qk + a.tiles * 16 * D, product_rows<D, false>(act, a_pitch(D), w_qkv[1], lane, bias4(bs + 7 * D + n0)));
    const float bv = bf16_to_f32(bs[8 * D + wave * 16 + lr]);
    const int ch = wave * 16;                        // the wave's channels
    store4(a.vt_out + pairs0 * D + ((ch / HD * ((a.tiles + 1) / 2) + tile / 2) * CT + ch % HD / 16) * 512 + lane * 8 + (tile & 1) * 4,
           product_rows<D, true>(act, a_pitch(D), w_qkv[2], lane, f32x4v{bv, bv, bv, bv}));
  }
}

// What fits the LDS of a compute unit runs here; however many trajectories are still active, so that a trajectory's result does not
// change with the prunes of its group or with the steps that are evaluated together.  A step with two blocks, us, a launch per
// layer / here:
//   width 128,  64 tokens:   4 trajectories  99 / 49   256: 173 / 58   4096: 1424 / 584
//   width 128,  90 tokens:   4 trajectories 100 / 60   256: 219 / 71   4096: 2031 / 754
//   width  64, 184 tokens:   4 trajectories  95 / 59   256: 243 / 70   4096: 2578 / 740
// A workgroup costs as much for 1 token as for 32, its smallest tile, where a launch per layer takes its time by the row.  So of up to
// 16 tokens (width 64: 14) only groups of few trajectories in all do, the number from which the layers are faster being about
// 1400 + 18 L^2 (width 64) and 896 + 8 L^2 (width 128).  Loops of three steps, us, a launch per layer / here:
//   width  64,  1 token:  1536 trajectories 339 / 334, 4096 443 / 778    8 tokens: 2560 520 / 511, 4096 668 / 776
//   width  64, 12 tokens: 4096 trajectories 793 / 776, 8192 1349 / 1502  15 tokens: 8192 1571 / 1498, 16384 3069 / 2990
//   width 128,  1 token:   768 trajectories 346 / 299, 4096 628 / 1409   8 tokens: 1280 505 / 478, 4096 961 / 1399
//   width 128, 16 tokens: 2560 trajectories 939 / 907, 4096 1314 / 1404  18 tokens: 4096 1589 / 1403, 16384 5387 / 5475
// Built for the two kinds of network whose blocks have this one sequence of layers.  Width 192 and 256, built the same way, were
// slower with 8 to 16 trajectories (width 256, 32 tokens, 4 blocks: 185 / 211): there a compute unit's reading of the weights (1.6 MB a
// block) is the longer part.
bool small_net_takes(const pg_ctx* c) {
  const pg_config& f = c->cfg;
  if ((f.net_kind != PG_NET_ADALN && f.net_kind != PG_NET_JOINT) || (f.D != 64 && f.D != 128) || f.C > 16 || tiles_for(f.D, c->L) == 0)
    return false;
  const int64_t L2 = (int64_t)c->L * c->L;
  return f.D == 64 ? c->L > 14 || c->M0 <= 1400 + 18 * L2 : c->L > 16 || c->M0 <= 896 + 8 * L2;
}

template <int D, int HD, int T>
static pg_status launch_small(const SmallNetArgs& a, hipStream_t s) {
  // the whole network as one product: its layers' flops and its attention's
  const double rows = (double)a.M * a.L, image = (double)a.M * a.Li;
  const int rec = prof_open(PROF_GEMM, a.blocks * rows * (24.0 * D * D + 4.0 * a.L * D) + 16.0 * image * D * a.C, s);
  small_net_kernel<D, HD, T><<<dim3(a.M), dim3(THREADS), 0, s>>>(a);
  prof_close(rec, s);
  PG_LAUNCH_CHECK("small_net_kernel");
  return PG_OK;
}
template <int HD>
static pg_status launch_width(const SmallNetArgs& a, int D, hipStream_t s) {
  switch (D * 100 + tiles_for(D, a.L)) {
    case 6402: return launch_small<64, HD, 2>(a, s);
    case 6404: return launch_small<64, HD, 4>(a, s);
    case 6408: return launch_small<64, HD, 8>(a, s);
    case 6412: return launch_small<64, HD, 12>(a, s);
    case 12802: return launch_small<128, HD, 2>(a, s);
    case 12804: return launch_small<128, HD, 4>(a, s);
    case 12806: return launch_small<128, HD, 6>(a, s);
  }
  return fail(PG_ESHAPE, "small network: %d tokens of width %d", a.L, D);
}

pg_status launch_small_net(const SmallNetArgs& a, int D, int hd, hipStream_t s) {
  if (a.C > 16 || a.Li < 1 || a.Li + a.Lc != a.L || (D != 64 && D != 128) || (hd != 32 && hd != 64))
    return fail(PG_ESHAPE, "small network: width %d, head width %d, %d channels", D, hd, a.C);
  return hd == 32 ? launch_width<32>(a, D, s) : launch_width<64>(a, D, s);
}

int small_rows_tiles(const pg_ctx* c) { return (c->L + 15) / 16; }

// A launch per block pays while its workgroups are about as many as the compute units hold; with more, they read the weights more
// often than one workgroup per trajectory does.  A compute unit holds one of width 128, two of width 64, so the lines lie at 256 and 512
// workgroups; a loop takes more of them than an evaluation alone, since its updates cost no launch, and one of few tokens fewer, since
// one workgroup per trajectory then is a short launch.  How many times as fast as one workgroup per trajectory, loops of six steps with a
// prune / evaluations alone, of 1, 2 and 4 blocks, row tiles x trajectories:
//   width 128, 2 tiles: 256 1.25 1.28 1.24 / 1.03 1.07 1.08, 288 1.09 1.03 0.96 / 0.82 0.79 0.75
//              4 tiles: 256 1.54 1.46 1.43 / 1.23 1.22 1.19, 512 1.21 1.13 1.03 / 0.84 0.82 0.80, 544 0.91 0.80 0.75 / 0.73 0.69 0.64
//              6 tiles: 504 1.37 1.34 1.25 / 0.99 0.98 0.96, 528 1.08 0.97 0.91 / 0.80 0.82 0.76
//   width  64, 2 tiles: 128 1.22 1.07 1.04 / 0.97 0.96 0.98, 256 1.20 1.05 1.01 / 1.07 0.99 0.87, 288 1.11 1.03 0.94 / 0.95 0.88 0.85
//              4 tiles: 128 1.27 1.22 1.15 / 1.04 0.94 0.99, 256 1.26 1.21 1.11 / 1.01 0.98 0.94, 352 1.19 1.05 0.93 / 0.88 0.85 0.78
//              8 tiles: 512 1.40 1.32 1.23 / 1.05 1.03 1.00, 544 1.26 1.19 1.06 / 0.91 0.87 0.82, 768 1.20 1.07 0.97 / 0.85 0.85 0.81
//             12 tiles: 480 1.67 1.57 1.50 / 1.13 1.16 1.14, 768 1.24 1.14 1.04 / 0.91 0.94 0.89
//   up to 16 tokens: width 128 512 1.45 1.36 1.36 / 1.24 1.35 1.34, 896 1.43 1.43 1.44 / 1.40 1.43 1.44; width 64 128 1.26 1.16 1.10 /
//              1.01 0.99 1.06, 896 1.59 1.60 1.66 / 1.48 1.55 1.64
bool small_rows_takes(const pg_ctx* c) {
  const int tiles = small_rows_tiles(c);
  const int most = tiles == 1 ? 1024 : c->cfg.D == 64 ? (tiles <= 4 ? 256 : tiles < 8 ? 512 : 64 * tiles) : tiles == 2 ? 256 : 512;
  return small_net_takes(c) && chunks_per_traj(c->d) <= 4 && (int64_t)c->M0 * tiles <= most;
}
bool small_rows_evaluates(const pg_ctx* c, int M) {
  const int tiles = small_rows_tiles(c);
  return small_rows_takes(c) && (int64_t)M * tiles <= (tiles == 1 ? 1024 : tiles > 4 ? 512 : c->cfg.D == 64 ? 128 : 256);
}

template <int D, int HD, int T, int KIND>
static pg_status launch_rows_kernel(const RowsArgs& a, int M, hipStream_t s) {
  small_rows_kernel<D, HD, T, KIND><<<dim3((unsigned)a.tiles, (unsigned)M), dim3(4 * D), 0, s>>>(a);
  PG_LAUNCH_CHECK("small_rows_kernel");
  return PG_OK;
}
template <int D, int HD, int T>
static pg_status launch_rows(const RowsArgs& a, int M, bool last, bool start, hipStream_t s) {
  if (!last) return launch_rows_kernel<D, HD, T, ROWS_BLOCK>(a, M, s);
  return start ? launch_rows_kernel<D, HD, T, ROWS_LAST_START>(a, M, s) : launch_rows_kernel<D, HD, T, ROWS_LAST>(a, M, s);
}
template <int HD>
static pg_status launch_rows_width(const RowsArgs& a, int M, int D, bool last, bool start, hipStream_t s) {
  switch (D * 100 + tiles_for(D, a.L)) {
    case 6402: return launch_rows<64, HD, 2>(a, M, last, start, s);
    case 6404: return launch_rows<64, HD, 4>(a, M, last, start, s);
    case 6408: return launch_rows<64, HD, 8>(a, M, last, start, s);
    case 6412: return launch_rows<64, HD, 12>(a, M, last, start, s);
    case 12802: return launch_rows<128, HD, 2>(a, M, last, start, s);
    case 12804: return launch_rows<128, HD, 4>(a, M, last, start, s);
    case 12806: return launch_rows<128, HD, 6>(a, M, last, start, s);
  }
  return fail(PG_ESHAPE, "small network: %d tokens of width %d", a.L, D);
}

// a layer's weights and bias lie where the kernel takes them to be
template <int D>
static bool rows_layout(const SmallNetArgs& n) {
  using LO = BlockLayout<D>;
  const uint16_t* w = n.qkv.w;
  auto at = [](const SmallLayer& l, const uint16_t* weights, const uint16_t* bias, int ld) { return l.w == weights && l.b == bias && l.ld == ld; };
  return at(n.qkv, w, w + LO::qkv_b, D) && at(n.out, w + LO::o_w, w + LO::o_b, D) && at(n.fc1, w + LO::fc1_w, w + LO::fc1_b, D) &&
         at(n.fc2, w + LO::fc2_w, w + LO::fc2_b, 4 * D) && at(n.embed, n.embed.w, n.embed.w + LO::pe_b, 64) && n.pos == n.embed.w + LO::pos &&
         n.fin.ld == D;
}

pg_status launch_small_rows(const SmallNetArgs& n, RowsArgs& a, int D, int hd, int block, bool start, hipStream_t s) {
  if (n.C > 16 || n.Li < 1 || n.Li + n.Lc != n.L || (D != 64 && D != 128) || (hd != 32 && hd != 64) || n.M < 1 ||
      !(D == 64 ? rows_layout<64>(n) : rows_layout<128>(n)))
    return fail(PG_ESHAPE, "small network: width %d, head width %d, %d channels", D, hd, n.C);
  const bool last = block + 1 == n.blocks;
  a.u = n.u; a.mod_of = n.mod_of; a.group_of = n.group_of; a.ctx_h = n.ctx_h;
  a.w = n.qkv.w + (int64_t)std::max(block, 0) * n.block_stride;
  a.w_next = block < 0 || last ? n.qkv.w : a.w + n.block_stride;
  a.embed = n.embed.w; a.fin = n.fin.w; a.fin_b = n.fin.b;
  a.mod = n.mod + (int64_t)std::max(block, 0) * 6 * D; a.fmod = n.fmod; a.mod_ld = n.blocks * 6 * D;
  a.tiles = (n.L + 15) / 16; a.L = n.L; a.Li = n.Li; a.Lc = n.Lc; a.C = n.C; a.H = n.H; a.W = n.W; a.scale_log2 = n.scale_log2;
  if (block < 0) {                                   // no attention in it
    if (D == 64) return hd == 32 ? launch_rows_kernel<64, 32, 2, ROWS_START>(a, n.M, s) : launch_rows_kernel<64, 64, 2, ROWS_START>(a, n.M, s);
    return hd == 32 ? launch_rows_kernel<128, 32, 2, ROWS_START>(a, n.M, s) : launch_rows_kernel<128, 64, 2, ROWS_START>(a, n.M, s);
  }
  return hd == 32 ? launch_rows_width<32>(a, n.M, D, last, start, s) : launch_rows_width<64>(a, n.M, D, last, start, s);
}

}  // namespace pg
