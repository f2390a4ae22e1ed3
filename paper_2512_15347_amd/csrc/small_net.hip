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
#include <cmath>
#include <type_traits>
#include "operands.hpp"
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

}  // namespace pg
