// The velocity / noise network evaluated on every active trajectory at every step (the drift input of
// paper Eq. 12): a patch-2 adaLN transformer in four variants (conditioning vector only, extra
// cross-attention over context tokens, context tokens joined to the sequence, and the dual-stream
// form of the latter with per-stream weights and RMS-normalised queries / keys).  This file holds the
// memory-bound glue kernels (patchify, conditioning GEMVs, LayerNorm + modulation, context rows) and
// the orchestration; the contractions live in gemm.hip and attention.hip.
//
// Activation layout: rows r = m * L + token for the M active trajectories (image tokens first, then
// context tokens in the joint variant).  The dual-stream variant keeps two planes instead, image rows
// m * Li + t first and context rows M * Li + m * Lc + j behind them, so that each stream is one contiguous
// GEMM operand; only q | k and V^T use the joint per-trajectory layout that attention reads.
// The residual stream h is fp32; every GEMM operand is bf16.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include "attention.hpp"
#include "ctx.hpp"
#include "gemm.hpp"
#include "operands.hpp"
#include "row_chain.hpp"
#include "small_net.hpp"

namespace pg {

__device__ __forceinline__ float bf2f(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float silu(float x) { return x / (1.0f + __expf(-x)); }

// ---- conditioning: c = MLP(sincos(t)) + y and the modulation vectors of every block ----
// Matrix-vector products bound by reading the weights once (fp32 accumulation).  A wave computes GEMV_ROWS outputs for up to
// PC inputs at a time: 16-byte weight loads, GEMV_ROWS of them in flight per column block, the inputs read once for all rows.
constexpr int GEMV_ROWS = 4, GEMV_OUT = 4 * GEMV_ROWS;      // outputs per wave, per workgroup of four waves

// acc[r][p] = sum_k w[r, k] in[p, k] in every lane; rows past `rows` repeat the last one, inputs past `P` the first
template <int PC>
__device__ __forceinline__ void gemv_rows(const uint16_t* __restrict__ w, int64_t ldw, int rows, const float* __restrict__ in,
                                          int64_t in_ld, int P, int K, float (&acc)[GEMV_ROWS][PC]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int r = 0; r < GEMV_ROWS; ++r)
#pragma unroll
    for (int p = 0; p < PC; ++p) acc[r][p] = 0.f;
  for (int k = lane * 8; k < K; k += WAVE * 8) {            // K is a multiple of 8
    uint4 q[GEMV_ROWS];
#pragma unroll
    for (int r = 0; r < GEMV_ROWS; ++r) q[r] = *reinterpret_cast<const uint4*>(w + (int64_t)min(r, rows - 1) * ldw + k);
#pragma unroll
    for (int p = 0; p < PC; ++p) {
      const float* v = in + (int64_t)(p < P ? p : 0) * in_ld + k;
      const float4 a = *reinterpret_cast<const float4*>(v), b = *reinterpret_cast<const float4*>(v + 4);
#pragma unroll
      for (int r = 0; r < GEMV_ROWS; ++r) {
        auto lo = [](uint32_t x) { return __builtin_bit_cast(float, x << 16); };
        auto hi = [](uint32_t x) { return __builtin_bit_cast(float, x & 0xFFFF0000u); };
        acc[r][p] += ((lo(q[r].x) * a.x + hi(q[r].x) * a.y) + (lo(q[r].y) * a.z + hi(q[r].y) * a.w)) +
                     ((lo(q[r].z) * b.x + hi(q[r].z) * b.y) + (lo(q[r].w) * b.z + hi(q[r].w) * b.w));
      }
    }
  }
#pragma unroll
  for (int r = 0; r < GEMV_ROWS; ++r)
#pragma unroll
    for (int p = 0; p < PC; ++p) acc[r][p] = wave_allsum(acc[r][p]);
}

// Sinusoidal embeddings of all step times, which the configuration fixes: row s of emb is
// emb[0:128] = cos(t_s f_i), emb[128:256] = sin(t_s f_i), f_i = 10000^(-i/128)
__global__ void timestep_embedding_kernel(const double* __restrict__ t_in, float* __restrict__ emb) {
  const int i = threadIdx.x, s = blockIdx.x;
  const double f = exp(-9.210340371976184 * (double)i / 128.0);     // fp64: t f reaches 1000 rad
  emb[256 * (size_t)s + i] = (float)cos(t_in[s] * f);
  emb[256 * (size_t)s + 128 + i] = (float)sin(t_in[s] * f);
}

// What a step's network evaluation can start from, in one launch (each part is a few microseconds of latency, and each
// used to be a launch or two): t1 = silu(W1 emb + b1) of the time embedding (of gridDim.y steps, where nothing else is asked
// for), the bf16 patch tokens of the latents,
//   tok[r, 4c + 2dy + dx] = bf16(x[m, c, 2py + dy, 2px + dx]), r = m * Li + py * Wp + px; columns >= 4C are zero,
// and the context rows of every trajectory, h[row_base + m * row_stride + j, :] = ctx_h[group_of[m], j, :].
struct StepInputs {
  const uint16_t* w1; int64_t ldw1; const uint16_t* b1; const float* emb; float* t1; int D;
  const float* x; uint16_t* tok; int M, C, H, W, Kp;
  const float* ctx_h; float* h; const int32_t* group_of; int64_t row_base; int row_stride, Lc;
  int t1_blocks, patch_blocks;                   // workgroups of the first two parts
};
__global__ __launch_bounds__(256) void step_inputs_kernel(const StepInputs a) {
  int blk = blockIdx.x;
  if (blk < a.t1_blocks) {
    const int n0 = blk * GEMV_OUT + (threadIdx.x >> 6) * GEMV_ROWS;
    if (n0 >= a.D) return;
    float acc[GEMV_ROWS][1];
    gemv_rows<1>(a.w1 + (int64_t)n0 * a.ldw1, a.ldw1, a.D - n0, a.emb + 256 * (int64_t)blockIdx.y, 0, 1, 256, acc);
    float* t1 = a.t1 + (int64_t)blockIdx.y * a.D;
    if ((threadIdx.x & 63) == 0)
      for (int r = 0; r < GEMV_ROWS && n0 + r < a.D; ++r) t1[n0 + r] = silu(acc[r][0] + bf2f(a.b1[n0 + r]));
    return;
  }
  blk -= a.t1_blocks;
  if (blk < a.patch_blocks) {
    const int Wp = a.W / 2, Hp = a.H / 2;
    const int cq = a.Kp / 4;                     // 4-column groups per row, channels first then padding
    const int64_t i = (int64_t)blk * 256 + threadIdx.x;
    if (i >= (int64_t)a.M * cq * Hp * Wp) return;
    const int px = (int)(i % Wp);
    const int py = (int)((i / Wp) % Hp);
    const int c = (int)((i / ((int64_t)Wp * Hp)) % cq);
    const int m = (int)(i / ((int64_t)Wp * Hp * cq));
    uint32_t lo = 0u, hi = 0u;
    if (c < a.C) {
      const float* src = a.x + ((int64_t)m * a.C + c) * a.H * a.W + (int64_t)(2 * py) * a.W + 2 * px;
      const float2 r0 = *reinterpret_cast<const float2*>(src);
      const float2 r1 = *reinterpret_cast<const float2*>(src + a.W);
      lo = (uint32_t)f2bf(r0.x) | ((uint32_t)f2bf(r0.y) << 16);
      hi = (uint32_t)f2bf(r1.x) | ((uint32_t)f2bf(r1.y) << 16);
    }
    *reinterpret_cast<uint2*>(a.tok + ((int64_t)m * Hp * Wp + (int64_t)py * Wp + px) * a.Kp + 4 * c) = uint2{lo, hi};
    return;
  }
  blk -= a.patch_blocks;
  const int D4 = a.D / 4;
  const int64_t i = (int64_t)blk * 256 + threadIdx.x;
  if (i >= (int64_t)a.M * a.Lc * D4) return;
  const int k = (int)(i % D4);
  const int j = (int)((i / D4) % a.Lc);
  const int m = (int)(i / ((int64_t)D4 * a.Lc));
  const float4 v = reinterpret_cast<const float4*>(a.ctx_h)[((int64_t)a.group_of[m] * a.Lc + j) * D4 + k];
  reinterpret_cast<float4*>(a.h)[(a.row_base + (int64_t)m * a.row_stride + j) * D4 + k] = v;
}

// sc[z, p, n] = silu(b[n] + sum_k W[n, k] t1[z, k] + y[p, n]) for step blockIdx.z; blockIdx.y: 64 groups, one per lane (1024
// groups of width 64: 4.8 us, 23.1 when a lane walked them)
__global__ __launch_bounds__(256) void condition_kernel(const uint16_t* __restrict__ W, int64_t ldw, const uint16_t* __restrict__ bias,
                                                        const float* __restrict__ t1, const float* __restrict__ y,
                                                        float* __restrict__ sc, int P, int D) {
  const int n0 = blockIdx.x * GEMV_OUT + (threadIdx.x >> 6) * GEMV_ROWS;
  if (n0 >= D) return;
  float acc[GEMV_ROWS][1];
  gemv_rows<1>(W + (int64_t)n0 * ldw, ldw, D - n0, t1 + (int64_t)blockIdx.z * D, 0, 1, D, acc);
  sc += (int64_t)blockIdx.z * P * D;
  const int p = blockIdx.y * WAVE + (threadIdx.x & 63);
  if (p < P)
#pragma unroll
    for (int r = 0; r < GEMV_ROWS; ++r)
      if (n0 + r < D) sc[(int64_t)p * D + n0 + r] = silu(acc[r][0] + bf2f(bias[n0 + r]) + y[(int64_t)p * D + n0 + r]);
}

// Every modulation vector of the network in one launch: blockIdx.y < sets * blocks walks the blocks of the one or two
// streams (out[set][p, block, 0:6D]), the last one the final layer's 2D outputs; blockIdx.z takes `span` groups, so that many
// groups of a narrow or shallow network are not walked by a few workgroups one after another (1024 groups, width 64, one block:
// 51 us, 1242 without the split).
struct Modulation {
  const uint16_t* w[2]; const uint16_t* b[2]; float* out[2];   // per stream, block 0
  int64_t ldw, block_stride;
  const uint16_t* fw; const uint16_t* fb; int64_t ldfw; float* fout;
  const float* sc; int P, D, blocks, sets, span;
};
template <int PC>
__global__ __launch_bounds__(256) void modulation_kernel(const Modulation a) {
  const int set = blockIdx.y / a.blocks, blk = blockIdx.y - set * a.blocks;
  const bool fin = set >= a.sets;
  const int N = fin ? 2 * a.D : 6 * a.D;
  const int n0 = blockIdx.x * GEMV_OUT + (threadIdx.x >> 6) * GEMV_ROWS;
  if (n0 >= N) return;
  const int64_t ld = fin ? a.ldfw : a.ldw;
  const uint16_t* w = (fin ? a.fw : a.w[set] + blk * a.block_stride) + (int64_t)n0 * ld;
  const uint16_t* b = fin ? a.fb : a.b[set] + blk * a.block_stride;
  float* out = fin ? a.fout : a.out[set] + (int64_t)blk * N;
  const int64_t out_ld = fin ? N : (int64_t)a.blocks * N;
  const int lane = threadIdx.x & 63;
  const int p_end = min(a.P, ((int)blockIdx.z + 1) * a.span);
  float bias[GEMV_ROWS];
#pragma unroll
  for (int r = 0; r < GEMV_ROWS; ++r) bias[r] = bf2f(b[min(r, N - 1 - n0) + n0]);
  for (int p0 = blockIdx.z * a.span; p0 < p_end; p0 += PC) {
    float acc[GEMV_ROWS][PC];
    gemv_rows<PC>(w, ld, N - n0, a.sc + (int64_t)p0 * a.D, a.D, a.P - p0, a.D, acc);
    if (lane == 0)
#pragma unroll
      for (int p = 0; p < PC; ++p)
        if (p0 + p < a.P)
#pragma unroll
          for (int r = 0; r < GEMV_ROWS; ++r)
            if (n0 + r < N) out[(int64_t)(p0 + p) * out_ld + n0 + r] = acc[r][p] + bias[r];
  }
}

// out[r', :] = bf16(LN(h[r, :]) * (1 + scale[g]) + shift[g]); one wave per row.  The row lives in registers (NV float4 per
// lane, D <= 256 NV; WHOLE: D = 256 NV, else the last float4 of some lanes lies past the row) so h is read once and every
// access is 16 bytes wide; NV = 0 is the generic route for wider rows (three cached passes of 4-byte accesses, which
// every width that is no multiple of 256 used to take).
// Rows: r' = m * L_out + t for t < L_out reads h row m * L_in + t (L_out < L_in drops the context rows).  From output row
// `rows0` on (dual-stream: the context plane) rows are read in place, L2 of them per trajectory, modulated by shift2 / scale2.
struct LnArgs {
  const float* h; uint16_t* out; const float* shift; const float* scale; int64_t mod_ld; const int32_t* group_of;
  int rows_out, L_in, L_out, D;
  int rows0; const float* shift2; const float* scale2; int L2;
};
template <int NV, bool WHOLE>
__global__ __launch_bounds__(256) void ln_modulate_kernel(const LnArgs a) {
  const int D = a.D;
  const int lane = threadIdx.x & 63;
  const int ro = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (ro >= a.rows_out) return;
  const bool second = ro >= a.rows0;
  const int m = second ? (ro - a.rows0) / a.L2 : ro / a.L_out;
  const float* hr = a.h + (second ? (int64_t)ro : (int64_t)m * a.L_in + (ro - m * a.L_out)) * D;
  uint16_t* orow = a.out + (int64_t)ro * D;
  const float* sh = nullptr;
  const float* sc = nullptr;
  if (a.shift) {
    const int64_t g = (int64_t)a.group_of[m] * a.mod_ld;
    sh = (second ? a.shift2 : a.shift) + g;
    sc = (second ? a.scale2 : a.scale) + g;
  }
  if (NV > 0) {
    float4 v[NV > 0 ? NV : 1];
    auto inside = [&](int i) { return WHOLE || i + 1 < NV || 4 * (lane + 64 * i) < D; };
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = inside(i) ? reinterpret_cast<const float4*>(hr)[lane + 64 * i] : float4{0.f, 0.f, 0.f, 0.f};
      s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    }
    const float mu = wave_allsum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i].x -= mu; v[i].y -= mu; v[i].z -= mu; v[i].w -= mu;
      const float qi = (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
      q += inside(i) ? qi : 0.f;
    }
    const float rstd = rsqrtf(wave_allsum(q) / (float)D + 1e-6f);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (!inside(i)) continue;
      float4 o = {v[i].x * rstd, v[i].y * rstd, v[i].z * rstd, v[i].w * rstd};
      if (sh) {
        const float4 a = reinterpret_cast<const float4*>(sc)[lane + 64 * i];
        const float4 b = reinterpret_cast<const float4*>(sh)[lane + 64 * i];
        o.x = o.x * (1.0f + a.x) + b.x; o.y = o.y * (1.0f + a.y) + b.y;
        o.z = o.z * (1.0f + a.z) + b.z; o.w = o.w * (1.0f + a.w) + b.w;
      }
      reinterpret_cast<uint2*>(orow)[lane + 64 * i] = pack_bf16x4(o);
    }
    return;
  }
  float s = 0.f;
  for (int k = lane; k < D; k += WAVE) s += hr[k];
  const float mu = wave_allsum(s) / (float)D;
  float q = 0.f;
  for (int k = lane; k < D; k += WAVE) { const float dv = hr[k] - mu; q += dv * dv; }
  const float rstd = rsqrtf(wave_allsum(q) / (float)D + 1e-6f);
  if (sh) {
    for (int k = lane; k < D; k += WAVE) orow[k] = f2bf((hr[k] - mu) * rstd * (1.0f + sc[k]) + sh[k]);
  } else {
    for (int k = lane; k < D; k += WAVE) orow[k] = f2bf((hr[k] - mu) * rstd);
  }
}

// ------------------------------------------------------------------------------------------------

static size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

pg_status net_plan(pg_ctx* c) {
  c->net = NetPlan{};
  const pg_config& f = c->cfg;
  if (f.net_kind == PG_NET_NONE) return PG_OK;
  const size_t R0 = (size_t)c->M0 * c->L, D = f.D;
  const size_t Lpad = ((size_t)c->L + 63) / 64 * 64, Lcpad = ((size_t)f.Lc + 63) / 64 * 64;
  const size_t Kp = ((size_t)4 * f.C + 63) / 64 * 64;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off = a256(off + bytes); return o; };
  NetPlan& n = c->net;
  n.h = take(R0 * D * 4);
  n.act = take(R0 * D * 2);
  n.qkv = take(R0 * 2 * D * 2);
  n.vt = take((size_t)c->M0 * D * Lpad * 2);
  n.att = take(R0 * D * 2);
  n.hid = take(R0 * 4 * D * 2);
  n.tok = take((size_t)c->M0 * c->Li * Kp * 2);
  // modulation vectors of several steps at a time, at most 64 vectors (or one step's)
  n.mod_steps = std::max(1, std::min(f.T, 64 / f.P));
  const size_t mod_rows = (size_t)n.mod_steps * f.P;
  n.mod = take(mod_rows * (f.blocks * 6 * D * (f.net_kind == PG_NET_MMDIT ? 2 : 1) + 2 * D) * 4);
  n.cond = take((n.mod_steps * D + mod_rows * D) * 4);
  n.rows = take(2 * sizeof(int32_t) * c->M0);
  if (f.net_kind == PG_NET_JOINT || f.net_kind == PG_NET_MMDIT) n.ctx_h = take((size_t)f.P * f.Lc * D * 4);
  if (f.net_kind == PG_NET_CROSS) {
    n.ckv = take((size_t)f.blocks * f.P * f.Lc * D * 2);
    n.ckvt = take((size_t)f.blocks * f.P * D * Lcpad * 2);
  }
  if (small_rows_takes(c)) {
    const size_t rows = (size_t)c->M0 * small_rows_tiles(c) * 16, pairs = (size_t)c->M0 * ((small_rows_tiles(c) + 1) & ~1) * 16;
    n.rows_h = take(rows * D * 4);
    for (int i = 0; i < 2; ++i) { n.rows_qk[i] = take(rows * 2 * D * 2); n.rows_vt[i] = take(pairs * D * 2); }
  }
  n.total = off;
  return PG_OK;
}

namespace {
struct Net {
  pg_ctx* c;
  hipStream_t s;
  char* base;
  const uint16_t* wts;
  template <class T> T* at(size_t off) const { return reinterpret_cast<T*>(base + off); }
  const uint16_t* w(int id, int block = 0) const {
    return wts + c->top[id].offset + (id >= PG_W_MOD_W ? c->block_stride * block : 0);
  }
  int ld(int id) const { return c->top[id].ld; }
};
}  // namespace

// time embeddings of all steps from their network times, both in the workspace (set-up, see pg_bind)
pg_status net_embed_times(pg_ctx* c, hipStream_t s) {
  timestep_embedding_kernel<<<dim3(c->cfg.T), dim3(128), 0, s>>>((const double*)((char*)c->buf.workspace + c->ws_tin),
                                                                (float*)((char*)c->buf.workspace + c->ws_emb));
  PG_LAUNCH_CHECK("timestep_embedding_kernel");
  return PG_OK;
}

// Step-independent work: projected context rows (joint) or per-block context keys / values (cross).
pg_status net_prepare(pg_ctx* c, const uint16_t* weights, hipStream_t s) {
  const pg_config& f = c->cfg;
  Net n{c, s, (char*)c->buf.workspace + c->ws_net, weights};
  const int D = f.D;
  if (f.net_kind == PG_NET_JOINT || f.net_kind == PG_NET_MMDIT) {
    GemmArgs g{};
    g.A = c->buf.ctx; g.lda = f.Dc; g.W = n.w(PG_W_CTX_W); g.ldw = n.ld(PG_W_CTX_W); g.bias = n.w(PG_W_CTX_B);
    g.M = f.P * f.Lc; g.N = D; g.K = f.Dc;
    g.outf = n.at<float>(c->net.ctx_h); g.ldo = D;
    PG_TRY(launch_gemm(g, EPI_F32, s));
  } else if (f.net_kind == PG_NET_CROSS) {
    const int Lcpad = (f.Lc + 63) / 64 * 64;
    for (int b = 0; b < f.blocks; ++b) {
      GemmArgs g{};
      g.A = c->buf.ctx; g.lda = f.Dc; g.W = n.w(PG_W_CKV_W, b); g.ldw = n.ld(PG_W_CKV_W); g.bias = n.w(PG_W_CKV_B, b);
      g.M = f.P * f.Lc; g.N = 2 * D; g.K = f.Dc;
      g.outb = n.at<uint16_t>(c->net.ckv) + (size_t)b * f.P * f.Lc * D; g.ldob = D;
      g.vt = n.at<uint16_t>(c->net.ckvt) + (size_t)b * f.P * D * Lcpad; g.v_start = D; g.Lpad = Lcpad; g.L = f.Lc;
      PG_TRY(launch_gemm(g, EPI_QKV, s));
    }
  }
  return PG_OK;
}

namespace {
// where the modulation vectors of a set of steps lie, and what the conditioning works on
struct ModPlan {
  float *mod, *fmod, *cmod, *t1, *sc;
  int64_t ld;                                       // floats from one vector set of a stream to the next
};
ModPlan mod_plan(const pg_ctx* c, const Net& n) {
  const pg_config& f = c->cfg;
  const size_t rows = (size_t)c->net.mod_steps * f.P;
  ModPlan m;
  m.ld = (int64_t)f.blocks * 6 * f.D;
  m.mod = n.at<float>(c->net.mod);
  m.fmod = m.mod + rows * m.ld;
  m.cmod = m.fmod + rows * 2 * f.D;                 // dual-stream variant: the context stream's modulation vectors
  m.t1 = n.at<float>(c->net.cond);
  m.sc = m.t1 + (size_t)c->net.mod_steps * f.D;
  return m;
}

StepInputs time_inputs(const pg_ctx* c, const Net& n, const ModPlan& m, int step) {
  StepInputs a{};
  a.w1 = n.w(PG_W_T_W1); a.ldw1 = n.ld(PG_W_T_W1); a.b1 = n.w(PG_W_T_B1); a.D = c->cfg.D;
  a.emb = reinterpret_cast<const float*>((char*)c->buf.workspace + c->ws_emb) + (size_t)step * 256; a.t1 = m.t1;
  a.t1_blocks = (c->cfg.D + GEMV_OUT - 1) / GEMV_OUT;
  return a;
}

// conditioning and modulation vectors of `steps` steps from their t1
pg_status launch_modulation(const pg_ctx* c, const Net& n, const ModPlan& m, int steps) {
  const pg_config& f = c->cfg;
  const int D = f.D;
  const bool dual = f.net_kind == PG_NET_MMDIT;
  condition_kernel<<<dim3((D + GEMV_OUT - 1) / GEMV_OUT, (f.P + WAVE - 1) / WAVE, steps), dim3(256), 0, n.s>>>(
      n.w(PG_W_T_W2), n.ld(PG_W_T_W2), n.w(PG_W_T_B2), m.t1, c->buf.y, m.sc, f.P, D);
  PG_LAUNCH_CHECK("condition_kernel");
  Modulation mo{};
  mo.w[0] = n.w(PG_W_MOD_W); mo.b[0] = n.w(PG_W_MOD_B); mo.out[0] = m.mod; mo.ldw = n.ld(PG_W_MOD_W); mo.block_stride = c->block_stride;
  if (dual) { mo.w[1] = n.w(PG_W_C_MOD_W); mo.b[1] = n.w(PG_W_C_MOD_B); mo.out[1] = m.cmod; }
  mo.fw = n.w(PG_W_FMOD_W); mo.fb = n.w(PG_W_FMOD_B); mo.ldfw = n.ld(PG_W_FMOD_W); mo.fout = m.fmod;
  const int P = steps * f.P;
  mo.sc = m.sc; mo.P = P; mo.D = D; mo.blocks = f.blocks; mo.sets = dual ? 2 : 1;
  // As many vectors at a time as leave 1024 workgroups (four to a compute unit): a wave adds up its lanes' sums for every vector and row,
  // which bounds a small network's launch (width 128, two blocks, ten vectors: 11.0 us with eight at a time, 4.9 with two).
  const int tiles = (6 * D + GEMV_OUT - 1) / GEMV_OUT, rows = mo.sets * f.blocks + 1;
  auto fills = [&](int pc) { return (int64_t)tiles * rows * ((P + pc - 1) / pc) >= 1024; };
  const int pc = P == 1 ? 1 : P > 4 && fills(8) ? 8 : P > 2 && fills(4) ? 4 : 2, passes = (P + pc - 1) / pc;
  // split the vectors until there are 2048 workgroups (eight to a compute unit) or one pass of `pc` vectors is left to each
  const int split = (int)std::min<int64_t>(passes, std::max<int64_t>(1, 2048 / ((int64_t)tiles * rows)));
  mo.span = (passes + split - 1) / split * pc;
  const dim3 grid(tiles, rows, (P + mo.span - 1) / mo.span);
  if (P == 1) modulation_kernel<1><<<grid, dim3(256), 0, n.s>>>(mo);
  else if (pc == 2) modulation_kernel<2><<<grid, dim3(256), 0, n.s>>>(mo);
  else if (pc == 4) modulation_kernel<4><<<grid, dim3(256), 0, n.s>>>(mo);
  else modulation_kernel<8><<<grid, dim3(256), 0, n.s>>>(mo);
  PG_LAUNCH_CHECK("modulation_kernel");
  return PG_OK;
}
}  // namespace

// Modulation vectors of steps [step, step + steps), steps <= mod_steps, for evaluations that name their row (NetBatch::mod_row).
// One step's are matrix-vector products bound by reading the weights, and three launches of latency: 24 blocks of width 1536
// 129 us a step, 519 us for ten steps together; two blocks of width 128 13 us a step, 19 for ten.
pg_status net_modulate(pg_ctx* c, int step, int steps, const uint16_t* weights, hipStream_t s) {
  Net n{c, s, (char*)c->buf.workspace + c->ws_net, weights};
  const ModPlan m = mod_plan(c, n);
  const StepInputs a = time_inputs(c, n, m, step);
  step_inputs_kernel<<<dim3((unsigned)a.t1_blocks, (unsigned)steps), dim3(256), 0, s>>>(a);
  PG_LAUNCH_CHECK("step_inputs_kernel");
  return launch_modulation(c, n, m, steps);
}

__global__ void batch_rows_kernel(const int32_t* __restrict__ group_of, int M, int steps, int P, int32_t* __restrict__ groups,
                                  int32_t* __restrict__ mods) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M * steps) return;
  const int g = group_of[i % M];
  groups[i] = g;
  mods[i] = (i / M) * P + g;
}

pg_status net_batch_steps(pg_ctx* c, int steps, NetBatch* batch, hipStream_t s) {
  int32_t* groups = reinterpret_cast<int32_t*>((char*)c->buf.workspace + c->ws_net + c->net.rows);
  int32_t* mods = groups + c->M0;
  const int M = c->M * steps;
  batch_rows_kernel<<<dim3((M + 255) / 256), dim3(256), 0, s>>>(c->buf.group_of, c->M, steps, c->cfg.P, groups, mods);
  PG_LAUNCH_CHECK("batch_rows_kernel");
  batch->M = M; batch->group_of = groups; batch->mod_of = mods; batch->mod_row = 0;
  return PG_OK;
}

namespace {
// what the narrow networks' kernels are given; mod, fmod: vectors of the batch's first row
SmallNetArgs small_args(const pg_ctx* c, const Net& n, const NetBatch& batch, const float* mod, const float* fmod) {
  const pg_config& f = c->cfg;
  auto layer = [&](int w, int b) { return SmallLayer{n.w(w), n.w(b), n.ld(w)}; };
  SmallNetArgs a{};
  a.x = batch.x; a.u = c->buf.u; a.group_of = batch.group_of; a.mod_of = batch.mod_of; a.M = batch.M;
  a.C = f.C; a.H = f.H; a.W = f.W; a.Li = c->Li; a.Lc = c->L - c->Li; a.L = c->L; a.blocks = f.blocks;
  if (a.Lc) a.ctx_h = n.at<float>(c->net.ctx_h);
  a.embed = layer(PG_W_PE_W, PG_W_PE_B); a.qkv = layer(PG_W_QKV_W, PG_W_QKV_B); a.out = layer(PG_W_O_W, PG_W_O_B);
  a.fc1 = layer(PG_W_FC1_W, PG_W_FC1_B); a.fc2 = layer(PG_W_FC2_W, PG_W_FC2_B); a.fin = layer(PG_W_F_W, PG_W_F_B);
  a.pos = n.w(PG_W_POS); a.mod = mod; a.fmod = fmod; a.block_stride = c->block_stride;
  a.scale_log2 = (float)(1.4426950408889634 / std::sqrt((double)(f.D / f.heads)));
  return a;
}
}  // namespace

pg_status net_rows(pg_ctx* c, const NetBatch& batch, const RowsPass& pass, const uint16_t* weights, hipStream_t s) {
  const pg_config& f = c->cfg;
  Net n{c, s, (char*)c->buf.workspace + c->ws_net, weights};
  const ModPlan mp = mod_plan(c, n);
  const int64_t row = (int64_t)std::max(0, batch.mod_row) * f.P;
  const int hd = f.D / f.heads;
  const SmallNetArgs net = small_args(c, n, batch, mp.mod + row * mp.ld, mp.fmod + row * 2 * f.D);
  RowsArgs a{};
  a.hs = n.at<float>(c->net.rows_h);
  auto launch = [&](int block, int to, bool start, const float* x, const RowsUpdate* update) -> pg_status {
    a.qk_in = n.at<uint16_t>(c->net.rows_qk[1 - to]); a.vt_in = n.at<uint16_t>(c->net.rows_vt[1 - to]);
    a.qk_out = n.at<uint16_t>(c->net.rows_qk[to]); a.vt_out = n.at<uint16_t>(c->net.rows_vt[to]);
    c->rows_buffer = to;
    a.x = x;
    a.mod_next = net.mod + (block < 0 ? 0 : f.P * mp.ld);
    a.update = update != nullptr;
    if (update) a.up = *update;
    return launch_small_rows(net, a, f.D, hd, block, start, s);
  };
  // the evaluation as one product: its layers' flops and its attention's
  const double rows = (double)batch.M * c->L, image = (double)batch.M * c->Li;
  const int rec = prof_open(PROF_GEMM, f.blocks * rows * (24.0 * f.D * f.D + 4.0 * c->L * f.D) + 16.0 * image * f.D * f.C, s);
  pg_status st = PG_OK;
  if (pass.begin) st = launch(-1, 0, true, pass.before ? pass.x_before : pass.x, pass.before);
  for (int b = 0; b < f.blocks && st == PG_OK; ++b) {
    const bool last = b + 1 == f.blocks;
    st = launch(b, 1 - c->rows_buffer, last && pass.start_next, pass.x, last ? pass.after : nullptr);
  }
  prof_close(rec, s);
  return st;
}

pg_status net_forward(pg_ctx* c, int step, const NetBatch& batch, const uint16_t* weights, hipStream_t s) {
  const pg_config& f = c->cfg;
  Net n{c, s, (char*)c->buf.workspace + c->ws_net, weights};
  const NetPlan& pl = c->net;
  const int D = f.D, M = batch.M, L = c->L, Li = c->Li, P = f.P, hd = D / f.heads;
  const int R = M * L, Ri = M * Li;
  const int Lpad = (L + 63) / 64 * 64, Lcpad = (f.Lc + 63) / 64 * 64, Kp = (4 * f.C + 63) / 64 * 64;
  if (M == 0) return PG_OK;
  float* h = n.at<float>(pl.h);
  uint16_t* act = n.at<uint16_t>(pl.act);
  uint16_t* qk = n.at<uint16_t>(pl.qkv);
  uint16_t* vt = n.at<uint16_t>(pl.vt);
  uint16_t* att = n.at<uint16_t>(pl.att);
  uint16_t* hid = n.at<uint16_t>(pl.hid);
  uint16_t* tok = n.at<uint16_t>(pl.tok);
  const ModPlan mp = mod_plan(c, n);
  const bool own_step = batch.mod_row < 0;          // this step's modulation vectors are made here
  const int64_t mod_ld = mp.ld;
  const float* mod = mp.mod + (own_step ? 0 : batch.mod_row) * P * mod_ld;
  const float* cmod = mp.cmod + (own_step ? 0 : batch.mod_row) * P * mod_ld;
  const float* fmod = mp.fmod + (int64_t)(own_step ? 0 : batch.mod_row) * P * 2 * D;
  const bool dual = f.net_kind == PG_NET_MMDIT;
  const int Rc = M * f.Lc;                          // context rows (dual-stream planes)
  const int32_t* group_of = batch.group_of;
  const int32_t* mod_of = batch.mod_of;
  const float scale_log2 = (float)(1.4426950408889634 / std::sqrt((double)hd));
  const bool small = small_net_takes(c);

  // ---- conditioning, patch tokens and context rows ----
  {
    StepInputs a = time_inputs(c, n, mp, step);
    if (!own_step) a.t1_blocks = 0;
    a.x = batch.x; a.tok = tok; a.M = M; a.C = f.C; a.H = f.H; a.W = f.W; a.Kp = Kp;
    const bool context = f.net_kind == PG_NET_JOINT || dual;
    a.h = h; a.group_of = group_of; a.Lc = context ? f.Lc : 0;
    if (context) a.ctx_h = n.at<float>(pl.ctx_h);
    a.row_base = dual ? (int64_t)Ri : (int64_t)Li; a.row_stride = dual ? f.Lc : L;
    a.patch_blocks = small ? 0 : (int)(((int64_t)M * (Kp / 4) * Li + 255) / 256);
    const int64_t context_blocks = small ? 0 : ((int64_t)M * a.Lc * (D / 4) + 255) / 256;
    const int64_t blocks = a.t1_blocks + a.patch_blocks + context_blocks;
    if (blocks > 0) {
      step_inputs_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(a);
      PG_LAUNCH_CHECK("step_inputs_kernel");
    }
    if (own_step) PG_TRY(launch_modulation(c, n, mp, 1));
  }

  // ---- narrow networks on short sequences: the rest in one launch, or one per block ----
  if (small) {
    if (small_rows_evaluates(c, M)) return net_rows(c, batch, RowsPass{batch.x, true, nullptr, nullptr, nullptr, false}, weights, s);
    return launch_small_net(small_args(c, n, batch, mod, fmod), D, hd, s);
  }

  // ---- patch embedding (+ position table) ----
  {
    GemmArgs g{};
    g.A = tok; g.lda = Kp; g.W = n.w(PG_W_PE_W); g.ldw = n.ld(PG_W_PE_W); g.bias = n.w(PG_W_PE_B);
    g.M = Ri; g.N = D; g.K = Kp; g.k_algo = 4 * f.C; g.outf = h; g.ldo = D; g.L = dual ? Li : L; g.Li = Li; g.pos = n.w(PG_W_POS);
    PG_TRY(launch_gemm(g, EPI_EMBED, s));
  }
  // act[m * L_out + t, :] = bf16(LN(h[m * L_in + t, :]) * (1 + scale) + shift), t < L_out
  auto ln = [&](const LnArgs& a) -> pg_status {
    if (a.rows_out <= 0) return PG_OK;
    const dim3 grid((a.rows_out + 3) / 4), block(256);
    auto run = [&](auto nv_c) {
      constexpr int NV = decltype(nv_c)::value;
      if (D == 256 * NV) ln_modulate_kernel<NV, true><<<grid, block, 0, s>>>(a);
      else ln_modulate_kernel<NV, false><<<grid, block, 0, s>>>(a);
    };
    switch ((D + 255) / 256) {                    // D is a multiple of 64: rows of h, out and the modulation vectors stay 16-byte aligned
      case 1: run(std::integral_constant<int, 1>{}); break;
      case 2: run(std::integral_constant<int, 2>{}); break;
      case 3: run(std::integral_constant<int, 3>{}); break;
      case 4: run(std::integral_constant<int, 4>{}); break;
      case 5: run(std::integral_constant<int, 5>{}); break;
      case 6: run(std::integral_constant<int, 6>{}); break;
      case 7: run(std::integral_constant<int, 7>{}); break;
      case 8: run(std::integral_constant<int, 8>{}); break;
      default: ln_modulate_kernel<0, false><<<grid, block, 0, s>>>(a);
    }
    PG_LAUNCH_CHECK("ln_modulate_kernel");
    return PG_OK;
  };
  auto layer_norm = [&](const float* shift, const float* scale, int64_t ld, int rows_out, int L_out) -> pg_status {
    return ln(LnArgs{h, act, shift, scale, ld, mod_of, rows_out, dual ? L_out : L, L_out, D, rows_out, nullptr, nullptr, 1});
  };
  // both planes of the dual-stream network in one launch
  auto layer_norm_pair = [&](const float* const* mods, int slot) -> pg_status {
    return ln(LnArgs{h, act, mods[0] + slot * D, mods[0] + (slot + 1) * D, mod_ld, mod_of, Ri + Rc, Li, Li, D,
                     Ri, mods[1] + slot * D, mods[1] + (slot + 1) * D, f.Lc});
  };

  const bool chain = row_chain_takes(D, c->M0, dual ? Li : L, dual ? f.Lc : 0);     // what lies between two attentions in one launch

  // ---- dual-stream blocks: two planes (image rows, context rows), joint q | k and V^T ----
  if (dual) {
    float* hs[2] = {h, h + (size_t)Ri * D};
    uint16_t* acts[2] = {act, act + (size_t)Ri * D};
    uint16_t* atts[2] = {att, att + (size_t)Ri * D};
    uint16_t* hids[2] = {hid, hid + (size_t)Ri * 4 * D};
    const int rows[2] = {Ri, Rc}, Ls[2] = {Li, f.Lc}, toff[2] = {0, Li};
    const int W_QN[2] = {PG_W_QN_G, PG_W_C_QN_G}, W_KN[2] = {PG_W_KN_G, PG_W_C_KN_G};
    const int W_QKV[2] = {PG_W_QKV_W, PG_W_C_QKV_W}, B_QKV[2] = {PG_W_QKV_B, PG_W_C_QKV_B};
    const int W_O[2] = {PG_W_O_W, PG_W_C_O_W}, B_O[2] = {PG_W_O_B, PG_W_C_O_B};
    const int W_FC1[2] = {PG_W_FC1_W, PG_W_C_FC1_W}, B_FC1[2] = {PG_W_FC1_B, PG_W_C_FC1_B};
    const int W_FC2[2] = {PG_W_FC2_W, PG_W_C_FC2_W}, B_FC2[2] = {PG_W_FC2_B, PG_W_C_FC2_B};
    for (int b = 0; b < f.blocks; ++b) {
      const float* mbs[2] = {mod + (size_t)b * 6 * D, cmod + (size_t)b * 6 * D};
      GemmArgs g[2];
      if (!chain) PG_TRY(layer_norm_pair(mbs, 0));
      for (int st = 0; st < 2 && !chain; ++st) {
        g[st] = GemmArgs{};
        g[st].A = acts[st]; g[st].lda = D; g[st].W = n.w(W_QKV[st], b); g[st].ldw = n.ld(W_QKV[st]); g[st].bias = n.w(B_QKV[st], b);
        g[st].M = rows[st]; g[st].N = 3 * D; g[st].K = D; g[st].outb = qk; g[st].ldob = 2 * D; g[st].vt = vt; g[st].v_start = 2 * D;
        g[st].Lpad = Lpad; g[st].L = Ls[st]; g[st].Lout = L; g[st].tok_off = toff[st];
        // queries and keys leave the projection RMS-normalised per head, queries also in the softmax's log2 units
        g[st].norm_hd = hd; g[st].qn_g = n.w(W_QN[st], b); g[st].kn_g = n.w(W_KN[st], b);
        g[st].out_scale = scale_log2; g[st].scale_cols = D;
      }
      ChainArgs r{};
      r.qk = qk; r.vt = vt; r.mod_ld = mod_ld; r.mod_of = mod_of; r.M = M; r.Lpad = Lpad; r.out_scale = scale_log2; r.norm_hd = hd;
      auto projection = [&](int st, int block, const float* norm) {
        ChainStream& t = r.s[st];
        t.h = hs[st]; t.L = Ls[st]; t.norm2 = norm;
        t.next_w = n.w(W_QKV[st], block); t.next_b = n.w(B_QKV[st], block); t.qn_g = n.w(W_QN[st], block); t.kn_g = n.w(W_KN[st], block);
      };
      if (!chain) PG_TRY(launch_gemm_pair(g[0], g[1], EPI_QKV, s));
      else if (b == 0) {
        for (int st = 0; st < 2; ++st) projection(st, 0, mbs[st]);
        PG_TRY(launch_row_chain(r, D, CHAIN_START, s));
      }
      AttnArgs a{};
      a.q = qk; a.ldq = 2 * D; a.k = qk + D; a.ldk = 2 * D; a.k_bstride = (int64_t)L * 2 * D;
      a.vt = vt; a.vt_bstride = (int64_t)D * Lpad; a.Lkpad = Lpad; a.out = atts[0]; a.ldo = D;
      a.split = Li; a.out2 = atts[1];
      a.B = M; a.Lq = L; a.Lk = L; a.heads = f.heads; a.scale_log2 = scale_log2; a.q_prescaled = 1; a.v_swapped = 1;
      PG_TRY(launch_attention(a, hd, s));
      if (chain) {                                   // the context's rows are not used any more after the last block
        const bool last = b + 1 == f.blocks;
        if (last) { r.norm_hd = 0; r.s[1].L = 0; }
        for (int st = 0; st < (last ? 1 : 2); ++st) {
          ChainStream& t = r.s[st];
          if (!last) projection(st, b + 1, mbs[st] + 6 * D);
          t.att = atts[st]; t.h = hs[st]; t.L = Ls[st];
          t.o_w = n.w(W_O[st], b); t.o_b = n.w(B_O[st], b); t.fc1_w = n.w(W_FC1[st], b); t.fc1_b = n.w(B_FC1[st], b);
          t.fc2_w = n.w(W_FC2[st], b); t.fc2_b = n.w(B_FC2[st], b);
          t.gate1 = mbs[st] + 2 * D; t.norm1 = mbs[st] + 3 * D; t.gate2 = mbs[st] + 5 * D;
        }
        PG_TRY(launch_row_chain(r, D, last ? CHAIN_LAST : CHAIN_BLOCK, s));
        continue;
      }
      // the layers that add into the residual stream: `gate` is the slot of their gates among the modulation vectors
      auto residual = [&](uint16_t* const* in, int K, const int* W, const int* B, int gate) -> pg_status {
        for (int st = 0; st < 2; ++st) {
          g[st] = GemmArgs{};
          g[st].A = in[st]; g[st].lda = K; g[st].W = n.w(W[st], b); g[st].ldw = n.ld(W[st]); g[st].bias = n.w(B[st], b);
          g[st].M = rows[st]; g[st].N = D; g[st].K = K; g[st].outf = hs[st]; g[st].ldo = D; g[st].L = Ls[st];
          g[st].gate = mbs[st] + gate * D; g[st].gate_ld = mod_ld; g[st].group_of = mod_of;
        }
        return launch_gemm_pair(g[0], g[1], EPI_RESID, s);
      };
      PG_TRY(residual(atts, D, W_O, B_O, 2));
      PG_TRY(layer_norm_pair(mbs, 3));
      for (int st = 0; st < 2; ++st) {
        g[st] = GemmArgs{};
        g[st].A = acts[st]; g[st].lda = D; g[st].W = n.w(W_FC1[st], b); g[st].ldw = n.ld(W_FC1[st]); g[st].bias = n.w(B_FC1[st], b);
        g[st].M = rows[st]; g[st].N = 4 * D; g[st].K = D; g[st].outb = hids[st]; g[st].ldob = 4 * D;
      }
      PG_TRY(launch_gemm_pair(g[0], g[1], EPI_GELU, s));
      PG_TRY(residual(hids, 4 * D, W_FC2, B_FC2, 5));
    }
  }

  // attention over the prompt's context tokens
  auto cross_attention = [&](int b) -> pg_status {
    AttnArgs a{};
    a.q = qk; a.ldq = D;
    a.k = n.at<uint16_t>(pl.ckv) + (size_t)b * P * f.Lc * D; a.ldk = D; a.k_bstride = (int64_t)f.Lc * D;
    a.vt = n.at<uint16_t>(pl.ckvt) + (size_t)b * P * D * Lcpad; a.vt_bstride = (int64_t)D * Lcpad; a.Lkpad = Lcpad;
    a.out = att; a.ldo = D; a.kv_map = group_of;
    a.B = M; a.Lq = L; a.Lk = f.Lc; a.heads = f.heads; a.scale_log2 = scale_log2; a.q_prescaled = 1; a.v_swapped = 1;
    return launch_attention(a, hd, s);
  };
  for (int b = 0; b < (dual ? 0 : f.blocks); ++b) {
    const float* mb = mod + (size_t)b * 6 * D;     // shift1, scale1, gate1, shift2, scale2, gate2
    // attention sub-block
    ChainArgs r{};
    r.qk = qk; r.vt = vt; r.mod_ld = mod_ld; r.mod_of = mod_of; r.M = M; r.Lpad = Lpad; r.out_scale = scale_log2;
    ChainStream& t = r.s[0];
    t.h = h; t.L = L;
    auto projection = [&](int block, const float* norm) {
      t.norm2 = norm; t.next_w = n.w(PG_W_QKV_W, block); t.next_b = n.w(PG_W_QKV_B, block);
    };
    if (chain && b == 0) {
      projection(0, mb);
      PG_TRY(launch_row_chain(r, D, CHAIN_START, s));
    }
    if (!chain) {
      PG_TRY(layer_norm(mb, mb + D, mod_ld, R, L));
      GemmArgs g{};
      g.A = act; g.lda = D; g.W = n.w(PG_W_QKV_W, b); g.ldw = n.ld(PG_W_QKV_W); g.bias = n.w(PG_W_QKV_B, b);
      g.M = R; g.N = 3 * D; g.K = D; g.outb = qk; g.ldob = 2 * D; g.vt = vt; g.v_start = 2 * D; g.Lpad = Lpad; g.L = L;
      g.out_scale = scale_log2; g.scale_cols = D;   // queries leave the projection already in the softmax's log2 units
      PG_TRY(launch_gemm(g, EPI_QKV, s));
    }
    {
      AttnArgs a{};
      a.q = qk; a.ldq = 2 * D; a.k = qk + D; a.ldk = 2 * D; a.k_bstride = (int64_t)L * 2 * D;
      a.vt = vt; a.vt_bstride = (int64_t)D * Lpad; a.Lkpad = Lpad; a.out = att; a.ldo = D;
      a.B = M; a.Lq = L; a.Lk = L; a.heads = f.heads; a.scale_log2 = scale_log2; a.q_prescaled = 1; a.v_swapped = 1;
      PG_TRY(launch_attention(a, hd, s));
    }
    if (chain) {
      const bool last = b + 1 == f.blocks;
      t.att = att; t.o_w = n.w(PG_W_O_W, b); t.o_b = n.w(PG_W_O_B, b); t.gate1 = mb + 2 * D;
      if (f.net_kind == PG_NET_CROSS) {
        t.next_w = n.w(PG_W_CQ_W, b); t.next_b = n.w(PG_W_CQ_B, b);
        PG_TRY(launch_row_chain(r, D, CHAIN_QUERIES, s));
        PG_TRY(cross_attention(b));
        t.o_w = n.w(PG_W_CO_W, b); t.o_b = n.w(PG_W_CO_B, b); t.gate1 = nullptr;
      }
      t.norm1 = mb + 3 * D; t.gate2 = mb + 5 * D;
      t.fc1_w = n.w(PG_W_FC1_W, b); t.fc1_b = n.w(PG_W_FC1_B, b); t.fc2_w = n.w(PG_W_FC2_W, b); t.fc2_b = n.w(PG_W_FC2_B, b);
      if (!last) projection(b + 1, mb + 6 * D);
      PG_TRY(launch_row_chain(r, D, last ? CHAIN_LAST : CHAIN_BLOCK, s));
      continue;
    }
    {
      GemmArgs o{};
      o.A = att; o.lda = D; o.W = n.w(PG_W_O_W, b); o.ldw = n.ld(PG_W_O_W); o.bias = n.w(PG_W_O_B, b);
      o.M = R; o.N = D; o.K = D; o.outf = h; o.ldo = D; o.L = L; o.gate = mb + 2 * D; o.gate_ld = mod_ld;
      o.group_of = mod_of;
      PG_TRY(launch_gemm(o, EPI_RESID, s));
    }
    // cross-attention sub-block over the prompt's context tokens
    if (f.net_kind == PG_NET_CROSS) {
      PG_TRY(layer_norm(nullptr, nullptr, 0, R, L));
      GemmArgs g{};
      g.A = act; g.lda = D; g.W = n.w(PG_W_CQ_W, b); g.ldw = n.ld(PG_W_CQ_W); g.bias = n.w(PG_W_CQ_B, b);
      g.M = R; g.N = D; g.K = D; g.outb = qk; g.ldob = D;
      g.out_scale = scale_log2; g.scale_cols = D;
      PG_TRY(launch_gemm(g, EPI_BF16, s));
      PG_TRY(cross_attention(b));
      GemmArgs o{};
      o.A = att; o.lda = D; o.W = n.w(PG_W_CO_W, b); o.ldw = n.ld(PG_W_CO_W); o.bias = n.w(PG_W_CO_B, b);
      o.M = R; o.N = D; o.K = D; o.outf = h; o.ldo = D; o.L = L; o.gate = nullptr; o.group_of = group_of;
      PG_TRY(launch_gemm(o, EPI_RESID, s));
    }
    // MLP sub-block
    PG_TRY(layer_norm(mb + 3 * D, mb + 4 * D, mod_ld, R, L));
    {
      GemmArgs g{};
      g.A = act; g.lda = D; g.W = n.w(PG_W_FC1_W, b); g.ldw = n.ld(PG_W_FC1_W); g.bias = n.w(PG_W_FC1_B, b);
      g.M = R; g.N = 4 * D; g.K = D; g.outb = hid; g.ldob = 4 * D;
      PG_TRY(launch_gemm(g, EPI_GELU, s));
      GemmArgs o{};
      o.A = hid; o.lda = 4 * D; o.W = n.w(PG_W_FC2_W, b); o.ldw = n.ld(PG_W_FC2_W); o.bias = n.w(PG_W_FC2_B, b);
      o.M = R; o.N = D; o.K = 4 * D; o.outf = h; o.ldo = D; o.L = L; o.gate = mb + 5 * D; o.gate_ld = mod_ld;
      o.group_of = mod_of;
      PG_TRY(launch_gemm(o, EPI_RESID, s));
    }
  }

  // ---- final layer on the image tokens, written straight into the latent layout ----
  PG_TRY(layer_norm(fmod, fmod + D, 2 * D, Ri, Li));
  GemmArgs g{};
  g.A = act; g.lda = D; g.W = n.w(PG_W_F_W); g.ldw = n.ld(PG_W_F_W); g.bias = n.w(PG_W_F_B);
  g.M = Ri; g.N = 4 * f.C; g.K = D; g.outf = c->buf.u; g.Li = Li; g.Wp = f.W / 2; g.HW = f.H * f.W; g.Wimg = f.W;
  return launch_gemm(g, EPI_UNPATCH, s);
}

}  // namespace pg
