// The layers between two attentions of a block (output projection, residual sum, LayerNorm, MLP, LayerNorm, queries / keys / values
// of the next block; in front of the first attention the last two) for networks of width 128, 192 and 256: a workgroup takes 16 or 32
// rows of one trajectory through all of them in one launch.  In the dual-stream network a workgroup's rows are image or context
// tokens, with the weights of their stream.
//
// Layer by layer each of them is a launch of 4 to 8 us with a microsecond of work in it (six of them and their gaps: 40 us).  They need
// nothing but their own rows, so the residual stream stays in registers, operands and hidden values in LDS, and what a workgroup
// reads is the weights, all of them: 24 D^2 bytes at what a compute unit reads from its L2, 64 bytes a cycle, is what bounds it.  A
// wave has 32 of the D columns of every product, so nobody else needs its weights: they come by direct loads, in pieces of 16 rows x
// 64 columns, through a ring of its own, asked for ahead across the barriers.
// A launch takes 8.6, 16 and 21 us (width 128, 192, 256; 2.6, 5.8 and 10.4 for the weights alone).  Of the 43000 cycles at width 256 the
// four quarters of the MLP are 19600 and the next projection 6700, 52 bytes a cycle; until the first product is done 10000 pass, most of
// them in waiting for attention's output and the first weights from beyond the L2, and the LayerNorms take 1600 and 3000.  Reads from LDS
// and MFMAs are in the shadow of the loads: 32 rows take as long as 16 at width 256 (21.1 us), and 13.9 us instead of 9.9 at 128, so where
// 16 would be more workgroups than compute units a workgroup has 32.
#include <algorithm>
#include <type_traits>
#include "operands.hpp"
#include "row_chain.hpp"

namespace pg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

namespace {
// products of a launch, each [rows, D] x [D, D]^T: the projection, then fc1 and fc2 by quarters of the hidden values, then the next ones
template <int KIND> constexpr int products() { return KIND == CHAIN_QUERIES ? 2 : KIND == CHAIN_BLOCK ? 12 : KIND == CHAIN_LAST ? 9 : 3; }

template <int D, int RT> struct Chain {
  static constexpr int WAVES = D / 32, THREADS = 64 * WAVES;
  static constexpr int PIECES = D / 32;              // of a product, per wave: 64 columns of 16 rows, the other 16 rows, the next 64 columns
  static constexpr int PIECE = 2048;                 // bytes
  static constexpr int SLOTS = D == 256 ? 4 : PIECES;        // of the ring: every product starts with its first one
  static constexpr int PITCH = D + 8, H_PITCH = D + 4;       // in elements: the 16 rows of a fragment start in different banks
};

__device__ __forceinline__ f32x4v widen(uint2 v) {
  return f32x4v{bf16_to_f32((uint16_t)v.x), bf16_to_f32((uint16_t)(v.x >> 16)), bf16_to_f32((uint16_t)v.y), bf16_to_f32((uint16_t)(v.y >> 16))};
}
__device__ __forceinline__ f32x4v four_of(const uint16_t* b) { return widen(*reinterpret_cast<const uint2*>(b)); }
__device__ __forceinline__ void put4(uint16_t* p, f32x4v v) { *reinterpret_cast<uint2*>(p) = pack_bf16x4({v[0], v[1], v[2], v[3]}); }
__device__ __forceinline__ int turn(int row) { return (row ^ (row >> 3)) & 7; }   // of a row's eight chunks in a piece

// a product's weights, from the wave's columns on; rows of D or 4 D columns
template <bool WIDE> struct Source { const uint16_t* w; };

// One wave's way through the weights of a launch.  RT: row tiles of 16.
template <int D, int RT>
struct Weights {
  using C = Chain<D, RT>;
  typedef bf16x8 Piece[2];
  typedef bf16x8 Rows[RT][D / 32];
  uint32_t off[2], off4[2];                          // the lane's bytes in a piece with rows of D and of 4 D columns
  const unsigned char* ring;
  uint32_t lds;
  int lane;

  __device__ __forceinline__ void init(unsigned char* smem, int wave, int lane_) {
    lane = lane_;
    ring = smem + wave * C::SLOTS * C::PIECE;
    lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + wave * C::SLOTS * C::PIECE);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = q * 8 + lane / 8, chunk = (lane & 7) ^ turn(row);
      off[q] = (uint32_t)(row * D + chunk * 8) * 2;
      off4[q] = (uint32_t)(row * 4 * D + chunk * 8) * 2;
    }
  }
  template <int I, bool WIDE> __device__ __forceinline__ void request(Source<WIDE> p) const {
    const uint16_t* base = p.w + (I & 1) * 16 * (WIDE ? 4 * D : D) + (I >> 1) * 64;
#pragma unroll
    for (int q = 0; q < 2; ++q) dma16(WIDE ? off4[q] : off[q], base, lds + I % C::SLOTS * C::PIECE + q * 1024);
  }
  template <int I = 0> __device__ __forceinline__ void begin(Source<false> p) const {
    if constexpr (I < C::SLOTS) { request<I>(p); begin<I + 1>(p); }
  }
  // The launch's weights (of the workgroup's stream) into the L2 of this XCD: its workgroups (every eighth of the grid) touch a share of
  // the 128-byte lines each.  They all run through the weights side by side, so without this nearly every piece of theirs was waited
  // for from beyond the L2.  The first product waits for these loads, too, so where few workgroups would have many each they are left
  // out: four blocks of width 256, 1, 4, 8, 64 trajectories of one stream and 100, 100, 256, 256 tokens, us with / without them 179 / 139,
  // 145 / 139, 143.6 / 144.7, 154 / 156; from eight workgroups to an XCD on they pay.  In the dual-stream network a share is that of the
  // workgroup's number among all, so some lines of either stream stay cold; every workgroup touching those of both streams takes
  // longer (8 of 128 tokens 138.5 / 144.8, 4 of 88 156 / 163).
  template <int KIND> __device__ __forceinline__ void warm(const ChainStream& a, unsigned char* touched, int wave) const {
    constexpr int LOADS = D * D * 2 / (128 * 64);    // of 64 lines, for the weights of a product
    const int id = blockIdx.y * gridDim.x + blockIdx.x, wgs = (gridDim.x * gridDim.y + 7) / 8;
    if (wgs < 8) return;
    const uint32_t to = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)touched);
    for (int k = id / 8 * C::WAVES + wave; k < products<KIND>() * LOADS; k += wgs * C::WAVES) {
      const int p = k / LOADS;
      const uint16_t* base = KIND == CHAIN_START ? a.next_w + p * D * D : p == 0 ? a.o_w
                             : KIND == CHAIN_QUERIES ? a.next_w : p < 5 ? a.fc1_w + (p - 1) * D * D
                             : p < 9 ? a.fc2_w + (p - 5) * D * D : a.next_w + (p - 9) * D * D;
      dma4(lane * 128u, base + (k - p * LOADS) * 64 * 64, to);
    }
  }
  // the lane's part of the workgroup's rows in LDS, columns of piece I and I + 1
  template <int I> __device__ __forceinline__ void read_rows(const uint16_t* A, Rows& x) const {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        x[t][I + ks] = *reinterpret_cast<const bf16x8*>(A + ((lane & 15) + t * 16) * C::PITCH + 8 * (lane >> 4) + I * 32 + 32 * ks);
  }
  template <int I = 0> __device__ __forceinline__ void read_all_rows(const uint16_t* A, Rows& x) const {
    if constexpr (I < C::PIECES) { read_rows<I>(A, x); read_all_rows<I + 2>(A, x); }
  }
  // piece I: awaited and read, with the rows' columns that it is multiplied by; `more`: pieces of the next product have been asked for
  template <bool LOAD, int I> __device__ __forceinline__ void fetch(const uint16_t* A, Piece& w, Rows& x, bool more) const {
    constexpr int asked = I + C::SLOTS - (I > 0);    // the first piece that was not asked for yet
    constexpr int behind = 2 * (asked - 1 - I);      // loads that were asked for behind this one
    if (asked <= C::PIECES || more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(behind) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int lr = lane & 15, lk = lane >> 4;
    const unsigned char* at = ring + I % C::SLOTS * C::PIECE + lr * 128;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) w[ks] = *reinterpret_cast<const bf16x8*>(at + ((4 * ks + lk) ^ turn(lr)) * 16);
    if constexpr (LOAD && I % 2 == 0) read_rows<I>(A, x);
  }
  // piece I multiplied while the next one is read, its slot given to the piece that comes SLOTS later
  template <bool TR, bool LOAD, int I, bool WIDE, bool NEXT_WIDE>
  __device__ __forceinline__ void step(Source<WIDE> p, Source<NEXT_WIDE> next, bool more, const uint16_t* A, Piece& now, Piece& after, Rows& x,
                                       f32x4v (&acc)[2][RT]) const {
    if constexpr (I + 1 < C::PIECES) fetch<LOAD, I + 1>(A, after, x, more);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const bf16x8 v = x[t][(I & ~1) + ks];
        acc[I & 1][t] = TR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, now[ks], acc[I & 1][t], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_16x16x32_bf16(now[ks], v, acc[I & 1][t], 0, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
    // the piece has been read: it is multiplied
    if constexpr (I + C::SLOTS < C::PIECES) request<I + C::SLOTS>(p);
    else if (more) request<I + C::SLOTS - C::PIECES>(next);
    if constexpr (I + 1 < C::PIECES) step<TR, LOAD, I + 1>(p, next, more, A, after, now, x, acc);
  }
  // acc += the workgroup's rows in LDS (x: the lane's part of them, LOAD: to be read) x the wave's 32 columns of product p; the first
  // pieces of `next` are asked for, where there is one (more).  TR: a lane gets four rows of one column, else four columns of one row.
  template <bool LOAD, bool TR = false, bool WIDE, bool NEXT_WIDE>
  __device__ __forceinline__ void product(Source<WIDE> p, Source<NEXT_WIDE> next, bool more, const uint16_t* A, Rows& x, f32x4v (&acc)[2][RT]) const {
    Piece a, b;
    fetch<LOAD, 0>(A, a, x, more);
    step<TR, LOAD, 0>(p, next, more, A, a, b, x, acc);
  }
};

// act[r, :] = bf16(LN(h[r, :]) (1 + scale) + shift), 16 lanes per row
template <int D, int RT>
__device__ __forceinline__ void normalise(const float* h, uint16_t* act, const float* shift, const float* scale) {
  using C = Chain<D, RT>;
  constexpr int V = D / 64;
  const int j = threadIdx.x & 15;
#pragma unroll 1
  for (int r = threadIdx.x >> 4; r < 16 * RT; r += C::THREADS / 16) {
    float4 v[V];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      v[i] = *reinterpret_cast<const float4*>(h + r * C::H_PITCH + 4 * j + 64 * i);
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
      put4(act + r * C::PITCH + n, f32x4v{v[i].x * rstd * (1.f + a.x) + b.x, v[i].y * rstd * (1.f + a.y) + b.y,
                                          v[i].z * rstd * (1.f + a.z) + b.z, v[i].w * rstd * (1.f + a.w) + b.w});
    }
  }
}

// DUAL: two streams with weights of their own, and normalised queries and keys
template <int D, int KIND, int RT, bool DUAL>
__global__ __launch_bounds__(2 * D, D == 128 ? 2 : 1) void row_chain_kernel(const ChainArgs args) {
  using C = Chain<D, RT>;
  constexpr bool START = KIND == CHAIN_START, MLP = KIND == CHAIN_BLOCK || KIND == CHAIN_LAST, NEXT = KIND == CHAIN_BLOCK || START;
  constexpr int ROWS = 16 * RT, NB = KIND == CHAIN_QUERIES ? 2 : KIND == CHAIN_BLOCK ? 9 : KIND == CHAIN_LAST ? 6 : 3;     // biases in units of D
  __shared__ __align__(16) unsigned char ring[C::WAVES * C::SLOTS * C::PIECE];
  __shared__ __align__(16) unsigned char both[ROWS * C::PITCH * 4];      // residual stream for the LayerNorm | hidden values, two quarters
  __shared__ __align__(16) uint16_t act[ROWS * C::PITCH];
  __shared__ __align__(16) float md[4 * D];          // shift, scale of the LayerNorm, shift, scale of the next block
  __shared__ __align__(16) uint16_t bs[NB * D];      // [projection,] [fc1, fc2,] [next]
  __shared__ __align__(16) unsigned char touched[256];
  __shared__ float squares[DUAL ? C::WAVES * ROWS : 1];     // of a wave's columns
  float* hl = reinterpret_cast<float*>(both);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles0 = DUAL ? (args.s[0].L + ROWS - 1) / ROWS : 0;
  const bool second = DUAL && (int)blockIdx.x >= tiles0;
  const ChainStream a = second ? args.s[1] : args.s[0];
  const int lr = lane & 15, lk = lane >> 4, m = blockIdx.y, t0 = (blockIdx.x - (second ? tiles0 : 0)) * ROWS;
  const int n0 = wave * 32 + 4 * lk;                 // the lane's columns: n0 .. n0 + 3 and 16 further
  const int64_t row0 = (int64_t)m * a.L;
  const int64_t mod_row = (int64_t)args.mod_of[m] * args.mod_ld;
  const int L_all = DUAL ? args.s[0].L + args.s[1].L : a.L, tok0 = second ? args.s[0].L : 0;       // the stream's tokens among all
  const int64_t all0 = (int64_t)m * L_all + tok0;

  // ---- asked for at once, in the order of use; rows past the end repeat the last one ----
  constexpr int AV = ROWS * D / 8 / C::THREADS;      // 16-byte chunks of attention's output per thread: RT
  u32x4v av[AV];
#pragma unroll
  for (int i = 0; i < AV && !START; ++i) {
    const int e = i * C::THREADS + tid, r = e / (D / 8), c = e - r * (D / 8);
    av[i] = *reinterpret_cast<const u32x4v*>(a.att + (row0 + min(t0 + r, a.L - 1)) * D + 8 * c);
  }
  u32x4v bias_in = {0u, 0u, 0u, 0u};
  const int bi = 8 * tid;                            // of the biases one after another
  if (bi < NB * D) {
    const uint16_t* p = START ? a.next_b + bi : bi < D ? a.o_b + bi : !MLP ? a.next_b + bi - D
                        : bi < 5 * D ? a.fc1_b + bi - D : bi < 6 * D ? a.fc2_b + bi - 5 * D : a.next_b + bi - 6 * D;
    bias_in = *reinterpret_cast<const u32x4v*>(p);
  }
  f32x4v h[2][RT];
  float* hp[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    hp[t] = a.h + (row0 + min(t0 + 16 * t + lr, a.L - 1)) * D + n0;
#pragma unroll
    for (int c = 0; c < 2; ++c) h[c][t] = *reinterpret_cast<const f32x4v*>(hp[t] + 16 * c);
  }
  f32x4v vec = {0.f, 0.f, 0.f, 0.f};
  if (tid < D) {                                     // of 4 D modulation values
    const int i = 4 * tid;
    if (i < 2 * D) { if (a.norm1) vec = *reinterpret_cast<const f32x4v*>(a.norm1 + mod_row + i); }
    else if (NEXT) vec = *reinterpret_cast<const f32x4v*>(a.norm2 + mod_row + i - 2 * D);
  }
  f32x4v gate1[2], gate2[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (!START) gate1[c] = a.gate1 ? *reinterpret_cast<const f32x4v*>(a.gate1 + mod_row + n0 + 16 * c) : f32x4v{1.f, 1.f, 1.f, 1.f};
    if (MLP) gate2[c] = *reinterpret_cast<const f32x4v*>(a.gate2 + mod_row + n0 + 16 * c);
  }
  __builtin_amdgcn_sched_barrier(0);
  Weights<D, RT> weights;
  weights.init(ring, wave, lane);
  const Source<false> w_out{a.o_w + wave * 32 * D}, w_next{a.next_w + wave * 32 * D};
  auto w_fc1 = [&](int j) { return Source<false>{a.fc1_w + (j * D + wave * 32) * D}; };
  auto w_fc2 = [&](int j) { return Source<true>{a.fc2_w + wave * 32 * 4 * D + j * D}; };
  weights.begin(START ? w_next : w_out);
  weights.template warm<KIND>(a, touched, wave);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < AV && !START; ++i) {
    const int e = i * C::THREADS + tid, r = e / (D / 8), c = e - r * (D / 8);
    *reinterpret_cast<u32x4v*>(act + r * C::PITCH + 8 * c) = av[i];
  }
  if (bi < NB * D) *reinterpret_cast<u32x4v*>(bs + bi) = bias_in;
  if (tid < D) *reinterpret_cast<f32x4v*>(md + 4 * tid) = vec;
  if (!START) __syncthreads();

  f32x4v acc[2][RT];
  typename Weights<D, RT>::Rows x;
  auto start = [&](f32x4v (&v)[2][RT], const uint16_t* bias) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const f32x4v b = four_of(bias + n0 + 16 * c);
#pragma unroll
      for (int t = 0; t < RT; ++t) v[c][t] = b;
    }
  };
  auto add_to_stream = [&](const f32x4v (&gate)[2], const f32x4v (&v)[2][RT]) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int t = 0; t < RT; ++t) h[c][t] = h[c][t] + gate[c] * v[c][t];
  };
  auto stream_to_lds = [&] {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int t = 0; t < RT; ++t) *reinterpret_cast<f32x4v*>(hl + (16 * t + lr) * C::H_PITCH + n0 + 16 * c) = h[c][t];
  };
  auto store_stream = [&] {
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if (t0 + 16 * t + lr < a.L)
#pragma unroll
        for (int c = 0; c < 2; ++c) *reinterpret_cast<f32x4v*>(hp[t] + 16 * c) = h[c][t];
  };
  // rows of the queries (and keys)
  auto store_rows = [&](uint16_t* dst, int ld, float scale) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
      if (t0 + 16 * t + lr < a.L)
#pragma unroll
        for (int c = 0; c < 2; ++c) put4(dst + (all0 + t0 + 16 * t + lr) * ld + n0 + 16 * c, acc[c][t] * scale);
  };
  // RMS norm of the rows' heads, which are the columns of this wave or of this one and its neighbour
  auto normalise_heads = [&](const uint16_t* g) {
    float ss[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      ss[t] = 0.f;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const f32x4v v = acc[c][t];
        ss[t] += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
      }
      ss[t] = across_rows(ss[t], [](float x, float y) { return x + y; });
    }
    if (args.norm_hd == 64) {
      __syncthreads();                               // the sums before these have been read
#pragma unroll
      for (int t = 0; t < RT; ++t)
        if (lk == 0) squares[wave * ROWS + 16 * t + lr] = ss[t];
      __syncthreads();
#pragma unroll
      for (int t = 0; t < RT; ++t) ss[t] = squares[(wave & ~1) * ROWS + 16 * t + lr] + squares[(wave | 1) * ROWS + 16 * t + lr];
    }
    const float inv_hd = args.norm_hd == 64 ? 1.f / 64.f : 1.f / 32.f;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const f32x4v scale = four_of(g + ((n0 + 16 * c) & (args.norm_hd - 1)));
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[c][t] = acc[c][t] * (rsqrtf(ss[t] * inv_hd + 1e-6f) * scale);
    }
  };

  if constexpr (!START) {
    start(acc, bs);
    weights.template product<true>(w_out, MLP ? w_fc1(0) : w_next, true, act, x, acc);
    add_to_stream(gate1, acc);
    stream_to_lds();
    __syncthreads();
    normalise<D, RT>(hl, act, md, md + D);
    __syncthreads();
  }

  if constexpr (KIND == CHAIN_QUERIES) {
    store_stream();
    start(acc, bs + D);
    weights.template product<true>(w_next, w_next, false, act, x, acc);
    store_rows(args.qk, D, args.out_scale);
  }
  if constexpr (MLP) {
    f32x4v sum[2][RT];
    start(sum, bs + 5 * D);
    weights.read_all_rows(act, x);
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {                    // quarters of the hidden values
      uint16_t* hid = reinterpret_cast<uint16_t*>(both) + (j & 1) * ROWS * C::PITCH;
      start(acc, bs + D + j * D);
      weights.template product<false>(w_fc1(j), w_fc2(j), true, act, x, acc);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const f32x4v v = acc[c][t];
          put4(hid + (16 * t + lr) * C::PITCH + n0 + 16 * c, f32x4v{gelu_tanh(v[0]), gelu_tanh(v[1]), gelu_tanh(v[2]), gelu_tanh(v[3])});
        }
      __syncthreads();                               // the other half is read by nobody any more, either
      typename Weights<D, RT>::Rows y;
      weights.template product<true>(w_fc2(j), j < 3 ? w_fc1(j + 1) : w_next, NEXT || j < 3, hid, y, sum);
    }
    add_to_stream(gate2, sum);
    if constexpr (!NEXT) store_stream();
    else __syncthreads();                            // the hidden values have been read
  }
  if constexpr (NEXT) {
    stream_to_lds();
    __syncthreads();
    normalise<D, RT>(hl, act, md + 2 * D, md + 3 * D);
    __syncthreads();
    if (!START) store_stream();                      // behind the last barrier, which would wait for it and for the ring's loads
    weights.read_all_rows(act, x);
    auto part = [&](int i) { return Source<false>{w_next.w + i * D * D}; };
#pragma unroll 1
    for (int i = 0; i < 2; ++i) {                    // queries, keys
      start(acc, bs + (NB - 3 + i) * D);
      weights.template product<false>(part(i), part(i + 1), true, act, x, acc);
      if constexpr (DUAL) normalise_heads(i ? a.kn_g : a.qn_g);
      store_rows(args.qk + i * D, 2 * D, i ? 1.f : args.out_scale);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const float b = bf16_to_f32(bs[(NB - 1) * D + wave * 32 + 16 * c + lr]);
#pragma unroll
      for (int t = 0; t < RT; ++t) acc[c][t] = f32x4v{b, b, b, b};
    }
    weights.template product<false, true>(part(2), part(2), false, act, x, acc);
    // tokens past the end, too, where nobody else's follow: a value row has room for whole tiles, and attention takes nothing from there
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        uint16_t* row = args.vt + ((int64_t)m * D + wave * 32 + 16 * c + lr) * args.Lpad;
        const int tok = t0 + 16 * t + 4 * lk;
        if (!DUAL || ((tok0 & 3) == 0 && tok + 4 <= a.L)) put4(row + value_slot(tok0 + tok), acc[c][t]);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (tok + e < a.L) row[value_slot(tok0 + tok + e)] = (uint16_t)pack_bf16x2(acc[c][t][e], 0.f);
      }
  }
}

template <int D, int KIND, bool DUAL>
pg_status launch_rows(const ChainArgs& a, hipStream_t s) {
  auto tiles = [&](int rows) { return (unsigned)((a.s[0].L + rows - 1) / rows + (DUAL ? (a.s[1].L + rows - 1) / rows : 0)); };
  if ((int64_t)a.M * tiles(16) <= 256) row_chain_kernel<D, KIND, 1, DUAL><<<dim3(tiles(16), (unsigned)a.M), dim3(2 * D), 0, s>>>(a);
  else row_chain_kernel<D, KIND, 2, DUAL><<<dim3(tiles(32), (unsigned)a.M), dim3(2 * D), 0, s>>>(a);
  PG_LAUNCH_CHECK("row_chain_kernel");
  return PG_OK;
}
template <int D>
pg_status launch_width(const ChainArgs& a, ChainKind kind, hipStream_t s) {
  if (kind == CHAIN_QUERIES) return launch_rows<D, CHAIN_QUERIES, false>(a, s);
  if (kind == CHAIN_LAST) return launch_rows<D, CHAIN_LAST, false>(a, s);
  if (kind == CHAIN_START) return a.s[1].L > 0 ? launch_rows<D, CHAIN_START, true>(a, s) : launch_rows<D, CHAIN_START, false>(a, s);
  return a.s[1].L > 0 ? launch_rows<D, CHAIN_BLOCK, true>(a, s) : launch_rows<D, CHAIN_BLOCK, false>(a, s);
}
}  // namespace

// Loops of four steps and four blocks (x: two), us, a launch per layer / here:
//   width 128:  8 trajectories of 200 tokens 638 / 394, 64 of 256 994 / 650, x 384 of 256 2154 / 1449, x 1152 of 256 6236 / 4108
//   width 192:  4 of 64 598 / 469, 64 of 256 1250 / 862, x 256 of 256 2040 / 1646, x 768 of 256 5598 / 4735
//   width 256: 16 of 100 727 / 601, 64 of 256 1386 / 1036, x 256 of 256 2529 / 2154, x 576 of 256 5159 / 4742
//   cross-attention: width 192, 9 of 88 876 / 630, width 256, 36 of 290 1687 / 1359, 4 of 88 960 / 875
//   dual-stream: width 128, 8 of 200 682 / 436, width 192, 64 of 256 1298 / 896, width 256, 4 of 88 695 / 678, 64 of 256 1420 / 1078
// A width of 320 won in a band of sizes alone (64 of 256 1683 / 1448, 4 of 88 722 / 880, x 384 of 256 4903 / 5480), and so did 384.
//
// Its time goes with the workgroups, that of a launch per layer with the rows, and a trajectory's last workgroup may have few: us a
// launch per layer / here, two blocks, width 192: 9344 trajectories of 16 tokens 1327 / 1687, 7488 of 20 1292 / 1464, 1472 of 100
// 1103 / 1128, 1344 of 110 1156 / 1068, 1088 of 132 1125 / 1075; few workgroups: 1024 of 8 160 / 193, 512 of 16 141 / 127, 384 of 1
// 100 / 105, 256 of 4 96 / 66; width 256: 1472 of 100 1417 / 1591, 1664 of 90 1512 / 1441, 4672 of 256 10966 / 10307; dual-stream, width
// 256: 1024 of 110 and 33 1544 / 1598, 384 of 64 and 5 368 / 312.  Hence at most so many workgroups of 32 rows: a number and,
// in thousandths, as many as the rows would fill without gaps, fitted to 557 sizes of 16 to 1200000 rows.  Of these 9 are slower here
// than by layer (by 11 % at most, 320 trajectories of 4 tokens) and 7 would be faster (by 6 %).
struct ChainLimit { int wgs, fill; };
constexpr ChainLimit CHAIN_LIMIT[3][2] = {{{950, 1625}, {1025, 2650}}, {{310, 1180}, {525, 1325}}, {{225, 1050}, {350, 1175}}};   // one stream, two
bool row_chain_has(int D, int64_t M) { return (D == 128 || D == 192 || D == 256) && M <= 65535; }       // of trajectories
bool row_chain_takes(int D, int64_t M, int L, int L2) {
  if (!row_chain_has(D, M)) return false;
  auto wgs = [&](int rows) { return M * ((L + rows - 1) / rows + (L2 + rows - 1) / rows); };
  const ChainLimit most = CHAIN_LIMIT[D / 64 - 2][L2 > 0];
  return wgs(16) <= 256 || 32000 * (wgs(32) - most.wgs) <= most.fill * M * (L + L2);      // up to 256, a compute unit each
}

pg_status launch_row_chain(const ChainArgs& a, int D, ChainKind kind, hipStream_t s) {
  const bool dual = a.s[1].L > 0, next = kind == CHAIN_BLOCK || kind == CHAIN_START, mlp = kind == CHAIN_BLOCK || kind == CHAIN_LAST;
  const int L = a.s[0].L + a.s[1].L;
  bool complete = row_chain_has(D, a.M) && a.M >= 1 && a.mod_of && (kind == CHAIN_LAST || a.qk) &&
                  (!next || (a.vt && a.Lpad % 64 == 0 && a.Lpad >= L)) && (dual ? next && (a.norm_hd == 32 || a.norm_hd == 64) : a.norm_hd == 0);
  for (int i = 0; i < (dual ? 2 : 1); ++i) {
    const ChainStream& c = a.s[i];
    complete = complete && c.L >= 1 && c.h && (kind == CHAIN_START || (c.att && c.o_w && c.o_b)) &&
               (kind == CHAIN_LAST || (c.next_w && c.next_b)) && (!mlp || (c.fc1_w && c.fc1_b && c.fc2_w && c.fc2_b && c.gate2)) &&
               (!next || c.norm2) && (!dual || (c.qn_g && c.kn_g));
  }
  if (!complete) return fail(PG_ESHAPE, "row chain: width %d, %d x %d rows", D, a.M, L);
  const double n = kind == CHAIN_QUERIES ? 2 : kind == CHAIN_BLOCK ? 12 : kind == CHAIN_LAST ? 9 : 3;
  const int rec = prof_open(PROF_GEMM, n * 2.0 * a.M * L * D * D, s);
  const pg_status st = D == 128 ? launch_width<128>(a, kind, s) : D == 192 ? launch_width<192>(a, kind, s) : launch_width<256>(a, kind, s);
  prof_close(rec, s);
  return st;
}

}  // namespace pg
