// Softmax attention on bf16 MFMA, the same code for self, joint and cross attention.  Two kernels: attention_kernel, first below, for
// head width 32 and for the public entry point, whose values are in natural key order; attention_fast_kernel for head width 64
// inside the network.  What follows describes the first, and the layout that both share.
//
// One workgroup = 4 wavefronts = 128 queries of one (batch, head); each wavefront owns 32 queries and
// walks the keys in tiles of 64 staged through LDS.  The score tile is computed TRANSPOSED,
// S^T = K Q^T, so that in the 32x32 MFMA accumulator layout every lane holds scores of ONE query
// (column) for 16 keys (rows): the online-softmax row statistics are in-lane reductions plus a single
// exchange with the other half-wave.  The probabilities then feed O^T = V^T P^T directly from the
// accumulator registers; the key order inside each 16-key contraction is permuted the same way in the
// V^T operand read from LDS, which is why V is stored transposed ([head dim][key]) by the QKV GEMM.
// The softmax's VALU work, not the MFMAs, sets the pace here, so it is kept minimal: the queries arrive
// pre-multiplied by log2(e)/sqrt(hd) (by the projection GEMM's epilogue), the score accumulators start
// at minus the running reference exponent, so a probability is a bare exp2 of the accumulator; the
// masking of keys past the end exists only in the code for the last, partial tile; a wavefront whose 32
// queries all lie past the end of the sequence (the ragged last query tile) still stages keys and values
// but skips the arithmetic.  (Feeding the reference exponent to the first score MFMA from a register block
// of its own, which saves the per-tile initialisation, measured 6 % slower: the vector ALU is not what
// the waves wait for.)
#include <cmath>
#include <type_traits>
#include "attention.hpp"
#include "operands.hpp"

namespace pg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int ATT_THREADS = 256;
constexpr int QTILE = 128, KTILE = 64;

// The value rows of the network keep their keys in the order in which the score accumulators hold them (VSWAP; value_slot),
// so that a lane reads its eight keys as one 16-byte chunk without bank conflicts instead of as two 8-byte pieces with two-way
// conflicts.  The public entry point takes them in natural order.  Key at a position of a value row:
template <bool VSWAP>
__device__ __forceinline__ int key_at(int position) { return VSWAP ? value_slot(position) : position; }
// zeroes the values of keys past the end in the chunk at position kc, a multiple of 8 (the padding may hold anything)
template <bool VSWAP>
__device__ __forceinline__ u32x4v zero_past_end(u32x4v v, int kc, int Lk) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t x = v[w];
    if (key_at<VSWAP>(kc + 2 * w) >= Lk) x &= 0xFFFF0000u;
    if (key_at<VSWAP>(kc + 2 * w + 1) >= Lk) x &= 0x0000FFFFu;
    v[w] = x;
  }
  return v;
}

template <int HD>
__device__ __forceinline__ int k_off(int row, int chunk) {       // K tile [64 keys][HD]
  if (HD == 64) return (row * 8 + (chunk ^ ((row ^ (row >> 3)) & 7))) * 16;
  return (row * 4 + (chunk ^ (((row >> 1) ^ (row >> 3)) & 3))) * 16;
}
__device__ __forceinline__ int v_off(int row, int chunk) {       // V^T tile [HD][64 keys]
  return (row * 8 + (chunk ^ ((row ^ (row >> 3)) & 7))) * 16;
}

template <int HD, bool VSWAP>
__global__ __launch_bounds__(ATT_THREADS, 2) void attention_kernel(const AttnArgs a) {
  constexpr int KCH = HD / 8;                  // 16-byte chunks per K row
  constexpr int K_PER_THREAD = KTILE * KCH / ATT_THREADS;        // 2 (HD 64) or 1 (HD 32)
  constexpr int V_PER_THREAD = HD * 8 / ATT_THREADS;             // 2 or 1
  constexpr int SLABS = HD / 16;               // k-slabs of the score MFMA
  constexpr int OT = HD / 32;                  // 32-row tiles of O^T
  __shared__ __align__(16) unsigned char sK[KTILE * HD * 2];
  __shared__ __align__(16) unsigned char sV[HD * KTILE * 2];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  // Workgroups are dealt to the 8 XCDs round-robin by id; the ids are permuted so that each XCD gets a
  // contiguous run of (batch, head, query tile): the query tiles of one head then share its keys and
  // values through one L2 instead of fetching them once per XCD.
  const int nq = (a.Lq + QTILE - 1) / QTILE;
  const int per_xcd = gridDim.x / 8;
  const int wg = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (wg >= nq * a.heads * a.B) return;
  const int b = wg / (nq * a.heads), h = (wg / nq) % a.heads;
  const int q0 = (wg % nq) * QTILE + wave * 32;
  const int kb = a.kv_map ? a.kv_map[b] : b;
  const uint16_t* kbase = a.k + (int64_t)kb * a.k_bstride + h * HD;
  const uint16_t* vbase = a.vt + (int64_t)kb * a.vt_bstride + (int64_t)h * HD * a.Lkpad;

  // Q fragments (B operand: column = query, k = head-dim index), kept in registers
  bf16x8 qf[SLABS];
  {
    const int qr = min(q0 + l32, a.Lq - 1);
    const uint16_t* qp = a.q + ((int64_t)b * a.Lq + qr) * a.ldq + h * HD + 8 * half;
#pragma unroll
    for (int s = 0; s < SLABS; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
    if (!a.q_prescaled) {
#pragma unroll
      for (int s = 0; s < SLABS; ++s)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[s][e] = (__bf16)((float)qf[s][e] * a.scale_log2);
    }
  }

  f32x16 o[OT];
#pragma unroll
  for (int t = 0; t < OT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[t][e] = 0.f;
  // Running softmax statistics in the log2 domain.  m_run is a reference exponent, not necessarily the
  // exact running maximum: after the first tile it is only raised (and the accumulators rescaled) when a
  // new score exceeds it by more than 2^8, so most tiles skip the rescale; probabilities stay below 2^8,
  // well inside bf16 / fp32 range, and the final division by l makes the result independent of the
  // reference.
  float m_run = 0.f, l_run = 0.f;
  const bool wave_has_queries = q0 < a.Lq;       // wave-uniform

  const int n_tiles = (a.Lk + KTILE - 1) / KTILE;
  u32x4v rk[K_PER_THREAD], rv[V_PER_THREAD];
  // per-lane staging positions (fixed), advanced by whole tiles
  int k_row[K_PER_THREAD], k_ch[K_PER_THREAD], v_row[V_PER_THREAD], v_ch[V_PER_THREAD];
#pragma unroll
  for (int i = 0; i < K_PER_THREAD; ++i) { const int cc = tid + i * ATT_THREADS; k_row[i] = cc / KCH; k_ch[i] = cc % KCH; }
#pragma unroll
  for (int i = 0; i < V_PER_THREAD; ++i) { const int cc = tid + i * ATT_THREADS; v_row[i] = cc >> 3; v_ch[i] = cc & 7; }

  // staging sources for tile 0; full tiles advance them by whole tiles with wave-uniform offsets
  const uint16_t* k_src[K_PER_THREAD];
  const uint16_t* v_src[V_PER_THREAD];
#pragma unroll
  for (int i = 0; i < K_PER_THREAD; ++i) k_src[i] = kbase + (int64_t)min(k_row[i], a.Lk - 1) * a.ldk + k_ch[i] * 8;
#pragma unroll
  for (int i = 0; i < V_PER_THREAD; ++i) v_src[i] = vbase + (int64_t)v_row[i] * a.Lkpad + v_ch[i] * 8;
  auto load_tile = [&](int kt) {
    const int k0 = kt * KTILE;
    if (k0 + KTILE <= a.Lk) {                    // full tile: no clamping, no masking
      const int64_t koff = (int64_t)k0 * a.ldk;
#pragma unroll
      for (int i = 0; i < K_PER_THREAD; ++i) rk[i] = *reinterpret_cast<const u32x4v*>(k_src[i] + koff);
#pragma unroll
      for (int i = 0; i < V_PER_THREAD; ++i) rv[i] = *reinterpret_cast<const u32x4v*>(v_src[i] + k0);
      return;
    }
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) {
      const int key = min(k0 + k_row[i], a.Lk - 1);
      rk[i] = *reinterpret_cast<const u32x4v*>(kbase + (int64_t)key * a.ldk + k_ch[i] * 8);
    }
#pragma unroll
    for (int i = 0; i < V_PER_THREAD; ++i) {
      const int kc = k0 + v_ch[i] * 8;
      u32x4v v = *reinterpret_cast<const u32x4v*>(vbase + (int64_t)v_row[i] * a.Lkpad + kc);
      if ((kc & ~15) + 16 > a.Lk) v = zero_past_end<VSWAP>(v, kc, a.Lk);
      rv[i] = v;
    }
  };
  auto store_tile = [&]() {
#pragma unroll
    for (int i = 0; i < K_PER_THREAD; ++i) *reinterpret_cast<u32x4v*>(sK + k_off<HD>(k_row[i], k_ch[i])) = rk[i];
#pragma unroll
    for (int i = 0; i < V_PER_THREAD; ++i) *reinterpret_cast<u32x4v*>(sV + v_off(v_row[i], v_ch[i])) = rv[i];
  };

  // one key tile; MASKED is the variant for a last tile that holds keys past the end
  auto tile = [&](int kt, auto masked_c) {
    constexpr bool MASKED = decltype(masked_c)::value;
    __syncthreads();                             // everyone is done reading the previous tile
    store_tile();
    __syncthreads();
    if (kt + 1 < n_tiles) load_tile(kt + 1);     // overlaps with the math below
    if (!wave_has_queries) return;               // staging and barriers above are the whole workgroup's

    const bool upper = !MASKED || kt * KTILE + 32 < a.Lk;            // wave-uniform: the last tile may end in its first half
    // ---- S^T = K Q^T - m_run : two 32-key tiles ----
    const float neg_m = -m_run;
    f32x16 s[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t == 1 && !upper) break;
#pragma unroll
      for (int e = 0; e < 16; ++e) s[t][e] = neg_m;
#pragma unroll
      for (int ks = 0; ks < SLABS; ++ks) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(sK + k_off<HD>(t * 32 + l32, 2 * ks + half));
        s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[t], 0, 0, 0);
      }
    }
    if (MASKED) {
      const int k0 = kt * KTILE;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (k0 + t * 32 + 8 * (e >> 2) + 4 * half + (e & 3) >= a.Lk) s[t][e] = -__builtin_huge_valf();
    }
    // ---- online softmax for this lane's query; scores are already relative to m_run ----
    float mx = s[0][0];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[t][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
    if (kt == 0 || __builtin_amdgcn_ballot_w64(mx > 8.0f) != 0ull) {   // wave-uniform: rare after the first tile
      const float delta = kt == 0 ? mx : fmaxf(mx, 0.f);               // the first tile sets the reference
      // (which may lie so far below zero that 2^-delta is infinite; there is nothing to rescale yet)
      const float alpha = kt == 0 ? 1.0f : __builtin_amdgcn_exp2f(-delta);
      m_run += delta;
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < OT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[t][e] *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) s[t][e] -= delta;
    }
    float psum = 0.f;
    bf16x8 pf[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(s[t][e]);
        const float p1 = __builtin_amdgcn_exp2f(s[t][e + 1]);
        const f32x2v pp = {p0, p1};
        const bf16x2 pb = __builtin_convertvector(pp, bf16x2);
        // the normaliser sums the probabilities as the value product sees them (rounded to bf16)
        psum = __builtin_amdgcn_fdot2_f32_bf16(pb, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, psum, false);
        pf[t][e >> 3][e & 7] = pb[0];
        pf[t][e >> 3][(e & 7) + 1] = pb[1];
      }
    l_run += psum;
    // ---- O^T += V^T P^T : contraction over 16 keys per MFMA, keys permuted as the accumulator holds them ----
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t == 1 && !upper) break;
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) {
        const int c0 = 4 * t + 2 * jj;
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
          const int row = ot * 32 + l32;
          bf16x8 vf;
          if constexpr (VSWAP) {
            vf = *reinterpret_cast<const bf16x8*>(sV + v_off(row, c0 + half));
          } else {
            const u32x2v lo = *reinterpret_cast<const u32x2v*>(sV + v_off(row, c0) + 8 * half);
            const u32x2v hi = *reinterpret_cast<const u32x2v*>(sV + v_off(row, c0 + 1) + 8 * half);
            vf = __builtin_bit_cast(bf16x8, u32x4v{lo[0], lo[1], hi[0], hi[1]});
          }
          o[ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[t][jj], o[ot], 0, 0, 0);
        }
      }
    }
  };

  load_tile(0);
  const int n_full = a.Lk / KTILE;               // tiles that lie wholly inside the keys
  for (int kt = 0; kt < n_full; ++kt) tile(kt, std::false_type{});
  if (n_full < n_tiles) tile(n_full, std::true_type{});

  // ---- normalise and store: lane holds head-dim rows 8*(e/4) + 4*half + e%4 of its query ----
  const float l_tot = l_run + __shfl_xor(l_run, 32, WAVE);
  const float inv = 1.0f / l_tot;
  const int qr = q0 + l32;
  if (qr < a.Lq) {
    uint16_t* op = (a.split > 0) ? (qr < a.split ? a.out + ((int64_t)b * a.split + qr) * a.ldo + h * HD
                                                 : a.out2 + ((int64_t)b * (a.Lq - a.split) + qr - a.split) * a.ldo + h * HD)
                                 : a.out + ((int64_t)b * a.Lq + qr) * a.ldo + h * HD;
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        bf16x4 w;
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = (__bf16)(o[ot][4 * q + t] * inv);
        *reinterpret_cast<bf16x4*>(op + ot * 32 + 8 * q + 4 * half) = w;
      }
  }
}

// ---- head width 64, values in the accumulators' order: what the network launches ----
// The kernel above waits: a key tile is a chain of LDS reads, scores, exponentials and value products between two barriers.  Here
// the chain is taken apart.  A wave owns QB blocks of 32 queries and walks the keys in steps of 32: the scores of the next step
// run on the matrix pipe beside this step's exponentials, operands are read from LDS a phase before they are used (keys while the
// value products run, values while the scores do), and keys and values come by direct loads a whole tile ahead, with one
// barrier per tile of 64 keys.  Two blocks share the operand reads.
// Ordinary scores need no running maximum: probabilities are 2^score as they are, which bf16 and fp32 hold with the same relative
// precision anywhere between 2^-60 and 2^60, so no reference has to be subtracted, compared or raised.  A block of 32 queries gets a
// reference exponent (raised by the rule of the kernel above) when the largest of a query's first 32 scores lies outside -40 .. 40, or
// after the tile that takes a normaliser past 2^60; a wave that holds such a block does the rest of its tiles one after another
// (`chained`).  Sharp scores (largest of a row 60 and more), us, always with a running maximum / blocks outside 2^-60 .. 2^60 done
// twice / now: 48 x 24 heads x 1178 714 / 1009 / 610, 24 x 12 x 1024 103 / 175 / 104, on 77 keys 28.5 / 35.1 / 28.6; every score
// moved by 70: 510 / 930 / 545.
// Done again from its first tile is only a block that leaves fp32's range all the same: a normaliser past 2^128 inside one tile, values
// whose sum is not finite or, below normalisers of 1, so small that products under 2^-126 could be missing from it.  All of this
// block by block, so that a query's result depends on its own block and not on QB.
// A step and wave costs 1024 cycles of MFMA and 850 of vector ALU (32 exponentials of eight) per 64 queries and 64 keys; taken apart
// like this it runs in about 2400 (2700 with the maximum, and with the keys read one fragment at a time before their MFMAs).  What
// is left is power (zero operands: 1040 TFLOP/s, random ones 870) and the part-filled tiles of queries and keys.  us, before / now:
// 48 x 24 heads x 1178 512 / 466, 24 x 24 x 1178 267 / 238, 24 x 12 x 1024 96 / 85, 24 x 12 x 1024 on 77 keys 28.5 / 24.8,
// 10 x 16 x 340 14.2 / 12.4.
constexpr int FAST_K = 2 * KTILE * 64 * 2, FAST_LDS = FAST_K + 3 * KTILE * 64 * 2;   // two key tiles, three value tiles
constexpr float S_PLAIN = 40.f, L_MIN = 0x1p-60f, L_MAX = 0x1p60f;
constexpr float O_MIN = 0x1p-96f;                // beside it, 2^16 lost products of 2^-126 are 2^-14

__device__ __forceinline__ float largest(const f32x16& s) {
  float mx = s[0];
#pragma unroll
  for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
  return mx;
}

// op over the two lanes of a query
template <class Op>
__device__ __forceinline__ float across_halves(float v, Op op) {
  const uint32_t b = __builtin_bit_cast(uint32_t, v);
  const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return op(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float max_of(float x, float y) { return fmaxf(x, y); }
__device__ __forceinline__ float sum_of(float x, float y) { return x + y; }

// the value exists from here on
__device__ __forceinline__ void pin(bf16x8& v) {
  u32x4v w = __builtin_bit_cast(u32x4v, v);
  asm volatile("" : "+v"(w));
  v = __builtin_bit_cast(bf16x8, w);
}

template <int QB>
__global__ __launch_bounds__(ATT_THREADS, QB == 2 ? 2 : 3) void attention_fast_kernel(const AttnArgs a) {
  constexpr int HD = 64, KS = 4, WQ = 32 * QB, QT = 4 * WQ;
  __shared__ __align__(16) unsigned char smem[FAST_LDS];
  __shared__ int left_over[4];                   // whether a wave has blocks to do again
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int nq = (a.Lq + QT - 1) / QT;
  const int per_xcd = gridDim.x / 8;
  const int wg = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;      // query tiles of one head share an L2, as above
  if (wg >= nq * a.heads * a.B) return;
  const int b = wg / (nq * a.heads), h = (wg / nq) % a.heads;
  const int q0 = (wg % nq) * QT + wave * WQ;
  const int kb = a.kv_map ? a.kv_map[b] : b;
  const uint16_t* kbase = a.k + (int64_t)kb * a.k_bstride + h * HD;
  const uint16_t* vbase = a.vt + (int64_t)kb * a.vt_bstride + (int64_t)h * HD * a.Lkpad;
  const bool wave_has_queries = q0 < a.Lq;       // wave-uniform

  // staging: a wave owns two of the eight 1 KB regions (8 rows) of either tile; lane l fills chunk l % 8 of row l / 8 of a
  // region with the source chunk that the swizzle puts there
  const int n_tiles = (a.Lk + KTILE - 1) / KTILE, n_full = a.Lk / KTILE;
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  int s_row[2], s_ch[2];
  int ka[KS], va[4];                             // operand addresses in a stage: the second 32 rows have the chunks permuted and lie 4 KB further
  auto addresses = [&](int lane) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      s_row[i] = (2 * wave + i) * 8 + (lane >> 3);
      s_ch[i] = (lane & 7) ^ ((s_row[i] ^ (s_row[i] >> 3)) & 7);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      ka[c] = k_off<HD>(lane & 31, 2 * c + (lane >> 5));
      va[c] = v_off(lane & 31, 2 * c + (lane >> 5));
    }
  };
  addresses(lane);
  auto k_stage = [](int kt) { return (kt & 1) * 8192; };
  auto v_stage = [](int kt) { return FAST_K + (kt % 3) * 8192; };
  auto request = [&](int kt) {
    const int k0 = kt * KTILE;
    const uint32_t kd = lds0 + k_stage(kt), vd = lds0 + v_stage(kt);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = min(s_row[i], a.Lk - 1 - k0);
      dma16((uint32_t)(row * (int)a.ldk + s_ch[i] * 8) * 2u, kbase + (int64_t)k0 * a.ldk, kd + (2 * wave + i) * 1024);
      dma16((uint32_t)(s_row[i] * a.Lkpad + s_ch[i] * 8) * 2u, vbase + k0, vd + (2 * wave + i) * 1024);
    }
  };
  // Tile kt, which this wave's loads have brought, is made whole: values of keys past the end (padding may hold anything) are
  // zeroed by the wave that fetched them.  Then everybody's part is there, and everybody is done with what was read before.
  auto publish = [&](int kt) {
    wait_dma();
    if (a.Lk - kt * KTILE < KTILE) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int kc = kt * KTILE + s_ch[i] * 8;
        if ((kc & ~15) + 16 > a.Lk) {
          u32x4v* at = reinterpret_cast<u32x4v*>(smem + v_stage(kt) + (2 * wave + i) * 1024 + lane * 16);
          *at = zero_past_end<true>(*at, kc, a.Lk);
        }
      }
    }
    __syncthreads();
  };
  // in tile kt, when its keys have been read: the next one is published, the one after it asked for
  auto turn = [&](int kt) {
    if (kt + 1 >= n_tiles) return;
    publish(kt + 1);
    if (kt + 2 < n_tiles) request(kt + 2);
  };
  request(0);
  if (n_tiles > 1) request(1);

  bf16x8 qf[QB][KS];
#pragma unroll
  for (int c = 0; c < QB; ++c) {
    const int qr = min(q0 + 32 * c + l32, a.Lq - 1);
    const uint16_t* qp = a.q + ((int64_t)b * a.Lq + qr) * a.ldq + h * HD + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[c][ks] = *reinterpret_cast<const bf16x8*>(qp + 16 * ks);
      if (!a.q_prescaled)
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[c][ks][e] = (__bf16)((float)qf[c][ks][e] * a.scale_log2);
    }
  }
  f32x16 o[QB][2];
  float l_run[QB], m_run[QB];                    // m_run: reference exponent of the lane's query, 0 in a block without
  bool ref[QB];                                  // wave-uniform: whether the block has one
#pragma unroll
  for (int c = 0; c < QB; ++c) {
    o[c][0] = o[c][1] = f32x16{};
    l_run[c] = m_run[c] = 0.f;
    ref[c] = false;
  }
  auto chain = [&] { return ref[0] || ref[QB - 1]; };
  // the first scores of a block
  auto look = [&](int c, const f32x16& s) {
    ref[c] = __builtin_amdgcn_ballot_w64(!(fabsf(across_halves(largest(s), max_of)) <= S_PLAIN)) != 0ull;
  };
  auto passed = [&] {
    bool over = false;
#pragma unroll
    for (int c = 0; c < QB; ++c) over = over || !(l_run[c] <= L_MAX);
    return __builtin_amdgcn_ballot_w64(over) != 0ull;
  };
  // after a tile: a reference that brings normalisers to 1 .. 2 for a block in which one has left the range
  auto settle = [&](int c) {
    if (ref[c] || __builtin_amdgcn_ballot_w64(!(l_run[c] <= L_MAX)) == 0ull) return;
    const int up = __builtin_amdgcn_frexp_expf(across_halves(l_run[c], sum_of)) - 1;
    ref[c] = true;
    m_run[c] = (float)up;
    l_run[c] = __builtin_amdgcn_ldexpf(l_run[c], -up);
#pragma unroll
    for (int ot = 0; ot < 2; ++ot)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[c][ot][e] = __builtin_amdgcn_ldexpf(o[c][ot][e], -up);
  };

  // keys / values of half t of a tile
  auto read_keys = [&](const unsigned char* st, int t, bf16x8 (&kf)[KS]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8*>(st + (t ? ka[ks ^ 2] + 4096 : ka[ks]));
  };
  auto read_values = [&](const unsigned char* st, int t, bf16x8 (&vf)[2][2]) {
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int ot = 0; ot < 2; ++ot) {
        const int g = 2 * t + jj;
        vf[jj][ot] = *reinterpret_cast<const bf16x8*>(st + (ot ? va[g ^ 2] + 4096 : va[g]));
      }
  };
  auto score_mfma = [&](f32x16& s, int c, int ks, const bf16x8 (&kf)[KS]) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[c][ks], ks ? s : f32x16{}, 0, 0, 0);
  };
  // probabilities 2 i and 2 i + 1 of a block
  auto probability_pair = [](const f32x16& s, bf16x8 (&pf)[2], int i) {
    const bf16x2 pb = __builtin_convertvector(f32x2v{__builtin_amdgcn_exp2f(s[2 * i]), __builtin_amdgcn_exp2f(s[2 * i + 1])}, bf16x2);
    pf[i >> 2][2 * (i & 3)] = pb[0];
    pf[i >> 2][2 * (i & 3) + 1] = pb[1];
  };
  // the normaliser sums the probabilities as the value product sees them (rounded to bf16)
  auto add_pair = [](const bf16x8 (&pf)[2], int i, float sum) {
    return __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[i >> 2][2 * (i & 3)], pf[i >> 2][2 * (i & 3) + 1]}, bf16x2{(__bf16)1.0f, (__bf16)1.0f},
                                           sum, false);
  };
  bf16x8 kf[KS];
  // One step of 32 keys: exponentials of `s`, beside them (NEXT) the scores of the following step from `kf`; then the value
  // products, beside them (READ) the reads of the keys after those.  Eight MFMAs of either kind with two blocks; the exponentials
  // of four scores and the packing after each score MFMA, one pair's sum after each value MFMA.
  auto step = [&](const f32x16 (&s)[QB], f32x16 (&next)[QB], const unsigned char* v_st, int t, float (&psum)[QB], auto next_c, auto between,
                  auto read_next) {
    constexpr bool NEXT = decltype(next_c)::value;
    bf16x8 vf[2][2], pf[QB][2];
    read_values(v_st, t, vf);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int c = 0; c < QB; ++c) {
        if (NEXT) score_mfma(next[c], c, ks, kf);
        probability_pair(s[c], pf[c], 2 * ks);
        probability_pair(s[c], pf[c], 2 * ks + 1);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int c = 0; c < QB; ++c)                 // made here, not where they are used: below the barrier nothing would run beside the scores
#pragma unroll
      for (int jj = 0; jj < 2; ++jj) pin(pf[c][jj]);
    between();
    read_next();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int c = 0; c < QB; ++c)
#pragma unroll
        for (int ot = 0; ot < 2; ++ot) {
          o[c][ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[jj][ot], pf[c][jj], o[c][ot], 0, 0, 0);
          psum[c] = add_pair(pf[c], 4 * jj + 2 * ot, psum[c]);
          psum[c] = add_pair(pf[c], 4 * jj + 2 * ot + 1, psum[c]);
          __builtin_amdgcn_sched_barrier(0);
        }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  const auto nothing = [] {};

  // a full tile; at entry s0 holds the scores of its first half and kf the keys of its second.  The barrier in the middle publishes
  // the next tile (LAST: the last full one, after which no scores are prepared)
  f32x16 s0[QB], s1[QB];
  auto full_tile = [&](int kt, auto last_c) {
    constexpr bool LAST = decltype(last_c)::value;
    const unsigned char* v_st = smem + v_stage(kt);
    const unsigned char* k_st = smem + k_stage(kt + 1);
    float psum[QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) psum[c] = 0.f;
    step(s0, s1, v_st, 0, psum, yes, [&] { turn(kt); }, [&] { if (!LAST) read_keys(k_st, 0, kf); });
    if constexpr (LAST) step(s1, s0, v_st, 1, psum, no, nothing, nothing);
    else step(s1, s0, v_st, 1, psum, yes, nothing, [&] { read_keys(k_st, 1, kf); });
#pragma unroll
    for (int c = 0; c < QB; ++c) l_run[c] += psum[c];
  };

  // The queries are here before the loop (a wait inside it would be one for the next tile, too), and with them the first two tiles,
  // which were asked for before them: loads return in order.
#pragma unroll
  for (int c = 0; c < QB; ++c)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) pin(qf[c][ks]);
  publish(0);
  int kt = 0;                                    // the next tile
  if (n_full > 0 && wave_has_queries) {
    read_keys(smem, 0, kf);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int c = 0; c < QB; ++c) score_mfma(s0[c], c, ks, kf);
    read_keys(smem, 1, kf);
#pragma unroll
    for (int c = 0; c < QB; ++c) look(c, s0[c]);
    bool plain = !chain();
    while (plain && kt + 1 < n_full) {
      full_tile(kt++, no);
      plain = !passed();
    }
    if (plain) full_tile(kt++, yes);
#pragma unroll
    for (int c = 0; c < QB; ++c) settle(c);
  }
  const int rest = a.Lk - n_full * KTILE;
  if (rest > 0 && wave_has_queries && !chain()) {    // the last, part-filled tile, published by the tile before it
    const unsigned char* k_st = smem + k_stage(n_full);
    float psum[QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) psum[c] = 0.f;
    for (int t = 0; t < 2 && 32 * t < rest; ++t) {
      if (t) read_keys(k_st, 1, kf);
      else read_keys(k_st, 0, kf);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int c = 0; c < QB; ++c) score_mfma(s0[c], c, ks, kf);
#pragma unroll
      for (int c = 0; c < QB; ++c)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (8 * (e >> 2) + (e & 3) >= rest - 32 * t - 4 * half) s0[c][e] = -__builtin_huge_valf();
      if (t) step(s0, s1, smem + v_stage(n_full), 1, psum, no, nothing, nothing);
      else step(s0, s1, smem + v_stage(n_full), 0, psum, no, nothing, nothing);
    }
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      l_run[c] += psum[c];
      settle(c);
    }
    ++kt;
  }

  // ---- the rest of the tiles where a block has a reference; waves without queries only fetch ----
  bool work[QB];
#pragma unroll
  for (int c = 0; c < QB; ++c) work[c] = wave_has_queries;
  // tile kt for N blocks from C0 on
  auto chained = [&](int kt, auto c0_c, auto n_c) {
    constexpr int C0 = decltype(c0_c)::value, N = decltype(n_c)::value;
    const unsigned char* k_st = smem + k_stage(kt);
    const unsigned char* v_st = smem + v_stage(kt);
    const int left = a.Lk - kt * KTILE;
    f32x16 s[N][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      read_keys(k_st, t, kf);
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const float neg_m = -m_run[C0 + n];
#pragma unroll
        for (int e = 0; e < 16; ++e) s[n][t][e] = neg_m;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) s[n][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[C0 + n][ks], s[n][t], 0, 0, 0);
      }
    }
    if (left < KTILE) {
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (8 * (e >> 2) + (e & 3) >= left - 32 * t - 4 * half) s[n][t][e] = -__builtin_huge_valf();
    }
    float mx[N];
    bool raise = false;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      mx[n] = fmaxf(largest(s[n][0]), largest(s[n][1]));
      raise = raise || (ref[C0 + n] && (kt == 0 || __builtin_amdgcn_ballot_w64(mx[n] > 8.0f) != 0ull));
    }
    if (raise)
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const int c = C0 + n;
        if (!ref[c] || (kt > 0 && __builtin_amdgcn_ballot_w64(mx[n] > 8.0f) == 0ull)) continue;
        const float top = across_halves(mx[n], max_of);
        const float delta = kt == 0 ? top : fmaxf(top, 0.f);             // the first tile sets the reference
        const float alpha = kt == 0 ? 1.0f : __builtin_amdgcn_exp2f(-delta);
        m_run[c] += delta;
        l_run[c] *= alpha;
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
          for (int e = 0; e < 16; ++e) o[c][ot][e] *= alpha;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int e = 0; e < 16; ++e) s[n][t][e] -= delta;
      }
    bf16x8 pf[N][2][2], vf[2][2];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      float psum = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) probability_pair(s[n][t], pf[n][t], i);
#pragma unroll
        for (int i = 0; i < 8; ++i) psum = add_pair(pf[n][t], i, psum);
      }
      l_run[C0 + n] += psum;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      read_values(v_st, t, vf);
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int ot = 0; ot < 2; ++ot)
            o[C0 + n][ot] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[jj][ot], pf[n][t][jj], o[C0 + n][ot], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) settle(C0 + n);
  };
  const bool kept = n_tiles <= 2;                // all tiles stay where they are
  float l_tot[QB];
  for (bool last_round = false;; last_round = true) {
    if (kt < n_tiles) {
      int lane_here = lane;
      asm volatile("" : "+v"(lane_here));        // computed anew: nothing is carried here through the loop above
      addresses(lane_here);
    }
    for (; kt < n_tiles; ++kt) {
      constexpr std::integral_constant<int, 0> c0{};
      constexpr std::integral_constant<int, 1> c1{};
      if (QB == 2 && work[0] && work[QB - 1]) {
        chained(kt, c0, std::integral_constant<int, QB>{});
      } else {
        if (work[0]) chained(kt, c0, c1);
        if constexpr (QB == 2)
          if (work[1]) chained(kt, c1, c1);
      }
      if (!kept || !last_round) turn(kt);
    }
    bool again[QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      l_tot[c] = across_halves(l_run[c], sum_of);
      float most[4] = {0.f, 0.f, 0.f, 0.f}, least = 1.f;     // of the lane's sums; NaN as soon as one of them is
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
          most[ot + (e & 2)] = __builtin_elementwise_maximum(most[ot + (e & 2)], __builtin_fabsf(o[c][ot][e]));
      most[0] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(most[0], most[1]), __builtin_elementwise_maximum(most[2], most[3]));
      if (__builtin_amdgcn_ballot_w64(l_tot[c] < 1.f) != 0ull)
#pragma unroll
        for (int ot = 0; ot < 2; ++ot)
#pragma unroll
          for (int e = 0; e < 16; ++e) least = __builtin_elementwise_minimum(least, __builtin_fabsf(o[c][ot][e]));
      const bool sound = l_tot[c] >= L_MIN && l_tot[c] <= L_MAX && most[0] < __builtin_huge_valf() && (l_tot[c] >= 1.f || least >= O_MIN);
      again[c] = wave_has_queries && __builtin_amdgcn_ballot_w64(!sound) != 0ull;
    }
    bool more = !last_round && (again[0] || again[QB - 1]);
    if (!kept && !last_round) {                  // all waves fetch
      if (lane == 0) left_over[wave] = more ? 1 : 0;
      __syncthreads();
      more = (left_over[0] | left_over[1] | left_over[2] | left_over[3]) != 0;
    }
    if (!more) break;
    kt = 0;
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      work[c] = again[c];
      if (!again[c]) continue;
      o[c][0] = o[c][1] = f32x16{};
      l_run[c] = m_run[c] = 0.f;
      ref[c] = true;
    }
    if (!kept) {
      request(0);
      request(1);
      publish(0);
    }
  }
  if (!wave_has_queries) return;

  // ---- normalise and store: lane holds head-dim rows 8*(e/4) + 4*half + e%4 of its queries ----
  int lane_out = lane;
  asm volatile("" : "+v"(lane_out));
#pragma unroll
  for (int c = 0; c < QB; ++c) {
    const float inv = 1.0f / l_tot[c];
    const int qr = q0 + 32 * c + (lane_out & 31);
    if (qr < a.Lq) {
      uint16_t* op = (a.split > 0) ? (qr < a.split ? a.out + ((int64_t)b * a.split + qr) * a.ldo + h * HD
                                                   : a.out2 + ((int64_t)b * (a.Lq - a.split) + qr - a.split) * a.ldo + h * HD)
                                   : a.out + ((int64_t)b * a.Lq + qr) * a.ldo + h * HD;
#pragma unroll
      for (int ot = 0; ot < 2; ++ot)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x4 w;
#pragma unroll
          for (int t = 0; t < 4; ++t) w[t] = (__bf16)(o[c][ot][4 * q + t] * inv);
          *reinterpret_cast<bf16x4*>(op + ot * 32 + 8 * q + 4 * (lane_out >> 5)) = w;
        }
    }
  }
}
constexpr int WIDE_QTILE = 256;

// Rounds of workgroups through the chip (two with 64 queries per wave or three with 32 per compute unit; a part-empty last round
// counts half as empty as it is) take about the same time per key tile with either, so the wide one wins where it needs clearly
// fewer and there are enough key tiles to share the reads of: from 0.8 of the narrow one's rounds down.  Narrow / wide, us:
// 48 x 24 heads x 1178 tokens 488 / 466 and 12 x 24 x 1178 122 / 115 at a ratio of 0.78, 30 x 4 x 2048 143 / 133 at 0.70, 64 x 4 x 512
// 27.8 / 27.3 at 0.6; but 24 x 12 x 1024 85 / 90 at 0.88, 96 x 10 x 410 70 / 72 at 0.78.
static bool use_wide(int64_t wgs, int64_t wide_wgs, int Lk) {
  auto rounds = [](double load) { return load <= 1.0 ? 1.0 : 0.5 * (load + ceil(load)); };
  return Lk >= 480 && rounds(wide_wgs / 512.0) <= 0.8 * rounds(wgs / 768.0);
}

int pick_attention(int B, int Lq, int Lk, int heads, int hd, int v_swapped) {
  const int64_t wgs = (int64_t)((Lq + QTILE - 1) / QTILE) * heads * B, wide_wgs = (int64_t)((Lq + WIDE_QTILE - 1) / WIDE_QTILE) * heads * B;
  return hd == 64 && v_swapped && use_wide(wgs, wide_wgs, Lk) ? 2 : 1;
}

pg_status launch_attention(const AttnArgs& a, int hd, hipStream_t s) {
  if (a.B <= 0 || a.Lq <= 0 || a.heads <= 0) return PG_OK;
  if (a.Lk <= 0) return fail(PG_EINVAL, "attention: no keys");
  if (hd != 32 && hd != 64) return fail(PG_ESHAPE, "attention: head width %d not supported (32 or 64)", hd);
  // the kernels read value rows in whole tiles of KTILE keys
  if (a.Lkpad % KTILE || a.Lkpad < a.Lk || a.ldq % 8 || a.ldk % 8 || a.ldo % 4 ||
      ((uintptr_t)a.q & 15) || ((uintptr_t)a.k & 15) || ((uintptr_t)a.vt & 15) || ((uintptr_t)a.out & 7))
    return fail(PG_ESHAPE, "attention: operands need 16-byte aligned rows, value rows a multiple of %d keys (%d)", KTILE, a.Lkpad);
  const int kernel = a.kernel ? a.kernel : pick_attention(a.B, a.Lq, a.Lk, a.heads, hd, a.v_swapped);
  const bool wide = kernel == 2;
  if (kernel < 1 || kernel > 2 || (wide && (hd != 64 || !a.v_swapped)))
    return fail(PG_EINVAL, "attention: kernel %d does not take head width %d", kernel, hd);
  const int q_tile = wide ? WIDE_QTILE : QTILE;
  const int64_t wgs = (int64_t)((a.Lq + q_tile - 1) / q_tile) * a.heads * a.B;
  if (wgs > (wide ? 1ll << 29 : 1ll << 30)) return fail(PG_ESHAPE, "attention: grid limit");
  const dim3 grid((unsigned)((wgs + 7) / 8 * 8)), block(ATT_THREADS);
  const int rec = prof_open(PROF_ATTENTION, 4.0 * a.B * (double)a.heads * a.Lq * (double)a.Lk * hd, s);
  if (wide) attention_fast_kernel<2><<<grid, block, 0, s>>>(a);
  else if (hd == 64 && a.v_swapped) attention_fast_kernel<1><<<grid, block, 0, s>>>(a);
  else if (hd == 64) attention_kernel<64, false><<<grid, block, 0, s>>>(a);
  else if (a.v_swapped) attention_kernel<32, true><<<grid, block, 0, s>>>(a);
  else attention_kernel<32, false><<<grid, block, 0, s>>>(a);
  prof_close(rec, s);
  PG_LAUNCH_CHECK("attention_kernel");
  return PG_OK;
}

}  // namespace pg

using namespace pg;

extern "C" pg_status pg_attention_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* vt, uint16_t* out,
                                       int32_t B, int32_t Lq, int32_t Lk, int32_t heads, int32_t hd,
                                       void* stream) {
  if (B < 0 || Lq < 0 || Lk < 0 || heads < 1) return fail(PG_EINVAL, "pg_attention_bf16: bad sizes");
  if (B == 0 || Lq == 0) return PG_OK;
  if (!q || !k || !vt || !out) return fail(PG_EINVAL, "pg_attention_bf16: null pointer");
  const int D = heads * hd;
  AttnArgs a{};
  a.q = q; a.ldq = D; a.k = k; a.ldk = D; a.k_bstride = (int64_t)Lk * D;
  a.vt = vt; a.Lkpad = (Lk + 63) / 64 * 64; a.vt_bstride = (int64_t)D * a.Lkpad;
  a.out = out; a.ldo = D; a.kv_map = nullptr;
  a.B = B; a.Lq = Lq; a.Lk = Lk; a.heads = heads;
  a.scale_log2 = (float)(1.4426950408889634 / sqrt((double)hd));
  return launch_attention(a, hd, (hipStream_t)stream);
}

extern "C" int32_t pg_attention_kernel(int32_t B, int32_t Lq, int32_t Lk, int32_t heads, int32_t hd) {
  return B < 1 || Lq < 1 || Lk < 1 || heads < 1 ? 0 : pick_attention(B, Lq, Lk, heads, hd, 1);
}

extern "C" pg_status pg_attention_network(const uint16_t* q, const uint16_t* k, const uint16_t* vt, uint16_t* out,
                                          int32_t B, int32_t Lq, int32_t Lk, int32_t Lk_pad, int32_t heads, int32_t hd,
                                          int32_t kernel, void* stream) {
  if (B < 0 || Lq < 0 || Lk < 0 || heads < 1) return fail(PG_EINVAL, "pg_attention_network: bad sizes");
  if (B == 0 || Lq == 0) return PG_OK;
  if (!q || !k || !vt || !out) return fail(PG_EINVAL, "pg_attention_network: null pointer");
  if (kernel < 0 || kernel > 2) return fail(PG_EINVAL, "pg_attention_network: kernel %d", kernel);
  const int D = heads * hd;
  AttnArgs a{};
  a.q = q; a.ldq = D; a.k = k; a.ldk = D; a.k_bstride = (int64_t)Lk * D;
  a.vt = vt; a.Lkpad = Lk_pad; a.vt_bstride = (int64_t)D * Lk_pad;
  a.out = out; a.ldo = D; a.kernel = kernel; a.q_prescaled = 1; a.v_swapped = 1;
  a.B = B; a.Lq = Lq; a.Lk = Lk; a.heads = heads;
  return launch_attention(a, hd, (hipStream_t)stream);
}
