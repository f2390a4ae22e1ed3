// bf16 MFMA GEMM for gfx950: C[M, N] = A[M, K] W[N, K]^T with a fused epilogue.  This is where the
// network evaluation of every denoising step spends its time (the noise-prediction row of the paper's
// cost table, Sec. 6.2).  Built around the 16x16x32 bf16 MFMA:
//   both operands are K-contiguous; 16-byte chunks go from global memory straight into LDS (no register
//   staging), a ring of two or three LDS stages of 64 columns per operand, one barrier per K step; the requests for
//   the tiles that take a freed stage are interleaved with the MFMAs that follow the barrier, and so are the reads of
//   the operand fragments, which are double buffered in registers and read one MFMA slab ahead, also across the
//   barrier; the K loop itself holds no branch (the last steps are peeled);
//   chunk positions are XOR-swizzled so that the 16-byte operand reads are bank-conflict free while the
//   direct loads still write 1 KB contiguous per instruction;
//   the epilogue goes through an LDS transpose so that every lane stores 16 contiguous bytes, with the
//   non-temporal hint; workgroup ids are spread so that the tiles resident on one XCD (one L2) form a
//   compact block of the output and share operand panels.
// The chip draws its power limit here, so energy per flop and not issue slots decides: with the branch-free loop and raised
// wave priority around the MFMAs the 16x16x32 instruction runs 56544 x 6144 x 1536 in 0.87 ms where 32x32x16 takes 0.93 ms
// (0.99 ms with the fragment reads in a burst before the MFMAs and a test around every request, as it was before); the
// smaller instruction also allows 16-row steps, so that every tile height keeps a 2 x 4 arrangement of waves.  Four waves with
// 128 x 128 wave tiles and accumulators in AGPRs read a third less from LDS, but one wave per SIMD exposes the epilogue:
// 0.92 ms (0.855 against 0.872 ms at K = 6144, N = 1536).  Storing the accumulators without the pass through LDS: 1.03 ms.
// A K step of a small tile, and of a large one whose rows come from beyond the L2, is shorter than a load takes (about 1 us under
// load), so two stages leave every step waiting: with a third one of both operands, or of A alone where LDS holds no more (192
// and 224 rows; 256 rows have no room), us before / now: 1296 x 1344 x 5376 + residual 48.4 / 29.9 (128 x 64), 648 x 384 x 1536
// 13.8 / 8.8 (64 x 64), 24576 x 768 x 3072 140.4 / 121.0 (160 rows), 18848 x 1536 x 6144 318 / 297 and 56544 rows 916 / 865
// (224 rows).  Six or eight stages of the small tiles are slower than three (35 and 48 us at the first shape): one workgroup
// per compute unit.
// Several tile shapes are instantiated (workgroup tile BM x BN x 64, WM x WN wavefronts, SA and SW stages); the launcher
// picks one (pick_tile).
#include <cmath>
#include <cstdlib>
#include <type_traits>
#include "gemm.hpp"
#include "operands.hpp"

namespace pg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

constexpr int GROUP_M = 8;                         // tile rows per raster band
constexpr int XCDS = 8;

constexpr int BK = 64, CH = BK / 8;                // columns per K step, 16-byte chunks per tile row
constexpr int MI = 16, KS = 32;                    // 16x16x32 MFMA: lane l holds row l % 16, 8 columns at 8 (l / 16)

// byte offset of 16-byte chunk `chunk` of tile row `row` inside an operand tile: the 16 rows of a fragment put one chunk
// of theirs into 16 different bank groups, and rows 16 apart share their swizzle
__device__ __forceinline__ int swz(int row) { return (row ^ ((row >> 3) & 1)) & 7; }
__device__ __forceinline__ int lds_off(int row, int chunk) { return (row * CH + (chunk ^ swz(row))) * 16; }

// dma16 (operands.hpp) with a 64-bit address per lane, for rows too far apart for a 32-bit offset
__device__ __forceinline__ void dma16_wide(const uint16_t* g, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_addr) : "memory");
}
constexpr int64_t NARROW_LD = 1 << 23;             // 255 rows of so many bf16, in bytes, fit 32 bits

// Outputs are written, and the residual stream is read, once per launch: they go through the caches
// with the non-temporal hint so that the operand panels shared by the tiles of an XCD stay resident.
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_stream(float* p, const float4 v) {
  __builtin_nontemporal_store(f32x4v{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4v*>(p));
}
__device__ __forceinline__ void store_stream(uint16_t* p, const uint2 v) {
  __builtin_nontemporal_store(u32x2v{v.x, v.y}, reinterpret_cast<u32x2v*>(p));
}
__device__ __forceinline__ float4 load_stream(const float* p) {
  const f32x4v v = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(p));
  return float4{v[0], v[1], v[2], v[3]};
}


// f(tag<I>, tag<n>) for consecutive groups of n = 4, 2 or 1 of the N row tiles while f returns true
template <int I> struct int_tag { static constexpr int value = I; };
template <int I, int N, class F>
__device__ __forceinline__ void for_row_groups(F&& f) {
  if constexpr (I < N) {
    constexpr int n = N - I >= 4 ? 4 : N - I >= 2 ? 2 : 1;
    if (f(int_tag<I>{}, int_tag<n>{})) for_row_groups<I + n, N>(f);
  }
}

// NP = 2: two problems of equal N and K in one launch, the tile rows of the second behind those of the first
template <int NP> struct GemmBatch { GemmArgs g[NP]; };
// The problem that a workgroup works on, chosen field by field: an array element picked at run time is read again from the
// kernel arguments at every use (32 scalar loads in the epilogue; QKV of 24576 + 3696 rows with the head norm 402 -> 398 us).
__device__ __forceinline__ GemmArgs chosen(const GemmBatch<1>& b, bool) { return b.g[0]; }
__device__ __forceinline__ GemmArgs chosen(const GemmBatch<2>& b, bool second) {
  const GemmArgs &x = b.g[0], &y = b.g[1];
  GemmArgs a = x;                                    // N, K, the head norm's width, the scaled columns and Lout are equal
#define PG_CHOOSE(field) a.field = second ? y.field : x.field
  PG_CHOOSE(A); PG_CHOOSE(lda); PG_CHOOSE(W); PG_CHOOSE(ldw); PG_CHOOSE(bias); PG_CHOOSE(M);
  PG_CHOOSE(outf); PG_CHOOSE(ldo); PG_CHOOSE(outb); PG_CHOOSE(ldob); PG_CHOOSE(L);
  PG_CHOOSE(vt); PG_CHOOSE(Lpad); PG_CHOOSE(gate); PG_CHOOSE(gate_ld); PG_CHOOSE(group_of);
  PG_CHOOSE(tok_off); PG_CHOOSE(qn_g); PG_CHOOSE(kn_g);
#undef PG_CHOOSE
  return a;
}

// Slabs of the residual stream that a wave loads ahead of the epilogue (EPI_RESID): the read half of its read-modify-write then
// runs beside the last MFMAs instead of after them, when every compute unit wants the memory at once.  The whole tile where
// registers allow it (24576 x 768 x 768 with 160-row tiles: 57.3 -> 50.0 us, 12288 rows 28.3 -> 24.1), a third of a 192-row
// tile (14136 x 1536 x 1536: 85.9 -> 82.3), nothing of taller ones (one slab of a 224-row tile spills: 437 -> 446 us).
constexpr int prefetched_slabs(int bm, int slabs) { return bm >= 224 ? 0 : bm == 192 ? 1 : slabs; }

template <int EPI, int BM, int BN, int WM, int WN, int MINW, int SA, int SW, bool WIDE, int NPROB>
__global__ __launch_bounds__(64 * WM * WN, MINW) void gemm_kernel(const GemmBatch<NPROB> batch) {
  constexpr int WAVES = WM * WN;
  constexpr int CW = BN / WN, FM = BM / WM / MI, FN = CW / MI, FR = FM + FN, MF = FM * FN;   // columns, fragments, MFMAs of a wave
  static_assert(CW == 32 || CW == 64, "the epilogue handles 32 or 64 columns per wave");
  static_assert((BM / WM) % MI == 0 && (BM / WM) % 8 == 0, "wave rows");
  // SA tiles of A and SW of W in LDS
  static_assert(SA == SW || (SA == 3 && SW == 2), "the counts of requests under way are worked out for these");
  constexpr int A_BYTES = BM * BK * 2, W_BYTES = BN * BK * 2, W_AT = SA * A_BYTES;
  constexpr int BIAS_AT = W_AT + SW * W_BYTES, BIAS_BYTES = BN < 128 ? 256 : 2 * BN;    // whole requests of 128 columns
  // of a fixed size, so that no launch depends on an attribute that a process would have to set once per device
  __shared__ __align__(16) unsigned char smem[BIAS_AT + BIAS_BYTES];
  const int per_xcd = gridDim.x / XCDS;
  const int b = (blockIdx.x % XCDS) * per_xcd + blockIdx.x / XCDS;
  // ---- which output tile: XCD-aware, banded raster ----
  const int rows0 = (batch.g[0].M + BM - 1) / BM;
  const int tiles_m = rows0 + (NPROB > 1 ? (batch.g[NPROB - 1].M + BM - 1) / BM : 0), tiles_n = (batch.g[0].N + BN - 1) / BN;
  const int total = tiles_m * tiles_n;
  if (b >= total) return;
  const int group_m = batch.g[0].group_m;
  const int band = group_m * tiles_n;
  const int first_m = (b / band) * group_m;
  const int gsz = min(tiles_m - first_m, group_m);
  const int tm = __builtin_amdgcn_readfirstlane(first_m + (b % band) % gsz);
  const int tn = __builtin_amdgcn_readfirstlane((b % band) / gsz);
  const bool second = NPROB > 1 && tm >= rows0;
  const GemmArgs a = chosen(batch, second);
  const int m0 = (second ? tm - rows0 : tm) * BM, n0 = tn * BN;
  const uint16_t* PA = a.A; const int64_t LDA = a.lda;
  const uint16_t* PW = a.W; const int64_t LDW = a.ldw;
  const uint16_t* PB = a.bias;
  const int MM = a.M, NN = a.N;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lr = lane % MI, lk = lane / MI;

  const int row_w = m0 + wm * (BM / WM), col_w = n0 + wn * CW;       // first row and column of this wave
  f32x4v acc[FM][FN];
  // EPI_RESID: PF slabs of 32 rows of the residual stream are loaded while the last one and a half K steps run (rows and columns
  // past the end repeat existing ones)
  constexpr int LPR = CW / 4, RPI = 64 / LPR, NP = 32 / RPI;     // epilogue: lanes per row, rows per access, accesses per slab
  constexpr int SLABS_M = (FM + 1) / 2;
  constexpr int PF = EPI != EPI_RESID ? 0 : prefetched_slabs(BM, SLABS_M);
  f32x4v hpre[PF > 0 ? PF : 1][NP];
  auto prefetch = [&] {
    const int n = col_w + (lane % LPR) * 4, rsub = lane / LPR;
    const float* base = a.outf + (n < NN ? n : 0);
#pragma unroll
    for (int i = 0; i < PF; ++i)
#pragma unroll
      for (int p = 0; p < (2 * i + 1 < FM ? NP : NP / 2); ++p)
        hpre[i][p] = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(
            base + (int64_t)min(row_w + 32 * i + RPI * p + rsub, MM - 1) * a.ldo));
  };

  {
    // ---- global -> LDS directly: a tile is regions of 1 KB (8 rows of it), dealt to the waves in turn, W's before A's ----
    constexpr int RPR = 64 / CH, A_REG = BM / RPR, W_REG = BN / RPR;
    constexpr int A_PER = (A_REG + WAVES - 1) / WAVES, W_PER = (W_REG + WAVES - 1) / WAVES, PER_WAVE = A_PER + W_PER;
    constexpr int A_LOW = A_REG / WAVES, W_LOW = W_REG / WAVES;    // what every wave has at least
    const int nk = a.K / BK;
    uint32_t g_off[WIDE ? 1 : PER_WAVE];
    const uint16_t* g_base[PER_WAVE];                // WIDE: per lane; else wave-uniform
    uint32_t g_lds[PER_WAVE];
    const uint32_t lds_base = (uint32_t)(uintptr_t)smem;
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
      const bool is_w = i < W_PER;
      const int rg = is_w ? min(wave + i * WAVES, W_REG - 1) : min(wave + (i - W_PER) * WAVES, A_REG - 1);  // wave-uniform
      const int row = rg * RPR + lane / CH;
      const int ch = (lane % CH) ^ swz(row);
      const int r = is_w ? min(row, NN - 1 - n0) : min(row, MM - 1 - m0);
      if (WIDE) {
        g_base[i] = (is_w ? PW + (int64_t)(n0 + r) * LDW : PA + (int64_t)(m0 + r) * LDA) + ch * 8;
      } else {
        g_base[i] = is_w ? PW + (int64_t)n0 * LDW : PA + (int64_t)m0 * LDA;
        g_off[WIDE ? 0 : i] = ((uint32_t)r * (uint32_t)(is_w ? LDW : LDA) + (uint32_t)(ch * 8)) * 2u;
      }
      g_lds[i] = __builtin_amdgcn_readfirstlane(lds_base + (is_w ? W_AT : 0) + rg * 1024);
    }
    // request region i of K tile `kt` into the stage of its ring that starts `at` bytes in
    auto request = [&](int i, int kt, int at) {
      if (i < W_PER ? (i + 1) * WAVES > W_REG && wave + i * WAVES >= W_REG
                    : (i - W_PER + 1) * WAVES > A_REG && wave + (i - W_PER) * WAVES >= A_REG) return;      // the last one of an uneven deal
      const uint32_t dst = g_lds[i] + at;
      if (WIDE) dma16_wide(g_base[i] + kt * BK, dst);
      else dma16(g_off[WIDE ? 0 : i], g_base[i] + kt * BK, dst);
    };
    // fragment addresses: 16 rows further down only add a constant, so one base per operand and slab serves all of them
    constexpr int SLABS = BK / KS;
    static_assert(SLABS == 2, "fragment buffers alternate per slab");
    const int pa0 = lds_off(wm * (BM / WM) + lr, lk), pa1 = lds_off(wm * (BM / WM) + lr, KS / 8 + lk);
    const int pw0 = W_AT + lds_off(wn * CW + lr, lk), pw1 = W_AT + lds_off(wn * CW + lr, KS / 8 + lk);
    struct Stage { int a, w; };                      // bytes into the two rings
    auto after = [&](Stage t) {
      return Stage{t.a + A_BYTES == SA * A_BYTES ? 0 : t.a + A_BYTES, t.w + W_BYTES == SW * W_BYTES ? 0 : t.w + W_BYTES};
    };
    bf16x8 fr[2][FR];
    auto fetch = [&](Stage t, int ks, int buf, int f) {
      const int at = f < FN ? (ks ? pw1 : pw0) + f * MI * CH * 16 + t.w : (ks ? pa1 : pa0) + (f - FN) * MI * CH * 16 + t.a;
      fr[buf][f] = *reinterpret_cast<const bf16x8*>(smem + at);
    };
    // One request after every EVERY-th MFMA and one fragment read after every FEV-th: a wave's request waits for the
    // texture path, which takes 1 KB every ~20 cycles, and in a burst the MFMAs queued behind it would wait too.
    static_assert(MF >= FR && MF >= PER_WAVE, "every fragment and every request has an MFMA to follow");
    constexpr int FEV = MF / FR, EVERY = MF / PER_WAVE;
    // K step kt, whose tiles lie at `cur`, the next one's at `next`.  At its last slab every read of its stage has been issued and
    // awaited, so the barrier that publishes tile kt+1 and frees the stage is passed before that slab's MFMAs; the first slab
    // of tile kt+1 is read, and the tiles that take the place of this one's are requested (REQ_W, REQ_A), while they run.
    // LEFT: requests of a wave that may still be under way when the ones of tile kt+1 have to have ended (-1: there is none).
    auto step = [&](int kt, Stage cur, Stage next, auto req_w, auto req_a, auto left_c) {
      constexpr bool REQ_W = decltype(req_w)::value, REQ_A = decltype(req_a)::value;
      constexpr int LEFT = decltype(left_c)::value;
      constexpr bool NEXT = LEFT >= 0;
#pragma unroll
      for (int ks = 0; ks < SLABS; ++ks) {
        const bool last = ks + 1 == SLABS;
        if (last && NEXT) {
          wait_dma<NEXT ? LEFT : 0>();
          __syncthreads();
          if (!REQ_W && LEFT == 0) prefetch();
        }
        const Stage from = last ? next : cur;
        const int to = (ks + 1) & 1;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
        int q = 0;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks & 1][FN + i], fr[ks & 1][j], acc[i][j], 0, 0, 0);
            if ((!last || NEXT) && q % FEV == 0 && q / FEV < FR) {
              __builtin_amdgcn_sched_barrier(0);
              fetch(from, last ? 0 : ks + 1, to, q / FEV);
              __builtin_amdgcn_sched_barrier(0);
            }
            if (last && q % EVERY == EVERY - 1 && q / EVERY < PER_WAVE && (q / EVERY < W_PER ? REQ_W : REQ_A)) {
              __builtin_amdgcn_sched_barrier(0);
              request(q / EVERY, kt + (q / EVERY < W_PER ? SW : SA), q / EVERY < W_PER ? cur.w : cur.a);
              __builtin_amdgcn_sched_barrier(0);
            }
            ++q;
          }
        __builtin_amdgcn_s_setprio(0);
      }
    };
    // The bias goes the same way as the operands, in front of them: a load into registers would be awaited with everything
    // that was requested after it.
    if (PB && wave * 128 < BN) {
      const int c = n0 + wave * 128 + 2 * lane;      // N is even
      dma4((uint32_t)min(c, NN - 2) * 2u, PB, lds_base + BIAS_AT + wave * 256);
    }
    static_assert(WAVES * 128 >= BN, "a wave asks for 128 columns of the bias");
#pragma unroll
    for (int t = 0; t < SA; ++t)
      if (t < nk)
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) {
          if (i < W_PER && t < SW) request(i, t, t * W_BYTES);
          if (i >= W_PER) request(i, t, t * A_BYTES);
        }
    if (nk >= SA) wait_dma<(SA - 1) * A_LOW + (SW - 1) * W_LOW>();
    else wait_dma();
    __syncthreads();
#pragma unroll
    for (int f = 0; f < FR; ++f) fetch(Stage{0, 0}, 0, 0, f);
    // The accumulators start at the bias: in each 16x16 tile a lane holds one column, so it is one value per tile instead of an
    // add per result in the epilogue.
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int cl = wn * CW + j * MI + lr;
      const float v = PB && n0 + cl < NN ? bf16_to_f32(*reinterpret_cast<const uint16_t*>(smem + BIAS_AT + 2 * cl)) : 0.f;
#pragma unroll
      for (int i = 0; i < FM; ++i) acc[i][j] = f32x4v{v, v, v, v};
    }
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    constexpr int LEFT = (SW - 2) * W_LOW + (SA == SW ? SW - 2 : SW - 1) * A_LOW;   // of a wave, behind those of tile kt+1
    Stage cur{0, 0};
    int kt = 0;
    auto run = [&](auto req_w, auto req_a, auto left_c) {
      const Stage next = after(cur);
      step(kt, cur, next, req_w, req_a, left_c);
      cur = next;
      ++kt;
    };
    while (kt + SA < nk) run(yes, yes, int_tag<LEFT>{});
    if (SA > SW && kt + SA == nk) run(yes, no, int_tag<LEFT>{});
    // the last SW steps, or all of them where there are fewer: T tiles behind kt+1
    auto drain = [&](auto&& self, auto t_c) -> void {
      constexpr int T = decltype(t_c)::value;
      if constexpr (T >= -1) {
        if (T == -1 && nk == 1) prefetch();
        if (kt + 2 + T == nk) run(no, no, int_tag<(T > 0 ? T * (A_LOW + W_LOW) : T)>{});
        self(self, int_tag<T - 1>{});
      }
    };
    drain(drain, int_tag<SW - 2>{});
  }

  // ---- epilogue: in each 16x16 accumulator tile a lane holds ONE column (lr) and rows 4 lk + t ----
  if constexpr (EPI != EPI_UNPATCH) {
    // ---- row-major epilogues: transpose each 32-row slab of the wave tile through LDS so that a lane
    // owns 4 consecutive columns of a row and every global access is 16 bytes wide (8 for bf16) ----
    constexpr int EST = CW + 4;                      // staging row stride in floats: 4 rows down are 16 banks on
    constexpr int VP = 72;                           // pitch of the transposed staging in bf16: 64 tokens + 8 (16-byte aligned rows)
    constexpr int STG = CW * VP * 2;                 // staging bytes per wave
    static_assert(32 * EST * 4 <= STG && WAVES * STG <= BIAS_AT, "the staging areas fit");
    __syncthreads();                                 // every wave has finished reading the last stage
    float* stg = reinterpret_cast<float*>(smem + wave * STG);
    int lane_e = lane;
    if (PF > 0) asm volatile("" : "+v"(lane_e));     // what follows from it is not carried through the K loop
    const int c4 = (lane_e % LPR) * 4, rsub = lane_e / LPR, n = col_w + c4;
    // columns written row-major: all of them, except the value channels of EPI_QKV
    const int n_rm = EPI == EPI_QKV ? a.v_start : NN;
    if (EPI == EPI_QKV) {
      // ---- value channels, stored TRANSPOSED: V^T[traj][channel][token].  In an accumulator tile a lane already
      // holds 4 consecutive tokens of ONE channel, so they are packed to bf16 and staged channel-major (8 bytes per
      // LDS write), up to 64 tokens at a time; then a lane owns 4 consecutive tokens of a channel row and 16
      // lanes write 64 consecutive tokens (128 bytes) of it.  A 32-column group is either all value
      // channels or none (v_start is a multiple of 32). ----
      uint16_t* stg16 = reinterpret_cast<uint16_t*>(stg);
      const int Dv = NN - n_rm;
      bool any_v = false;
#pragma unroll
      for (int j = 0; j < FN; ++j) any_v = any_v || (col_w + j * MI >= n_rm && col_w + j * MI < NN);   // wave-uniform
      if (any_v) {
        const bool all_v = col_w >= n_rm && col_w + CW <= NN;
        // Trajectories of whole units of four tokens: a lane's four belong to one, also where a group of rows spans several
        // (256 trajectories of 16 tokens, width 512: 19.4 -> 11.8 us; other lengths are stored token by token there, since lanes of
        // both kinds in one wave take longer than that: loops of 50 tokens 825 us against 841).
        const bool units = ((a.L | a.tok_off | MM) & 3) == 0;
        for_row_groups<0, FM>([&](auto first, auto count) {
          constexpr int i0 = decltype(first)::value, nt = decltype(count)::value;    // row tiles staged together
          const int row0 = row_w + i0 * MI;          // first token row of the group, wave-uniform
          if (row0 >= MM) return false;
#pragma unroll
          for (int ii = 0; ii < nt; ++ii)
#pragma unroll
            for (int j = 0; j < FN; ++j) {
              const f32x4v t = acc[i0 + ii][j];
              *reinterpret_cast<uint2*>(stg16 + (j * MI + lr) * VP + ii * MI + 4 * lk) = pack_bf16x4({t[0], t[1], t[2], t[3]});
            }
          wave_lds_sync();
          constexpr int lpr = 4 * nt, rpa = 64 / lpr;    // lanes per channel row, channel rows per access
          const int t4 = (lane % lpr) * 4, csub = lane / lpr;
          const int traj_w = row0 / a.L, tok_w = row0 - traj_w * a.L, at_w = a.tok_off + tok_w;     // wave-uniform
          if (all_v && row0 + nt * MI <= MM && tok_w + nt * MI <= a.L && (at_w & 1) == 0) {
            // the whole group is one trajectory's: 8 bytes per lane, or two pairs where its tokens start in the middle of four.
            // No streaming hint: a wave's rows end inside a 128-byte line unless the tile has 256 or 128 of them, and the L2 puts
            // the parts together (12288 x 2304 x 768 with 224-row tiles 50.2 us with the hint, 44.0 without).
            const int at = at_w + t4;
            uint16_t* dst = a.vt + ((int64_t)traj_w * Dv + (col_w - n_rm) + csub) * a.Lpad;
            const uint16_t* src = stg16 + csub * VP + t4;
            const int64_t step_v = (int64_t)rpa * a.Lpad;
            if ((at_w & 3) == 0) {
              dst += value_slot(at);
#pragma unroll
              for (int p = 0; p < CW / rpa; ++p, dst += step_v)
                *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(src + p * rpa * VP);
            } else {
              uint16_t* dst2 = dst + value_slot(at + 2);
              dst += value_slot(at);
#pragma unroll
              for (int p = 0; p < CW / rpa; ++p, dst += step_v, dst2 += step_v) {
                const uint2 pk = *reinterpret_cast<const uint2*>(src + p * rpa * VP);
                *reinterpret_cast<uint32_t*>(dst) = pk.x;
                *reinterpret_cast<uint32_t*>(dst2) = pk.y;
              }
            }
          } else {
            const int r = row0 + t4;                 // the lane's first token row
            const int traj0 = r / a.L, tok0 = r - traj0 * a.L;
#pragma unroll 1
            for (int p = 0; p < CW / rpa; ++p) {
              const int cl = p * rpa + csub;         // channel row inside the wave's columns
              const int ch = col_w + cl - n_rm;
              if (ch < 0 || ch >= Dv) continue;
              const uint2 pk = *reinterpret_cast<const uint2*>(stg16 + cl * VP + t4);
              if (units) {
                if (r < MM) store_stream(a.vt + ((int64_t)traj0 * Dv + ch) * a.Lpad + value_slot(a.tok_off + tok0), pk);
                continue;
              }
              const uint16_t e[4] = {(uint16_t)pk.x, (uint16_t)(pk.x >> 16), (uint16_t)pk.y, (uint16_t)(pk.y >> 16)};
              int traj = traj0, tok = tok0;
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                if (r + k < MM) {
                  if (tok >= a.L) { tok -= a.L; ++traj; }
                  a.vt[((int64_t)traj * Dv + ch) * a.Lpad + value_slot(a.tok_off + tok)] = e[k];
                  ++tok;
                }
              }
            }
          }
          wave_lds_sync();
          return true;
        });
      }
      if (col_w >= n_rm) return;                     // nothing row-major in this wave's columns
    }
    const bool n_ok = n < n_rm;                      // N is a multiple of 4
    const float col_scale = n < a.scale_cols ? a.out_scale : 1.f;   // e.g. queries pre-multiplied by the softmax scale
    const float inv_hd = a.norm_hd == 64 ? 1.f / 64.f : 1.f / 32.f;
    float4 ng4 = {1.f, 1.f, 1.f, 1.f};               // norm scales of this lane's 4 columns
    if (EPI == EPI_QKV && a.norm_hd > 0 && n_ok) {
      const uint2 raw = *reinterpret_cast<const uint2*>((n < a.scale_cols ? a.qn_g : a.kn_g) + n % a.norm_hd);
      ng4 = {bf16_to_f32((uint16_t)raw.x), bf16_to_f32((uint16_t)(raw.x >> 16)), bf16_to_f32((uint16_t)raw.y),
             bf16_to_f32((uint16_t)(raw.y >> 16))};
    }
    // The row map of the layers that have one is linear inside a trajectory: row r = traj * per_traj + tok of the problem goes
    // to row r + shift + traj * gap.  A slab of 32 rows touches at most two trajectories when one has at least 32 rows; a
    // division per row and access (`per_row`) is left to shorter ones.
    const bool mapped = EPI == EPI_EMBED || (EPI == EPI_QKV && a.Lout > 0);
    const int per_traj = EPI == EPI_EMBED ? a.Li : a.L;
    const int gap = EPI == EPI_EMBED ? a.L - a.Li : a.Lout - a.L, shift = EPI == EPI_QKV ? a.tok_off : 0;
    const bool per_row = per_traj < 32;
    constexpr bool F32 = EPI == EPI_F32 || EPI == EPI_EMBED || EPI == EPI_RESID;
    typedef std::conditional_t<F32, float, uint16_t> out_t;
    const int64_t ld = F32 ? a.ldo : a.ldob;
    out_t* const out_w = [&] { if constexpr (F32) return a.outf; else return a.outb; }() + (int64_t)(row_w + rsub) * ld + n;
    // FULL: every row of the wave's tile and every column of the lane exist, so no access is masked
    auto slabs = [&](auto full_c) {
      constexpr bool FULL = decltype(full_c)::value;
#pragma unroll
      for (int i = 0; i < FM; i += 2) {
        const int slab0 = row_w + i * MI;                          // wave-uniform
        if (!FULL && slab0 >= MM) break;
        const int np = i + 1 < FM ? NP : NP / 2;                   // an odd last row tile is half a slab
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
          if (i + ii < FM)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
              for (int t = 0; t < 4; ++t) stg[(ii * MI + 4 * lk + t) * EST + j * MI + lr] = acc[i + ii < FM ? i + ii : 0][j][t];
        float4 v[NP];
#pragma unroll
        for (int p = 0; p < np; ++p) {
          v[p] = *reinterpret_cast<const float4*>(stg + (RPI * p + rsub) * EST + c4);
          if (EPI == EPI_QKV && a.norm_hd > 0) {
            // RMS norm over the head chunk this lane's 4 columns belong to (norm_hd / 4 adjacent lanes of the row)
            const float ss = (v[p].x * v[p].x + v[p].y * v[p].y) + (v[p].z * v[p].z + v[p].w * v[p].w);
            const float rstd = rsqrtf(head_sum(ss, a.norm_hd == 64) * inv_hd + 1e-6f);
            v[p].x *= rstd * ng4.x; v[p].y *= rstd * ng4.y; v[p].z *= rstd * ng4.z; v[p].w *= rstd * ng4.w;
          }
          if (EPI == EPI_BF16 || EPI == EPI_QKV) { v[p].x *= col_scale; v[p].y *= col_scale; v[p].z *= col_scale; v[p].w *= col_scale; }
        }
        auto exists = [&](int p) { return FULL || (slab0 + RPI * p + rsub < MM && n_ok); };
        out_t* const out_i = out_w + (int64_t)(i * MI) * ld;
        // trajectory of the slab's first row, and the first row of the next one
        const int traj0 = EPI == EPI_RESID || mapped ? slab0 / per_traj : 0, split = (traj0 + 1) * per_traj;
        if constexpr (EPI == EPI_RESID) {
          // gates are per (group, column).  All loads of the slab are issued before its stores.
          float4 g0 = {1.f, 1.f, 1.f, 1.f}, g1 = g0;
          if (a.gate && !per_row && n_ok) {
            const int last = (MM - 1) / a.L;
            g0 = *reinterpret_cast<const float4*>(a.gate + (int64_t)a.group_of[traj0] * a.gate_ld + n);
            g1 = *reinterpret_cast<const float4*>(a.gate + (int64_t)a.group_of[min(traj0 + 1, last)] * a.gate_ld + n);
          }
          float4 hv[NP], gv[NP];
#pragma unroll
          for (int p = 0; p < np; ++p) {
            const int r = slab0 + RPI * p + rsub;
            if (i / 2 < PF) hv[p] = __builtin_bit_cast(float4, hpre[i / 2 < PF ? i / 2 : 0][p]);
            else hv[p] = exists(p) ? load_stream(out_i + (int64_t)(RPI * p) * ld) : float4{0.f, 0.f, 0.f, 0.f};
            gv[p] = r < split ? g0 : g1;
            if (a.gate && per_row && exists(p))
              gv[p] = *reinterpret_cast<const float4*>(a.gate + (int64_t)a.group_of[r / a.L] * a.gate_ld + n);
          }
#pragma unroll
          for (int p = 0; p < np; ++p)
            if (exists(p))
              store_stream(out_i + (int64_t)(RPI * p) * ld, float4{hv[p].x + gv[p].x * v[p].x, hv[p].y + gv[p].y * v[p].y,
                                                                   hv[p].z + gv[p].z * v[p].z, hv[p].w + gv[p].w * v[p].w});
        } else {
#pragma unroll
          for (int p = 0; p < np; ++p) {
            if (!exists(p)) continue;
            out_t* dst = out_i + (int64_t)(RPI * p) * ld;
            const int r = slab0 + RPI * p + rsub;
            const int traj = mapped && per_row ? r / per_traj : r < split ? traj0 : traj0 + 1;
            if (mapped) dst += ((int64_t)traj * gap + shift) * ld;
            if constexpr (EPI == EPI_F32) {
              store_stream(dst, v[p]);
            } else if constexpr (EPI == EPI_EMBED) {
              const uint2 raw = *reinterpret_cast<const uint2*>(a.pos + (int64_t)(r - traj * a.Li) * a.N + n);
              store_stream(dst, float4{v[p].x + bf16_to_f32((uint16_t)raw.x), v[p].y + bf16_to_f32((uint16_t)(raw.x >> 16)),
                                       v[p].z + bf16_to_f32((uint16_t)raw.y), v[p].w + bf16_to_f32((uint16_t)(raw.y >> 16))});
            } else if constexpr (EPI == EPI_GELU) {
              store_stream(dst, pack_bf16x4({gelu_tanh(v[p].x), gelu_tanh(v[p].y), gelu_tanh(v[p].z), gelu_tanh(v[p].w)}));
            } else {
              store_stream(dst, pack_bf16x4(v[p]));
            }
          }
        }
      }
    };
    // Plain fp32 output keeps its masks: rows that do not end on a 128-byte line share lines with their neighbours, and waves with and
    // without masks in one workgroup get further apart in them (24576 x 1000 x 256 36.9 us, with masks alone 34.6; no difference
    // for 1024 or 2048 columns).
    if (EPI != EPI_F32 && row_w + BM / WM <= MM && col_w + CW <= n_rm) slabs(std::true_type{});
    else slabs(std::false_type{});
    return;
  }
  // ---- unpatchify: per-element scatter into the latent layout (small: N = 4C columns) ----
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int r0 = row_w + i * MI + 4 * lk;          // rows r0 + t
    if (r0 >= a.M) continue;
    const int traj0 = r0 / a.Li, tok0 = r0 - traj0 * a.Li;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = col_w + j * MI + lr;
      if (n >= a.N) continue;
      int traj = traj0, tok = tok0;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (r0 + t >= a.M) break;
        if (tok >= a.Li) { tok -= a.Li; ++traj; }
        const int py = tok / a.Wp, px = tok - py * a.Wp;
        const int c = n >> 2, dy = (n >> 1) & 1, dx = n & 1;
        a.outf[(int64_t)traj * ((int64_t)(a.N >> 2) * a.HW) + (int64_t)c * a.HW + (2 * py + dy) * a.Wimg + 2 * px + dx] =
            acc[i][j][t];
        ++tok;
      }
    }
  }
}

template <int EPI, int BM, int BN, int WM, int WN, int MINW, int SA, int SW, bool WIDE = false, int NPROB>
static pg_status launch_tile(const GemmBatch<NPROB>& batch, hipStream_t s) {
  int tiles_m = 0;
  for (const GemmArgs& g : batch.g) tiles_m += (g.M + BM - 1) / BM;
  const int tiles = tiles_m * ((batch.g[0].N + BN - 1) / BN);
  const int grid = (tiles + XCDS - 1) / XCDS * XCDS;
  gemm_kernel<EPI, BM, BN, WM, WN, MINW, SA, SW, WIDE, NPROB><<<dim3(grid), dim3(64 * WM * WN), 0, s>>>(batch);
  PG_LAUNCH_CHECK("gemm_kernel");
  return PG_OK;
}

// Tile choice: the shape with the smallest estimated time.  A compute unit works through w = tiles / 256 tiles (the last
// round, part empty, counts half as empty as it is: tiles of a long launch drift apart), each an edge (prologue and epilogue,
// by what the epilogue does) and K / 64 steps; where it holds several tiles at a time (`several`), a lone one's steps take
// their latency (`idle`) whatever else there is, otherwise they rise from `idle` to `full` as the chip fills.  The constants are
// microseconds fitted to every tile's time in 1892 layers (256 to 450000 rows, 16 widths from 64 to 1536); with the chosen tile a block
// of the network takes 0.2 % longer than with the best one, layer by layer, and 8 % at most.
struct TileShape { int bm, bn; bool several; double fixed, resid, qkv, out, idle, full; };
constexpr TileShape TILES[9] = {
    {256, 256, false, 0, 11.7, 11.3, 7.16, 1.76, 1.44},
    {192, 256, false, 0, 8.42, 8.79, 6.22, 0.396, 1.14},
    {128, 128, true, 3.41, 2.58, 1.98, 1.66, 0.83, 0.479},
    {160, 256, false, 0, 7.29, 8.98, 5.48, 0.801, 0.969},
    {224, 256, false, 0, 10.2, 9.5, 6.72, 0.976, 1.32},
    {128, 64, true, 3.76, 2.04, 1.5, 1.24, 0.23, 0.28},
    {64, 64, true, 4.13, 0.844, 0.295, 0.131, 0.304, 0.196},
    {128, 256, false, 0, 7.28, 9.94, 5.89, 0.457, 0.763},
    {64, 64, true, 4.3, 0.897, 0.413, 0.293, 0.204, 0.169}};
template <int NPROB>
static int pick_tile(const GemmBatch<NPROB>& batch, int epilogue) {
  const GemmArgs& a = batch.g[0];
  const double nk = a.K / BK;
  const bool whole_heads = epilogue == EPI_QKV && a.norm_hd > 32;   // the fused norm needs a whole head inside one wave's columns
  int best = 0;
  double best_us = 0.0;
  for (int i = 0; i < 9; ++i) {
    const TileShape& t = TILES[i];
    if (whole_heads && t.bm == 64) continue;      // 32 columns per wave
    double tile_rows = 0.0;
    for (const GemmArgs& g : batch.g) tile_rows += ceil((double)g.M / t.bm);
    const double load = tile_rows * ceil((double)a.N / t.bn) / 256.0;
    const double w = load <= 1.0 ? 1.0 : 0.5 * (load + ceil(load));
    const double edge = epilogue == EPI_RESID ? t.resid : epilogue == EPI_QKV ? t.qkv : t.out;
    const double full = t.bm == 256 && a.K > a.N ? 1.08 * t.full : t.full;    // two tiles of A ahead are too few for a cold A
    const double alone = t.several ? t.idle : t.idle + (full - t.idle) * fmin(1.0, load / 0.75);
    const double us = t.fixed + fmax(edge + nk * alone, w * (edge + nk * full));
    if (i == 0 || us < best_us) { best = i; best_us = us; }
  }
  return best;
}

template <int EPI, int NPROB>
static pg_status launch_one(const GemmBatch<NPROB>& batch, hipStream_t s, int tile = 0) {
  // operand rows so far apart that their byte offsets inside a tile need 64 bits (pg_gemm_bf16 alone takes any)
  if constexpr (EPI == EPI_F32)
    if (batch.g[0].lda > NARROW_LD || batch.g[0].ldw > NARROW_LD) return launch_tile<EPI_F32, 128, 128, 2, 2, 2, 2, 2, true>(batch, s);
  switch (tile ? tile - 1 : pick_tile(batch, EPI)) {
    case 0: return launch_tile<EPI, 256, 256, 2, 4, 2, 2, 2>(batch, s);
    case 1: return launch_tile<EPI, 192, 256, 2, 4, 2, 3, 2>(batch, s);
    case 2: return launch_tile<EPI, 128, 128, 2, 2, 2, 2, 2>(batch, s);
    case 3: return launch_tile<EPI, 160, 256, 2, 4, 2, 3, 3>(batch, s);
    case 4: return launch_tile<EPI, 224, 256, 2, 4, 2, 3, 2>(batch, s);
    case 5: return launch_tile<EPI, 128, 64, 4, 1, 2, 3, 3>(batch, s);
    case 6: return launch_tile<EPI, 64, 64, 2, 2, 4, 2, 2>(batch, s);
    case 7: return launch_tile<EPI, 128, 256, 2, 4, 2, 3, 3>(batch, s);
    default: return launch_tile<EPI, 64, 64, 2, 2, 3, 3, 3>(batch, s);
  }
}

// what the kernels assume of one problem
static pg_status check_gemm(const GemmArgs& a, int epilogue) {
  if (a.K <= 0 || a.K % 64) return fail(PG_ESHAPE, "GEMM K = %d must be a positive multiple of 64", a.K);
  if (a.lda % 8 || a.ldw % 8 || a.lda < a.K || a.ldw < a.K || ((uintptr_t)a.A & 15) || ((uintptr_t)a.W & 15))
    return fail(PG_ESHAPE, "GEMM operands need 16-byte aligned rows (lda %lld, ldw %lld)", (long long)a.lda, (long long)a.ldw);
  if (!a.A || !a.W) return fail(PG_EINVAL, "GEMM: null operand");
  if (epilogue != EPI_UNPATCH) {
    // the row-major epilogues write 4 consecutive columns per lane
    const int n_rm = epilogue == EPI_QKV ? a.v_start : a.N;
    if (n_rm % 4) return fail(PG_ESHAPE, "GEMM N = %d must be a multiple of 4", n_rm);
    if ((a.outf && (a.ldo % 4 || ((uintptr_t)a.outf & 15))) || (a.outb && (a.ldob % 4 || ((uintptr_t)a.outb & 7))) ||
        (a.bias && ((uintptr_t)a.bias & 7)) || (a.gate && (a.gate_ld % 4 || ((uintptr_t)a.gate & 15))) ||
        (a.pos && ((uintptr_t)a.pos & 7)))
      return fail(PG_ESHAPE, "GEMM output / bias / gate rows need 16-byte (bf16: 8-byte) alignment");
  }
  if (epilogue == EPI_QKV && a.norm_hd > 0) {
    if ((a.norm_hd != 32 && a.norm_hd != 64) || !a.qn_g || !a.kn_g || a.v_start % a.norm_hd || a.scale_cols % a.norm_hd ||
        ((uintptr_t)a.qn_g & 7) || ((uintptr_t)a.kn_g & 7))
      return fail(PG_ESHAPE, "GEMM: bad fused head norm (width %d)", a.norm_hd);
  }
  if (epilogue == EPI_QKV) {
    const int vs = a.v_start;
    if (!a.vt || a.L < 1 || a.tok_off + a.L > a.Lpad || (a.Lpad & 15) || ((uintptr_t)a.vt & 7) || vs < 0 || vs > a.N || vs % 32 ||
        (a.N - vs) % 32 || !a.outb)
      return fail(PG_ESHAPE, "GEMM: bad transposed-value output (L %d, Lpad %d, v_start %d)", a.L, a.Lpad, a.v_start);
  }
  return PG_OK;
}

// bands of 8 tile rows; of 4 when the output is at most six tiles wide (the D-wide residual GEMMs of the 1536-wide network:
// a band then still spans the whole width, and 0.7 % of the loop's GEMM time goes away)
static int raster_band(int N) { return (N + 255) / 256 <= 6 ? GROUP_M / 2 : GROUP_M; }
static double gemm_flops(const GemmArgs& a) { return 2.0 * a.M * (double)a.N * (a.k_algo > 0 ? a.k_algo : a.K); }

pg_status launch_gemm(const GemmArgs& a_in, int epilogue, hipStream_t s, int tile) {
  GemmBatch<1> batch{{a_in}};
  GemmArgs& a = batch.g[0];
  a.group_m = raster_band(a.N);
  if (a.M <= 0 || a.N <= 0) return PG_OK;
  PG_TRY(check_gemm(a, epilogue));
  const int rec = prof_open(PROF_GEMM, gemm_flops(a), s);
  pg_status st = PG_EINVAL;
  switch (epilogue) {
    case EPI_F32: st = launch_one<EPI_F32>(batch, s, tile); break;
    case EPI_EMBED: st = launch_one<EPI_EMBED>(batch, s); break;
    case EPI_BF16: st = launch_one<EPI_BF16>(batch, s); break;
    case EPI_QKV: st = launch_one<EPI_QKV>(batch, s); break;
    case EPI_GELU: st = launch_one<EPI_GELU>(batch, s); break;
    case EPI_RESID: st = launch_one<EPI_RESID>(batch, s, tile); break;
    case EPI_UNPATCH: st = launch_one<EPI_UNPATCH>(batch, s); break;
    default: st = fail(PG_EINVAL, "unknown GEMM epilogue %d", epilogue);
  }
  prof_close(rec, s);
  return st;
}

// Two problems of equal N and K (the same layer of the two streams of the dual-stream network) in one launch: the context
// stream alone is a few dozen tiles, which left most of the 256 compute units idle for as long as the image stream's tiles take.
pg_status launch_gemm_pair(const GemmArgs& first, const GemmArgs& second, int epilogue, hipStream_t s) {
  if (first.M <= 0 || second.M <= 0) return launch_gemm(first.M > 0 ? first : second, epilogue, s);
  if (first.N != second.N || first.K != second.K || first.norm_hd != second.norm_hd || first.out_scale != second.out_scale ||
      first.scale_cols != second.scale_cols || first.v_start != second.v_start || first.Lout != second.Lout)
    return fail(PG_EINVAL, "GEMM pair: different layers");
  GemmBatch<2> batch{{first, second}};
  for (GemmArgs& g : batch.g) {
    PG_TRY(check_gemm(g, epilogue));
    if (g.lda > NARROW_LD || g.ldw > NARROW_LD) return fail(PG_ESHAPE, "GEMM pair: operand rows too far apart");
    g.group_m = raster_band(g.N);
  }
  const int rec = prof_open(PROF_GEMM, gemm_flops(first) + gemm_flops(second), s);
  pg_status st = PG_EINVAL;
  switch (epilogue) {
    case EPI_QKV: st = launch_one<EPI_QKV>(batch, s); break;
    case EPI_GELU: st = launch_one<EPI_GELU>(batch, s); break;
    case EPI_RESID: st = launch_one<EPI_RESID>(batch, s); break;
    default: st = fail(PG_EINVAL, "GEMM pair: epilogue %d", epilogue);
  }
  prof_close(rec, s);
  return st;
}

// Measurement hook: bf16 MFMAs on registers alone.  Eight independent 32x32 accumulators per wave keep the pipe
// full (an MFMA may not follow one that writes the accumulator it reads without waiting for it).
constexpr int PROBE_ACC = 8;
__global__ __launch_bounds__(256) void mfma_probe_kernel(float* __restrict__ out, int iters, float scale) {
  bf16x8 a, b;
  uint32_t h = (threadIdx.x + 1u) * 2654435761u + blockIdx.x * 40503u;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    h = h * 1664525u + 1013904223u;
    a[e] = (__bf16)(((int)(h >> 8) % 2001 - 1000) * 1e-3f * scale);
    h = h * 1664525u + 1013904223u;
    b[e] = (__bf16)(((int)(h >> 8) % 2001 - 1000) * 1e-3f * scale);
  }
  f32x16 acc[PROBE_ACC];
#pragma unroll
  for (int i = 0; i < PROBE_ACC; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < PROBE_ACC; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
  }
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < PROBE_ACC; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) sum += acc[i][e];
  out[blockIdx.x * blockDim.x + threadIdx.x] = sum;
}

}  // namespace pg

using namespace pg;

extern "C" pg_status pg_mfma_probe(int32_t blocks, int32_t iters, float operand_scale, float* out, double* flops,
                                   void* stream) {
  if (blocks < 1 || blocks > 65536 || iters < 1 || iters > 10000000) return fail(PG_EINVAL, "pg_mfma_probe: blocks %d, iters %d", blocks, iters);
  if (!out) return fail(PG_EINVAL, "pg_mfma_probe: out is NULL");
  mfma_probe_kernel<<<dim3(blocks), dim3(256), 0, (hipStream_t)stream>>>(out, iters, operand_scale);
  PG_LAUNCH_CHECK("mfma_probe_kernel");
  if (flops) *flops = (double)blocks * 4.0 * iters * PROBE_ACC * 32768.0;
  return PG_OK;
}

// C = A W^T + bias, or C += it
static pg_status plain_gemm(const uint16_t* A, int64_t lda, const uint16_t* W, int64_t ldw, const uint16_t* bias, float* C, int64_t ldc,
                            int64_t M, int64_t N, int64_t K, bool accumulate, int tile, hipStream_t s) {
  if (M < 0 || N < 0 || M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return fail(PG_EINVAL, "pg_gemm_bf16: bad sizes");
  if (M == 0 || N == 0) return PG_OK;
  if (!C || ldc < N) return fail(PG_EINVAL, "pg_gemm_bf16: bad output");
  GemmArgs a{};
  a.A = A; a.lda = lda; a.W = W; a.ldw = ldw; a.bias = bias;
  a.M = (int)M; a.N = (int)N; a.K = (int)K; a.L = (int)M;
  a.outf = C; a.ldo = ldc;
  return launch_gemm(a, accumulate ? EPI_RESID : EPI_F32, s, tile);
}

extern "C" pg_status pg_gemm_bf16(const uint16_t* A, int64_t lda, const uint16_t* W, int64_t ldw,
                                  const uint16_t* bias, float* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                                  void* stream) {
  return plain_gemm(A, lda, W, ldw, bias, C, ldc, M, N, K, false, 0, (hipStream_t)stream);
}

extern "C" int32_t pg_gemm_tile(int64_t M, int64_t N, int64_t K, int32_t accumulate) {
  if (M < 1 || N < 1 || K < 1 || M > INT32_MAX || N > INT32_MAX || K > INT32_MAX) return 0;
  GemmBatch<1> batch{};
  batch.g[0].M = (int)M; batch.g[0].N = (int)N; batch.g[0].K = (int)K;
  return pick_tile(batch, accumulate ? EPI_RESID : EPI_F32) + 1;
}

extern "C" pg_status pg_gemm_bf16_tile(const uint16_t* A, int64_t lda, const uint16_t* W, int64_t ldw,
                                       const uint16_t* bias, float* C, int64_t ldc, int64_t M, int64_t N, int64_t K,
                                       int32_t accumulate, int32_t tile, void* stream) {
  if (tile < 0 || tile > (int)(sizeof(TILES) / sizeof(TILES[0]))) return fail(PG_EINVAL, "pg_gemm_bf16_tile: tile %d", tile);
  if (lda > NARROW_LD || ldw > NARROW_LD) return fail(PG_ESHAPE, "pg_gemm_bf16_tile: operand rows too far apart");
  return plain_gemm(A, lda, W, ldw, bias, C, ldc, M, N, K, accumulate != 0, tile, (hipStream_t)stream);
}
