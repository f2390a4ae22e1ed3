// Narrow networks on short sequences: the whole network evaluation of a trajectory in one workgroup.
#pragma once
#include "ctx.hpp"
#include "logprob.hpp"

namespace pg {

// One layer's weights: bf16 [rows, K] with row length `ld`, bias bf16 [rows]; block b of a per-block layer lies b * stride further.
struct SmallLayer { const uint16_t* w; const uint16_t* b; int ld; };
struct SmallNetArgs {
  const float* x; float* u;                        // latents and network output [M, C, H, W]
  const int32_t* group_of; const int32_t* mod_of;  // per trajectory: its group, and its row of the modulation vectors
  const float* ctx_h;                              // projected context rows [P, Lc, D] (joint network)
  SmallLayer embed, qkv, out, fc1, fc2, fin;       // per-block ones: block 0
  const uint16_t* pos;                             // bf16 [Li, D]
  const float* mod; const float* fmod;             // modulation vectors [rows][blocks][6 D], [rows][2 D]
  int64_t block_stride;
  int M, C, H, W, Li, Lc, L, blocks;
  float scale_log2;
};

// whether the networks of this context run that way; a property of its configuration, not of how many trajectories are active
bool small_net_takes(const pg_ctx* c);
pg_status launch_small_net(const SmallNetArgs& a, int D, int hd, hipStream_t s);

// The same networks with a workgroup per 16 rows of a trajectory and a launch per block, for few trajectories
// (small_rows_takes).  A step is ROWS_START (patch embedding, queries / keys / values of the first block), then one launch per
// block, each with the queries / keys / values of the block after it; the last one writes u, may make the sampler's update and may
// start the next step.
struct RowsUpdate {                                // x_out = A x[src] + B u[src] + C xi, log-prob from the sum of xi^2
  float A, B, C;
  uint32_t k0, k1, step;
  const int32_t* src; const int32_t* orig_id;      // src NULL: the same row
  float* x_out; float* hist_next;                  // [M, C, H, W]; by original id, or NULL
  const double* sums;                              // of this step, by original id
  LogProb out;
};
struct RowsArgs {
  const float* x; float* u; float* hs;             // latents, output; residual stream [M][16 tiles][D]
  const uint16_t* qk_in; const uint16_t* vt_in;    // queries, keys [M][2][16 tiles][D] and values [M][D][16 tiles, an even number] of this
                                                   // block, in the order in which attention holds them
  uint16_t* qk_out; uint16_t* vt_out;              // of the next one: other buffers, as workgroups of this launch still read these
  const uint16_t* w; const uint16_t* w_next;       // the block's tensors from its QKV weights on, and those of the next one
  const uint16_t* embed; const uint16_t* fin; const uint16_t* fin_b;
  const float* mod; const float* mod_next; const float* fmod;      // row 0 of the block, of the step that is started, of the final layer
  const int32_t* mod_of; const int32_t* group_of; const float* ctx_h;
  int mod_ld, tiles, L, Li, Lc, C, H, W;
  float scale_log2;
  int update;                                      // whether `up` is made
  RowsUpdate up;
};
bool small_rows_takes(const pg_ctx* c);                // whether a loop in one call runs that way
bool small_rows_evaluates(const pg_ctx* c, int M);     // whether an evaluation of M trajectories alone does (the same bits either way)
int small_rows_tiles(const pg_ctx* c);
// block -1: a step's first rows; start: the last block's launch starts the next step (an update goes with it).  The caller sets x, hs,
// the buffers, mod_next and the update.
pg_status launch_small_rows(const SmallNetArgs& n, RowsArgs& a, int D, int hd, int block, bool start, hipStream_t s);
// One network evaluation that way (dit_kernels.hip).
struct RowsPass {
  const float* x;                                  // the latents that are evaluated
  bool begin;                                      // start the step; else the pass before has
  const RowsUpdate* before; const float* x_before; // the update of x_before that `begin` makes first, giving x (or NULL)
  const RowsUpdate* after;                         // the update of x that follows u (or NULL)
  bool start_next;                                 // start the next step with it (the next row of the modulation vectors)
};
pg_status net_rows(pg_ctx* c, const NetBatch& batch, const RowsPass& pass, const uint16_t* weights, hipStream_t s);

}  // namespace pg
