// Narrow networks on short sequences: the whole network evaluation of a trajectory in one workgroup.
#pragma once
#include "ctx.hpp"

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

}  // namespace pg
