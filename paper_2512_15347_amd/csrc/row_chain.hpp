// The layers between two attentions of a block, which work on a row at a time, in one launch.
#pragma once
#include "common.hpp"

namespace pg {

// What follows an attention: the output projection with its residual sum, and then
enum ChainKind {
  CHAIN_QUERIES = 0,   // LayerNorm and the queries of the cross-attention
  CHAIN_BLOCK = 1,     // LayerNorm, MLP with its residual sum, LayerNorm and queries | keys | values of the next block
  CHAIN_LAST = 2,      // LayerNorm, MLP with its residual sum
  CHAIN_START = 3      // and, in front of the first one: LayerNorm and queries | keys | values of the first block
};
struct ChainStream {
  const uint16_t* att; float* h;                   // attention's output and the residual stream, [M L, D]
  const uint16_t* o_w; const uint16_t* o_b; const uint16_t* fc1_w; const uint16_t* fc1_b; const uint16_t* fc2_w; const uint16_t* fc2_b;
  const uint16_t* next_w; const uint16_t* next_b;  // rows of D (fc2: 4 D) columns, no padding
  // of modulation row 0: gate of the projection (NULL: 1), shift and scale of the LayerNorm behind it (NULL: 0, 0), gate of the MLP,
  // shift and scale of the next block
  const float* gate1; const float* norm1; const float* gate2; const float* norm2;
  const uint16_t* qn_g; const uint16_t* kn_g;      // scales of the normalised queries and keys of the next block (ChainArgs::norm_hd)
  int L;                                           // rows of a trajectory
};
struct ChainArgs {
  ChainStream s[2];                                // the second one with L > 0: CHAIN_BLOCK or CHAIN_START, its tokens follow the first one's
  uint16_t* qk; uint16_t* vt;                      // CHAIN_QUERIES: [M L, D]; CHAIN_BLOCK, CHAIN_START: [M L, 2 D] and transposed values (EPI_QKV), L of both
  int64_t mod_ld; const int32_t* mod_of;
  int M, Lpad;
  float out_scale;                                 // of the queries
  int norm_hd;                                     // head width of queries and keys that are RMS-normalised (EPI_QKV), or 0
};
// whether networks of this width, for at most M trajectories of L (and L2, of the second stream) tokens, run that way
bool row_chain_takes(int D, int64_t M, int L, int L2);
pg_status launch_row_chain(const ChainArgs& a, int D, ChainKind kind, hipStream_t s);

}  // namespace pg
