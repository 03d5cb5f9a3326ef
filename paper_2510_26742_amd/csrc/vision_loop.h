// Parameters of the persistent kernel that runs the vision tower's layers (vision_persistent.hip).
#pragma once
#include "exec_ctx.h"
#include "pi0_internal.h"

struct VisionLoopParams {
  // operations of layer 0, filled as for the launches; what changes per layer is derived in the kernel from the strides below
  GemmParams qkv, o, up, down;
  AttnParams att;
  int att_items;
  int layers;
  size_t layer_stride;            // bytes between consecutive layers' weights, biases and column sums
  size_t gain_stride;             // bytes between consecutive layers' gain vectors
  const float* g_attn0;           // gain vector of layer 0's first norm (what follows the down projection of the layer before)
  const float* g_mlp0;            // ... of its second norm
  const float* g_final;
  int planes_rest;                // planes of row statistics that the residual projections leave (o, down)
  // Ring of per-layer buffers (layer l at ring + l * ring_stride): every activation that one block writes and another reads
  // has a place that nothing has read before in this launch and whose cache lines are each written by one block
  // (exec_ctx.h, BULK_CACHED).  Byte offsets inside a slot: gain-scaled bf16 copy of the residual stream and row statistics
  // after the O and the down projection; the QKV projection's outputs; the attention's; the up projection's.  What the slots
  // hold before the launch does not matter.  (The residual stream itself stays where it is: a block reads the tile that it wrote.)
  char* ring;
  size_t ring_stride;
  unsigned r_xb_o, r_st_o, r_xb_d, r_st_d, r_q, r_k, r_v, r_attn, r_mid;
  unsigned* sync;                 // GB_WORDS words for each turn (GB_TURNS), those from GB_START on zeroed before the launch
  const char* arena;              // the ring and the residual stream lie in [arena, arena + arena_bytes)
  unsigned arena_bytes;
  unsigned most_blocks;           // that take part at most (GridBarrierT::init_some); 0: all, which are resident
  unsigned spin_limit;            // bound of one barrier wait, in polls
};

// Tiles that the kernel for `views` views is built for, as gemm_stream_tile chooses them for the launches.
// steps: k16 steps of a part, 0: any number, the parts of one size
struct VisionTile {
  int mb, nb, parts, steps;
  bool takes(int k_pad) const { return steps != 0 ? (k_pad >> 4) == steps * parts : (k_pad >> 4) % parts == 0; }
};
struct VisionTiles { VisionTile qkv, resid, up; };
constexpr int VISION_LOOP_VIEWS = 3;                      // most views that the kernel takes
bool vision_loop_tiles(int views, VisionTiles* out);
int vision_loop_planes(int views);                        // planes of row statistics that it adds up
int vision_loop_attention_items(int views, int heads);

hipError_t vision_loop_init_attributes();
hipError_t vision_loop_max_blocks_per_cu(int* out);
bool vision_loop_takes(int views, const VisionLoopParams& P, int blocks);   // the kernel covers this shape
// d_params: device memory for one VisionLoopParams (16-byte aligned), written by a small launch ahead of the kernel
hipError_t launch_vision_loop(hipStream_t s, int views, const VisionLoopParams& P, VisionLoopParams* d_params, int blocks);
