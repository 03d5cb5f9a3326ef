// Parameters of the persistent kernel that runs the prefix transformer's layers (prefix_persistent.hip).
#pragma once
#include "exec_ctx.h"
#include "pi0_internal.h"

struct PrefixLoopParams {
  // operations of layer 0, filled as for the launches; what changes per layer is derived in the kernel from the strides below
  GemmParams qkv, o, gu, dn;
  ReduceParams red;
  AttnParams att;
  int att_tiles;                  // query tiles of the attention, of 16 or 32 rows
  int gu_blocks;                  // tiles of gate||up, rounded up to eighths
  int dn_blocks;                  // tiles of one k range of down, rounded up to eighths where a die has no range to itself
  int layers;                     // whole layers: all of the stack but the last, which only leaves keys and values
  size_t layer_stride;            // bytes between consecutive layers' weights
  size_t gain_stride;             // bytes between consecutive layers' gain vectors
  size_t kcache_stride, vcache_stride;   // bytes between consecutive layers of the cache
  // Ring of per-layer buffers (layer l at ring + l * ring_stride), as VisionLoopParams has it: gain-scaled bf16 copy of the residual stream and row
  // statistics after the O and the down projection, queries, the attention's output, the GeGLU product.  Layer 0's queries
  // are there before the launch.  (The residual stream and down's partial sums stay where they are: they are read past the caches.  So are
  // the row statistics after the down projection: an item of the reduction leaves half a cache line of each plane, the next block the other.)
  char* ring;
  size_t ring_stride;
  unsigned r_xb_o, r_st_o, r_xb_d, r_st_d, r_q, r_attn, r_mid;
  unsigned* sync;                 // GB_WORDS words for each turn (GB_TURNS), those from GB_START on zeroed before the launch
  const char* arena;              // everything that blocks exchange lies in [arena, arena + arena_bytes)
  unsigned arena_bytes;
  unsigned spin_limit;            // bound of one barrier wait, in polls
  unsigned most_blocks;           // that take part at most (GridBarrierT::init_some); 0: all, which are resident
};

// What a variant of the kernel is built for, to be compared with the launches' own choices for the shape
struct PrefixTiles {
  struct { int mb, nb, parts, steps; } qkv, o;   // gemm_stream_tile's; steps: k16 steps of a part
  struct { int mt, nt; } gu, dn;                 // gemm_lds_tile's
  int gu_height;                                 // gemm_cols_height's of gate||up; not 0: instead of the tile gu
  int gu_tile_rows() const { return gu_height != 0 ? 32 * gu_height : 64 * gu.mt; }
  int gu_tile_features() const { return gu_height != 0 ? 8 : 2 * gu.nt; }   // of 32
  bool walk;                                     // gate||up: a block's tiles one after the other in the same rows
  int att_rows, att_chunks;                      // query rows of an attention item, most chunks of keys
  int o_groups;                                  // groups in which the planes of the O projection's row statistics are added
  bool gu_rows;                                  // gate||up by gemm_rows_body
};
int prefix_loop_variants();
PrefixTiles prefix_loop_tiles(int variant);
constexpr int PREFIX_LOOP_CHUNKS = 24;            // most chunks of 32 tokens that a variant takes
constexpr int PREFIX_QKV_PLANES = 8;              // planes of row statistics that the reduction behind down leaves

hipError_t prefix_loop_init_attributes();
hipError_t prefix_loop_max_blocks_per_cu(int* out);
bool prefix_loop_takes(int variant, const PrefixLoopParams& P, int blocks);   // the variant covers this shape
// d_params: device memory for one PrefixLoopParams (16-byte aligned), written by a small launch ahead of the kernel
hipError_t launch_prefix_loop(hipStream_t s, int variant, const PrefixLoopParams& P, PrefixLoopParams* d_params, int blocks);
