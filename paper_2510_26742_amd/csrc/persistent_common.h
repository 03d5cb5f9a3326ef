// What the persistent kernels share (expert_persistent.hip, vision_persistent.hip, prefix_persistent.hip): reading their parameter block, handing out items.
#pragma once
#include "exec_ctx.h"
#include "pi0_internal.h"

// block: this block's place in the order in which the operation's items are handed out; blocks: that take part
template <class F>
__device__ __forceinline__ void for_items(int n_items, F&& f, int block = (int)blockIdx.x, int blocks = (int)gridDim.x) {
  bool first = true;
  for (int it = block; it < n_items; it += blocks) {
    if (!first) __syncthreads();   // shared memory of the item before is free
    f(it);
    first = false;
  }
}

// The same for an operation with an item for every block of the grid, of which usually each takes one: block < N
template <int N, class F>
__device__ __forceinline__ void for_all_items(F&& f, int block, int blocks) {
  for (int it = block;;) {
    f(it);
    it += blocks;
    if (__builtin_expect(it >= N, 1)) break;
    __syncthreads();   // shared memory of the item before is free
  }
}

// Reads part `part` of `nparts` of n16 16-byte pieces, piece i at addr(i), into the caches: 16 bytes per lane, 8 loads in flight; the
// values are folded into a word that the caller stores only if it equals a constant, so no result depends on them.
template <int THREADS, class F>
__device__ __forceinline__ unsigned read_ahead_part(unsigned n16, int part, int nparts, int tid, unsigned fold, F&& addr) {
  const unsigned per = (n16 + (unsigned)nparts - 1) / (unsigned)nparts;
  const unsigned beg = (unsigned)part * per;
  const unsigned end = beg + per < n16 ? beg + per : n16;
  for (unsigned i = beg + (unsigned)tid; i < end; i += 8 * THREADS) {
    u32x4_t v[8];
#pragma unroll
    for (int j = 0; j < 8; j++) {
      const unsigned idx = i + (unsigned)j * THREADS;
      v[j] = *reinterpret_cast<const u32x4_t*>(addr(idx < end ? idx : end - 1));   // clamped, unconditional
    }
#pragma unroll
    for (int j = 0; j < 8; j++) fold ^= v[j][0] ^ v[j][1] ^ v[j][2] ^ v[j][3];
  }
  return fold;
}

// The parameter block lives in device memory and every operation reads its own part afresh: taken by value, the
// operations' pointers and sizes stay live across the whole loop and the kernel spills hundreds of registers.  It is read
// through the constant address space (scalar loads; as generic memory it was read with FLAT vector loads that queued
// behind the prefetches in flight), and the pointers in it are declared global.
template <class P>
using ParamsPtr = const __attribute__((address_space(4))) P*;
template <class P>
__device__ __forceinline__ const P& fresh(ParamsPtr<P> p) {
  asm volatile("" : "+s"(p));   // nothing read through the pointer before this point is reused after it
  return *(const P*)p;
}
__device__ __forceinline__ GemmParams global(const GemmParams& src) {
  GemmParams p = src;
  p.X = as_global(p.X);
  p.W.w = as_global(p.W.w);
  p.bias = as_global(p.bias);
  p.colsum = as_global(p.colsum);
  p.rowstat = as_global(p.rowstat);
  p.stat_out = as_global(p.stat_out);
  p.gain = as_global(p.gain);
  p.out_f32 = as_global(p.out_f32);
  p.out_bf16 = as_global(p.out_bf16);
  p.resid = as_global(p.resid);
  p.kfrag = as_global(p.kfrag);
  p.vfrag = as_global(p.vfrag);
  p.rope = as_global(p.rope);
  p.xsplit_ml = as_global(p.xsplit_ml);
  return p;
}
__device__ __forceinline__ AttnParams global(const AttnParams& src) {
  AttnParams p = src;
  p.k0 = as_global(p.k0);
  p.v0 = as_global(p.v0);
  return p;
}
