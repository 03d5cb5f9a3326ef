// The action expert's whole denoise loop as ONE persistent kernel (Section 5.2 of the paper: software barriers
// in place of kernel boundaries, operands requested across the synchronisation points; Section 6.2 names the
// persistent megakernel as the way to take the expert's per-kernel overhead out).
//
// 256 blocks of 8 waves, one per compute unit, walk the operation list of Table 2's action-expert rows - state
// token; per Euler step the folded action/time embedding and its second linear layer; per layer QKV + RoPE,
// attention over [prefix cache ; own keys], O projection + residual, gate||up GeGLU, down + residual; final norm,
// output projection and the Euler update - with one grid barrier between consecutive operations.  Every operation
// is the same body that the per-operation launches run (gemm_common.h, attention_body.h, embed_bodies.h), cut
// into the same work items, so the results agree with that path bit for bit; a block takes the work items
// block index, block index + 256, ... of each operation and then arrives at the barrier.
// What the persistent form buys: a body requests its weights (constant during the kernel, ordinary loads) and
// the other constants BEFORE it waits for the operation before to complete everywhere, so the weights' trip
// from HBM overlaps the barrier; and there is no dispatch, no cold instruction / argument fetch, no end-of-kernel
// cache write-back per operation.  What it costs: data that crosses blocks must be written through to memory
// and read past the per-die L2 or from places never read before (exec_ctx.h), and a barrier costs two store-to-poll hops,
// one inside a die and one between dies.
#include "attention_body.h"
#include "expert_loop.h"
#include "persistent_common.h"

namespace {

constexpr int PK_THREADS = 512;
// Shared memory of a block: first the weights of one of gate||up's two feature tiles, which wait there, and then the partial
// tiles of the 32-feature bodies; behind it the attention and the partial tiles of O and down, which run meanwhile.
constexpr int PK_TAIL = (2 * 16 * 64 + 64) * SK_WAVES * 4;
static_assert(PK_TAIL >= SK_WAVES * 8 * 1024 && ATTN_SUFFIX_SMEM >= SK_WAVES * 64 * 4 * 4, "the staged weights; the partial tiles of O and down");

// Reading ahead inside the loop.  The expert's weights (623 MB) cycle through the 256 MB memory-side cache once per Euler
// step, so an operation's weight request - issued when the operation before ends - goes all the way to HBM (the same loop
// run on one layer's weights throughout, i.e. from that cache, is 0.46 ms faster).  The attention has 64 items for 256
// blocks: the blocks without one use the time to read the weights that the following operations will ask for, which puts
// them into the memory-side cache (read_ahead_part; 8 loads in flight: 4 finish too late, 16 disturb the working blocks' loads more than
// they gain, pi0_denoise 5.47 / 5.42 / 5.48 ms on one device, before the flag barrier).
// A packed weight matrix of n_tiles 32-feature tiles of kc16 KiB is shared out so that a block reads what
// blocks of its own die will ask for (their L2 then holds it: the second request is one die-local round trip).  Work
// items go to blocks in turn and consecutive blocks to different dies, so items u, u + 8, ... share a die.  UNIT: what
// consecutive items take: 2 = pairs of tiles (gate||up), 1 = a tile (QKV), 0 = half a tile, i.e. 16 of its 32 features
// (O and down).  Where the counts are no multiples of 8 the matrix is shared out without regard to dies.
template <int UNIT>
__device__ __forceinline__ unsigned read_ahead_weights(const bf16* w, int n_tiles, int kc16, int part, int nparts, bool by_die, int tid, unsigned fold) {
  const char* base = reinterpret_cast<const char*>(w);
  const unsigned unit16 = UNIT == 0 ? (unsigned)kc16 * 32u : (unsigned)UNIT * (unsigned)kc16 * 64u;   // 16-byte pieces per unit
  const unsigned units = UNIT == 0 ? 2u * (unsigned)n_tiles : (unsigned)(n_tiles / UNIT);
  unsigned u0 = 0, du = 1, n = units;
  if (by_die && units % 8u == 0u) {
    u0 = (unsigned)part & 7u;
    du = 8;
    n = units / 8u;
    part >>= 3;
    nparts >>= 3;
  }
  return read_ahead_part<PK_THREADS>(n * unit16, part, nparts, tid, fold, [&](unsigned i) {
    const unsigned j = i / unit16, c = i - j * unit16, u = u0 + j * du;
    if (UNIT == 0) return base + (size_t)(u >> 1) * (unsigned)kc16 * 1024u + (c >> 5) * 1024u + ((c >> 4) & 1u) * 512u + (u & 1u) * 256u + (c & 15u) * 16u;
    return base + (size_t)u * unit16 * 16u + (size_t)c * 16u;
  });
}

// The out-projection's context where every block computes the rows of x that it goes on with: they come from one buffer and go
// to LDS and, from one block, to another buffer.
template <bool TRACE>
struct EulerCtx : PersistCtxT<true, TRACE> {
  const float* from;
  float* to;
  float* lds;
  int first;      // element of x that comes first in LDS
  bool publish;
  float* actions;   // not null: instead of `to`, and not for other blocks
  __device__ __forceinline__ EulerCtx(const PersistCtxT<true, TRACE>& c, const float* from_, float* to_, float* lds_, int first_, bool publish_, float* actions_)
      : PersistCtxT<true, TRACE>(c), from(from_), to(to_), lds(lds_), first(first_), publish(publish_), actions(actions_) {}
  using PersistCtxT<true, TRACE>::st;
  __device__ __forceinline__ void st(float* p, const float& v) const {
    const int i = (int)(p - from);
    lds[i - first] = v;
    if (publish && actions != nullptr) actions[i] = v;
    else if (publish) PersistCtxT<true, TRACE>::st(to + i, v);
  }
};

// parameter block to device memory and barrier words to zero (the error word, first, stays as it is), a piece per thread, and the call's
// inputs.  Three launches before, with the copy of the actions that the loop now stores itself; pi0_denoise over two layers, one view, with the state token's
// operation taken in as well 484.6 -> 482.1 us (a launch of that size costs 1 us between others, whatever its own 4.7 us in a trace)
constexpr int PREP_THREADS = 256;
static_assert(sizeof(ExpertLoopParams) % 4 == 0 && (GB_WORDS - GB_START) % 4 == 0, "whole pieces");
__global__ __launch_bounds__(PREP_THREADS) void expert_loop_prepare_kernel(ExpertLoopParams P, ExpertLoopParams* dst, unsigned* sync, CopyArgs inputs) {
  if (blockIdx.y != 0) {
    copy_segment(inputs.seg[blockIdx.y - 1], blockIdx.x * PREP_THREADS + threadIdx.x, gridDim.x * PREP_THREADS);
    return;
  }
  const unsigned i = blockIdx.x * PREP_THREADS + threadIdx.x;
  if (i < sizeof(ExpertLoopParams) / 4) reinterpret_cast<unsigned*>(dst)[i] = reinterpret_cast<const unsigned*>(&P)[i];
  if (i < (GB_WORDS - GB_START) / 4) reinterpret_cast<uint4*>(sync + GB_START)[i] = uint4{0u, 0u, 0u, 0u};
}

// DN_NS: k steps per wave of the down projection, 16 or 8.  A kernel for each: the other one's code, never run, pushed the
// kernel over the 64 KB of instruction cache that two compute units share (pi0_denoise +25 us).
template <bool TRACE, int DN_NS>
__global__ __launch_bounds__(PK_THREADS) void expert_loop_kernel(const ExpertLoopParams* __restrict__ params) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  using PersistCtx = PersistCtxT<false, TRACE>;
  GridBarrierT<TRACE> bar;
  const ParamsPtr<ExpertLoopParams> Pg = (ParamsPtr<ExpertLoopParams>)params;
  const ExpertLoopParams& P = fresh<ExpertLoopParams>(Pg);
  // The attention's items start at the first block without a QKV item: such a block requests its share of the prefix
  // cache when the QKV projection begins, and has it when the projection ends.
  const int att_off = P.qkv.n_tiles * 2 < (int)gridDim.x ? P.qkv.n_tiles * 2 : 0;
  const int att_block = (int)blockIdx.x >= att_off ? (int)blockIdx.x - att_off : (int)blockIdx.x + (int)gridDim.x - att_off;
  const bool idle = att_block >= P.att_items;   // no item in the attention
  const int part_die = (att_off | P.att_items | (int)gridDim.x) & 7;   // 0: consecutive idle blocks are on consecutive dies, starting with item 0's
  bar.init(P.sync, P.spin_limit, att_block >= P.att_items);
  PersistCtx cx;
  cx.arena = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(P.arena), 0, (int)P.arena_bytes, 0x00020000);
  cx.arena_base = P.arena;
  cx.bar = &bar;
  cx.bx = cx.by = cx.bz = 0;
  cx.thread = (int)threadIdx.x;
  long long* const trace = as_global(P.trace);
  const int trace_ops = P.trace_ops;
  int opi = 0;
  // timeline, 8 samples per (operation, block): 0 at the start of an operation, 1 by the barrier when the wait ends,
  // 2 after the body, 3 after arrive, 4 .. 7 by the body itself (cx.mark)
  auto op_begin = [&]() {
    if (TRACE && trace != nullptr && opi < trace_ops) {
      long long* slot = trace + ((size_t)opi * gridDim.x + blockIdx.x) * 8;
      bar.trace = slot + 1;
      if (threadIdx.x == 0) { slot[0] = (long long)wall_clock64(); slot[1] = slot[4] = slot[5] = slot[6] = slot[7] = 0; }
    } else if (TRACE) {
      bar.trace = nullptr;
    }
  };
  auto op_end = [&]() {
    if (!TRACE) {
      bar.arrive();
      return;
    }
    long long* slot = trace != nullptr && opi < trace_ops ? trace + ((size_t)opi * gridDim.x + blockIdx.x) * 8 : nullptr;
    if (slot != nullptr && threadIdx.x == 0) slot[2] = (long long)wall_clock64();
    bar.trace = nullptr;
    bar.arrive();
    if (slot != nullptr && threadIdx.x == 0) slot[3] = (long long)wall_clock64();
    opi++;
  };
  auto op_skip = [&]() {   // an operation of the timeline's numbering that nobody has an item in
    if (TRACE && trace != nullptr && opi < trace_ops && threadIdx.x < 8) trace[((size_t)opi * gridDim.x + blockIdx.x) * 8 + threadIdx.x] = 0;
    if (TRACE) opi++;
  };
  auto item = [&](int bx, int by, int bz) {
    PersistCtx c = cx;
    c.bx = bx; c.by = by; c.bz = bz;
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    c.thread = t;
    return c;
  };

  op_skip();   // C0, the state token, is part of the first embedding: an operation less in the chain

  const int emb_cols = (P.emb.a.X + 255) / 256;
  const int steps = P.steps, layers = P.layers;
  // ---- C9 of step k: final RMS -> out-projection (+bias), Euler update x <- x + dt * v; C1 of step k + 1: folded action/time
  // embedding + SiLU, suffix row 0 <- state token.  One operation: the 32 rows of x that hold a block's row are one item of
  // the out-projection, which every block computes for itself (64 KB behind the wait, as for QKV) and leaves in LDS; one block
  // of each half also writes them out.  As two operations they were 3.4 + 0.6 + 3.1 us, ten times.  k = -1: the embedding alone, and in front of it
  // C0, the state token, by the blocks that need it at once (their own columns of it).
  auto euler_embed = [&](int k) {
    const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
    const bool more = k + 1 < steps;
    ActionEmbedArgs a = F.emb.a;
    a.wfold = as_global(a.wfold);
    a.gain = as_global(a.gain);
    a.bias_k = as_global(a.bias_k) + (size_t)(k + 1) * a.X;
    GemmParams u = global(F.outp);
    char* slot = as_global(F.ring) + (size_t)(max(k, 0) * layers + layers - 1) * F.ring_stride;
    u.X = reinterpret_cast<const bf16*>(slot + F.r_yb_d);
    u.rowstat = reinterpret_cast<const float*>(slot + F.r_st_d);
    float* const written = F.emb.x_rw[(steps - 1 - k) & 1];
    const float* const read = k <= 0 ? F.noise : F.emb.x_rw[(steps - k) & 1];
    u.out_f32 = const_cast<float*>(read);
    float* const xs = reinterpret_cast<float*>(smem_raw + PK_TAIL);   // [32 rows][A]
    for_items(emb_cols * (a.chunk + 1), [&](int it) {
      const int bx = it % emb_cols, r = it / emb_cols, half = (r + 1) >> 5;   // x row r is suffix row r + 1
      const bool row = r < a.chunk, publish = bx == 0 && (r == 0 || ((r + 1) & 31) == 0);
      if (!more && !(row && publish)) return;
      const PersistCtx c = item(bx, r, 0);
      ActionEmbedWeights e;
      if (more) action_embed_load(a, c, e);
      if (k < 0 && !row) {
        state_token_body(F.stok, c);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // it is where action_embed_finish reads it
      }
      if (k >= 0 && row) {
        gemm_skinny_body<PRO_RMS, EPI_EULER, 1>(u, EulerCtx<TRACE>(item(0, 0, half).template as<true>(), read, written, xs, (32 * half - 1) * a.A, publish, more ? nullptr : as_global(F.actions)), smem_raw);
      } else {
        bar.wait();
        if (row && c.thread < a.A) xs[((r + 1) & 31) * a.A + c.thread] = cx.ld(read + (size_t)r * a.A + c.thread);
      }
      __syncthreads();
      if (more) action_embed_finish(a, c, e, [&](int j) { return xs[((r + 1) & 31) * a.A + j]; });
    });
  };
  for (int k = -1; k < steps; k++) {
    if (k >= 0) {
      op_begin();
      // ---- C2: second linear of the action/time MLP -> suffix rows 1 .. chunk --------------------------
      {
        const GemmParams t = global(fresh<ExpertLoopParams>(Pg).tout);
        for_items(t.n_tiles * 2, [&](int it) { gemm_skinny_body<PRO_NONE, EPI_RESID, 1>(t, item(it % t.n_tiles, 0, it / t.n_tiles), smem_raw); });
      }
      op_end();
      for (int l = 0; l < layers; l++) {
        op_begin();
        {  // ---- C3: RMS -> QKV, RoPE at positions P .. P + 63 -------------------------------------
          const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
          GemmParams q = global(F.qkv);
          q.W.w += (size_t)l * F.w_stride;
          char* slot = as_global(F.ring) + (size_t)(k * layers + l) * F.ring_stride;
          q.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_q);
          q.kfrag = reinterpret_cast<bf16*>(slot + F.r_k);
          q.vfrag = reinterpret_cast<bf16*>(slot + F.r_v);
          if (l == 0) {   // input: the step's embedding (two operations wrote its rows)
            q.rowstat_parts = F.parts_first;
            for_items(q.n_tiles * 2, [&](int it) { gemm_skinny_body<PRO_RMS, EPI_QKV, 1>(q, item(it % q.n_tiles, 0, it / q.n_tiles), smem_raw); });
          } else {
            q.rowstat_parts = F.parts_rest;
            q.X = reinterpret_cast<const bf16*>(slot - F.ring_stride + F.r_yb_d);
            q.rowstat = reinterpret_cast<const float*>(slot - F.ring_stride + F.r_st_d);
            for_items(q.n_tiles * 2, [&](int it) {
              gemm_skinny_body<PRO_RMS, EPI_QKV, 1>(q, item(it % q.n_tiles, 0, it / q.n_tiles).template as<true>(), smem_raw);
            });
          }
          if (att_block >= F.att_items && (int)blockIdx.x >= q.n_tiles * 2 && (F.read_ahead & 48)) {   // no item here nor in the attention
            const int tid = item(0, 0, 0).thread;
            const int idle = (int)gridDim.x - (q.n_tiles * 2 > att_off + F.att_items ? q.n_tiles * 2 : att_off + F.att_items);
            const int part = (int)gridDim.x - 1 - (int)blockIdx.x;
            unsigned fold = 0;
            if (F.read_ahead & 16) fold = read_ahead_weights<0>(as_global(F.o.W.w) + (size_t)l * F.w_stride, F.o.n_tiles, F.o.W.k_pad >> 4, part, idle, false, tid, fold);
            if (fold == 0x9e3779b9u) as_global(F.sync)[GB_SINK] = fold;
          }
          op_end();
        }
        op_begin();
        {  // ---- C4 + C5: scores, block mask, softmax, PV over [cache ; own keys] ---------------------
          const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
          AttnParams a = global(F.att);
          a.k0 += (size_t)l * F.kcache_stride;
          a.v0 += (size_t)l * F.vcache_stride;
          char* slot = as_global(F.ring) + (size_t)(k * layers + l) * F.ring_stride;
          a.q = reinterpret_cast<const bf16*>(slot + F.r_q);
          a.k1 = reinterpret_cast<const bf16*>(slot + F.r_k);
          a.v1 = reinterpret_cast<const bf16*>(slot + F.r_v);
          a.out = reinterpret_cast<bf16*>(slot + F.r_attn);
          if (a.ml_out != nullptr) a.ml_out = reinterpret_cast<float*>(slot + F.r_ml);
          const int att_gx = F.att_gx, att_gxy = F.att_gx * a.heads;
          for_items(F.att_items, [&](int it) {
            attention_suffix_body(a, item(it % att_gx, (it % att_gxy) / att_gx, it / att_gxy).template as<true>(), smem_raw + PK_TAIL);
          }, att_block);
          if (att_block >= F.att_items && (F.read_ahead & 15)) {   // no item: read ahead (constants only, no wait needed)
            const int part = att_block - F.att_items, nparts = (int)gridDim.x - F.att_items;
            const int ln = l + 1 < layers ? l + 1 : 0;
            const bool by_die = part_die == 0 && nparts % 8 == 0 && (F.read_ahead & 32) != 0;
            const int tid = item(0, 0, 0).thread;
            unsigned fold = 0;
            if (F.read_ahead & 1) fold = read_ahead_weights<2>(as_global(F.gu.W.w) + (size_t)l * F.w_stride, F.gu.n_tiles, F.gu.W.k_pad >> 4, part, nparts, by_die, tid, fold);
            if (F.read_ahead & 2) fold = read_ahead_weights<0>(as_global(F.dn.W.w) + (size_t)l * F.w_stride, F.dn.n_tiles, F.dn.W.k_pad >> 4, part, nparts, by_die, tid, fold);
            if (F.read_ahead & 4) fold = read_ahead_weights<1>(as_global(F.qkv.W.w) + (size_t)ln * F.w_stride, F.qkv.n_tiles, F.qkv.W.k_pad >> 4, part, nparts, by_die, tid, fold);
            if (F.read_ahead & 8) fold = read_ahead_weights<0>(as_global(F.o.W.w) + (size_t)ln * F.w_stride, F.o.n_tiles, F.o.W.k_pad >> 4, part, nparts, by_die, tid, fold);
            if (fold == 0x9e3779b9u) as_global(F.sync)[GB_SINK] = fold;
          }
          op_end();
          // Behind the arrival, so behind nothing that anybody waits for: the first of the two feature tiles of this block's
          // gate||up item, straight into LDS.  A gate||up block takes 128 KB of weights through its compute unit, 2.5 us between
          // two operations that are 1.8 apart; half of them ahead, by the 160 .. 192 blocks that are idle here, take its span from
          // 4.1 to 3.6 us and the hand-over in front of it from 1.5 to 0.6 (the others find the lines in their die's L2).  All of
          // them, or the attention blocks' too, cost the attention's own loads more than they give: 1 / 3 views 3.66 .. 3.85 ms /
          // 3.98 .. 4.2, none 3.71 / 4.05, half 3.63 / 3.95.  Ahead of the arrival or of the down weights it is slower.
          // Not a block that leads its die: its arrival ends with the whole die's, so the request would stand in front of its
          // out-projection weights while the others have theirs, and everybody waits for it (1 / 1+7 / 3 views 3.605 / 3.620 /
          // 3.927 ms, without 3.585 / 3.600 / 3.927; requested ahead of the arrival instead, along with those weights, +20 .. +50 us).
          if (idle && !bar.leader && (int)blockIdx.x < F.gu.n_tiles)
            skinny_stage_weights(as_global(F.gu.W.w) + (size_t)l * F.w_stride, F.gu.W.k_pad, (int)blockIdx.x % (F.gu.n_tiles / 2) * 2, lds_address(smem_raw), item(0, 0, 0).thread);
        }
        op_begin();
        {  // ---- C6: O projection + residual ------------------------------------------------------
          const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
          GemmParams o = global(F.o);
          o.W.w += (size_t)l * F.w_stride;
          o.gain = as_global(F.g_mlp0) + (size_t)l * F.gain_stride;
          char* slot = as_global(F.ring) + (size_t)(k * layers + l) * F.ring_stride;
          o.X = reinterpret_cast<const bf16*>(slot + F.r_attn);
          if (o.xsplits > 1) o.xsplit_ml = reinterpret_cast<const float*>(slot + F.r_ml);
          o.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_yb_o);
          o.stat_out = reinterpret_cast<float*>(slot + F.r_st_o);
          const int nx = o.n_tiles * 2;
          for_items(nx * F.m16, [&](int it) { gemm_skinny16_body<8>(o, item(it % nx, it / nx, 0).template as<true>(), smem_raw + PK_TAIL); });
          op_end();
        }
        op_begin();
        {  // ---- C7: RMS -> gate||up, fused gate -----------------------------------------------------
          const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
          GemmParams g = global(F.gu);
          g.W.w += (size_t)l * F.w_stride;
          char* slot = as_global(F.ring) + (size_t)(k * layers + l) * F.ring_stride;
          g.X = reinterpret_cast<const bf16*>(slot + F.r_yb_o);
          g.rowstat = reinterpret_cast<const float*>(slot + F.r_st_o);
          g.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_mid);
          // two feature tiles x one token block per item: the same sums as one tile x both token blocks, half the
          // activation bytes per block behind the wait
          const int pairs = g.n_tiles / 2;
          for_items(pairs * 2, [&](int it) {
            auto c = item(it % pairs, 0, it / pairs).template as<true>();
            c.staged = idle && !bar.leader && it == (int)blockIdx.x;
            gemm_skinny_body<PRO_RMS, EPI_GEGLU, 2>(g, c, smem_raw);
          });
          op_end();
        }
        op_begin();
        {  // ---- C8: down + residual -----------------------------------------------------------------
          const ExpertLoopParams& F = fresh<ExpertLoopParams>(Pg);
          GemmParams d = global(F.dn);
          d.W.w += (size_t)l * F.w_stride;
          d.gain = as_global(l + 1 < F.layers ? F.g_attn0 + (size_t)(l + 1) * F.gain_stride : F.g_final);
          char* slot = as_global(F.ring) + (size_t)(k * layers + l) * F.ring_stride;
          d.X = reinterpret_cast<const bf16*>(slot + F.r_mid);
          d.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_yb_d);
          d.stat_out = reinterpret_cast<float*>(slot + F.r_st_d);
          const int nx = d.n_tiles * 2;
          for_items(nx * F.m16, [&](int it) { gemm_skinny16_body<DN_NS>(d, item(it % nx, it / nx, 0).template as<true>(), smem_raw + PK_TAIL); });
          op_end();
        }
      }
    }
    op_begin();
    euler_embed(k);   // one copy of its code
    op_end();
    if (k >= 0 && k + 1 < steps) op_skip();   // the embedding was part of it
  }
}

}  // namespace

int expert_loop_smem_bytes() { return PK_TAIL + ATTN_SUFFIX_SMEM; }

namespace {
const void* const kernels[4] = {reinterpret_cast<const void*>(&expert_loop_kernel<false, 8>), reinterpret_cast<const void*>(&expert_loop_kernel<false, 16>),
                                reinterpret_cast<const void*>(&expert_loop_kernel<true, 8>), reinterpret_cast<const void*>(&expert_loop_kernel<true, 16>)};
}

hipError_t expert_loop_init_attributes() {
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, expert_loop_smem_bytes());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t expert_loop_max_blocks_per_cu(int* out) {
  *out = 1 << 30;
  for (const void* k : kernels) {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, PK_THREADS, expert_loop_smem_bytes());
    if (e != hipSuccess) return e;
    if (n < *out) *out = n;
  }
  return hipSuccess;
}

// Host-side checks of everything the kernel's indexing assumes.
hipError_t prepare_expert_loop(hipStream_t s, const ExpertLoopParams& P, ExpertLoopParams* d_params, int blocks, const CopyArgs& inputs) {
  if (inputs.n < 0 || inputs.n > 4 || P.actions == nullptr) return hipErrorInvalidValue;
  if (d_params == nullptr || (reinterpret_cast<uintptr_t>(d_params) & 15) != 0) return hipErrorInvalidValue;
  if (blocks < 1 || blocks > GB_MAX_BLOCKS || P.sync == nullptr || (reinterpret_cast<uintptr_t>(P.sync) & 15) != 0 || P.arena == nullptr || P.arena_bytes == 0 || P.spin_limit == 0)
    return hipErrorInvalidValue;
  if (P.layers < 1 || P.steps < 1 || P.x_elems < 1) return hipErrorInvalidValue;
  // every buffer that blocks exchange lies inside the arena (offsets are 32-bit)
  auto in_arena = [&](const void* p, size_t bytes) {
    const char* c = reinterpret_cast<const char*>(p);
    return p != nullptr && c >= P.arena && c + bytes <= P.arena + P.arena_bytes;
  };
  const GemmParams* gs[6] = {&P.qkv, &P.o, &P.gu, &P.dn, &P.tout, &P.outp};
  for (const GemmParams* g : gs) {
    if (g->X == nullptr || g->W.w == nullptr || g->M < 1 || g->M > 64 || g->W.k_pad % 64 != 0 || g->n_tiles * 32 != g->W.n_pad)
      return hipErrorInvalidValue;
    if (g->ldx < g->W.k_pad || g->ldx % 16 != 0 || !in_arena(g->X, (size_t)64 * g->ldx * 2)) return hipErrorInvalidValue;
    if (g->pf.blocks != 0 || g->progress != nullptr) return hipErrorInvalidValue;
  }
  const GemmParams* sk[4] = {&P.qkv, &P.gu, &P.tout, &P.outp};   // 32-feature tiles, k <= 1024 split over 8 waves
  for (const GemmParams* g : sk) {
    if (g->k_per_split != g->W.k_pad || g->W.k_pad > SK_KMAX || g->m_tiles != 1) return hipErrorInvalidValue;
  }
  if (P.read_ahead < 0 || P.read_ahead > 63) return hipErrorInvalidValue;
  if (P.gu.n_tiles % 2 != 0 || P.gu.M <= 32 || P.gu.bias != nullptr) return hipErrorInvalidValue;   // gate||up: pairs of feature tiles, two token blocks
  if (P.qkv.rowstat == nullptr || P.gu.rowstat == nullptr || P.outp.rowstat == nullptr) return hipErrorInvalidValue;
  if (P.parts_first < 1 || P.parts_first > 8 * SK_WAVES || P.parts_rest < 1 || P.parts_rest > 8 * SK_WAVES) return hipErrorInvalidValue;
  if (P.gu.rowstat_parts < 1 || P.gu.rowstat_parts > 8 * SK_WAVES || P.outp.rowstat_parts < 1 || P.outp.rowstat_parts > 8 * SK_WAVES)
    return hipErrorInvalidValue;
  if (!in_arena(P.qkv.rowstat, (size_t)8 * SK_WAVES * 64 * 8)) return hipErrorInvalidValue;
  if (P.qkv.rope == nullptr || P.qkv.out_bf16 == nullptr || P.qkv.kfrag == nullptr || P.qkv.vfrag == nullptr) return hipErrorInvalidValue;
  const GemmParams* s16[2] = {&P.o, &P.dn};   // 16 x 16 tiles over the whole k range
  for (const GemmParams* g : s16) {
    const int kc16 = g->W.k_pad >> 4;
    if ((kc16 != 128 && kc16 != 256) || g->out_f32 == nullptr || g->out_bf16 == nullptr || g->resid == nullptr || g->ldo % 4 != 0 ||
        g->ldo2 % 16 != 0 || g->stat_out == nullptr)
      return hipErrorInvalidValue;
  }
  if ((P.o.W.k_pad >> 4) != 128 || P.dn_ns != ((P.dn.W.k_pad >> 4) == 256 ? 16 : 8) || P.m16 != (P.o.M + 15) / 16) return hipErrorInvalidValue;
  if (P.o.xsplits > 1 && (P.o.xsplits > 4 || P.o.xsplit_ml == nullptr || P.o.xsplit_stride < (size_t)64 * P.o.ldx)) return hipErrorInvalidValue;
  // attention: head dim 256, at most 10 prefix chunks per share, the suffix's own 2 chunks as second segment
  const AttnParams& a = P.att;
  if (a.q == nullptr || a.k0 == nullptr || a.v0 == nullptr || a.k1 == nullptr || a.v1 == nullptr || a.out == nullptr) return hipErrorInvalidValue;
  if (a.head_dim != 256 || a.Tq != 64 || a.chunks1 != 2 || a.heads < 1 || a.chunks0 < 1 || a.valid0 < 1 || a.valid0 > a.chunks0 * 32)
    return hipErrorInvalidValue;
  const int shares = a.key_splits > 1 ? a.key_splits : 1;
  const int n0 = shares > 1 ? a.chunks_per_split : a.chunks0;
  if (!attn_suffix_ok(a, n0)) return hipErrorInvalidValue;
  if (shares > 4 || (shares > 1 && (a.ml_out == nullptr || (shares - 1) * a.chunks_per_split >= a.chunks0 ||
                                    shares * a.chunks_per_split < a.chunks0)))
    return hipErrorInvalidValue;
  const int vs = a.v_split > 1 ? a.v_split : 1;
  if (P.att_gx != 4 * vs || P.att_items != 4 * vs * a.heads * shares || a.pf.blocks != 0) return hipErrorInvalidValue;
  if (!in_arena(a.q, 2) || !in_arena(a.k1, 2) || !in_arena(a.v1, 2) || !in_arena(a.out, 2)) return hipErrorInvalidValue;
  if (P.emb.a.X % 32 != 0 || P.emb.a.gain == nullptr || P.emb.a.stat_parts == nullptr) return hipErrorInvalidValue;
  // x: 63 rows of at most 32 values, one tile of the out-projection
  if (P.emb.a.chunk != 63 || P.emb.a.A < 1 || P.emb.a.A > 32 || P.x_elems != 63 * P.emb.a.A || P.outp.n_tiles != 1 || P.outp.M != 64 || P.outp.ldo != P.emb.a.A ||
      P.outp.n_valid != P.emb.a.A || P.emb.x_rw[0] == P.emb.x_rw[1])
    return hipErrorInvalidValue;
  if (!in_arena(P.emb.x_rw[0], (size_t)P.x_elems * 4) || !in_arena(P.emb.x_rw[1], (size_t)P.x_elems * 4) || !in_arena(P.noise, (size_t)P.x_elems * 4) || !in_arena(P.stok.out, (size_t)P.stok.X * 4)) return hipErrorInvalidValue;
  if (P.stok.sd < 1 || P.stok.sd > 32) return hipErrorInvalidValue;
  if (P.ring == nullptr || P.ring_stride % 256 != 0 || !in_arena(P.ring, P.ring_stride * (size_t)P.layers * P.steps)) return hipErrorInvalidValue;
  if (P.r_mid >= P.ring_stride || P.r_attn >= P.ring_stride) return hipErrorInvalidValue;
  constexpr int pieces = (int)sizeof(ExpertLoopParams) / 4 > (GB_WORDS - GB_START) / 4 ? (int)sizeof(ExpertLoopParams) / 4 : (GB_WORDS - GB_START) / 4;
  const unsigned rows = (unsigned)ceil_div(pieces, PREP_THREADS), wide = copy_blocks(inputs);
  hipLaunchKernelGGL(expert_loop_prepare_kernel, dim3(rows > wide ? rows : wide, 1 + inputs.n), dim3(PREP_THREADS), 0, s, P, d_params, P.sync, inputs);
  return hipGetLastError();
}

hipError_t launch_expert_loop(hipStream_t s, const ExpertLoopParams* d_params, int dn_ns, bool trace, int blocks) {
  if (d_params == nullptr || blocks < 1 || blocks > GB_MAX_BLOCKS) return hipErrorInvalidValue;
  void* args[] = {&d_params};
  return hipLaunchKernel(kernels[(trace ? 2 : 0) + (dn_ns == 16 ? 1 : 0)], dim3(blocks), dim3(PK_THREADS), args, expert_loop_smem_bytes(), s);
}
