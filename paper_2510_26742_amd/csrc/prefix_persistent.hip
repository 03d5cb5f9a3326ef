// The prefix transformer's layers as ONE persistent kernel (Section 5.2 of the paper: software barriers in place of kernel boundaries).
//
// 256 blocks of four waves, one per compute unit, walk per layer attention, O projection + residual, gate||up with its gate, down as
// partial sums, their reduction + residual, and the next layer's QKV projection, with a grid barrier (exec_ctx.h) between consecutive
// operations.  The GEMM bodies are those of the launches with the same tiles, k ranges and order of every sum, so the results
// agree with the launches bit for bit.  The first layer's QKV projection and the last one's, which only leaves keys and values, stay launches.
//
// What bounds it: gate||up and down, which are two thirds of it, as in gemm_tile.hip (at one view what a compute unit's shared memory and
// memory path hand out, beyond the clock that the matrix cores' power leaves).  Between two operations lie 1.0 .. 1.5 us from the
// last block's end to the first block's release, where launches have a boundary, cold code and arguments, and from 257 tokens on a
// launch that adds up row statistics; the partial sums of down take another 5 .. 8 us to reach memory at two and three views.
// Per layer with what lies between it and the next operation, at 1 / 2 / 3 views, us (profiles/loop_timeline_prefill_full_pi0.txt): attention
// 6.3 / 11.7 / 16.3, O 8.4 / 12.6 / 16.5, gate||up 38.6 (gemm_rows_body) / 59.7 / 90.7, down 26.0 / 40.6 / 54.4, its reduction 6.5 / 6.2 / 7.3, QKV
// 10.3 / 14.8 / 16.0.  pi0_infer, one device, ms, launches -> here: 1 view 6.408 -> 6.259 (-> 6.18 with gemm_rows_body), 1 view + 7 tokens 6.640 -> 6.511,
// 2 views 7.837 -> 7.752, 3 views 9.252 -> 9.061; with gemm_cols_body for gate||up 515 tokens 8.25 -> 7.96, 560 tokens 8.37 -> 8.09.  Not beyond 768 tokens: 816 tokens 9.867 -> 9.843 .. 9.89 with the tiles that range
// then had (256 x 256 for gate||up in two rounds, 192 x 256 for down).  Beyond 320 tokens the kernel is larger than the instruction cache (80 .. 135 KB).
#include "attention_body.h"
#include "gemm_stream_body.h"
#include "gemm_tile_body.h"
#include "persistent_common.h"
#include "prefix_loop.h"

namespace {

constexpr int PL_THREADS = 256, PREFIX_LOOP_BLOCKS = 256;
static_assert(PREFIX_LOOP_BLOCKS == WALK_BLOCKS, "gate||up walks with as many");

// Variants by number of prefix tokens, with the full model's feed-forward: 193 .. 256, 257 .. 320, 385 .. 512, 641 .. 768 and, the last one, 513 .. 576
// (what lies between has other tiles and runs as launches; a narrower feed-forward sends fewer than 193 to the first one too, and 513 .. 576 to the
// fourth where gate||up has no use for tiles of nine blocks: gemm_cols_height).  Stream GEMMs: tile, parts of the
// k range (two per wave where there are eight), stages in flight (the most that do not spill), groups of the row statistics' sum as
// the launch has them, k16 steps of a part.
template <int MB_, int NB_, int W_, int D_, int SG_, int NS_>
struct StreamOp { static constexpr int MB = MB_, NB = NB_, W = W_, V = W_ / 4, D = D_, SG = SG_, NS = NS_; };
template <int MT_, int NT_>
struct TileOp { static constexpr int MT = MT_, NT = NT_; };
template <class QKV, class O, class GU, class DN, bool WALK_, int ATT_CM_, int O_GROUPS_, bool ROWS_ = false, int GU_HEIGHT_ = 0>
struct Variant {
  using Qkv = QKV;
  using Out = O;
  using Gu = GU;
  using Dn = DN;
  static constexpr bool WALK = WALK_, ROWS = ROWS_;   // ROWS: gemm_rows_body for gate||up
  static constexpr int GU_HEIGHT = GU_HEIGHT_;        // not 0: gemm_cols_body for gate||up
  static constexpr int ATT_CM = ATT_CM_, O_GROUPS = O_GROUPS_;   // ATT_CM: 0: 16 query rows over at most 10 chunks, else 32 over at most 4 ATT_CM
};
template <int I> struct Variants;
template <> struct Variants<0> { using T = Variant<StreamOp<2, 2, 8, 8, 8, 16>, StreamOp<1, 2, 8, 9, 1, 16>, TileOp<4, 2>, TileOp<2, 2>, false, 0, 1, true>; };
template <> struct Variants<1> { using T = Variant<StreamOp<2, 2, 8, 8, 8, 16>, StreamOp<3, 1, 8, 8, 1, 16>, TileOp<5, 2>, TileOp<3, 2>, false, 0, 8>; };
template <> struct Variants<2> { using T = Variant<StreamOp<2, 3, 8, 5, 8, 16>, StreamOp<2, 2, 8, 6, 1, 16>, TileOp<4, 4>, TileOp<4, 2>, false, 4, 8>; };
template <> struct Variants<3> { using T = Variant<StreamOp<2, 3, 8, 5, 8, 16>, StreamOp<3, 2, 8, 5, 1, 16>, TileOp<3, 4>, TileOp<5, 2>, false, 5, 8>; };
template <> struct Variants<4> { using T = Variant<StreamOp<2, 4, 4, 8, 4, 32>, StreamOp<3, 2, 8, 5, 1, 16>, TileOp<3, 4>, TileOp<3, 4>, true, 6, 8>; };
template <> struct Variants<5> { using T = Variant<StreamOp<2, 3, 8, 5, 8, 16>, StreamOp<3, 2, 8, 5, 1, 16>, TileOp<0, 0>, TileOp<5, 2>, false, 5, 8, false, 9>; };
constexpr int VARIANTS = 6;
constexpr int ATT_EARLY = 5, ATT_RING = 12;

constexpr int PREP_THREADS = 256;
static_assert(sizeof(PrefixLoopParams) % 4 == 0 && (GB_WORDS - GB_START) % 4 == 0, "whole pieces");
// parameter block to device memory and barrier words to zero
__global__ __launch_bounds__(PREP_THREADS) void prefix_loop_prepare_kernel(PrefixLoopParams P, PrefixLoopParams* dst, int turns) {
  const unsigned i = blockIdx.x * PREP_THREADS + threadIdx.x;
  if (i < sizeof(PrefixLoopParams) / 4) reinterpret_cast<unsigned*>(dst)[i] = reinterpret_cast<const unsigned*>(&P)[i];
  gb_clear(P.sync, turns, i);
}

template <int VARIANT>
__global__ __launch_bounds__(PL_THREADS) __attribute__((amdgpu_waves_per_eu(1, 1))) void prefix_loop_kernel(const PrefixLoopParams* __restrict__ params) {
  using C = typename Variants<VARIANT>::T;
  constexpr bool LEAN = C::GU_HEIGHT != 0;   // (gate||up takes every register)
  using Cx = PersistCtxT<true, false, LEAN>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const ParamsPtr<PrefixLoopParams> Pg = (ParamsPtr<PrefixLoopParams>)params;
  GridBarrierT<false, LEAN> bar;
  Cx cx;
  int layers, begin, end = 0, first = 0, blocks = 0;   // begin, end: the turn's layers
  {
    const PrefixLoopParams& P = fresh<PrefixLoopParams>(Pg);
    cx.arena = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(P.arena), 0, (int)P.arena_bytes, 0x00020000);
    cx.arena_base = P.arena;
  }
  cx.bar = &bar;
  cx.by = cx.bz = 0;
  auto item = [&](int bx, int by) {
    Cx c = cx;
    c.bx = bx;
    c.by = by;
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    c.thread = t;
    return c;
  };
  auto each = [&](int n_items, auto&& f) { for_items(n_items, f, first, blocks); };   // this block's items
  auto each_block = [&](auto&& f) { for_all_items<PREFIX_LOOP_BLOCKS>(f, first, blocks); };
  auto moved = [](const auto* p, size_t bytes) { return reinterpret_cast<decltype(p)>(reinterpret_cast<const char*>(p) + bytes); };

  const bool may_lead = (int)(blockIdx.x >> 3) == 31;
  do {
    {
      const PrefixLoopParams& P = fresh<PrefixLoopParams>(Pg);
      layers = P.layers;
      if (!bar.init_some(P.sync, P.spin_limit, may_lead, P.most_blocks, reinterpret_cast<unsigned*>(smem_raw), layers, first, blocks, begin, end)) return;
    }
    for (int l = begin; l < end; l++) {
      {  // ---- attention, whole prefix visible ---------------------------------------------------------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        AttnParams a = F.att;
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        a.q = reinterpret_cast<const bf16*>(slot + F.r_q);
        a.k0 = moved(as_global(a.k0), (size_t)l * F.kcache_stride);
        a.v0 = moved(as_global(a.v0), (size_t)l * F.vcache_stride);
        a.out = reinterpret_cast<bf16*>(slot + F.r_attn);
        const int tiles = F.att_tiles;
        each(tiles * a.heads, [&](int it) {
          const Cx c = item(it % tiles, it / tiles);
          c.wait_inputs();
          if constexpr (C::ATT_CM == 0) attention_prefix16_body(a, c, smem_raw);
          else attention_prefix32_body<C::ATT_CM, ATT_EARLY, ATT_RING>(a, c, smem_raw);
        });
        bar.arrive();
      }
      {  // ---- O projection + residual -----------------------------------------------------------------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        GemmParams o = global(F.o);
        o.W.w = moved(o.W.w, (size_t)l * F.layer_stride);
        o.gain = moved(o.gain, (size_t)l * F.gain_stride);
        o.X = reinterpret_cast<const bf16*>(slot + F.r_attn);
        o.bias = nullptr;
        o.resid_mod = o.row_offset = 0;
        __builtin_assume(o.gain != nullptr && o.resid != nullptr);
        o.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_xb_o);
        o.stat_out = reinterpret_cast<float*>(slot + F.r_st_o);
        using O = typename C::Out;
        each_block([&](int it) { gemm_stream_body<O::MB, O::NB, O::W, O::V, O::D, O::SG, 1, O::NS, PRO_NONE, EPI_RESID>(o, item(it, 0), smem_raw); });
        bar.arrive();
      }
      {  // ---- RMS -> gate||up, fused gate -------------------------------------------------------------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        GemmParams g = global(F.gu);
        g.W.w = moved(g.W.w, (size_t)l * F.layer_stride);
        g.X = reinterpret_cast<const bf16*>(slot + F.r_xb_o);
        g.rowstat = reinterpret_cast<const float*>(slot + F.r_st_o);
        g.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_mid);
        using G = typename C::Gu;
        if constexpr (C::ROWS) {
          static_assert(G::MT == 4 && G::NT == 2 && C::O_GROUPS == 1, "the same tile and order of the planes");
          each(F.gu_blocks, [&](int it) { gemm_rows_body(g, item(it, 0), smem_raw); });
        } else if constexpr (C::GU_HEIGHT != 0) {
          each(F.gu_blocks, [&](int it) { gemm_cols_item<C::GU_HEIGHT, C::O_GROUPS, EPI_GEGLU>(g, item(it, 0), smem_raw); });
        } else if constexpr (C::WALK) {
          each_block([&](int it) { gemm_lds_body<G::MT, G::NT, C::O_GROUPS, PRO_RMS, EPI_GEGLU, true>(g, item(it, 0), smem_raw); });
        } else {
          each(F.gu_blocks, [&](int it) { gemm_lds_body<G::MT, G::NT, C::O_GROUPS, PRO_RMS, EPI_GEGLU, false>(g, item(it, 0), smem_raw); });
        }
        bar.arrive();
      }
      {  // ---- down, partial sums of each k range ------------------------------------------------------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        GemmParams d = global(F.dn);
        d.W.w = moved(d.W.w, (size_t)l * F.layer_stride);
        d.X = reinterpret_cast<const bf16*>(as_global(F.ring) + (size_t)l * F.ring_stride + F.r_mid);
        using G = typename C::Dn;
        const int gx = F.dn_blocks, z = F.red.Z;
        const bool ranges = d.range_per_die != 0;
        each(gx * z, [&](int it) {
          gemm_lds_body<G::MT, G::NT, 1, PRO_NONE, EPI_PARTIAL, false>(d, ranges ? item(it >> 3, it & 7) : item(it % gx, it / gx), smem_raw);
        });
        bar.arrive();
      }
      {  // ---- their sum + residual --------------------------------------------------------------------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        ReduceParams r = F.red;
        r.part = as_global(r.part);
        r.resid = as_global(r.resid);
        r.out_f32 = as_global(r.out_f32);
        r.bias = nullptr;
        r.resid_mod = 0;
        r.gain = moved(as_global(r.gain), (size_t)l * F.gain_stride);
        __builtin_assume(r.gain != nullptr && r.resid != nullptr);
        r.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_xb_d);
        r.stat_out = reinterpret_cast<float*>(slot + F.r_st_d);
        const int rows = (r.M + 7) >> 3;
        each(rows * PREFIX_QKV_PLANES, [&](int it) {
          tile_reduce_body<PL_THREADS>(r, item(it % rows, it / rows), reinterpret_cast<float2 (*)[8]>(smem_raw));
        });
        bar.arrive();
      }
      if (l + 1 < layers) {  // ---- RMS -> next layer's QKV, RoPE, keys and values into the cache ---------
        const PrefixLoopParams& F = fresh<PrefixLoopParams>(Pg);
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        GemmParams q = global(F.qkv);
        q.W.w = moved(q.W.w, (size_t)(l + 1) * F.layer_stride);
        q.bias = nullptr;
        __builtin_assume(q.rope != nullptr);
        q.X = reinterpret_cast<const bf16*>(slot + F.r_xb_d);
        q.rowstat = reinterpret_cast<const float*>(slot + F.r_st_d);
        q.out_bf16 = reinterpret_cast<bf16*>(slot + F.ring_stride + F.r_q);
        q.kfrag = reinterpret_cast<bf16*>(reinterpret_cast<char*>(q.kfrag) + (size_t)(l + 1) * F.kcache_stride);
        q.vfrag = reinterpret_cast<bf16*>(reinterpret_cast<char*>(q.vfrag) + (size_t)(l + 1) * F.vcache_stride);
        using O = typename C::Qkv;
        each_block([&](int it) { gemm_stream_body<O::MB, O::NB, O::W, O::V, O::D, O::SG, PREFIX_QKV_PLANES, O::NS, PRO_RMS, EPI_QKV, true>(q, item(it, 0), smem_raw); });
        bar.arrive();
      }
    }
  } while (end < layers);
}

constexpr int max_int(int a, int b) { return a > b ? a : b; }
template <class C>
constexpr int smem_of() {
  using Q = typename C::Qkv;
  using O = typename C::Out;
  constexpr int att = C::ATT_CM == 0 ? ATTN_PREFIX16_SMEM : attn_prefix32_smem(C::ATT_CM == 0 ? 1 : C::ATT_CM);
  return max_int(max_int(stream_body_smem<Q::MB, Q::NB, Q::W, Q::SG, EPI_QKV>(), stream_body_smem<O::MB, O::NB, O::W, O::SG, EPI_RESID>()),
                 max_int(att, LT_SMEM));
}
struct Kernel {
  const void* f;
  int smem;
  PrefixTiles tiles;
};
template <int I>
Kernel kernel_of() {
  using C = typename Variants<I>::T;
  using Q = typename C::Qkv;
  using O = typename C::Out;
  return Kernel{reinterpret_cast<const void*>(&prefix_loop_kernel<I>), smem_of<C>(),
                PrefixTiles{{Q::MB, Q::NB, Q::W, Q::NS}, {O::MB, O::NB, O::W, O::NS}, {C::Gu::MT, C::Gu::NT}, {C::Dn::MT, C::Dn::NT}, C::GU_HEIGHT, C::WALK,
                            C::ATT_CM == 0 ? 16 : 32, C::ATT_CM == 0 ? ATT_SHARE : 4 * C::ATT_CM, C::O_GROUPS, C::ROWS}};
}
Kernel kernel_for(int v) {
  switch (v) {
    case 0: return kernel_of<0>();
    case 1: return kernel_of<1>();
    case 2: return kernel_of<2>();
    case 3: return kernel_of<3>();
    case 4: return kernel_of<4>();
    default: return kernel_of<5>();
  }
}

}  // namespace

int prefix_loop_variants() { return VARIANTS; }
PrefixTiles prefix_loop_tiles(int variant) { return kernel_for(variant).tiles; }

hipError_t prefix_loop_init_attributes() {
  for (int v = 0; v < VARIANTS; v++) {
    const Kernel k = kernel_for(v);
    const hipError_t e = hipFuncSetAttribute(k.f, hipFuncAttributeMaxDynamicSharedMemorySize, k.smem);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t prefix_loop_max_blocks_per_cu(int* out) {
  *out = 1 << 30;
  for (int v = 0; v < VARIANTS; v++) {
    const Kernel k = kernel_for(v);
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k.f, PL_THREADS, k.smem);
    if (e != hipSuccess) return e;
    if (n < *out) *out = n;
  }
  return hipSuccess;
}

// Everything that the kernel's indexing assumes, so that what is not covered takes the launches
bool prefix_loop_takes(int variant, const PrefixLoopParams& P, int blocks) {
  if (variant < 0 || variant >= VARIANTS) return false;
  const PrefixTiles T = prefix_loop_tiles(variant);
  if (blocks != PREFIX_LOOP_BLOCKS || P.sync == nullptr || (reinterpret_cast<uintptr_t>(P.sync) & 15) != 0 || P.spin_limit == 0)
    return false;
  if (P.layers < 1 || P.ring == nullptr || (reinterpret_cast<uintptr_t>(P.ring) & 255) != 0 || P.ring_stride % 256 != 0 || P.arena == nullptr || P.arena_bytes == 0 ||
      P.layer_stride % 16 != 0 || P.gain_stride % 16 != 0 || P.kcache_stride % 16 != 0 || P.vcache_stride % 16 != 0)
    return false;
  auto in_arena = [&](const void* p, size_t bytes) {
    const char* c = reinterpret_cast<const char*>(p);
    return p != nullptr && c >= P.arena && c + bytes <= P.arena + P.arena_bytes;
  };
  if (!in_arena(P.ring, P.ring_stride * (size_t)P.layers)) return false;
  const int M = P.qkv.M, chunks = ceil_div(M, 32);
  const GemmParams* gs[4] = {&P.qkv, &P.o, &P.gu, &P.dn};
  for (const GemmParams* g : gs) {
    if (g->M != M || M < 1 || g->W.w == nullptr || g->bias != nullptr || g->pf.blocks != 0) return false;
    if (g->W.k_pad < 64 || g->W.k_pad % 64 != 0 || g->n_tiles < 1 || g->n_tiles * 32 != g->W.n_pad || g->ldx < g->W.k_pad || g->ldx % 16 != 0) return false;
    if ((size_t)g->W.k_pad * 64 > 0x7fffffffu) return false;
  }
  // stream GEMMs: one round of blocks, parts of the k range as built
  if (P.qkv.m_tiles != ceil_div(M, T.qkv.mb * 32) || ceil_div(P.qkv.n_tiles, T.qkv.nb) * P.qkv.m_tiles > blocks || P.qkv.W.k_pad != 16 * T.qkv.steps * T.qkv.parts) return false;
  if (P.o.m_tiles != ceil_div(M, T.o.mb * 32) || ceil_div(P.o.n_tiles, T.o.nb) * P.o.m_tiles > blocks || P.o.W.k_pad != 16 * T.o.steps * T.o.parts) return false;
  const int value_tile = (P.qkv.q_cols + P.qkv.k_cols) / 32;
  if (P.qkv.rope == nullptr || P.qkv.head_dim != 256 || P.qkv.dqk_pad != 256 || P.qkv.nvb != 8 || P.qkv.kv_heads != 1 || P.qkv.k_cols != 256 || P.qkv.q_cols % 256 != 0 ||
      P.qkv.n_tiles != value_tile + 8 || value_tile % T.qkv.nb != 0 || P.qkv.kv_chunks < chunks || P.qkv.q_mbs != chunks || P.qkv.pos0 != 0)
    return false;
  const size_t cache = (size_t)chunks * 16384;   // of a layer, in use
  if (P.kcache_stride < cache || P.vcache_stride < cache || !in_arena(P.qkv.kfrag, P.kcache_stride * (size_t)(P.layers - 1) + cache) ||
      !in_arena(P.qkv.vfrag, P.vcache_stride * (size_t)(P.layers - 1) + cache))
    return false;
  const int E = P.o.W.n_pad;
  if (E != 256 * PREFIX_QKV_PLANES || P.qkv.W.k_pad != E || P.gu.W.k_pad != E || P.dn.W.n_pad != E || P.qkv.ldx != E || P.gu.ldx != E || P.qkv.k_true != E || P.gu.k_true != E) return false;
  if (P.qkv.stat_rows < M || P.qkv.stat_rows % 2 != 0 || P.o.stat_rows != P.qkv.stat_rows || P.gu.stat_rows != P.qkv.stat_rows || P.red.stat_rows != P.qkv.stat_rows) return false;
  if (P.gu.rowstat_parts != ceil_div(P.o.n_tiles, T.o.nb) || P.gu.rowstat_parts < 2) return false;
  if (P.o.ldo != E || P.o.ldo2 != E || P.o.n_valid != E || P.o.gain == nullptr || P.o.resid != P.o.out_f32 || !in_arena(P.o.out_f32, (size_t)M * E * 4)) return false;
  // gate||up and down
  const int gu_total = ceil_div(P.gu.n_tiles, T.gu_tile_features()) * P.gu.m_tiles, dn_total = ceil_div(P.dn.n_tiles, 2 * T.dn.nt) * P.dn.m_tiles;
  if (P.gu.m_tiles != ceil_div(M, T.gu_tile_rows()) || P.dn.m_tiles != ceil_div(M, T.dn.mt * 64) || P.gu_blocks != 8 * ceil_div(gu_total, 8) || P.dn_blocks != (P.dn.range_per_die ? dn_total : 8 * ceil_div(dn_total, 8))) return false;
  if (P.gu.W.k_pad % 128 != 0 || P.gu.k_per_split != P.gu.W.k_pad || P.dn.k_per_split % 128 != 0 || P.dn.W.k_pad % 128 != 0 || P.red.Z < 1 || P.dn.range_per_die != (P.red.Z == LDS_DIES) ||
      P.dn.k_per_split % lds_tile_group(T.dn.mt, T.dn.nt) != 0 || (P.dn.W.k_pad - P.dn.k_per_split * (P.red.Z - 1)) % lds_tile_group(T.dn.mt, T.dn.nt) != 0 ||
      (long)P.dn.k_per_split * P.red.Z < P.dn.W.k_pad || (long)P.dn.k_per_split * (P.red.Z - 1) >= P.dn.W.k_pad)
    return false;
  if (T.gu_height != 0 && P.gu.W.k_pad % (16 * COLS_GROUP) != 0) return false;
  if (T.gu_rows && (M > 256 || P.gu.W.k_pad % (16 * ROWS_GROUP) != 0 || P.gu.rowstat_parts > ROWS_PARTS)) return false;
  if (T.walk && (WALK_BLOCKS / 8 % P.gu.m_tiles != 0)) return false;   // a block's tiles are in the same rows
  if (P.gu.ldo * 2 != P.gu.W.n_pad || P.dn.ldx != P.gu.ldo || P.dn.W.k_pad != P.gu.ldo) return false;
  if (P.red.M != M || P.red.N != E || P.red.ldp != E || P.red.ldo != E || P.red.ldo2 != E || P.red.part != P.dn.out_f32 || P.red.out_f32 != P.o.out_f32 ||
      P.red.resid != P.o.out_f32 || P.red.bias != nullptr || P.red.gain == nullptr || P.red.out8 != nullptr || !in_arena(P.red.part, (size_t)P.red.Z * chunks * 32 * E * 4))
    return false;
  const AttnParams& a = P.att;
  if (a.Tq != M || a.chunks0 != chunks || a.valid0 != M || a.chunks1 != 0 || a.heads * 256 != P.qkv.q_cols || a.head_dim != 256 || a.view_tokens != 0 || a.key_splits > 1 ||
      a.v_split > 1 || a.kv_head_stride0 != 0 || a.v_head_stride0 != 0 || a.q_head_stride != chunks * 8192 || a.out_ld != a.heads * 256 || P.o.W.k_pad != a.out_ld || P.o.ldx != a.out_ld ||
      a.k0 != P.qkv.kfrag || a.v0 != P.qkv.vfrag || chunks > T.att_chunks || chunks > PREFIX_LOOP_CHUNKS || P.att_tiles != ceil_div(M, T.att_rows) || P.att_tiles * a.heads > blocks)
    return false;
  // every buffer of a slot lies inside it
  const size_t rows = (size_t)chunks * 32;
  const size_t ends[7] = {P.r_xb_o + rows * E * 2, P.r_xb_d + rows * E * 2, P.r_st_o + (size_t)P.gu.rowstat_parts * P.o.stat_rows * 8,
                          P.r_st_d + (size_t)PREFIX_QKV_PLANES * P.o.stat_rows * 8, P.r_q + rows * a.out_ld * 2, P.r_attn + rows * a.out_ld * 2, P.r_mid + rows * P.gu.ldo * 2};
  for (size_t e : ends) {
    if (e > P.ring_stride) return false;
  }
  // ... on cache lines of its own, planes of row statistics too
  for (unsigned at : {P.r_xb_o, P.r_st_o, P.r_xb_d, P.r_st_d, P.r_q, P.r_attn, P.r_mid}) {
    if (at % 128 != 0) return false;
  }
  if (P.o.stat_rows * 8 % 128 != 0) return false;
  return true;
}

hipError_t launch_prefix_loop(hipStream_t s, int variant, const PrefixLoopParams& P, PrefixLoopParams* d_params, int blocks) {
  if (d_params == nullptr || (reinterpret_cast<uintptr_t>(d_params) & 15) != 0 || !prefix_loop_takes(variant, P, blocks)) return hipErrorInvalidValue;
  const int turns = P.most_blocks != 0 ? gb_turns(P.layers) : 1, pieces = std::max((int)sizeof(PrefixLoopParams) / 4, (GB_WORDS - GB_START) / 4 * turns);
  hipLaunchKernelGGL(prefix_loop_prepare_kernel, dim3(ceil_div(pieces, PREP_THREADS)), dim3(PREP_THREADS), 0, s, P, d_params, turns);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const Kernel k = kernel_for(variant);
  void* args[] = {&d_params};
  return hipLaunchKernel(k.f, dim3(blocks), dim3(PL_THREADS), args, k.smem, s);
}
