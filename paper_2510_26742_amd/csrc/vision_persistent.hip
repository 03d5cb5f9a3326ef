// The vision tower's layers as ONE persistent kernel (Section 5.2 of the paper: software barriers in place of kernel boundaries).
//
// 256 blocks, one per compute unit, walk per layer QKV, attention, O projection + residual, up + GELU, down + residual, with a
// grid barrier (exec_ctx.h) between consecutive operations.  The GEMM bodies are those of the launches with the same tiles and the same
// order of every sum, so the results agree with the launches bit for bit.
//
// What bounds it: per operation the compute unit's memory path (64 bytes per clock; (MB + NB) KiB per k16 step), then the epilogue's
// instructions, then 1.5 us from the last block's stores to everybody's first loads.  A launch spent 1.4 .. 2.0 us between the last
// block of the one before and its first, and 3.1 .. 5.0 us until its first operands were there: arguments, code and weights cold.
// Here weights wait in registers (the first stages) and in the die's L2 (the readers), code in the instruction cache.
// Per operation with what lies between it and the next, us at 1 / 2 / 3 views, launches -> here (profiles/loop_timeline_prefill_full_pi0.txt):
//   QKV        9.4 / 13.7 / 16.7 -> 6.1 / 8.9 / 11.8
//   attention  6.6 /  8.5 /  9.8 -> 4.9 / 5.2 /  7.2
//   O          6.5 /  8.0 /  8.9 -> 4.7 / 7.3 /  8.8
//   up        11.5 / 17.9 / 20.9 -> 7.3 / 11.5 / 14.1   (launches: with the statistics' launch at 2 and 3 views)
//   down      13.5 / 17.8 / 19.7 -> 11.3 / 17.2 / 18.1
// pi0_infer 6605 / 8015 / 9395 us -> 6279 / 7645 / 8953.  Without the readers' L2 lines 6600 -> 6490 at 1 view on a slower device (then
// the polls of a barrier return behind 2 us of cold weights); the die's tiles cut by tokens too, so that it reads half of the activations and
// twice the weights: -20 .. +60 us.
#include "attention_body.h"
#include "gemm_stream_body.h"
#include "persistent_common.h"
#include "vision_loop.h"

namespace {

// Per number of views: waves of a block (4 where tiles of 12 and more need 512 registers; the residual projections then take the launches'
// eight parts of k as two per wave), planes of row statistics, query tiles of an attention item (two at three views: 192 items instead of
// 384 for 256 blocks); per operation its tile, parts of k and parts per wave (gemm_stream_body), stages in
// flight (the most that do not spill), groups of the row statistics' sum (two views and more: the eight of row_sums_kernel behind an O
// projection), k steps of a part.
template <int VIEWS> struct Cfg;
template <> struct Cfg<1> {
  static constexpr int WAVES = 8, PARTS = 18, QT = 1;
  static constexpr bool READERS_ATTEND = false;
  struct Qkv { static constexpr int MB = 2, NB = 2, W = 8, V = 1, D = 9, SG = 8, NS = 9; };
  struct Resid { static constexpr int MB = 1, NB = 2, W = 8, V = 1, D = 9, SG = 1; };
  struct Up { static constexpr int MB = 2, NB = 3, W = 8, V = 1, D = 5, SG = 8, NS = 9; };
};
template <> struct Cfg<2> {
  static constexpr int WAVES = 4, PARTS = 36, QT = 1;
  static constexpr bool READERS_ATTEND = true;    // 256 items
  struct Qkv { static constexpr int MB = 2, NB = 4, W = 4, V = 1, D = 7, SG = 4, NS = 18; };
  struct Resid { static constexpr int MB = 3, NB = 1, W = 8, V = 2, D = 7, SG = 1; };
  struct Up { static constexpr int MB = 3, NB = 4, W = 4, V = 1, D = 5, SG = 8, NS = 18; };
};
template <> struct Cfg<3> {
  static constexpr int WAVES = 4, PARTS = 18, QT = 2;
  static constexpr bool READERS_ATTEND = false;
  struct Qkv { static constexpr int MB = 3, NB = 4, W = 4, V = 1, D = 7, SG = 2, NS = 18; };
  struct Resid { static constexpr int MB = 2, NB = 2, W = 8, V = 2, D = 5, SG = 1; };
  struct Up { static constexpr int MB = 4, NB = 4, W = 4, V = 1, D = 5, SG = 8, NS = 18; };
};

// Blocks 27 .. 30 of each die, which have no item but at two views in the attention (27 blocks a die are the most that the GEMMs use),
// read the weights of the operations ahead into the die's L2.  Block 31 leads the die's barrier.
constexpr int READER_RANK = 27, LEADER_RANK = 31, VISION_LOOP_BLOCKS = 8 * (LEADER_RANK + 1);

template <class O, int EPI>
constexpr int op_smem() { return stream_body_smem<O::MB, O::NB, O::W, O::SG, EPI>(); }
constexpr int max_int(int a, int b) { return a > b ? a : b; }
template <int VIEWS>
constexpr int vision_smem() {
  using C = Cfg<VIEWS>;
  return max_int(max_int(op_smem<typename C::Qkv, EPI_QKV>(), op_smem<typename C::Resid, EPI_RESID>()),
                 max_int(op_smem<typename C::Up, EPI_BF16>(), attn_view_smem(C::QT)));
}

constexpr int PREP_THREADS = 256;
static_assert(sizeof(VisionLoopParams) % 4 == 0 && (GB_WORDS - GB_START) % 4 == 0, "whole pieces");
// parameter block to device memory and barrier words to zero
__global__ __launch_bounds__(PREP_THREADS) void vision_loop_prepare_kernel(VisionLoopParams P, VisionLoopParams* dst, int turns) {
  const unsigned i = blockIdx.x * PREP_THREADS + threadIdx.x;
  if (i < sizeof(VisionLoopParams) / 4) reinterpret_cast<unsigned*>(dst)[i] = reinterpret_cast<const unsigned*>(&P)[i];
  gb_clear(P.sync, turns, i);
}

template <int VIEWS>
__global__ __launch_bounds__(64 * Cfg<VIEWS>::WAVES) __attribute__((amdgpu_waves_per_eu(Cfg<VIEWS>::WAVES / 4, Cfg<VIEWS>::WAVES / 4)))
void vision_loop_kernel(const VisionLoopParams* __restrict__ params) {
  using C = Cfg<VIEWS>;
  using Cx = PersistCtxT<true, false>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const ParamsPtr<VisionLoopParams> Pg = (ParamsPtr<VisionLoopParams>)params;
  GridBarrierT<false> bar;
  Cx cx;
  int begin, end = 0, first = 0, blocks = 0;   // begin, end: the turn's layers
  {
    const VisionLoopParams& P = fresh<VisionLoopParams>(Pg);
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
  auto moved = [](const auto* p, size_t bytes) { return reinterpret_cast<decltype(p)>(reinterpret_cast<const char*>(p) + bytes); };

  auto attention = [&](int l) {   // ---- attention inside each view
    const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
    AttnParams a = F.att;
    char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
    a.q = reinterpret_cast<const bf16*>(slot + F.r_q);
    a.k0 = reinterpret_cast<const bf16*>(slot + F.r_k);
    a.v0 = reinterpret_cast<const bf16*>(slot + F.r_v);
    a.out = reinterpret_cast<bf16*>(slot + F.r_attn);
    for_items(F.att_items, [&](int it) {
      const Cx c = item(it / a.heads, it % a.heads);
      c.wait_inputs();
      attention_view_body<C::WAVES, C::QT>(a, c, smem_raw);
    }, first, blocks);
    bar.arrive();
  };

  // the columns of the up projection's output that only pad the down projection's k
  auto clear_padding = [&](int l, int begin, int step) {
    const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
    const int kc16 = F.down.ldx >> 4, pad16 = (F.down.ldx - F.up.n_valid) >> 4;
    char* const mid = as_global(F.ring) + ((size_t)l * F.ring_stride + F.r_mid);
    for (int mb = begin; mb < F.down.M >> 5; mb += step) {
      for (int i = (int)threadIdx.x; i < pad16 * 64; i += 64 * C::WAVES)
        cx.st(reinterpret_cast<u32x4_t*>(mid + ((size_t)(mb + 1) * kc16 - pad16) * 1024u + (unsigned)i * 16u), u32x4_t{0u, 0u, 0u, 0u});
    }
  };

  const int rank = (int)blockIdx.x >> 3;
  const bool may_lead = rank == LEADER_RANK;   // (no item but at two views in the attention)
  do {
    {
      const VisionLoopParams& P = fresh<VisionLoopParams>(Pg);
      if (!bar.init_some(P.sync, P.spin_limit, may_lead, P.most_blocks, reinterpret_cast<unsigned*>(smem_raw), P.layers, first, blocks, begin, end)) return;
    }
    const bool all = blocks == VISION_LOOP_BLOCKS;   // fewer than all of the grid share the items of all and read nothing ahead
    if (all && rank >= READER_RANK && rank < LEADER_RANK) {
      unsigned fold = 0;
      for (int op = 5 * begin; op < 5 * end; op++) {   // QKV, attention, O, up, down
        const int l = op / 5, k = op - l * 5;
        if constexpr (C::READERS_ATTEND) {
          if (k == 1) {
            attention(l);
            continue;
          }
        }
        if (k == 0 && rank == READER_RANK) clear_padding(l, (int)blockIdx.x & 7, 8);
        bar.arrive();   // nobody waits for what is read here
        // QKV, attention: up.  O, up: down.  Down: the next layer's QKV and O, and where the attention leaves no time to read a part of its up
        for (int i = 0; i < (k < 4 ? 1 : l + 1 == end ? 0 : C::READERS_ATTEND ? 3 : 2); i++) {
          // part num of den of what the blocks of this die will ask for, in gemm_stream_body's order of items
          const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
          const GemmParams& g = k < 2 || i == 2 ? F.up : k < 4 ? F.down : i == 1 ? F.o : F.qkv;
          const int nb = k < 2 || i == 2 ? C::Up::NB : k < 4 || i == 1 ? C::Resid::NB : C::Qkv::NB;
          const int den = k == 4 && i < 2 ? 1 : 2, num = k == 4 ? 0 : C::READERS_ATTEND && k == 0 ? 1 : k & 1;
          int first, count;
          stream_share((int)blockIdx.x & 7, (g.n_tiles + nb - 1) / nb * g.m_tiles, first, count);
          const int t0 = first / g.m_tiles * nb, t1 = min(((first + count - 1) / g.m_tiles + 1) * nb, g.n_tiles);
          const unsigned tile16 = (unsigned)(g.W.k_pad >> 4) * 64u;
          const char* const base = reinterpret_cast<const char*>(as_global(g.W.w)) + ((size_t)(l + (k == 4)) * F.layer_stride + (size_t)t0 * tile16 * 16u);
          int t = (int)threadIdx.x;
          asm volatile("" : "+v"(t));
          constexpr int READERS = LEADER_RANK - READER_RANK;
          fold = read_ahead_part<64 * C::WAVES>((unsigned)(t1 - t0) * tile16, rank - READER_RANK + READERS * num, READERS * den, t, fold,
                                                [&](unsigned i) { return base + (size_t)i * 16u; });
        }
        bar.wait();   // the next operation begins
      }
      if (fold == 0x9e3779b9u) as_global(fresh<VisionLoopParams>(Pg).sync)[GB_SINK] = fold;
      return;
    }

    for (int l = begin; l < end; l++) {
      if (!all) clear_padding(l, first, blocks);
      {  // ---- LN -> QKV, keys and values in the attention's fragment order ----------------------------
        const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
        GemmParams q = global(F.qkv);
        char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
        q.W.w = moved(q.W.w, (size_t)l * F.layer_stride);
        q.bias = moved(q.bias, (size_t)l * F.layer_stride);
        q.colsum = moved(q.colsum, (size_t)l * F.layer_stride);
        q.rope = nullptr;   // (the launch checks it, and what follows below: no code for the other cases)
        __builtin_assume(q.bias != nullptr);
        q.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_q);
        q.kfrag = reinterpret_cast<bf16*>(slot + F.r_k);
        q.vfrag = reinterpret_cast<bf16*>(slot + F.r_v);
        if (l != 0) {
          q.X = reinterpret_cast<const bf16*>(slot - F.ring_stride + F.r_xb_d);
          q.rowstat = reinterpret_cast<const float*>(slot - F.ring_stride + F.r_st_d);
        }
        using O = typename C::Qkv;
        for_all_items<VISION_LOOP_BLOCKS>([&](int it) { gemm_stream_body<O::MB, O::NB, O::W, O::V, O::D, O::SG, C::PARTS, O::NS, PRO_LN, EPI_QKV>(q, item(it, 0), smem_raw); }, first, blocks);
        bar.arrive();
      }
      attention(l);
      using O = typename C::Resid;
      // the two residual projections: one copy of their code
      for (int second = 0; second < 2; second++) {
        {
          const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
          char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
          GemmParams o = global(second ? F.down : F.o);
          o.W.w = moved(o.W.w, (size_t)l * F.layer_stride);
          o.bias = moved(o.bias, (size_t)l * F.layer_stride);
          if (second) {
            o.X = reinterpret_cast<const bf16*>(slot + F.r_mid);
            o.gain = l + 1 < F.layers ? moved(as_global(F.g_attn0), (size_t)(l + 1) * F.gain_stride) : as_global(F.g_final);
          } else {
            o.X = reinterpret_cast<const bf16*>(slot + F.r_attn);
            o.gain = moved(as_global(F.g_mlp0), (size_t)l * F.gain_stride);
          }
          o.resid_mod = o.row_offset = 0;
          __builtin_assume(o.bias != nullptr && o.gain != nullptr && o.resid != nullptr);
          o.out_bf16 = reinterpret_cast<bf16*>(slot + (second ? F.r_xb_d : F.r_xb_o));
          o.stat_out = reinterpret_cast<float*>(slot + (second ? F.r_st_d : F.r_st_o));
          for_all_items<VISION_LOOP_BLOCKS>([&](int it) { gemm_stream_body<O::MB, O::NB, O::W, O::V, O::D, O::SG, 1, 0, PRO_NONE, EPI_RESID>(o, item(it, 0), smem_raw); }, first, blocks);
          bar.arrive();
        }
        if (second) break;
        {  // ---- LN -> up, GELU -------------------------------------------------------------------------
          const VisionLoopParams& F = fresh<VisionLoopParams>(Pg);
          char* const slot = as_global(F.ring) + (size_t)l * F.ring_stride;
          GemmParams u = global(F.up);
          u.W.w = moved(u.W.w, (size_t)l * F.layer_stride);
          u.bias = moved(u.bias, (size_t)l * F.layer_stride);
          u.colsum = moved(u.colsum, (size_t)l * F.layer_stride);
          u.act = ACT_GELU;
          __builtin_assume(u.bias != nullptr);
          u.X = reinterpret_cast<const bf16*>(slot + F.r_xb_o);
          u.rowstat = reinterpret_cast<const float*>(slot + F.r_st_o);
          u.out_bf16 = reinterpret_cast<bf16*>(slot + F.r_mid);
          using U = typename C::Up;
          for_all_items<VISION_LOOP_BLOCKS>([&](int it) { gemm_stream_body<U::MB, U::NB, U::W, U::V, U::D, U::SG, C::PARTS, U::NS, PRO_LN, EPI_BF16>(u, item(it, 0), smem_raw); }, first, blocks);
          bar.arrive();
        }
      }
    }
  } while (end < fresh<VisionLoopParams>(Pg).layers);
}

struct Kernel { const void* f; int threads, smem; };
template <int VIEWS>
Kernel kernel_of() { return Kernel{reinterpret_cast<const void*>(&vision_loop_kernel<VIEWS>), 64 * Cfg<VIEWS>::WAVES, vision_smem<VIEWS>()}; }
Kernel kernel_for(int views) { return views == 1 ? kernel_of<1>() : views == 2 ? kernel_of<2>() : kernel_of<3>(); }

template <int VIEWS>
VisionTiles tiles_of() {
  using C = Cfg<VIEWS>;
  return VisionTiles{{C::Qkv::MB, C::Qkv::NB, C::Qkv::W, C::Qkv::NS}, {C::Resid::MB, C::Resid::NB, C::Resid::W, 0}, {C::Up::MB, C::Up::NB, C::Up::W, C::Up::NS}};
}

}  // namespace

int vision_loop_planes(int views) { return views == 1 ? Cfg<1>::PARTS : views == 2 ? Cfg<2>::PARTS : Cfg<3>::PARTS; }
int vision_loop_attention_items(int views, int heads) {
  return views * 8 / (views == 1 ? Cfg<1>::QT : views == 2 ? Cfg<2>::QT : Cfg<3>::QT) * heads;
}

bool vision_loop_tiles(int views, VisionTiles* out) {
  if (views < 1 || views > VISION_LOOP_VIEWS) return false;
  *out = views == 1 ? tiles_of<1>() : views == 2 ? tiles_of<2>() : tiles_of<3>();
  return true;
}

hipError_t vision_loop_init_attributes() {
  for (int v = 1; v <= VISION_LOOP_VIEWS; v++) {
    const Kernel k = kernel_for(v);
    const hipError_t e = hipFuncSetAttribute(k.f, hipFuncAttributeMaxDynamicSharedMemorySize, k.smem);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t vision_loop_max_blocks_per_cu(int* out) {
  *out = 1 << 30;
  for (int v = 1; v <= VISION_LOOP_VIEWS; v++) {
    const Kernel k = kernel_for(v);
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k.f, k.threads, k.smem);
    if (e != hipSuccess) return e;
    if (n < *out) *out = n;
  }
  return hipSuccess;
}

// Everything that the kernel's indexing and its division of the blocks assume, so that what is not covered takes the launches
bool vision_loop_takes(int views, const VisionLoopParams& P, int blocks) {
  VisionTiles T;
  if (!vision_loop_tiles(views, &T)) return false;
  if (blocks != VISION_LOOP_BLOCKS || P.sync == nullptr || (reinterpret_cast<uintptr_t>(P.sync) & 15) != 0 || P.spin_limit == 0) return false;
  if (P.layers < 1 || P.ring == nullptr || (reinterpret_cast<uintptr_t>(P.ring) & 255) != 0 || P.ring_stride % 256 != 0 ||
      P.arena == nullptr || P.arena_bytes == 0 || P.ring < P.arena || P.ring + P.ring_stride * (size_t)P.layers > P.arena + P.arena_bytes || P.layer_stride % 16 != 0 || P.gain_stride % 16 != 0)
    return false;
  const int M = P.qkv.M;
  const GemmParams* gs[4] = {&P.qkv, &P.o, &P.up, &P.down};
  const VisionTile* ts[4] = {&T.qkv, &T.resid, &T.up, &T.resid};
  for (int i = 0; i < 4; i++) {
    const GemmParams& g = *gs[i];
    const int m_tiles = ceil_div(g.M, ts[i]->mb * 32);
    if (g.M != M || g.X == nullptr || g.W.w == nullptr || g.bias == nullptr || g.pf.blocks != 0 || g.m_tiles != m_tiles) return false;
    if (g.W.k_pad < 64 || g.W.k_pad % 64 != 0 || g.n_tiles < 1 || g.n_tiles * 32 != g.W.n_pad || g.ldx < g.W.k_pad || g.ldx % 16 != 0) return false;
    if ((size_t)g.W.k_pad * 64 > 0x7fffffffu) return false;
    if (ceil_div(g.n_tiles, ts[i]->nb) * m_tiles > 8 * READER_RANK) return false;   // one round of the blocks that run GEMM items
    if (!ts[i]->takes(g.W.k_pad)) return false;
  }
  if (M % 32 != 0 || P.qkv.colsum == nullptr || P.up.colsum == nullptr || P.qkv.rowstat == nullptr) return false;
  if (P.up.ldo != P.down.ldx || P.up.n_valid % 16 != 0 || P.up.n_valid > P.down.ldx || P.up.n_valid != P.up.W.n_pad) return false;
  const int most = vision_loop_planes(views);
  if (P.qkv.rowstat_parts != most || P.planes_rest != most || P.qkv.stat_rows < M || P.up.stat_rows < M ||
      P.planes_rest != ceil_div(P.o.n_tiles, T.resid.nb) || P.down.n_tiles != P.o.n_tiles)
    return false;
  if (P.o.ldo % 4 != 0 || P.o.ldo2 % 16 != 0 || P.down.ldo != P.o.ldo || P.down.ldo2 != P.o.ldo2 || P.o.stat_rows != P.up.stat_rows || P.down.stat_rows != P.qkv.stat_rows ||
      P.o.out_f32 == nullptr || P.o.resid != P.o.out_f32 || P.down.resid != P.o.resid || P.down.out_f32 != P.o.out_f32 ||
      reinterpret_cast<const char*>(P.o.out_f32) < P.arena || reinterpret_cast<const char*>(P.o.out_f32 + (size_t)M * P.o.ldo) > P.arena + P.arena_bytes || P.o.resid_mod != 0 || P.o.row_offset != 0 || P.down.resid_mod != 0 || P.down.row_offset != 0 || P.g_attn0 == nullptr ||
      P.g_mlp0 == nullptr || P.g_final == nullptr)
    return false;
  // no block of the QKV projection straddles the boundary of keys and values, 8 features lie in one head
  const int value_tile = (P.qkv.q_cols + P.qkv.k_cols) / 32;
  if ((P.qkv.q_cols + P.qkv.k_cols) % 32 != 0 || value_tile % T.qkv.nb != 0 || P.qkv.head_dim % 8 != 0 || P.qkv.rope != nullptr || P.up.act != ACT_GELU) return false;
  const AttnParams& a = P.att;
  if (a.view_tokens != 256 || M != views * 256 || a.Tq != M || a.chunks0 != M / 32 || a.valid0 != M || a.chunks1 != 0 || a.heads < 1 || a.head_dim <= 64 || a.head_dim > 80 ||
      a.head_dim % 4 != 0 || a.out_ld % 16 != 0 || a.out_ld < a.heads * a.head_dim || a.key_splits > 1 || a.v_split > 1 || P.att_items != vision_loop_attention_items(views, a.heads) || (views != 2 && P.att_items > READER_RANK * 8))
    return false;
  // every buffer of a slot lies inside it
  const size_t rows = (size_t)M, planes = (size_t)P.planes_rest * P.qkv.stat_rows * 8, head = (size_t)a.heads * (M / 32);
  const size_t ends[9] = {P.r_xb_o + rows * P.o.ldo2 * 2, P.r_xb_d + rows * P.o.ldo2 * 2,
                           P.r_st_o + planes, P.r_st_d + planes, P.r_q + head * 5 * 1024, P.r_k + head * 5 * 1024, P.r_v + head * 3 * 2048,
                           P.r_attn + rows * a.out_ld * 2, P.r_mid + rows * P.down.ldx * 2};
  for (size_t e : ends) {
    if (e > P.ring_stride) return false;
  }
  // ... on cache lines of its own, planes of row statistics too
  for (unsigned at : {P.r_xb_o, P.r_st_o, P.r_xb_d, P.r_st_d, P.r_q, P.r_k, P.r_v, P.r_attn, P.r_mid}) {
    if (at % 128 != 0) return false;
  }
  if (P.o.stat_rows * 8 % 128 != 0) return false;
  return true;
}

hipError_t launch_vision_loop(hipStream_t s, int views, const VisionLoopParams& P, VisionLoopParams* d_params, int blocks) {
  if (d_params == nullptr || (reinterpret_cast<uintptr_t>(d_params) & 15) != 0 || !vision_loop_takes(views, P, blocks)) return hipErrorInvalidValue;
  const int turns = P.most_blocks != 0 ? gb_turns(P.layers) : 1, pieces = std::max((int)sizeof(VisionLoopParams) / 4, (GB_WORDS - GB_START) / 4 * turns);
  hipLaunchKernelGGL(vision_loop_prepare_kernel, dim3(ceil_div(pieces, PREP_THREADS)), dim3(PREP_THREADS), 0, s, P, d_params, turns);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const Kernel k = kernel_for(views);
  void* args[] = {&d_params};
  return hipLaunchKernel(k.f, dim3(blocks), dim3(k.threads), args, k.smem, s);
}
