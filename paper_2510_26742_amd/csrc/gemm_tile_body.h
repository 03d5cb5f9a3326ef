// Body of the prefix's large bf16 GEMMs (gemm_tile.hip says what they are), for an execution context (exec_ctx.h): the launches of
// gemm_tile.hip, and the prefix as one persistent kernel (prefix_persistent.hip), where the weights of the first stages are requested
// ahead of the wait for the inputs.
#pragma once
#include "pi0_internal.h"

#include <utility>

#include "gemm_common.h"

template <int V>
struct Int {
  static constexpr int value = V;
};
template <class F, int... I>
__device__ __forceinline__ void for_each_in(F&& f, std::integer_sequence<int, I...>) {
  (f(Int<I>{}), ...);
}
// f(Int<0>), f(Int<1>), ...: an unrolled loop whose index is a constant for assembly operands
template <int N, class F>
__device__ __forceinline__ void for_each(F&& f) {
  for_each_in(f, std::make_integer_sequence<int, N>{});
}

// Zero, which the compiler does not know as such.  A constant it writes once for the loop and once for the last turn without one (there are as many
// writes as registers, behind the wait for the first stage), keeps the accumulators of the two apart and moves all of them from the one to the other:
// 500 instructions of a 256 x 256 tile, and a quarter of its code.  OPAQUE = false: the constant, where the registers do not suffice otherwise (the
// persistent kernel with nine blocks of rows).  Constant -> this, in turn, us, and what the runs of one side differ by: pi0_infer at 2 views 7727 -> 7678 (0.3 %),
// 3 views 9038 -> 9001 (0.0 %), 3 views + 48 tokens 9478 -> 9429 (0.1 %), two-stream frame at 2 views 7146 -> 7120 (0.1 %); 1 view 6237 -> 6230 (0.5 %, nothing).
template <bool OPAQUE = true>
__device__ __forceinline__ void zero_accumulator(f32x16& a) {
#pragma unroll
  for (int r = 0; r < 16; r++) a[r] = 0.f;
  if (OPAQUE) asm volatile("" : "+a"(a));
}

constexpr int lds_tile_stages(int MT, int NT) { return MT * NT <= 6 ? 8 : 4; }   // stages in LDS
constexpr int WALK_BLOCKS = 256;               // that walk (WALK), a compute unit's each
constexpr int LT_KC = 2;                       // k16 steps of a stage
constexpr int lds_tile_group(int MT, int NT) { return 16 * LT_KC * lds_tile_stages(MT, NT); }   // of k, of a turn of the loop: k ranges are multiples of it

constexpr int lds_tile_fragments(int MT, int NT) { return 2 * (MT + NT) * LT_KC; }   // of a stage
constexpr int LT_SMEM = 160 * 1024;             // of a compute unit, which a block has to itself
constexpr int lds_tile_stat_bytes(int MT) { return (2 * MT * 32 * 8 + 1023) / 1024 * 1024; }   // row statistics, whole requests of 1 KiB
constexpr int lds_tile_smem(int MT, int NT) { return (MT * NT <= 6 ? 0 : lds_tile_stat_bytes(MT)) + lds_tile_stages(MT, NT) * lds_tile_fragments(MT, NT) * 1024; }
// planes of partial row statistics that fit behind the three stages requested first (the last request may be half empty)
constexpr int lds_tile_planes(int MT, int NT) {
  return (LT_SMEM - lds_tile_stat_bytes(MT) - (lds_tile_stages(MT, NT) - 1) * lds_tile_fragments(MT, NT) * 1024 - 1024) / (2 * MT * 32 * 8);
}
// tiles of a launch as in gemm_stream.hip: consecutive block ids on different dies, a die takes a contiguous eighth
__device__ __forceinline__ void lds_tile_share(int die, int tiles, int& first, int& count) {
  first = die * (tiles >> 3) + min(die, tiles & 7);
  count = (tiles >> 3) + (die < (tiles & 7) ? 1 : 0);
}

// SG: groups in which planes of row statistics are added (group g: planes g, g + SG, ...; then the groups in order).
// cx.bx, cx.by: the tile, in the order of stream_share unless p.range_per_die, and the k range.
template <int MT, int NT, int SG, int PRO, int EPI, bool WALK, class Cx>
__device__ __forceinline__ void gemm_lds_body(const GemmParams& p, const Cx& cx, unsigned char* smem) {
  constexpr int W = 4, LT_STAGES = lds_tile_stages(MT, NT), LT_GROUP = LT_STAGES * LT_KC;
  constexpr int XB = 2 * MT, WB = 2 * NT;        // 32-row blocks of the two operands
  constexpr int NF = lds_tile_fragments(MT, NT);
  constexpr int L = NF / W;                      // fragments a wave requests per stage
  static_assert(NF % W == 0, "even shares");
  constexpr int ROWS = XB * 32;
  // shared memory: row statistics, then [stage][fragment][1 KiB]; in the persistent kernel the stages first
  float2* sstat = reinterpret_cast<float2*>(smem + (Cx::kPersistent ? LT_STAGES * NF * 1024 : 0));
  unsigned char* const smem_raw = smem + (Cx::kPersistent || PRO == PRO_NONE ? 0 : (WALK ? 2 : 1) * lds_tile_stat_bytes(MT));

  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = w & 1, wn = w >> 1;
  const int lq = lane & 31;
  const int lh = lane >> 5;

  // tiles as in gemm_stream.hip: consecutive ids on different dies, a die takes a contiguous eighth, token tiles fastest
  const int total = (p.n_tiles + WB - 1) / WB * p.m_tiles;
  // ... or in order, where a die has a k range to itself
  const bool ranges = EPI == EPI_PARTIAL && p.range_per_die != 0;
  const int die = cx.bx & 7, die_rank = ranges ? cx.bx : cx.bx >> 3;
  const int first = ranges ? 0 : die * (total >> 3) + min(die, total & 7), of_die = ranges ? total : (total >> 3) + (die < (total & 7) ? 1 : 0);
  if (die_rank >= of_die) return;
  const int nb = (first + die_rank) / p.m_tiles;
  const int mt = (first + die_rank) - nb * p.m_tiles;
  const int m0 = mt * ROWS;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4, XKC16 = p.ldx >> 4;
  const int kbeg = cx.by * (p.k_per_split >> 4);
  const int groups = (min(kbeg + (p.k_per_split >> 4), KC16) - kbeg) / LT_GROUP;

  // The wave's fragment i of a stage is fragment w + 4 i of the block's: operand block f / 2 (tokens first), k16 step f % 2;
  // blocks beyond the operands repeat the last one and are not stored
  const char* src[L];
  auto set_sources = [&](int nb, int m0) {
#pragma unroll
    for (int i = 0; i < L; i++) {
      const int f = w + W * i, b = f / LT_KC, k = f % LT_KC;
      const char* base = b < XB ? reinterpret_cast<const char*>(p.X) + (size_t)min((m0 >> 5) + b, mb_last) * XKC16 * 1024
                                : reinterpret_cast<const char*>(p.W.w) + (size_t)min(nb * WB + (b - XB), p.n_tiles - 1) * KC16 * 1024;
      src[i] = base + (size_t)(kbeg + k) * 1024;
    }
  };
  set_sources(nb, m0);
  const unsigned lds0 = lds_address(smem_raw) + (unsigned)w * 1024u;
  // Where a round of blocks reads the whole weight matrix (one token tile), all blocks would ask for the same k of their own
  // weight rows, a power of two apart: each starts elsewhere in its range and goes round (prefill at 256 / 263 tokens
  // 3.133 / 3.348 -> 3.099 / 3.338 ms).  With more token tiles the blocks that share weights set the pace, and 816 tokens are
  // 25 us slower that way
  int turn = p.m_tiles == 1 || (EPI == EPI_PARTIAL && p.M <= 320) ? (int)((unsigned)nb % (unsigned)groups) : 0;
  const unsigned vfirst = (unsigned)lane * 16u + 4096u;
  unsigned voff = vfirst + (unsigned)turn * (LT_GROUP * 1024u);      // of the current group: stages 0 .. 3 are at 2048 q - 4096, a 13-bit constant
  // request the wave's fragment I of stage Q of the group at v; the constant counts towards both addresses
  auto issue = [&](auto Q, auto I, unsigned v) {
    constexpr int q = decltype(Q)::value, i = decltype(I)::value;
    const unsigned l0 = lds0;
    const char* const s = src[i];
    constexpr int off = q % 4 * 2048 - 4096;
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::"s"(l0), "v"(v + (unsigned)(q / 4) * 8192u), "s"(s),
                 "n"((q * NF + W * i) * 1024 - off), "n"(off)
                 : "memory", "scc");
  };
  // Row statistics: whole-row sums, or partial sums in planes, one per block column of the producer, which the thread of the
  // row adds up.  They go to LDS like the operands and in front of them: loaded into registers behind the first stages, as
  // they were, they kept every block until all of those stages had come, a burst of 18 - 25 MB from memory (start of a block
  // to its first product 4.3 us at 256 and 512 tokens, as against 1.9 without statistics;
  // prefill at 512 / 768 / 816 tokens 4.432 / 5.822 / 6.350 -> 4.414 / 5.790 / 6.310 ms).
  constexpr int PAIRS = ROWS / 2, RR = (ROWS + 64 * W - 1) / (64 * W);
  constexpr int PLANES = lds_tile_planes(MT, NT);
  static_assert(PRO == PRO_NONE || PLANES >= 1, "room for a plane");
  float2 sum[RR] = {};
  const int parts = PRO != PRO_NONE ? p.rowstat_parts : 0;
  unsigned char* const planes = smem_raw + (LT_STAGES - 1) * NF * 1024;
  auto request_planes = [&](int m0, int first_plane, int n, unsigned char* to) {   // 16 bytes per lane: two rows
    const int last = (p.M - 1) & ~1;
    for (int q = w; q * 64 < n * PAIRS; q += W) {
      const int u = min(q * 64 + lane, n * PAIRS - 1), pl = u / PAIRS;
      const int row = min(m0 + 2 * (u - pl * PAIRS), last);
      request_to_lds(reinterpret_cast<const char*>(p.rowstat), (unsigned)((first_plane + pl) * p.stat_rows + row) * 8u, lds_address(to) + (unsigned)q * 1024u);
    }
  };
  auto add_planes = [&](int n) {
    const float2* const v = reinterpret_cast<const float2*>(planes);
#pragma unroll
    for (int i = 0; i < RR; i++) {
      const int r = min(t + i * 64 * W, ROWS - 1);
#pragma unroll 8
      for (int j = 0; j < n; j++) {
        const float2 x = v[j * ROWS + r];
        sum[i].x += x.x;
        sum[i].y += x.y;
      }
    }
  };
  int plane = 0;
  constexpr int LX = XB * LT_KC / W;   // of the wave's fragments of a stage, those of the tokens: the first ones
  static_assert(!Cx::kPersistent || XB * LT_KC % W == 0, "tokens and weights apart");
  if constexpr (Cx::kPersistent) {   // the weights of the first stages are constant: ahead of the wait for the inputs
    for_each<LT_STAGES - 1>([&](auto Q) { for_each<L - LX>([&](auto I) { issue(Q, Int<LX + decltype(I)::value>{}, voff); }); });
    cx.wait_inputs();
  }
  // Added in groups (the sum of squares is all that RMS wants), planes go to registers: a wave takes two groups of all rows.  In one
  // round trip with the stages behind them; through LDS 64 planes of 320 rows took three turns, 7.2 us to the first product.
  constexpr int RC = ROWS / 64;
  float gsum[SG > 1 ? 2 : 1][SG > 1 ? RC : 1] = {};
  float gv[SG > 1 ? 2 : 1][SG > 1 ? SG : 1][SG > 1 ? RC : 1];
  static_assert(SG == (PRO != PRO_NONE && Cx::kPersistent ? 2 * W : 1), "in the persistent kernel planes in groups, two for each wave");
  if constexpr (SG > 1) {
#pragma unroll
    for (int g = 0; g < 2; g++)
#pragma unroll
      for (int j = 0; j < SG; j++)
#pragma unroll
        for (int c = 0; c < RC; c++)
          gv[g][j][c] = cx.ld_bulk(p.rowstat + 2 * ((size_t)min(w + W * g + SG * j, parts - 1) * p.stat_rows + min(m0 + 64 * c + lane, p.M - 1)) + 1);   // clamped, unconditional
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  } else if (PRO != PRO_NONE) {
    if (parts > 1) {
      for (; parts - plane > PLANES; plane += PLANES) {   // more than fit: in turns
        request_planes(m0, plane, PLANES, planes);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        add_planes(PLANES);
        __syncthreads();
      }
      request_planes(m0, plane, parts - plane, planes);
    } else {
      request_planes(m0, 0, 1, smem);
    }
  }
  constexpr int LF = Cx::kPersistent ? LX : L;   // requests of a first stage that are behind the planes
  for_each<LT_STAGES - 1>([&](auto Q) { for_each<LF>([&](auto I) { issue(Q, I, voff); }); });
  if constexpr (SG > 1) {
    float* const groups = reinterpret_cast<float*>(planes);   // [SG][ROWS]
#pragma unroll
    for (int g = 0; g < 2; g++)
#pragma unroll
      for (int c = 0; c < RC; c++) {
#pragma unroll
        for (int j = 0; j < SG; j++) gsum[g][c] += w + W * g + SG * j < parts ? gv[g][j][c] : 0.f;
        groups[(w + W * g) * ROWS + 64 * c + lane] = gsum[g][c];
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < RR; i++) {
      const int r = min(t + i * 64 * W, ROWS - 1);
      float a = groups[r];
#pragma unroll
      for (int g = 1; g < SG; g++) a += groups[g * ROWS + r];
      sstat[r] = make_float2(0.f, a);   // the last row's extra threads store the same
    }
  } else if (PRO != PRO_NONE && parts > 1) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((LT_STAGES - 1) * LF) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    add_planes(parts - plane);
#pragma unroll
    for (int i = 0; i < RR; i++) sstat[min(t + i * 64 * W, ROWS - 1)] = sum[i];   // the last row's extra threads store the same
  }

  // WALK: a block takes its tiles one after the other, and the next one's first stages and row statistics (in the other of two
  // places) are on their way during the epilogue.  The persistent kernel walks where the tiles of a block are in the same
  // rows, and keeps the statistics.
  int nb_now = nb, m0_now = m0;
  for (int next = die_rank + WALK_BLOCKS / 8;; next += WALK_BLOCKS / 8) {
    f32x16 acc[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int i = 0; i < MT; i++) zero_accumulator<!Cx::kLean>(acc[j][i]);

    bf16x8 xf[2][MT], wf[2][NT];
    constexpr int R = MT + NT, P = MT * NT;        // reads and products of a step
    const unsigned char* const xs = smem_raw + lane * 16 + wm * MT * LT_KC * 1024;
    const unsigned char* const ws = smem_raw + lane * 16 + (XB + wn * NT) * LT_KC * 1024;
    // read r of step s of a group, in the order in which the products need them: x0, w0 .. , x1 ..
    auto read = [&](int u, int s, int r) {
      const int o = (s / LT_KC) * NF * 1024 + (s % LT_KC) * 1024;
      if (r == 0) xf[u][0] = *reinterpret_cast<const bf16x8*>(xs + o);
      else if (r <= NT) wf[u][r - 1] = *reinterpret_cast<const bf16x8*>(ws + o + (r - 1) * LT_KC * 1024);
      else xf[u][r - NT] = *reinterpret_cast<const bf16x8*>(xs + o + (r - NT) * LT_KC * 1024);
    };
    // stage 0 (the other stages requested may be on their way) and the row statistics are complete for everybody; where the weights went
    // ahead stage 1 too, because the count in front of it below takes its requests for whole ones
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(Cx::kPersistent ? LX : (LT_STAGES - 2) * L) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; r++) read(0, 0, r);

    // One group of LT_STAGES stages; LAST: nothing beyond it is requested.  Step s multiplies the fragments of set s % 2 and reads
    // those of step s + 1 into the other set.  In the second step of stage q the next stage must be complete for everybody
    // (LT_STAGES - 3 more may be on their way); everybody has then read stage q - 1, whose place stage q + LT_STAGES - 1 takes.
    auto group = [&](auto last_group) {
      constexpr bool LAST = decltype(last_group)::value != 0;
      turn = turn + 1 == groups ? 0 : turn + 1;
      const unsigned vnext = vfirst + (unsigned)turn * (LT_GROUP * 1024u);
      for_each<LT_GROUP>([&](auto SS) {
        constexpr int s = decltype(SS)::value, q = s / LT_KC, u = s & 1;
        constexpr bool boundary = u == 1 && !(LAST && q == LT_STAGES - 1);
        constexpr bool request = u == 1 && (!LAST || q == 0);
        constexpr bool more = !(LAST && s == LT_GROUP - 1);
        if constexpr (boundary) {
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"((LAST && q > 1 ? LT_STAGES - 2 - q : LT_STAGES - 3) * L) : "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
        for_each<P>([&](auto MM) {
          constexpr int m = decltype(MM)::value;
#pragma unroll
          for (int r = 0; r < R; r++)
            if (r * P / R == m && more) read(u ^ 1, (s + 1) % LT_GROUP, r);
          if constexpr (request) {
            for_each<L>([&](auto I) {
              if constexpr ((2 * decltype(I)::value + 1) * P / (2 * L) == m) issue(Int<(q + LT_STAGES - 1) % LT_STAGES>{}, I, q == 0 ? voff : vnext);
            });
          }
          acc[m % NT][m / NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][m % NT], xf[u][m / NT], acc[m % NT][m / NT], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);   // this order
        });
      });
      voff = vnext;
    };
    for (int g = 0; g + 1 < groups; g++) group(Int<0>{});
    group(Int<1>{});
    const float2* const stat = sstat;
    int nb_next = 0, m0_next = 0;
    if (WALK && next < of_die) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();   // everybody has read the last stage
      nb_next = (first + next) / p.m_tiles;
      m0_next = ((first + next) - nb_next * p.m_tiles) * ROWS;
      set_sources(nb_next, m0_next);
      if constexpr (!Cx::kPersistent) {
        sstat = reinterpret_cast<float2*>(smem + (sstat == reinterpret_cast<float2*>(smem) ? lds_tile_stat_bytes(MT) : 0));
        if (PRO != PRO_NONE) request_planes(m0_next, 0, 1, reinterpret_cast<unsigned char*>(sstat));
      }
      voff = vfirst;
      for_each<LT_STAGES - 1>([&](auto Q) { for_each<L>([&](auto I) { issue(Q, I, voff); }); });
    }
    if constexpr (EPI == EPI_PARTIAL) {   // whole tiles, see partial_tile_at; rows beyond the last are never read
      const int mbs = (p.M + 31) >> 5;
#pragma unroll
      for (int i = 0; i < MT; i++) {
        const int mb = (m0_now >> 5) + wm * MT + i;
#pragma unroll
        for (int j = 0; j < NT; j++) {
          const int nt = nb_now * WB + wn * NT + j;
          if (mb < mbs && nt < p.n_tiles) {   // uniform
            float* const dst = p.out_f32 + (((size_t)cx.by * mbs + mb) * p.n_tiles + nt) * 1024 + lane * 4;
#pragma unroll
            for (int q = 0; q < 4; q++) cx.st(reinterpret_cast<f32x4*>(dst + q * 256), f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]});
          }
        }
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < MT; i++) {
      const int row = (wm * MT + i) * 32 + lq, m = m0_now + row;
      if (m < p.M) {
        float ssum = 0.f, ssq = 0.f;
        if (PRO != PRO_NONE) {
          const float2 v = stat[row];
          ssum = v.x;
          ssq = v.y;
        }
#pragma unroll
        for (int j = 0; j < NT; j++) {
          const int nt = nb_now * WB + wn * NT + j;
          if (nt < p.n_tiles) {
            EpiOps ops;
            epilogue_preload<PRO, EPI>(p, nt, m, lh, ops, cx);
            epilogue_tile<PRO, EPI>(p, acc[j][i], nt, m, lh, ssum, ssq, cx.by, ops, cx);
          }
        }
      }
    }
    if (!WALK || next >= of_die) return;
    nb_now = nb_next;
    m0_now = m0_next;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the counts below take no stores
  }
}

// gate||up of up to 256 rows: the four waves split the rows (two blocks of 32 each) and share four feature tiles.  A wave's
// activations are nobody else's and go from memory straight into registers, sixteen steps ahead; the weights go to LDS, eight stages.  A step
// then takes 20 KiB through LDS instead of the 36 of gemm_lds_body<4, 2>, which need longer than its 256 cycles of products.  Same tile,
// order of k and of the row statistics' planes, so the same bits.  In the persistent prefix (2048 x 32768 at 256 tokens, pi0_infer): 6396 -> 6320 us;
// as a launch, behind whose start everything waits for, it is 1.3 us slower than gemm_lds_body and does not exist.
constexpr int ROWS_STAGES = 8, ROWS_NT = 4, ROWS_PARTS = 32;   // stages, feature tiles, most planes of row statistics
constexpr int ROWS_GROUP = 16;   // k16 steps of a turn of the loop
constexpr int GEMM_ROWS_SMEM = ROWS_STAGES * ROWS_NT * LT_KC * 1024 + 256 * 4;
static_assert(GEMM_ROWS_SMEM <= LT_SMEM, "what the persistent kernel asks for");
template <class Cx>
__device__ __forceinline__ void gemm_rows_body(const GemmParams& p, const Cx& cx, unsigned char* smem) {
  constexpr int W = 4, MT = 2, NT = ROWS_NT, SF = NT * LT_KC, L = SF / W;   // fragments of a stage, of a wave's share of it
  static_assert(SF % W == 0, "even shares");
  float* const ssq = reinterpret_cast<float*>(smem + ROWS_STAGES * SF * 1024);   // [256]
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;
  const int total = (p.n_tiles + NT - 1) / NT;
  int first, of_die;
  const int die_rank = cx.bx >> 3;
  lds_tile_share(cx.bx & 7, total, first, of_die);
  if (die_rank >= of_die) return;
  const int nb = first + die_rank;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4, XKC16 = p.ldx >> 4;
  const int groups = KC16 / ROWS_GROUP, halves = 2 * groups;

  const char* wsrc[L];
#pragma unroll
  for (int i = 0; i < L; i++) {
    const int f = w + W * i;
    wsrc[i] = reinterpret_cast<const char*>(p.W.w) + ((size_t)min(nb * NT + f / LT_KC, p.n_tiles - 1) * KC16 + f % LT_KC) * 1024;
  }
  const char* xsrc[MT];
#pragma unroll
  for (int i = 0; i < MT; i++) xsrc[i] = reinterpret_cast<const char*>(p.X) + ((size_t)min(w * MT + i, mb_last) * XKC16) * 1024;
  const unsigned lds0 = lds_address(smem) + (unsigned)w * 1024u;
  // all blocks read the whole k range of their own weight rows, a power of two apart: each starts elsewhere and goes round.  In halves of
  // a group, as gemm_lds_body's groups are: stages 0 .. 3 and steps 0 .. 7 at va, the rest at vb
  int turn = (int)((unsigned)nb % (unsigned)halves);
  const unsigned vfirst = (unsigned)lane * 16u + 4096u;
  auto half_at = [&](int h) { return vfirst + (unsigned)(h >= halves ? h - halves : h) * (ROWS_GROUP * 512u); };
  unsigned va = half_at(turn), vb = half_at(turn + 1);
  auto request = [&](auto Q, auto I, unsigned v) {   // the wave's fragment I of stage Q of the half at v
    constexpr int q = decltype(Q)::value, i = decltype(I)::value, off = q % 4 * 2048 - 4096;
    const unsigned l0 = lds0;
    const char* const s = wsrc[i];
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::"s"(l0), "v"(v), "s"(s),
                 "n"((q * SF + W * i) * 1024 - off), "n"(off)
                 : "memory", "scc");
  };
  bf16x8 xr[ROWS_GROUP][MT];
  auto load_x = [&](int s, int i, unsigned v) { xr[s][i] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(xsrc[i] + (v - 4096u) + s % 8 * 1024)); };

  for_each<ROWS_STAGES - 1>([&](auto Q) { for_each<L>([&](auto I) { request(Q, I, decltype(Q)::value < 4 ? va : vb); }); });
  if constexpr (Cx::kPersistent) cx.wait_inputs();
  const int parts = p.rowstat_parts > 1 ? p.rowstat_parts : 1;
  float gv[ROWS_PARTS];   // the sum of squares is all that RMS wants; clamped, unconditional
#pragma unroll
  for (int j = 0; j < ROWS_PARTS; j++) gv[j] = cx.ld_bulk(p.rowstat + 2 * ((size_t)min(j, parts - 1) * p.stat_rows + min(t, p.M - 1)) + 1);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < ROWS_GROUP; s++)
#pragma unroll
    for (int i = 0; i < MT; i++) load_x(s, i, s < 8 ? va : vb);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  {
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < ROWS_PARTS; j++) a += j < parts ? gv[j] : 0.f;
    ssq[t] = a;
  }

  f32x16 acc[NT][MT];
#pragma unroll
  for (int j = 0; j < NT; j++)
#pragma unroll
    for (int i = 0; i < MT; i++) zero_accumulator(acc[j][i]);
  bf16x8 wf[2][NT];
  const unsigned char* const ws = smem + lane * 16;
  auto read = [&](int u, int s, int j) { wf[u][j] = *reinterpret_cast<const bf16x8*>(ws + (((s / LT_KC) * NT + j) * LT_KC + s % LT_KC) * 1024); };
  // stage 0 is complete for everybody; the other stages' requests and the activations are behind it
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((ROWS_STAGES - 2) * L + ROWS_GROUP * MT) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int j = 0; j < NT; j++) read(0, 0, j);
  // One group of eight stages.  Step s multiplies the weights of set s % 2 and reads those of step s + 1 into the other set.  In the
  // second step of stage q the next stage must be complete for everybody.  Behind its requests are, at least: the activations
  // of 2 (ROWS_STAGES - 2) steps (LAST asks for none: not counted) and the requests of ROWS_STAGES - 3 stages.
  auto group = [&](auto last_group) {
    constexpr bool LAST = decltype(last_group)::value != 0;
    turn = turn + 2 >= halves ? turn + 2 - halves : turn + 2;
    const unsigned na = half_at(turn), nb_ = half_at(turn + 1);
    for_each<ROWS_GROUP>([&](auto SS) {
      constexpr int s = decltype(SS)::value, q = s / LT_KC, u = s & 1, P = NT * MT;
      if constexpr (u == 1 && !(LAST && q == ROWS_STAGES - 1)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LAST ? (q > 1 ? ROWS_STAGES - 2 - q : ROWS_STAGES - 3) * L : 2 * MT * (ROWS_STAGES - 2) + (ROWS_STAGES - 3) * L) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if constexpr (!LAST || q == 0) {
          for_each<L>([&](auto I) { request(Int<(q + ROWS_STAGES - 1) % ROWS_STAGES>{}, I, q == 0 ? vb : q - 1 < 4 ? na : nb_); });
        }
      }
      for_each<P>([&](auto MM) {
        constexpr int m = decltype(MM)::value;
        if constexpr (m < NT && !(LAST && s == ROWS_GROUP - 1)) read(u ^ 1, (s + 1) % ROWS_GROUP, m);
        if constexpr (m == NT && !LAST) load_x(s, 0, s < 8 ? na : nb_);
        acc[m % NT][m / NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][m % NT], xr[s][m / NT], acc[m % NT][m / NT], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);   // this order
      });
      if constexpr (!LAST) load_x(s, 1, s < 8 ? na : nb_);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    });
    va = na;
    vb = nb_;
  };
  for (int g = 0; g + 1 < groups; g++) group(Int<0>{});
  group(Int<1>{});

#pragma unroll
  for (int i = 0; i < MT; i++) {
    const int row = (w * MT + i) * 32 + lq;
    if (row < p.M) {
#pragma unroll
      for (int j = 0; j < NT; j++) {
        const int nt = nb * NT + j;
        if (nt < p.n_tiles) {
          EpiOps ops;
          epilogue_preload<PRO_RMS, EPI_GEGLU>(p, nt, row, lh, ops, cx);
          epilogue_tile<PRO_RMS, EPI_GEGLU>(p, acc[j][i], nt, row, lh, 0.f, ssq[row], 0, ops, cx);
        }
      }
    }
  }
}

// gate||up and down of more than 512 rows: H blocks of 32 rows, which the four waves share, and eight feature tiles, two to a wave.  A
// wave's weights are nobody else's and go from memory straight into registers, a turn of the loop ahead; the activations go to LDS, four
// stages of four k16 steps.  What it is for is the height: such a GEMM runs at the clock that the matrix cores' power leaves, so rows that
// are only there to fill a tile cost as much as others, and H may be any number up to what the accumulators allow (nine blocks are 288 of a
// lane's 512 registers; gemm_lds_body has none left at ten), with a lower body for the rows that are left over.  A step takes 5 H KiB through
// LDS (gemm_lds_body 6 (MT + NT)).  At heights that gemm_lds_body has it is no quicker: prefill at 512 tokens 4.26 -> 4.28 ms, 768 5.43 -> 5.46.
// An accumulator's order of k is gemm_lds_body's with several token tiles, so the bits are the same.
// SG: as in gemm_lds_body.
constexpr int COLS_STAGES = 4, COLS_KS = 4, COLS_GROUP = COLS_STAGES * COLS_KS;   // stages, k16 steps of a stage, of a turn
constexpr int COLS_NT = 2, COLS_TILES = 4 * COLS_NT;                              // feature tiles of a wave, of a block
constexpr int cols_smem(int H) { return COLS_STAGES * COLS_KS * H * 1024 + H * 32 * 4; }
template <int H, int SG, int EPI, class Cx>
__device__ __forceinline__ void gemm_cols_body(const GemmParams& p, const Cx& cx, unsigned char* smem, int nb, int m0) {
  static_assert(EPI == EPI_GEGLU || EPI == EPI_PARTIAL, "RMS in front of the one, nothing in front of the other");
  static_assert(cols_smem(H) <= LT_SMEM, "what the kernels ask for");
  constexpr int W = 4, S = COLS_STAGES, KS = COLS_KS, G = COLS_GROUP, NT = COLS_NT, ROWS = H * 32;
  constexpr bool STATS = EPI == EPI_GEGLU;
  constexpr int SB = H * KS * 1024;                      // bytes of a stage: [row block][k16 step][1 KiB]
  constexpr int RX = 8, AHEAD = H < 6 ? H : 6;           // activation fragments in registers, of them requested ahead of the products
  static_assert(G * H % RX == 0 && AHEAD < RX, "what is read ahead is in a stage's last step");
  float* const ssq = reinterpret_cast<float*>(smem + S * SB);   // [ROWS]
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4, XKC16 = p.ldx >> 4;
  const int kbeg = EPI == EPI_PARTIAL ? cx.by * (p.k_per_split >> 4) : 0;
  const int groups = ((EPI == EPI_PARTIAL ? min(kbeg + (p.k_per_split >> 4), KC16) : KC16) - kbeg) / G;

  const char* wsrc[NT];
#pragma unroll
  for (int j = 0; j < NT; j++) wsrc[j] = reinterpret_cast<const char*>(p.W.w) + ((size_t)min(nb * COLS_TILES + w * NT + j, p.n_tiles - 1) * KC16 + kbeg) * 1024;
  const char* xsrc[H];   // the wave requests k16 step w of every stage; blocks beyond the rows repeat the last one and are not stored
#pragma unroll
  for (int b = 0; b < H; b++) xsrc[b] = reinterpret_cast<const char*>(p.X) + ((size_t)min((m0 >> 5) + b, mb_last) * XKC16 + kbeg + w) * 1024;
  const unsigned lds0 = lds_address(smem) + (unsigned)w * 1024u;
  // stages 0 .. 3 of a group are at 4096 q - 4096 behind v, v + 8192: a 13-bit constant, which counts towards both addresses
  unsigned voff = (unsigned)lane * 16u + 4096u;
  auto request = [&](auto Q, auto B, unsigned v) {
    constexpr int q = decltype(Q)::value, b = decltype(B)::value, off = q % 2 * 4096 - 4096;
    const unsigned l0 = lds0;
    const char* const s = xsrc[b];
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::"s"(l0), "v"(v + (unsigned)(q / 2) * 8192u), "s"(s),
                 "n"((q * H + b) * KS * 1024 - off), "n"(off)
                 : "memory", "scc");
  };
  bf16x8 wr[G][NT];
  auto pinned = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_w = [&](int s, unsigned v) {
#pragma unroll
    for (int j = 0; j < NT; j++) wr[s][j] = *reinterpret_cast<const bf16x8*>(wsrc[j] + (v - 4096u) + s * 1024);
  };
  constexpr int EARLY = Cx::kPersistent ? G : 0;   // the weights are constant: ahead of the wait for the inputs
  if constexpr (Cx::kPersistent) {
#pragma unroll
    for (int s = 0; s < EARLY; s++) load_w(s, voff);
    pinned();
    cx.wait_inputs();
  }
  // row statistics, of which RMS wants the sum of squares: whole-row sums, or planes of partial sums added in groups (a wave takes two)
  constexpr int RR = (ROWS + 64 * W - 1) / (64 * W), RC = (ROWS + 63) / 64;
  static_assert(SG == (STATS && Cx::kPersistent ? 2 * W : 1), "in the persistent kernel planes in groups, two for each wave");
  float gv[SG > 1 ? 2 : 1][SG > 1 ? SG : 1][SG > 1 ? RC : RR];
  const int parts = STATS ? p.rowstat_parts : 0;
  if constexpr (SG > 1) {
#pragma unroll
    for (int g = 0; g < 2; g++)
#pragma unroll
      for (int j = 0; j < SG; j++)
#pragma unroll
        for (int c = 0; c < RC; c++)   // clamped, unconditional
          gv[g][j][c] = cx.ld_bulk(p.rowstat + 2 * ((size_t)min(w + W * g + SG * j, parts - 1) * p.stat_rows + min(m0 + min(64 * c + lane, ROWS - 1), p.M - 1)) + 1);
  } else if constexpr (STATS) {
#pragma unroll
    for (int i = 0; i < RR; i++) gv[0][0][i] = p.rowstat[2 * (size_t)min(m0 + min(t + i * 64 * W, ROWS - 1), p.M - 1) + 1];
  }
  pinned();
  for_each<2>([&](auto Q) { for_each<H>([&](auto B) { request(Q, B, voff); }); });
#pragma unroll
  for (int s = EARLY; s < G; s++) load_w(s, voff);
  pinned();
  for_each<H>([&](auto B) { request(Int<2>{}, B, voff); });
  if constexpr (SG > 1) {
    float* const sums = reinterpret_cast<float*>(smem + (S - 1) * SB);   // [SG][ROWS], where the last stage will be
#pragma unroll
    for (int g = 0; g < 2; g++)
#pragma unroll
      for (int c = 0; c < RC; c++) {
        float a = 0.f;
#pragma unroll
        for (int j = 0; j < SG; j++) a += w + W * g + SG * j < parts ? gv[g][j][c] : 0.f;
        sums[(w + W * g) * ROWS + min(64 * c + lane, ROWS - 1)] = a;   // the last row's extra lanes store the same
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < RR; i++) {
      const int r = min(t + i * 64 * W, ROWS - 1);
      float a = sums[r];
#pragma unroll
      for (int g = 1; g < SG; g++) a += sums[g * ROWS + r];
      ssq[r] = a;
    }
  } else if constexpr (STATS) {
#pragma unroll
    for (int i = 0; i < RR; i++) ssq[min(t + i * 64 * W, ROWS - 1)] = gv[0][0][i];
  }

  f32x16 acc[NT][H];
#pragma unroll
  for (int j = 0; j < NT; j++)
#pragma unroll
    for (int b = 0; b < H; b++) {
      if (b < 8) {
        zero_accumulator<!Cx::kLean>(acc[j][b]);
      } else {
#pragma unroll
        for (int r = 0; r < 16; r++) acc[j][b][r] = 0.f;
      }
    }
  bf16x8 xf[RX];
  // an LDS read reaches 64 KiB: a base for each (left alone, the compiler keeps an address in a register for every read beyond the first)
  unsigned base[(S * SB + 65535) / 65536];
#pragma unroll
  for (int i = 0; i < (S * SB + 65535) / 65536; i++) {
    base[i] = (unsigned)lane * 16u + (unsigned)i * 65536u;
    asm volatile("" : "+v"(base[i]));
  }
  auto read = [&](int f) {   // fragment f of a group: k16 step f / H, row block f % H
    const int s = f / H, b = f % H, at = ((s / KS * H + b) * KS + s % KS) * 1024;
    xf[f % RX] = *reinterpret_cast<const bf16x8*>(smem + base[at >> 16] + (at & 65535));
  };
  // the first two stages are complete for everybody; the third one's requests and the other weights are behind them
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(H + (G - EARLY) * NT) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int f = 0; f < AHEAD; f++) read(f);

  // One group of four stages; LAST: nothing beyond it is requested.  AHEAD products in front of a stage's end, where the next one is first
  // read, that one must be complete for everybody, and everybody is through with the one before, whose place the stage three on takes.
  // Behind the next stage's requests are, at least: those of one stage (LAST, from its second on: of none that it asked for itself) and
  // the weights of seven steps, of which six are counted (LAST: of four, then none; three counted).  The first group
  // finds its second stage complete, and behind the third one's requests the loads of its own six steps.
  auto group = [&](auto last_group) {
    constexpr bool LAST = decltype(last_group)::value != 0;
    const unsigned vnext = voff + (unsigned)G * 1024u;
    for_each<G * H>([&](auto FF) {
      constexpr int f = decltype(FF)::value, s = f / H, b = f % H, q = s / KS, at = f - ((q + 1) * KS * H - AHEAD);
      if constexpr (at == 0 && !(LAST && q == S - 1)) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(!LAST ? H + 12 : q == 0 ? H + 6 : q == 1 ? H : 0) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      if constexpr (!LAST || f + AHEAD < G * H) read((f + AHEAD) % (G * H));
      if constexpr (at >= 0 && (!LAST || q == 0)) {
        for_each<H>([&](auto B) {
          if constexpr (decltype(B)::value * AHEAD / H == at) request(Int<(q + S - 1) % S>{}, B, q == 0 ? voff : vnext);
        });
      }
#pragma unroll
      for (int j = 0; j < NT; j++) {
        // The ninth block's accumulators are ordinary vector registers, written down as such (the compiler keeps them all in the other
        // half, 256 of a lane, and spills).  It leaves no wait states behind them, so nothing but the next product may name those registers here:
        // test_gpu_cols_gemm.py looks at the code as built
        if constexpr (b < 8) acc[j][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[s][j], xf[f % RX], acc[j][b], 0, 0, 0);
        else asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[j][b]) : "v"(wr[s][j]), "v"(xf[f % RX]));
        __builtin_amdgcn_sched_barrier(0);   // this order
      }
      if constexpr (!LAST && b == H - 1) {
        load_w(s, vnext);
        pinned();
      }
    });
    voff = vnext;
  };
  for (int g = 0; g + 1 < groups; g++) group(Int<0>{});
  group(Int<1>{});
  if constexpr (H > 8) asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[0][8]), "+v"(acc[1][8]));   // products that the compiler does not know as such: written by now
  if constexpr (EPI == EPI_PARTIAL) {   // whole tiles, see partial_tile_at; rows beyond the last are never read
    const int mbs = (p.M + 31) >> 5;
#pragma unroll
    for (int b = 0; b < H; b++) {
      const int mb = (m0 >> 5) + b;
#pragma unroll
      for (int j = 0; j < NT; j++) {
        const int nt = nb * COLS_TILES + w * NT + j;
        if (mb < mbs && nt < p.n_tiles) {   // uniform
          float* const dst = p.out_f32 + (((size_t)cx.by * mbs + mb) * p.n_tiles + nt) * 1024 + lane * 4;
#pragma unroll
          for (int q = 0; q < 4; q++) cx.st(reinterpret_cast<f32x4*>(dst + q * 256), f32x4{acc[j][b][4 * q], acc[j][b][4 * q + 1], acc[j][b][4 * q + 2], acc[j][b][4 * q + 3]});
        }
      }
    }
  } else {
#pragma unroll
    for (int b = 0; b < H; b++) {
      const int row = b * 32 + lq, m = m0 + row;
      if (m < p.M) {
        const float sq = ssq[row];
#pragma unroll
        for (int j = 0; j < NT; j++) {
          const int nt = nb * COLS_TILES + w * NT + j;
          if (nt < p.n_tiles) {
            EpiOps ops;
            epilogue_preload<PRO_RMS, EPI_GEGLU>(p, nt, m, lh, ops, cx);
            epilogue_tile<PRO_RMS, EPI_GEGLU>(p, acc[j][b], nt, m, lh, 0.f, sq, 0, ops, cx);
          }
        }
      }
    }
  }
}

// Height of the rows that are left over: five blocks (769 .. 800 and 816 tokens behind three tiles of seven), eight (513 .. 544 behind one of nine)
constexpr int cols_short(int H) { return H == 7 ? 5 : H - 1; }
template <int H, int SG, int EPI, class Cx>
__device__ __forceinline__ void gemm_cols_item(const GemmParams& p, const Cx& cx, unsigned char* smem) {
  // tiles as in gemm_lds_body; partial sums: in order, a k range (cx.by) for each die
  const int total = (p.n_tiles + COLS_TILES - 1) / COLS_TILES * p.m_tiles;
  int first = 0, of_die = total, rank = cx.bx;
  if (EPI != EPI_PARTIAL) {
    lds_tile_share(cx.bx & 7, total, first, of_die);
    rank = cx.bx >> 3;
  }
  if (rank >= of_die) return;
  const int nb = (first + rank) / p.m_tiles, m0 = ((first + rank) - nb * p.m_tiles) * H * 32;
  if (p.M - m0 <= cols_short(H) * 32) gemm_cols_body<cols_short(H), SG, EPI>(p, cx, smem, nb, m0);
  else gemm_cols_body<H, SG, EPI>(p, cx, smem, nb, m0);
}
