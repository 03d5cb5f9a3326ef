// The prefix's large bf16 GEMMs (gate||up, and down as split-K partial sums): one wave per SIMD, both operands through LDS.
//
// Orientation and epilogues as in gemm.hip.  A block of 4 waves owns 2 MT * 32 tokens x 2 NT * 32 features, a wave MT x NT
// tiles of 32 x 32.  Operands are in fragment order in memory, so a stage (2 k16 steps) is a list of 1 KiB fragments; they
// go from memory straight to LDS (global_load_lds_dwordx4: lane l's 16 bytes land at base + 16 l) and come back as whole
// fragments, one k16 step ahead of the products.  Four stages rotate: one is being multiplied, the next is complete, two are
// on their way.
// What bounds it: with a single wave per SIMD everything between two products is time the matrix cores stand still, so the
// loop is straight-line code over a group of four stages - every LDS offset, every memory offset within a group and every
// wait count is a constant, and reads and requests are issued one by one between the products (in front of them, the eight
// reads of a step alone cost 200 of its 512 cycles; with stage indices computed at run time the step took 1240).  At 512
// tokens the loop takes 537 cycles per 16 products of 32 cycles; the chip then clocks at 1.25 - 1.4 GHz instead of 2.4, so
// the rest is power.  The requests are written as assembly because the compiler makes every LDS read wait for all LDS-bound
// loads in flight; their completion is counted here.
// gate||up (32768 x 2048), cold weights, us, against the register-staged tiles of gemm.hip: 256 tokens 42.7 (47 - 51),
// 304 48 (56), 512 65 (82), 768 100 (106), 816 124 (140).
#include "pi0_internal.h"

#include <utility>

#include "gemm_common.h"

namespace {

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

constexpr int LT_STAGES = 4;                   // stages in LDS
constexpr int LT_KC = 2;                       // k16 steps of a stage
constexpr int LT_GROUP = LT_STAGES * LT_KC;    // k16 steps of a turn of the loop: k ranges are multiples of 128

constexpr int lds_tile_fragments(int MT, int NT) { return 2 * (MT + NT) * LT_KC; }   // of a stage
constexpr int LT_SMEM = 160 * 1024;             // of a compute unit, which a block has to itself
constexpr int lds_tile_stat_bytes(int MT) { return (2 * MT * 32 * 8 + 1023) / 1024 * 1024; }   // row statistics, whole requests of 1 KiB
constexpr int lds_tile_smem(int MT, int NT) { return lds_tile_stat_bytes(MT) + LT_STAGES * lds_tile_fragments(MT, NT) * 1024; }
// planes of partial row statistics that fit behind the three stages requested first (the last request may be half empty)
constexpr int lds_tile_planes(int MT, int NT) {
  return (LT_SMEM - lds_tile_stat_bytes(MT) - (LT_STAGES - 1) * lds_tile_fragments(MT, NT) * 1024 - 1024) / (2 * MT * 32 * 8);
}

template <int MT, int NT, int PRO, int EPI, bool WALK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_lds_kernel(GemmParams p) {
  constexpr int W = 4;
  constexpr int XB = 2 * MT, WB = 2 * NT;        // 32-row blocks of the two operands
  constexpr int NF = lds_tile_fragments(MT, NT);
  constexpr int L = NF / W;                      // fragments a wave requests per stage
  static_assert(NF % W == 0, "even shares");
  constexpr int ROWS = XB * 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];          // row statistics, then [stage][fragment][1 KiB]
  float2* sstat = reinterpret_cast<float2*>(smem);
  unsigned char* const smem_raw = smem + (WALK ? 2 : 1) * lds_tile_stat_bytes(MT);

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = w & 1, wn = w >> 1;
  const int lq = lane & 31;
  const int lh = lane >> 5;

  // tiles as in gemm_stream.hip: consecutive ids on different dies, a die takes a contiguous eighth, token tiles fastest
  const int total = (p.n_tiles + WB - 1) / WB * p.m_tiles;
  const int die = (int)blockIdx.x & 7, die_rank = (int)blockIdx.x >> 3;
  const int first = die * (total >> 3) + min(die, total & 7), of_die = (total >> 3) + (die < (total & 7) ? 1 : 0);
  if (die_rank >= of_die) return;
  const int nb = (first + die_rank) / p.m_tiles;
  const int mt = (first + die_rank) - nb * p.m_tiles;
  const int m0 = mt * ROWS;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4, XKC16 = p.ldx >> 4;
  const int kbeg = (int)blockIdx.y * (p.k_per_split >> 4);
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
  int turn = p.m_tiles == 1 ? (int)((unsigned)nb % (unsigned)groups) : 0;
  const unsigned vfirst = (unsigned)lane * 16u + 4096u;
  unsigned voff = vfirst + (unsigned)turn * (LT_GROUP * 1024u);      // of the current group: its stage q is at 2048 q - 4096, a 13-bit constant
  // request the wave's fragment I of stage Q of the group at v; the constant counts towards both addresses
  auto issue = [&](auto Q, auto I, unsigned v) {
    constexpr int q = decltype(Q)::value, i = decltype(I)::value;
    const unsigned l0 = lds0;
    const char* const s = src[i];
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::"s"(l0), "v"(v), "s"(s),
                 "n"((q * NF + W * i) * 1024 - (q * 2048 - 4096)), "n"(q * 2048 - 4096)
                 : "memory", "scc");
  };
  // Row statistics: whole-row sums, or partial sums in planes, one per block column of the producer, which the thread of the
  // row adds up.  They go to LDS like the operands and in front of them: loaded into registers behind the first stages, as
  // they were, they kept every block until all of those stages had come, a burst of 18 - 25 MB from memory (start of a block
  // to its first product 4.3 us at 256 and 512 tokens, as against 1.9 without statistics;
  // prefill at 512 / 768 / 816 tokens 4.432 / 5.822 / 6.350 -> 4.414 / 5.790 / 6.310 ms).
  constexpr int PLANES = lds_tile_planes(MT, NT), PAIRS = ROWS / 2, RR = (ROWS + 64 * W - 1) / (64 * W);
  static_assert(PLANES >= 1, "room for a plane");
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
  if (PRO != PRO_NONE) {
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
  for_each<LT_STAGES - 1>([&](auto Q) { for_each<L>([&](auto I) { issue(Q, I, voff); }); });
  if (PRO != PRO_NONE && parts > 1) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((LT_STAGES - 1) * L) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    add_planes(parts - plane);
#pragma unroll
    for (int i = 0; i < RR; i++) sstat[min(t + i * 64 * W, ROWS - 1)] = sum[i];   // the last row's extra threads store the same
  }

  // WALK: a block takes its tiles one after the other, and the next one's first stages and row statistics (in the other of two
  // places) are on their way during the epilogue
  int nb_now = nb, m0_now = m0;
  for (int next = die_rank + ((int)gridDim.x >> 3);; next += (int)gridDim.x >> 3) {
    f32x16 acc[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int i = 0; i < MT; i++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[j][i][r] = 0.f;

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
    // stage 0 (stages 1 and 2 may be on their way) and the row statistics are complete for everybody
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * L) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; r++) read(0, 0, r);

    // One group of four stages; LAST: nothing beyond it is requested.  Step s multiplies the fragments of set s % 2 and reads
    // those of step s + 1 into the other set.  In the second step of stage q the next stage must be complete for everybody
    // (one more may be on its way); everybody has then read stage q - 1, whose place stage q + 3 takes.
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
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LAST && q == LT_STAGES - 2 ? 0 : L) : "memory");
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
              if constexpr ((2 * decltype(I)::value + 1) * P / (2 * L) == m) issue(Int<(q + 3) % LT_STAGES>{}, I, q == 0 ? voff : vnext);
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
      sstat = reinterpret_cast<float2*>(smem + (sstat == reinterpret_cast<float2*>(smem) ? lds_tile_stat_bytes(MT) : 0));
      if (PRO != PRO_NONE) request_planes(m0_next, 0, 1, reinterpret_cast<unsigned char*>(sstat));
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
            float* const dst = p.out_f32 + (((size_t)blockIdx.y * mbs + mb) * p.n_tiles + nt) * 1024 + lane * 4;
#pragma unroll
            for (int q = 0; q < 4; q++) *reinterpret_cast<f32x4*>(dst + q * 256) = f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
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
            epilogue_preload<PRO, EPI>(p, nt, m, lh, ops);
            epilogue_tile<PRO, EPI>(p, acc[j][i], nt, m, lh, ssum, ssq, blockIdx.y, ops);
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

// tiles (MT, NT): 256 x 128, 320 x 128, 192 x 256, 256 x 256 (tokens x features).  One token tile of 320 takes a view and its
// prompt, one of 256 a view; four of 192 take three views.
#define LDS_TILES(X) X(4, 2) X(5, 2) X(3, 4) X(4, 4)

// Time of a launch in microseconds, for the choice of the tile and of the number of k ranges.  A round of 256 blocks takes
// the larger of the operands' way to the compute units (46 KB per us and unit with all of them asking; a round that leaves
// units idle is quicker, gate||up down to 3/4, partial sums 0.9) and the products (32 cycles each at the 1.35 GHz the chip
// then runs at), and 3 us plus the epilogue, which goes with the tile (0.8 us per 32 x 32 tile and wave with the gate, 0.12 us
// for partial sums).  The partial sums are then read and written once more (5 TB/s, a launch, and
// 3 us for each round trip of eight ranges beyond the first: 533 tokens, prefill in ms with 7 / 8 / 9 / 10 ranges 4.870 / 4.816 /
// 4.862 / 4.974).  It ranks tiles and ranges; it does not predict a time.  In a traced pass at 256 / 512 / 768 / 816 tokens gate||up
// takes 42.5 / 59.9 / 87.7 / 112.4 us, the formula says 42.8 / 64.3 / 103.1 / 128.7 (1 % high, then 7 .. 18 %); down with its reduction
// takes 35.6 / 51.4 / 69.5 / 74.8, the formula says 41.6 / 55.8 / 68.5 / 75.7 (17 and 9 % high, then within 1.5 %: the GEMM alone
// 13 .. 25 % low, the reduction 1.8 .. 2.7 times too long).
// Number of ranges, prefill in ms at 256 tokens with 8 / 10 / 11 / 12 / 16 ranges:
// 3.078 / 3.046 / 3.024 / 3.030 / 3.031; 512 with 6 / 7 / 8 / 10 / 12: 4.336 / 4.306 / 4.248 / 4.300 / 4.208 .. 4.31; 768 with
// 5 / 6 / 7 / 8 / 9: 5.523 / 5.451 / 5.393 / 5.393 / 5.425; 816 with 5 / 6 / 7 / 8: 5.998 / 5.948 / 6.033 / 6.038.
float lds_tile_cost(int MT, int NT, int M, int n_tiles, int k_per_split, int z, bool partial) {
  const int blocks = ceil_div(M, 2 * MT * 32) * ceil_div(n_tiles, 2 * NT) * z;
  const int rounds = ceil_div(blocks, 256);
  const float steps = (float)(k_per_split >> 4);
  const float feed = 2.f * (float)(MT + NT) / 46.f, products = (float)(MT * NT) * 0.0237f;
  const float full = steps * (feed > products ? feed : products);
  const float fill = (float)blocks / (256.f * (float)rounds), least = partial ? 0.9f : 0.75f;
  float us = (float)rounds * (full * (fill > least ? fill : least) + 3.f + (partial ? 0.12f : 0.8f) * (float)(MT * NT));
  if (partial) us += (float)z * (float)M * (float)n_tiles * 32.f * 8.f / 5.0e6f + 5.f + (float)((z - 1) / 8) * 3.f;
  return us;
}

template <int MT, int NT, int PRO, int EPI>
hipError_t lds_tile_launch(hipStream_t s, GemmParams p, int z) {
  p.m_tiles = ceil_div(p.M, 2 * MT * 32);
  const int total = ceil_div(p.n_tiles, 2 * NT) * p.m_tiles;
  // More tiles than compute units: blocks that stay and walk save the start of the second round, 2 of 88 us at 768 tokens
  // (prefill at 533 / 768 tokens 4.650 / 5.280 -> 4.621 / 5.255 ms).  Where one round is enough the same code is slower (3.23 -> 3.28 ms
  // at 256 tokens): its registers take part in the loop.  Tiles of 256 x 256 have none left for it and spill: 816 tokens
  // alone 20 us faster, beside a denoise loop on half of the chip 9.50 -> 9.55 ms
  if constexpr (EPI == EPI_GEGLU && MT * NT <= 12) {
    if (total > 256 && p.m_tiles > 1 && p.rowstat_parts <= 1) {
      gemm_lds_kernel<MT, NT, PRO, EPI, true><<<dim3(256), dim3(256), LT_SMEM, s>>>(p);
      return hipGetLastError();
    }
  }
  gemm_lds_kernel<MT, NT, PRO, EPI, false><<<dim3(8 * ceil_div(total, 8), z), dim3(256), PRO != PRO_NONE ? LT_SMEM : lds_tile_smem(MT, NT), s>>>(p);
  return hipGetLastError();
}

}  // namespace

bool gemm_lds_ok(int k_pad) { return k_pad % (16 * LT_GROUP) == 0; }

int gemm_lds_splits(int M, int n_tiles, int k_pad, int z_max) {
  int best_z = 1;
  float best = -1.f;
  for (int z = 1; z <= z_max; z++) {
    const int kps = round_up(ceil_div(k_pad, z), 16 * LT_GROUP);
    if (ceil_div(k_pad, kps) != z) continue;   // a range would be empty
#define X(MT, NT)                                                                       \
  {                                                                                     \
    const float c = lds_tile_cost(MT, NT, M, n_tiles, kps, z, true);                    \
    if (best < 0.f || c < best) { best = c; best_z = z; }                               \
  }
    LDS_TILES(X)
#undef X
  }
  return best_z;
}

hipError_t gemm_lds_init_attributes() {
  hipError_t e = hipSuccess;
#define X(MT, NT)                                                                                                                       \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_RMS, EPI_GEGLU, false>),             \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, LT_SMEM);                                    \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_NONE, EPI_PARTIAL, false>),          \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_tile_smem(MT, NT));
  LDS_TILES(X)
#undef X
#define X(MT, NT)                                                                                                                       \
  if constexpr (MT * NT <= 12)                                                                                                          \
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_RMS, EPI_GEGLU, MT * NT <= 12>), \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LT_SMEM);
  LDS_TILES(X)
#undef X
  return e;
}

hipError_t launch_gemm_lds(hipStream_t s, int pro, int epi, const GemmParams& p, int z) {
  // everything the kernel's indexing assumes
  if (p.X == nullptr || p.W.w == nullptr || p.M <= 0 || p.pf.blocks != 0 || z < 1) return hipErrorInvalidValue;
  if (!gemm_lds_ok(p.W.k_pad) || p.W.k_pad < 128 || !gemm_lds_ok(p.k_per_split) || p.k_per_split < 128) return hipErrorInvalidValue;
  if ((long)p.k_per_split * z < p.W.k_pad || (long)p.k_per_split * (z - 1) >= p.W.k_pad) return hipErrorInvalidValue;
  if (p.n_tiles < 1 || p.n_tiles * 32 != p.W.n_pad || p.ldx < p.W.k_pad || p.ldx % 16 != 0) return hipErrorInvalidValue;
  if ((size_t)p.W.k_pad * 64 > 0x7fffffffu) return hipErrorInvalidValue;   // a row of fragments is addressed with 32 bits
  if (pro == PRO_RMS && epi == EPI_GEGLU) {
    if (z != 1 || p.rowstat == nullptr || p.out_bf16 == nullptr || p.bias != nullptr) return hipErrorInvalidValue;
    // statistics are read two rows at a time
    if (p.rowstat_parts > 1 && (p.stat_rows < p.M || p.stat_rows % 2 != 0)) return hipErrorInvalidValue;
  } else if (pro != PRO_NONE || epi != EPI_PARTIAL || p.out_f32 == nullptr) {
    return hipErrorInvalidValue;
  }
  hipError_t (*best)(hipStream_t, GemmParams, int) = nullptr;
  float cost = 0.f;
#define X(MT, NT)                                                                                            \
  {                                                                                                          \
    const float c = lds_tile_cost(MT, NT, p.M, p.n_tiles, p.k_per_split, z, epi == EPI_PARTIAL);             \
    if (best == nullptr || c < cost) {                                                                       \
      cost = c;                                                                                              \
      best = epi == EPI_PARTIAL ? &lds_tile_launch<MT, NT, PRO_NONE, EPI_PARTIAL> : &lds_tile_launch<MT, NT, PRO_RMS, EPI_GEGLU>; \
    }                                                                                                        \
  }
  LDS_TILES(X)
#undef X
  return best(s, p, z);
}
