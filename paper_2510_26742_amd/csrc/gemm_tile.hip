// The prefix's large bf16 GEMMs (gate||up, and down as split-K partial sums): one wave per SIMD, both operands through LDS.
//
// Orientation and epilogues as in gemm.hip.  A block of 4 waves owns 2 MT * 32 tokens x 2 NT * 32 features, a wave MT x NT
// tiles of 32 x 32.  Operands are in fragment order in memory, so a stage (2 k16 steps) is a list of 1 KiB fragments; they
// go from memory straight to LDS (global_load_lds_dwordx4: lane l's 16 bytes land at base + 16 l) and come back as whole
// fragments, one k16 step ahead of the products.  The stages rotate: one is being multiplied, the next is complete, the others are
// on their way; four, or eight with tiles small enough (down at one view, four stages: loop 22.1 us, eight: 18.3).
// What bounds it: with a single wave per SIMD everything between two products is time the matrix cores stand still, so the
// loop is straight-line code over a group of all stages - every LDS offset, every memory offset within a group and every
// wait count is a constant, and reads and requests are issued one by one between the products (in front of them, the eight
// reads of a step alone cost 200 of its 512 cycles; with stage indices computed at run time the step took 1240).  At 512
// tokens the loop takes 537 cycles per 16 products of 32 cycles; the chip then clocks at 1.25 - 1.4 GHz instead of 2.4, so
// the rest is power.  The requests are written as assembly because the compiler makes every LDS read wait for all LDS-bound
// loads in flight; their completion is counted here.
// The other bound is what shared memory hands out: a step of (MT, NT) writes 2 (MT + NT) KiB and reads twice that, and loops whose
// products do not fill the time run at 87 .. 99 bytes per clock of it.
// Since it is power, rows that only fill a tile cost what others cost: gemm_cols_body has tiles of seven and nine blocks of 32 rows.
// gate||up (32768 x 2048), cold weights, us, against the register-staged tiles of gemm.hip: 256 tokens 42.7 (47 - 51),
// 304 48 (56), 512 65 (82), 768 100 (106), 816 124 (140).
#include "pi0_internal.h"

#include "gemm_tile_body.h"

namespace {
template <int MT, int NT, int PRO, int EPI, bool WALK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_lds_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  LaunchCtx cx{(int)blockIdx.x, (int)blockIdx.y, 0};
  if (EPI == EPI_PARTIAL && p.range_per_die) cx = LaunchCtx{(int)blockIdx.x >> 3, (int)blockIdx.x & 7, 0};
  gemm_lds_body<MT, NT, 1, PRO, EPI, WALK>(p, cx, smem);
}

template <int H, int EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_cols_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (EPI == EPI_PARTIAL) gemm_cols_item<H, 1, EPI>(p, LaunchCtx{(int)blockIdx.x >> 3, (int)blockIdx.x & 7, 0}, smem);
  else gemm_cols_item<H, 1, EPI>(p, LaunchCtx{(int)blockIdx.x, 0, 0}, smem);
}
// heights of gemm_cols_body in blocks of 32 rows, of gate||up and of down
#define COLS_HEIGHTS(X) X(7, EPI_GEGLU) X(9, EPI_GEGLU) X(7, EPI_PARTIAL)

// tiles (MT, NT): 256 x 128, 320 x 128, 192 x 256, 256 x 256 (tokens x features).  One token tile of 320 takes a view and its
// prompt, one of 256 a view; four of 192 take three views.
#define LDS_TILES(X) X(4, 2) X(5, 2) X(3, 4) X(4, 4)
// Partial sums over eight k ranges: a die takes all tiles of one range, so its L2 fetches an eighth of the activations instead of all of
// them, and the tile is the one that fills its 32 compute units (2 x 2: 256 tokens, 3 x 2: 257 .. 384).  pi0_prefill with as many ranges
// as the cost below asked for (13 up to 304 tokens) and all dies on all ranges -> this, ms: 256 tokens 3.040 -> 2.932, 263 3.278 -> 3.189,
// 304 3.387 -> 3.272, 512 4.346 -> 4.297, 533 4.829 -> 4.811, 560 4.909 -> 4.844, 768 5.568 -> 5.449.
#define LDS_RANGE_TILES(X) X(2, 2) X(3, 2) X(4, 2) X(5, 2) X(3, 4) X(4, 4)

// Time of a launch in microseconds, for the choice of the tile and of the number of k ranges.  A round of 256 blocks takes
// the larger of the operands' way to the compute units (46 KB per us and unit with all of them asking; a round that leaves
// units idle is quicker, gate||up down to 3/4, partial sums 0.9) and the products (32 cycles each at the 1.35 GHz the chip
// then runs at), and 3 us plus the epilogue, which goes with the tile (0.8 us per 32 x 32 tile and wave with the gate, 0.12 us
// for partial sums).  The partial sums are then read and written once more (5 TB/s, a launch, and
// 3 us for each round trip of eight ranges beyond the first: 533 tokens, prefill in ms with 7 / 8 / 9 / 10 ranges 4.870 / 4.816 /
// 4.862 / 4.974).  It ranks tiles and ranges; it does not predict a time.  In a traced pass at 256 / 512 / 768 / 816 tokens gate||up
// takes 42.5 / 59.9 / 87.7 / 112.4 us, the formula says 42.8 / 64.3 / 103.1 / 128.7 (1 % high, then 7 .. 18 %); down with its reduction, when all dies took all ranges,
// 35.6 / 51.4 / 69.5 / 74.8, the formula says 41.6 / 55.8 / 68.5 / 75.7 (17 and 9 % high, then within 1.5 %: the GEMM alone
// 13 .. 25 % low, the reduction 1.8 .. 2.7 times too long).
// Number of ranges when all dies took all of them, prefill in ms at 512 tokens with 6 / 7 / 8 / 10 / 12: 4.336 / 4.306 / 4.248 / 4.300 /
// 4.208 .. 4.31; 768 with 5 / 6 / 7 / 8 / 9: 5.523 / 5.451 / 5.393 / 5.393 / 5.425; 816 with 5 / 6 / 7 / 8: 5.998 / 5.948 / 6.033 / 6.038.
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
      gemm_lds_kernel<MT, NT, PRO, EPI, true><<<dim3(WALK_BLOCKS), dim3(256), LT_SMEM, s>>>(p);
      return hipGetLastError();
    }
  }
  p.range_per_die = EPI == EPI_PARTIAL && z == LDS_DIES;
  gemm_lds_kernel<MT, NT, PRO, EPI, false><<<p.range_per_die ? dim3(8 * total) : dim3(8 * ceil_div(total, 8), z), dim3(256), PRO != PRO_NONE ? LT_SMEM : lds_tile_smem(MT, NT), s>>>(p);
  return hipGetLastError();
}

template <int H, int EPI>
hipError_t cols_launch(hipStream_t s, GemmParams p) {
  p.m_tiles = ceil_div(p.M, 32 * H);
  const int total = ceil_div(p.n_tiles, COLS_TILES) * p.m_tiles;
  gemm_cols_kernel<H, EPI><<<dim3(EPI == EPI_PARTIAL ? 8 * total : 8 * ceil_div(total, 8)), dim3(256), LT_SMEM, s>>>(p);
  return hipGetLastError();
}

}  // namespace

bool gemm_lds_ok(int k_pad) { return k_pad % 128 == 0; }

// Eight ranges, one for each die, unless the cost finds fewer better.
// The line was drawn at 2048 features and k = 16384.  At other widths, pi0_prefill with as many ranges as the cost asks for up to 16, all dies
// on all of them -> this, features x k, 256 .. 768 tokens: where the cost asked for more than eight (k 16384 and 32768) +11 .. -2 % in speed, 1024 x 16384
// 685 / 773 / 972 / 1252 -> 692 / 710 / 915 / 1203 us at 256 / 263 / 512 / 768 tokens, 2048 x 32768 1412 / 1582 -> 1428 / 1611 at 256 / 263; with eight both
// times (512 and 1024 x 2048 .. 8192) mostly +1 .. +7 %.  Slower by more than 2 % is only a range of less than 1024 that
// keeps all units of a die busy, whose reduction then waits for the partial sums: 1024 x 4096 at 768 tokens 781 -> 825, 1280 x 4096 at 512
// 718 -> 764, 768 x 4096 at 544 629 -> 645, 1024 x 6144 at 768 858 -> 882; next to them, 1280 x 4096 at 544, the same rule gains (809 -> 795).
int gemm_lds_splits(int M, int n_tiles, int k_pad, int z_max, bool cols) {
  int best_z = 1;
  float best = -1.f;
  for (int z = 1; z <= z_max && z <= LDS_DIES; z++) {
    const int kps = round_up(ceil_div(k_pad, z), 128);
    if (ceil_div(k_pad, kps) != z) continue;   // a range would be empty
#define X(MT, NT)                                                                       \
  {                                                                                     \
    const float c = lds_tile_cost(MT, NT, M, n_tiles, kps, z, true);                    \
    if (best < 0.f || c < best) { best = c; best_z = z; }                               \
  }
    LDS_TILES(X)
#undef X
  }
  // where eight ranges fit gemm_cols_body's height, they are the better choice (the same 1024 rows of k as above)
  const int kps = round_up(ceil_div(k_pad, LDS_DIES), 128);
  if (cols && z_max >= LDS_DIES && kps >= 1024 && ceil_div(k_pad, kps) == LDS_DIES && gemm_cols_height(M, n_tiles, k_pad, kps, LDS_DIES, true) != 0) return LDS_DIES;
  return best_z;
}

void gemm_lds_tile(int M, int n_tiles, int k_pad, int k_per_split, int z, bool partial, int* mt, int* nt) {
  if (partial && z == LDS_DIES) {
    int best = 0, rounds_best = 0;   // (whole turns of the loop in every range)
#define X(MT, NT)                                                                                                     \
  {                                                                                                                   \
    const int rounds = ceil_div(ceil_div(M, 64 * MT) * ceil_div(n_tiles, 2 * NT), 32), c = rounds * MT * NT;          \
    if (k_per_split % lds_tile_group(MT, NT) == 0 && k_pad % lds_tile_group(MT, NT) == 0 && (best == 0 || c < best || (c == best && rounds < rounds_best))) { \
      best = c; rounds_best = rounds; *mt = MT; *nt = NT;                                                             \
    }                                                                                                                 \
  }
    LDS_RANGE_TILES(X)
#undef X
    return;
  }
  float best = -1.f;
#define X(MT, NT)                                                                       \
  {                                                                                     \
    const float c = lds_tile_cost(MT, NT, M, n_tiles, k_per_split, z, partial);         \
    if (best < 0.f || c < best) { best = c; *mt = MT; *nt = NT; }                       \
  }
  LDS_TILES(X)
#undef X
}

// Height of gemm_cols_body's tiles where a compute unit then gets fewer products than with the tile of gemm_lds_tile (rounds of the chip's, or a
// die's, blocks x products of a wave and step), else 0.  2048 features, k 2048 (gate||up) and 16384 (down), pi0_prefill in ms, gemm_lds_body -> this:
//   513 .. 576 tokens  gate||up 2 x 12 -> 18:             515 4.67 -> 4.47, 533 4.77 -> 4.54, 560 4.79 -> 4.58
//   769 .. 896         gate||up 2 x 16 -> 2 x 14:         771 6.09 -> 5.92, 816 6.26 -> 5.98
//                      down, eight ranges, 16 -> 14:      771 5.91 -> 5.78, 816 5.99 -> 5.88 (six ranges of gemm_lds_body: 5.98)
// Not up to 512 tokens: the persistent prefix has gemm_lds_body's tiles there.
int gemm_cols_height(int M, int n_tiles, int k_pad, int k_per_split, int z, bool partial) {
  if (M <= 512 || k_pad % (16 * COLS_GROUP) != 0 || k_per_split % (16 * COLS_GROUP) != 0 || (partial && z != LDS_DIES)) return 0;
  const int units = partial ? 256 / LDS_DIES : 256;
  int mt, nt;
  gemm_lds_tile(M, n_tiles, k_pad, k_per_split, z, partial, &mt, &nt);
  int best = 0, cost = ceil_div(ceil_div(M, 64 * mt) * ceil_div(n_tiles, 2 * nt), units) * mt * nt;
#define X(H, EPI)                                                                                                       \
  if (partial == (EPI == EPI_PARTIAL)) {                                                                                \
    const int c = ceil_div(ceil_div(M, 32 * H) * ceil_div(n_tiles, COLS_TILES), units) * H * COLS_NT;                   \
    if (c < cost) { cost = c; best = H; }                                                                               \
  }
  COLS_HEIGHTS(X)
#undef X
  return best;
}

hipError_t gemm_lds_init_attributes() {
  hipError_t e = hipSuccess;
#define X(MT, NT)                                                                                                                       \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_RMS, EPI_GEGLU, false>),             \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, LT_SMEM);
  LDS_TILES(X)
#undef X
#define X(MT, NT)                                                                                                                       \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_NONE, EPI_PARTIAL, false>),          \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_tile_smem(MT, NT));
  LDS_RANGE_TILES(X)
#undef X
#define X(MT, NT)                                                                                                                       \
  if constexpr (MT * NT <= 12)                                                                                                          \
    if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_lds_kernel<MT, NT, PRO_RMS, EPI_GEGLU, MT * NT <= 12>), \
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LT_SMEM);
  LDS_TILES(X)
#undef X
#define X(H, EPI)                                                                                                                          \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_cols_kernel<H, EPI>), hipFuncAttributeMaxDynamicSharedMemorySize, LT_SMEM);
  COLS_HEIGHTS(X)
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
  // (partial row statistics beyond 512 rows: only where pi0_tune leaves out the launch that adds them up)
  const int height = epi == EPI_GEGLU && p.rowstat_parts > 1 ? 0 : gemm_cols_height(p.M, p.n_tiles, p.W.k_pad, p.k_per_split, z, epi == EPI_PARTIAL);
#define X(H, EPI) if (height == H && epi == EPI) return cols_launch<H, EPI>(s, p);
  COLS_HEIGHTS(X)
#undef X
  int mt, nt;
  gemm_lds_tile(p.M, p.n_tiles, p.W.k_pad, p.k_per_split, z, epi == EPI_PARTIAL, &mt, &nt);
#define X(MT, NT)                                                                                            \
  if (epi == EPI_GEGLU && mt == MT && nt == NT) return lds_tile_launch<MT, NT, PRO_RMS, EPI_GEGLU>(s, p, z);
  LDS_TILES(X)
#undef X
#define X(MT, NT)                                                                                            \
  if (epi == EPI_PARTIAL && mt == MT && nt == NT) return lds_tile_launch<MT, NT, PRO_NONE, EPI_PARTIAL>(s, p, z);
  LDS_RANGE_TILES(X)
#undef X
  return hipErrorInvalidValue;
}
