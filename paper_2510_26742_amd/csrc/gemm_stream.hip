// Mid-size bf16 GEMMs of the vision tower and the prefix (256 .. 816 tokens): the k range is split over the waves of a
// block, and every wave streams its operands straight into MFMA registers.
//
// Orientation and epilogues as in gemm.hip (weights are the A operand, tokens the B operand, both in fragment order).
// A block owns MB x NB tiles of 32 tokens x 32 features over the WHOLE k range; each of its W waves accumulates all of
// them over its own k16 steps (w, w + W, ...), the partial tiles meet in LDS and are added in wave order.  Since no two
// waves of a block read the same operand bytes there is nothing to stage through LDS: no barrier, no LDS traffic in the
// main loop, and a wave's D stages in flight are hidden by nothing but its own wait counter.  The block pulls
// (MB + NB) * 32 * k * 2 bytes through its compute unit's vector-memory path, the least that a tile of its size can.
// That path is the bound: 30 .. 75 GB/s per compute unit (the longer k, the more), a 32 KB L1 over the latency of what
// it misses; deeper stages, non-temporal loads and another order of loads and products change nothing.
// Measured against what ran before (LDS-staged tiles, split-K with a reduction launch for the residual projections), us per
// launch in a graph with cold weights at 256 / 512 / 768 tokens: vision QKV 10.5 / 13.8 / 20.1 -> 8.8 / 12.1 / 16.9, up
// 13.1 / 19.4 / 20.6 -> 11.2 / 16.4 / 18.6, O 7.6 / 13.6 / 20.4 -> 6.0 / 7.6 / 8.4, down 17.4 / 23.2 / 31.3 -> 13.8 / 18.6 / 19.4,
// prefix QKV 15.0 / 18.4 / 24.2 -> 11.1 / 14.3 / 17.2, prefix O 11.3 / 20.7 / 25.5 -> 9.5 / 12.0 / 16.4.  Not for the prefix's
// feed-forward GEMMs, which are large enough to be bound by the matrix pipe.
#include "pi0_internal.h"

#include "gemm_common.h"

namespace {

constexpr int STREAM_RED_BYTES = 128 * 1024;   // partial tiles of one round: W waves x TPR tiles x 4 KiB
constexpr int STREAM_PARTS_MAX = 64;           // most planes of partial row statistics

template <int MB, int NB, int W, int D, int PRO, int EPI>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void gemm_stream_kernel(GemmParams p) {
  constexpr int TILES = MB * NB;
  constexpr int ROUNDS = (TILES * W * 4096 + STREAM_RED_BYTES - 1) / STREAM_RED_BYTES;
  constexpr int TPR = (TILES + ROUNDS - 1) / ROUNDS;                      // tiles per round
  constexpr int PIECES = EPI == EPI_RESID ? 1 : (W >= 4 * TPR ? 4 : W >= 2 * TPR ? 2 : 1);   // waves that share a tile's epilogue
  constexpr int UPW = (TPR * PIECES + W - 1) / W;                         // pieces a wave finishes per round
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  float* red = reinterpret_cast<float*>(smem_raw);                        // [W][TPR][4][64][4]
  float2* sstat = reinterpret_cast<float2*>(smem_raw + W * TPR * 4096);   // [groups][MB * 32]
  float* cols = reinterpret_cast<float*>(sstat + 64 * W);                 // [bias, column sums, gain][NB * 32]

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;

  // Consecutive block ids go to different dies (an L2 each).  A die takes a contiguous eighth of the tiles, token tiles
  // fastest: the tiles that share a weight panel meet in one L2, and no die has more than one tile more than another
  // (whole panels dealt to dies in turn gave 18 panels x 12 token tiles as 36 blocks to two dies of 32 compute units).
  const int nblocks_n = (p.n_tiles + NB - 1) / NB;
  const int total = nblocks_n * p.m_tiles;
  const int die = (int)blockIdx.x & 7, die_rank = (int)blockIdx.x >> 3;
  const int first = die * (total >> 3) + min(die, total & 7);
  if (die_rank >= (total >> 3) + (die < (total & 7) ? 1 : 0)) return;
  const int nb = (first + die_rank) / p.m_tiles;
  const int mt = (first + die_rank) - nb * p.m_tiles;
  const int nt0 = nb * NB;
  const int m0 = mt * MB * 32;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4;
  const int XKC16 = p.ldx >> 4;
  const int per = (KC16 + W - 1) / W;
  const int n = max(0, min(per, KC16 - w * per));   // this wave's k16 steps: w * per .. + n - 1

  const char* wb[NB];
  const char* xb[MB];
#pragma unroll
  for (int j = 0; j < NB; j++) wb[j] = reinterpret_cast<const char*>(p.W.w) + (size_t)min(nt0 + j, p.n_tiles - 1) * KC16 * 1024;
#pragma unroll
  for (int i = 0; i < MB; i++) xb[i] = reinterpret_cast<const char*>(p.X) + (size_t)min((m0 >> 5) + i, mb_last) * XKC16 * 1024;
  const unsigned voff = (unsigned)(min(w * per, KC16 - 1) * 1024 + lane * 16);
  // Blocks and waves start at different steps of their range and wrap around: in step, the 32 compute units of a die ask
  // for addresses that are a power of two apart and meet in the same few cache channels (vision down at 512 tokens
  // 22.0 -> 18.5 us, prefix QKV at 256 tokens 12.4 -> 11.1 us).
  const int rot = (int)((unsigned)(nb * 3 + mt * 5 + w * 7) % (unsigned)max(n, 1));

  bf16x8 wr[D][NB], xr[D][MB];
  auto issue = [&](int u, int i) {
    const int k = i + rot;
    const unsigned off = voff + (unsigned)(k < n ? k : max(k - n, 0)) * 1024u;
#pragma unroll
    for (int j = 0; j < NB; j++) wr[u][j] = *reinterpret_cast<const bf16x8*>(wb[j] + off);
#pragma unroll
    for (int b = 0; b < MB; b++) xr[u][b] = *reinterpret_cast<const bf16x8*>(xb[b] + off);
  };
  f32x16 acc[TILES];   // tile b * NB + j
#pragma unroll
  for (int k = 0; k < TILES; k++)
#pragma unroll
    for (int r = 0; r < 16; r++) acc[k][r] = 0.f;
  auto multiply = [&](int u) {
#pragma unroll
    for (int b = 0; b < MB; b++)
#pragma unroll
      for (int j = 0; j < NB; j++)
        acc[b * NB + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[u][j], xr[u][b], acc[b * NB + j], 0, 0, 0);
  };

#pragma unroll
  for (int u = 0; u < D; u++) issue(u, max(0, min(u, n - 1)));
  // Row statistics of the block's rows, behind the first stages: whole-row sums, or one partial sum per 32-column tile
  // of the producer (thread group g adds planes g, g + G, ...; the groups are added in order in the epilogue)
  constexpr int G = 64 * W / (MB * 32);
  constexpr int PPG = (STREAM_PARTS_MAX + G - 1) / G;
  if (PRO != PRO_NONE && t < G * MB * 32) {
    const int row = t % (MB * 32), g = t / (MB * 32);
    const size_t rowg = (size_t)min(m0 + row, p.M - 1);
    const int parts = p.rowstat_parts > 1 ? p.rowstat_parts : 1;
    float a = 0.f, b = 0.f;
    float2 v[PPG];
#pragma unroll
    for (int jj = 0; jj < PPG; jj++) {
      v[jj] = make_float2(0.f, 0.f);
      if (g + G * jj < parts) v[jj] = *reinterpret_cast<const float2*>(p.rowstat + 2 * ((size_t)(g + G * jj) * p.stat_rows + rowg));
    }
#pragma unroll
    for (int jj = 0; jj < PPG; jj++) {
      a += v[jj].x;
      b += v[jj].y;
    }
    sstat[g * (MB * 32) + row] = make_float2(a, b);
  }

  // column vectors and RoPE rows of the epilogue, behind the first stages too (residual rows this early cost the small
  // tiles more than the round trip they save at the end: vision O at 256 tokens 6.0 -> 6.4 us)
  if (t < NB * 32) {
    const int col = min(nt0 * 32 + t, p.W.n_pad - 1);
    if (p.bias != nullptr) cols[t] = p.bias[col];
    if (PRO == PRO_LN) cols[NB * 32 + t] = p.colsum[col];
    if (EPI == EPI_RESID && p.gain != nullptr) cols[2 * NB * 32 + t] = p.gain[min(col, p.n_valid - 1)];
  }
  f32x4 rope[ROUNDS][UPW][4 / PIECES];
  if (EPI == EPI_QKV && p.rope != nullptr) {
#pragma unroll
    for (int rd = 0; rd < ROUNDS; rd++)
#pragma unroll
      for (int v = 0; v < UPW; v++) {
        const int unit = w + W * v, tile = rd * TPR + unit / PIECES, pc = unit % PIECES;
        const int m = m0 + (tile / NB) * 32 + lq;
#pragma unroll
        for (int q = 0; q < 4 / PIECES; q++) {
          const int n4 = (nt0 + tile % NB) * 32 + 8 * (pc * (4 / PIECES) + q) + 4 * lh;
          if (unit < TPR * PIECES && tile < TILES && m < p.M && n4 < p.q_cols + p.k_cols) {
            const int nl = n4 < p.q_cols ? n4 : n4 - p.q_cols;
            rope[rd][v][q] = *reinterpret_cast<const f32x4*>(p.rope + ((size_t)(p.pos0 + m) * 128 + ((nl & 255) >> 1)) * 2);
          }
        }
      }
  }

  int i = 0;
  for (; i + 2 * D <= n; i += D) {
#pragma unroll
    for (int u = 0; u < D; u++) {
      multiply(u);
      issue(u, i + u + D);
    }
  }
  // the last D .. 2 D - 1 steps (all of them if there are fewer)
#pragma unroll
  for (int u = 0; u < D; u++) {
    if (i + u < n) {
      multiply(u);
      if (i + u + D < n) issue(u, i + u + D);
    }
  }
#pragma unroll
  for (int u = 0; u < D - 1; u++) {
    if (i + u + D < n) multiply(u);
  }

  // ---- partial tiles -> LDS, fixed-order sums, epilogue --------------------------------------------
#pragma unroll
  for (int rd = 0; rd < ROUNDS; rd++) {
    f32x4 resid[UPW][4];   // requested here: their round trip overlaps the sums through LDS
    if (EPI == EPI_RESID && p.resid != nullptr) {
#pragma unroll
      for (int v = 0; v < UPW; v++) {
        const int unit = w + W * v, tile = rd * TPR + unit;
        const int m = m0 + (tile / NB) * 32 + lq;
        const int rr = p.resid_mod > 0 ? m % p.resid_mod : m;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int n4 = (nt0 + tile % NB) * 32 + 8 * q + 4 * lh;
          if (unit < TPR && tile < TILES && m < p.M && n4 < p.n_valid)
            resid[v][q] = *reinterpret_cast<const f32x4*>(p.resid + (size_t)rr * p.ldo + n4);
        }
      }
    }
    if (rd) __syncthreads();   // the readers of the round before are done
#pragma unroll
    for (int k = 0; k < TPR; k++) {
      if (rd * TPR + k < TILES) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const f32x16& a = acc[rd * TPR + k < TILES ? rd * TPR + k : 0];
          const f32x4 v4 = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
          *reinterpret_cast<f32x4*>(red + ((((size_t)w * TPR + k) * 4 + q) * 64 + lane) * 4) = v4;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < UPW; v++) {
      const int unit = w + W * v, tile = rd * TPR + unit / PIECES, pc = unit % PIECES;
      const int nt = nt0 + tile % NB, row = (tile / NB) * 32 + lq, m = m0 + row;
      if (unit < TPR * PIECES && tile < TILES && nt < p.n_tiles && m < p.M) {
        float ssum = 0.f, ssq = 0.f;
        if (PRO != PRO_NONE) {
#pragma unroll
          for (int g = 0; g < G; g++) {
            const float2 s2 = sstat[g * (MB * 32) + row];
            ssum += s2.x;
            ssq += s2.y;
          }
        }
        constexpr int NSTEP = 4 / PIECES;
        const int ib = pc * NSTEP;
        f32x16 sum;
#pragma unroll
        for (int r = 0; r < 16; r++) sum[r] = 0.f;
#pragma unroll
        for (int ww = 0; ww < W; ww++)
#pragma unroll
          for (int q = 0; q < NSTEP; q++) {
            const f32x4 v4 = *reinterpret_cast<const f32x4*>(red + ((((size_t)ww * TPR + unit / PIECES) * 4 + ib + q) * 64 + lane) * 4);
#pragma unroll
            for (int jj = 0; jj < 4; jj++) sum[4 * q + jj] += v4[jj];
          }
        EpiOps ops;
#pragma unroll
        for (int q = 0; q < NSTEP; q++) {
          const float* c4 = cols + (tile % NB) * 32 + 8 * (ib + q) + 4 * lh;
          ops.bias[q] = p.bias != nullptr ? *reinterpret_cast<const f32x4*>(c4) : f32x4{0.f, 0.f, 0.f, 0.f};
          if (PRO == PRO_LN) ops.colsum[q] = *reinterpret_cast<const f32x4*>(c4 + NB * 32);
          if (EPI == EPI_RESID && p.gain != nullptr) ops.gain[q] = *reinterpret_cast<const f32x4*>(c4 + 2 * NB * 32);
          if (EPI == EPI_RESID) ops.aux[q] = resid[v][q];
          if (EPI == EPI_QKV) ops.aux[q] = rope[rd][v][q];
        }
        epilogue_tile<PRO, EPI, 0, NSTEP>(p, sum, nt, m, lh, ssum, ssq, 0, ops, LaunchCtx{}, ib);
      }
    }
  }
}

template <int MB, int NB, int W>
constexpr int stream_smem_bytes() {
  constexpr int tiles = MB * NB, rounds = (tiles * W * 4096 + STREAM_RED_BYTES - 1) / STREAM_RED_BYTES;
  return W * ((tiles + rounds - 1) / rounds) * 4096 + 64 * W * 8 + 3 * NB * 32 * 4;
}

// Tiles that exist: X(token blocks, feature tiles, waves, stages in flight).  8 waves of 256 registers for up to 8
// accumulator tiles, 4 waves of 512 beyond.
#define STREAM_WIDE(X) X(2, 2, 8, 6) X(2, 3, 8, 4) X(2, 4, 4, 8) X(3, 3, 4, 8) X(3, 4, 4, 6) X(4, 4, 4, 5)
#define STREAM_NARROW(X) X(1, 2, 8, 9) X(2, 1, 8, 9) X(3, 1, 8, 8) X(2, 2, 8, 6) X(3, 2, 8, 5) X(4, 2, 8, 3)
// Y(PRO, EPI, its tiles): residual projections are narrow (1152 or 2048 features), QKV and up are wide
#define STREAM_KINDS(Y)                  \
  Y(PRO_LN, EPI_QKV, STREAM_WIDE)        \
  Y(PRO_RMS, EPI_QKV, STREAM_WIDE)       \
  Y(PRO_LN, EPI_BF16, STREAM_WIDE)       \
  Y(PRO_NONE, EPI_RESID, STREAM_NARROW)  \
  Y(PRO_LN, EPI_RESID, STREAM_NARROW)

// Estimated time of a launch in us, fitted to a sweep of single launches over the vision and prefix shapes at 256 / 512 / 768
// tokens: a compute unit pulls one KiB fragment per 14.5 ns whatever the tile (70 GB/s: what its 32 KB L1 can have
// in flight over the latency beyond it), an accumulator tile costs 0.5 us of sums and epilogue, and a launch of more
// blocks than compute units takes a whole further round.  It ranks tiles and does not predict a time: in a traced pass at
// 256 .. 816 tokens it reads low by 6 .. 24 % for QKV and up, 3 .. 13 % for vision O and down together, 21 .. 28 % for prefix O
// and 29 .. 47 % for the projector (8.9 us at 256 tokens, 17.5 at 768).
float stream_cost(int mb, int nb, int m, int n_tiles, int kc16) {
  const int blocks = ceil_div(ceil_div(m, 32), mb) * ceil_div(n_tiles, nb);
  return (float)ceil_div(blocks, 256) * ((float)((mb + nb) * kc16) * 0.0145f + (float)(mb * nb) * 0.5f + 1.0f);
}

template <int MB, int NB, int W, int D, int PRO, int EPI>
hipError_t stream_launch(hipStream_t s, GemmParams p) {
  p.m_tiles = ceil_div(p.M, MB * 32);
  const int total = ceil_div(p.n_tiles, NB) * p.m_tiles;
  gemm_stream_kernel<MB, NB, W, D, PRO, EPI><<<dim3(8 * ceil_div(total, 8)), dim3(64 * W), stream_smem_bytes<MB, NB, W>(), s>>>(p);
  return hipGetLastError();
}

// whole-row sums of partial row statistics [planes][stat_rows][2]: 32 rows per block, 8 thread groups share the planes
__global__ __launch_bounds__(256) void row_sums_kernel(const float* parts, int planes, int stat_rows, int M, float* out) {
  __shared__ float2 sums[8][32];
  const int r = threadIdx.x & 31, g = threadIdx.x >> 5;
  const int m = min((int)blockIdx.x * 32 + r, M - 1);
  float a = 0.f, b = 0.f;
  for (int j0 = g; j0 < planes; j0 += 64) {   // 8 loads in flight: one round trip for up to 64 planes
    float2 v[8];
#pragma unroll
    for (int j = 0; j < 8; j++)
      v[j] = *reinterpret_cast<const float2*>(parts + 2 * ((size_t)min(j0 + 8 * j, planes - 1) * stat_rows + m));   // clamped, unconditional
#pragma unroll
    for (int j = 0; j < 8; j++) {
      if (j0 + 8 * j < planes) {
        a += v[j].x;
        b += v[j].y;
      }
    }
  }
  sums[g][r] = make_float2(a, b);
  __syncthreads();
  if (g != 0 || (int)blockIdx.x * 32 + r >= M) return;
#pragma unroll
  for (int i = 1; i < 8; i++) {
    a += sums[i][r].x;
    b += sums[i][r].y;
  }
  *reinterpret_cast<float2*>(out + 2 * (size_t)m) = make_float2(a, b);
}

}  // namespace

hipError_t launch_row_sums(hipStream_t s, const float* parts, int planes, int stat_rows, int M, float* out) {
  if (parts == nullptr || out == nullptr || planes < 1 || M < 1 || stat_rows < M) return hipErrorInvalidValue;
  hipLaunchKernelGGL(row_sums_kernel, dim3(ceil_div(M, 32)), dim3(256), 0, s, parts, planes, stat_rows, M, out);
  return hipGetLastError();
}

hipError_t gemm_stream_init_attributes() {
  hipError_t e = hipSuccess;
#define X(MB, NB, W, D) \
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_stream_kernel<MB, NB, W, D, SPRO, SEPI>), hipFuncAttributeMaxDynamicSharedMemorySize, stream_smem_bytes<MB, NB, W>());
#define Y(PRO, EPI, TILES_) { constexpr int SPRO = PRO, SEPI = EPI; TILES_(X) }
  STREAM_KINDS(Y)
#undef Y
#undef X
  return e;
}

hipError_t launch_gemm_stream(hipStream_t s, int pro, int epi, const GemmParams& p) {
  // everything the kernel's indexing assumes
  if (p.X == nullptr || p.W.w == nullptr || p.M <= 0 || p.pf.blocks != 0) return hipErrorInvalidValue;
  if (p.W.k_pad < 64 || p.W.k_pad % 64 != 0 || p.n_tiles < 1 || p.n_tiles * 32 != p.W.n_pad || p.ldx < p.W.k_pad || p.ldx % 16 != 0) return hipErrorInvalidValue;
  if ((size_t)p.W.k_pad * 64 > 0x7fffffffu) return hipErrorInvalidValue;   // a row of fragments is addressed with 32 bits
  if (pro != PRO_NONE && (p.rowstat == nullptr || p.rowstat_parts > STREAM_PARTS_MAX || (p.rowstat_parts > 1 && p.stat_rows < p.M))) return hipErrorInvalidValue;
  if (pro == PRO_LN && p.colsum == nullptr) return hipErrorInvalidValue;
  if (epi == EPI_RESID && (p.out_f32 == nullptr || p.out_bf16 == nullptr || p.ldo % 4 != 0 || p.ldo2 % 16 != 0 || (p.stat_out != nullptr && p.stat_rows < p.M + p.row_offset)))
    return hipErrorInvalidValue;
  const int kc16 = p.W.k_pad >> 4;
  hipError_t (*best)(hipStream_t, GemmParams) = nullptr;
  float cost = 0.f;
#define X(MB, NB, W, D)                                                   \
  {                                                                       \
    const float c = stream_cost(MB, NB, p.M, p.n_tiles, kc16);            \
    if (best == nullptr || c < cost) { cost = c; best = &stream_launch<MB, NB, W, D, SPRO, SEPI>; } \
  }
#define Y(PRO, EPI, TILES_) if (pro == PRO && epi == EPI) { constexpr int SPRO = PRO, SEPI = EPI; TILES_(X) }
  STREAM_KINDS(Y)
#undef Y
#undef X
  return best == nullptr ? hipErrorInvalidValue : best(s, p);
}
