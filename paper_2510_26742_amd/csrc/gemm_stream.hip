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
// Measured, when they came, against what ran before (LDS-staged tiles, split-K with a reduction launch for the residual projections), us per
// launch in a graph with cold weights at 256 / 512 / 768 tokens: vision QKV 10.5 / 13.8 / 20.1 -> 8.8 / 12.1 / 16.9, up
// 13.1 / 19.4 / 20.6 -> 11.2 / 16.4 / 18.6, O 7.6 / 13.6 / 20.4 -> 6.0 / 7.6 / 8.4, down 17.4 / 23.2 / 31.3 -> 13.8 / 18.6 / 19.4,
// prefix QKV 15.0 / 18.4 / 24.2 -> 11.1 / 14.3 / 17.2, prefix O 11.3 / 20.7 / 25.5 -> 9.5 / 12.0 / 16.4.  Not for the prefix's
// feed-forward GEMMs, which are large enough to be bound by the matrix pipe.
// The epilogue (partial tiles through LDS, sums, norm, activation, stores) then took 2 .. 7 us of these: a tile's columns by
// lane put 16-byte pieces of 32 rows into every store of a residual row, half of the waves had nothing to do, and each
// element cost some 25 instructions of one wave per SIMD.  Traced passes of both on one device (a traced launch reads up to 1.5 us
// longer), us per launch at 256 / 512 / 768 tokens, before -> now: vision O 7.5 / 8.2 / 9.1 -> 6.6 / 7.7 / 8.5, down
// 14.4 / 17.9 / 19.4 -> 13.3 / 17.2 / 18.7, up 11.2 / 16.5 / 18.7 -> 11.0 / 15.1 / 18.3, prefix O 10.6 / 13.2 / 17.8 -> 9.5 / 12.1 / 15.8,
// projector 9.1 / 10.2 / 17.8 -> 7.8 / 10.0 / 12.8.  QKV gained nothing, except vision's at three views: vision 8.9 / 13.2 / 18.3 -> 8.9 / 13.2 / 16.7,
// prefix 11.9 / 15.7 / 19.3 -> 11.9 / 15.5 / 19.7.
#include "pi0_internal.h"

#include "gemm_stream_body.h"

namespace {

constexpr int STREAM_PARTS_MAX = 64;           // most planes of partial row statistics

// groups in which a launch adds up the planes of row statistics: one per group of threads that covers the block's rows
template <int MB, int W>
constexpr int stream_groups() { return 64 * W / (MB * 32); }

template <int MB, int NB, int W, int D, int PRO, int EPI>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void gemm_stream_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  LaunchCtx cx{(int)blockIdx.x, 0, 0};
  gemm_stream_body<MB, NB, W, 1, D, stream_groups<MB, W>(), STREAM_PARTS_MAX, 0, PRO, EPI>(p, cx, smem_raw);
}

template <int MB, int NB, int W, int EPI>
constexpr int stream_smem_bytes() {
  return stream_body_smem<MB, NB, W, stream_groups<MB, W>(), EPI>();
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
// blocks than compute units takes a whole further round.  It ranks tiles and does not predict a time: against traced passes at
// 256 / 512 / 768 / 816 tokens it reads 5 .. 20 % low for QKV and up, 13 .. 22 % for vision O, 10 .. 20 % for prefix O, 28 .. 34 % for
// the projector, and 1 .. 6 % high for vision down.
float stream_cost(int mb, int nb, int m, int n_tiles, int kc16) {
  const int blocks = ceil_div(ceil_div(m, 32), mb) * ceil_div(n_tiles, nb);
  return (float)ceil_div(blocks, 256) * ((float)((mb + nb) * kc16) * 0.0145f + (float)(mb * nb) * 0.5f + 1.0f);
}

template <int MB, int NB, int W, int D, int PRO, int EPI>
hipError_t stream_launch(hipStream_t s, GemmParams p) {
  p.m_tiles = ceil_div(p.M, MB * 32);
  const int total = ceil_div(p.n_tiles, NB) * p.m_tiles;
  gemm_stream_kernel<MB, NB, W, D, PRO, EPI><<<dim3(8 * ceil_div(total, 8)), dim3(64 * W), stream_smem_bytes<MB, NB, W, EPI>(), s>>>(p);
  return hipGetLastError();
}

struct StreamChoice {
  hipError_t (*launch)(hipStream_t, GemmParams);
  int mb, nb, parts;   // token blocks and feature tiles of a block, waves
};
// value_tile: feature tile of QKV's output that the values start at, where the last 32-token chunk is incomplete, else 0.  Blocks of
// nothing but values then store the rest of the chunk as zeros (zero_values says why), so no block may straddle that boundary;
// the same stores in the blocks that straddle it would cost every QKV launch their code (3 views 9.704 -> 9.741 ms)
StreamChoice stream_choose(int pro, int epi, int M, int n_tiles, int kc16, int value_tile = 0) {
  StreamChoice best{nullptr, 0, 0, 0};
  float cost = 0.f;
#define X(MB, NB, W, D)                                                   \
  {                                                                       \
    const float c = stream_cost(MB, NB, M, n_tiles, kc16);                \
    if (value_tile % NB == 0 && (best.launch == nullptr || c < cost)) { cost = c; best = StreamChoice{&stream_launch<MB, NB, W, D, SPRO, SEPI>, MB, NB, W}; } \
  }
#define Y(PRO, EPI, TILES_) if (pro == PRO && epi == EPI) { constexpr int SPRO = PRO, SEPI = EPI; TILES_(X) }
  STREAM_KINDS(Y)
#undef Y
#undef X
  return best;
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
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_stream_kernel<MB, NB, W, D, SPRO, SEPI>), hipFuncAttributeMaxDynamicSharedMemorySize, stream_smem_bytes<MB, NB, W, SEPI>());
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
  const int value_tile = epi == EPI_QKV && p.M % 32 != 0 ? (p.q_cols + p.k_cols) / 32 : 0;
  if (value_tile != 0 && (p.q_cols + p.k_cols) % 32 != 0) return hipErrorInvalidValue;   // (views are whole chunks, a prefix has heads of 256)
  const StreamChoice c = stream_choose(pro, epi, p.M, p.n_tiles, p.W.k_pad >> 4, value_tile);
  return c.launch == nullptr ? hipErrorInvalidValue : c.launch(s, p);
}

int gemm_stream_stat_planes(int pro, int M, int n_tiles, int k_pad) {
  const StreamChoice c = stream_choose(pro, EPI_RESID, M, n_tiles, k_pad >> 4);
  return c.launch == nullptr ? 0 : ceil_div(n_tiles, c.nb);
}

bool gemm_stream_tile(int pro, int epi, int M, int n_tiles, int k_pad, int* mb, int* nb, int* parts, int value_tile) {
  const StreamChoice c = stream_choose(pro, epi, M, n_tiles, k_pad >> 4, value_tile);
  *mb = c.mb;
  *nb = c.nb;
  *parts = c.parts;
  return c.launch != nullptr;
}
