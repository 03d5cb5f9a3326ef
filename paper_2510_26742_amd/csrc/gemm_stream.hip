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

#include "gemm_common.h"

namespace {

constexpr int STREAM_RED_BYTES = 144 * 1024;   // partial tiles of one round: W waves x TPR tiles x 4 KiB, at most this much
constexpr int STREAM_PARTS_MAX = 64;           // most planes of partial row statistics

// Rounds through LDS and tiles of a round; the residual epilogue takes whole token blocks, so that a row's columns are in one round
template <int MB, int NB, int W, int EPI>
struct StreamRounds {
  static constexpr int TILES = MB * NB;
  static constexpr int RB = STREAM_RED_BYTES / (NB * W * 4096) < MB ? STREAM_RED_BYTES / (NB * W * 4096) : MB;
  static constexpr int ROUNDS = EPI == EPI_RESID ? (MB + RB - 1) / RB : (TILES * W * 4096 + STREAM_RED_BYTES - 1) / STREAM_RED_BYTES;
  static constexpr int TPR = EPI == EPI_RESID ? RB * NB : (TILES + ROUNDS - 1) / ROUNDS;
};

// sum over groups of 16 adjacent lanes (sum8_dpp, then the other half of the row of 16)
__device__ __forceinline__ float sum16_dpp(float v) {
  v = sum8_dpp(v);
  return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));
}

template <int MB, int NB, int W, int D, int PRO, int EPI>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) void gemm_stream_kernel(GemmParams p) {
  using Rounds = StreamRounds<MB, NB, W, EPI>;
  constexpr int TILES = MB * NB, ROUNDS = Rounds::ROUNDS, TPR = Rounds::TPR;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  float* red = reinterpret_cast<float*>(smem_raw);                        // [W][TPR][8 groups of 4 columns][32 rows, rotated by the group][4]
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
  // Row statistics of the block's rows, behind the first stages: whole-row sums, or partial sums in planes, one per range of
  // columns that a block of the producer owned (thread group g adds planes g, g + G, ...; the groups are added in order in the epilogue)
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
    cols[t] = p.bias != nullptr ? p.bias[col] : 0.f;
    if (PRO == PRO_LN) cols[NB * 32 + t] = p.colsum[col];
    if (EPI == EPI_RESID) cols[2 * NB * 32 + t] = p.gain != nullptr ? p.gain[min(col, p.n_valid - 1)] : 1.f;
  }
  // A block of nothing but value features: 16-byte stores into the value fragments (2-byte ones otherwise)
  const bool values = EPI == EPI_QKV && nt0 * 32 >= p.q_cols + p.k_cols;

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
  // A tile lies in LDS as 8 groups of 4 consecutive accumulator rows, each group's 32 lanes rotated by its number: lanes
  // that go through the columns of a row (residual epilogue) then meet different banks, like those that go through the rows.
  auto part = [&](int ww, int k, int c4, int r) {
    return reinterpret_cast<f32x4*>(red + (((size_t)ww * TPR + k) * 8 + c4) * 128 + (((r + c4) & 31) * 4));
  };
  auto stat_sums = [&](int row, float& ssum, float& ssq) {
    ssum = ssq = 0.f;
#pragma unroll
    for (int g = 0; g < G; g++) {
      const float2 s2 = sstat[g * (MB * 32) + row];
      ssum += s2.x;
      ssq += s2.y;
    }
  };
  // of the norm in front: 1 / deviation and mean of a row
  const float inv_k = 1.0f / (float)p.k_true;
  auto scale_of = [&](int row, float& rs, float& mu) {
    rs = 1.f;
    mu = 0.f;
    if (PRO == PRO_NONE) return;
    float ssum, ssq;
    stat_sums(row, ssum, ssq);
    if (PRO == PRO_LN) mu = ssum * inv_k;
    rs = rsqrtf(PRO == PRO_LN ? fmaxf(ssq * inv_k - mu * mu, 0.f) + 1e-6f : ssq * inv_k + 1e-6f);
  };
#pragma unroll
  for (int rd = 0; rd < ROUNDS; rd++) {
    // residual epilogue: a unit is 8 / NB rows x all of the block's columns, a lane 4 columns of one row, so that rows are
    // read and written in whole cache lines
    constexpr int RL = 8 * NB, RU = TPR / NB * 4 * NB, RUPW = EPI == EPI_RESID ? (RU + W - 1) / W : 1;
    f32x4 resid[RUPW];   // requested here: their round trip overlaps the sums through LDS
    auto resid_at = [&](int v, int& k, int& row, int& c4, int& n4) {
      const int unit = w + W * v, bl = unit / (4 * NB), c = lane % RL;
      k = bl * NB + (c >> 3);
      c4 = c & 7;
      row = (rd * (TPR / NB) + bl) * 32 + unit % (4 * NB) * (8 / NB) + lane / RL;
      n4 = (nt0 + (c >> 3)) * 32 + 4 * c4;
      return unit < RU && row < MB * 32;
    };
    if (EPI == EPI_RESID && p.resid != nullptr) {
#pragma unroll
      for (int v = 0; v < RUPW; v++) {
        int k, row, c4, n4;
        const bool have = resid_at(v, k, row, c4, n4);
        const int m = m0 + row, rr = p.resid_mod > 0 ? m % p.resid_mod : m;
        if (have && m < p.M && n4 < p.n_valid) resid[v] = *reinterpret_cast<const f32x4*>(p.resid + (size_t)rr * p.ldo + n4);
      }
    }
    if (rd) __syncthreads();   // the readers of the round before are done
#pragma unroll
    for (int k = 0; k < TPR; k++) {
      if (rd * TPR + k < TILES) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const f32x16& a = acc[rd * TPR + k < TILES ? rd * TPR + k : 0];
          *part(w, k, 2 * q + lh, lq) = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
        }
      }
    }
    __syncthreads();
    if constexpr (EPI == EPI_RESID) {
      constexpr int VG = TILES < 8 ? RUPW : 1;   // units at a time: 8 accumulator tiles leave registers for one
#pragma unroll
      for (int v0 = 0; v0 < RUPW; v0 += VG) {
        f32x4 pt[VG][W], bias[VG], gain[VG];
        float rs[VG], mu[VG];
#pragma unroll
        for (int v = 0; v < VG; v++) {
          int k, row, c4, n4;
          resid_at(v0 + v, k, row, c4, n4);
#pragma unroll
          for (int ww = 0; ww < W; ww++) pt[v][ww] = *part(ww, min(k, TPR - 1), c4, row & 31);
          const float* const c = cols + n4 - nt0 * 32;
          bias[v] = *reinterpret_cast<const f32x4*>(c);
          gain[v] = *reinterpret_cast<const f32x4*>(c + 2 * NB * 32);
          scale_of(min(row, MB * 32 - 1), rs[v], mu[v]);
        }
        __builtin_amdgcn_sched_barrier(0);   // every read in flight (left alone they are read and added one by one)
#pragma unroll
        for (int v = 0; v < VG; v++) {
          int k, row, c4, n4;
          const bool have = resid_at(v0 + v, k, row, c4, n4);
          const int m = m0 + row, mo = m + p.row_offset;
          const bool live = have && m < p.M && n4 < p.n_valid;
          f32x4 x = pt[v][0];
#pragma unroll
          for (int ww = 1; ww < W; ww++) x += pt[v][ww];
          if (PRO == PRO_RMS) x *= rs[v];
          if (PRO == PRO_LN) x = rs[v] * (x - mu[v] * *reinterpret_cast<const f32x4*>(cols + n4 - nt0 * 32 + NB * 32));
          x += bias[v];
          if (p.resid != nullptr) x += resid[v0 + v];
          const f32x4 y = x * gain[v];
          float st_a = 0.f, st_b = 0.f;
          if (live) {
            *reinterpret_cast<f32x4*>(p.out_f32 + (size_t)mo * p.ldo + n4) = x;
            *reinterpret_cast<bf16x4*>(p.out_bf16 + xf_index(mo, n4, p.ldo2 >> 4)) = bf16x4{(bf16)y[0], (bf16)y[1], (bf16)y[2], (bf16)y[3]};
#pragma unroll
            for (int j = 0; j < 4; j++) {
              st_a += x[j];
              st_b += x[j] * x[j];
            }
          }
          if (p.stat_out != nullptr) {   // the row's sums over the block's columns, one plane per block column
            st_a = NB == 2 ? sum16_dpp(st_a) : sum8_dpp(st_a);
            st_b = NB == 2 ? sum16_dpp(st_b) : sum8_dpp(st_b);
            if (lane % RL == 0 && have && m < p.M)
              *reinterpret_cast<float2*>(p.stat_out + ((size_t)nb * p.stat_rows + mo) * 2) = make_float2(st_a, st_b);
          }
        }
      }
    } else {
      // What bounds this part is the number of instructions (one or two waves per SIMD, 4 cycles per vector instruction, 16 for
      // an exponential or a reciprocal) and the size of the code, which every launch fetches anew: whatever a unit's lanes
      // share is computed in scalar registers, an address is a uniform base plus 32 bits, row scales and column vectors are
      // fetched once, and every read of a group of units is in flight before the first sum.
      float rs[MB], mu[MB];
#pragma unroll
      for (int b = 0; b < MB; b++) scale_of(b * 32 + lq, rs[b], mu[b]);
      if (EPI == EPI_QKV && values) {   // uniform
        // A unit is 16 tokens of a tile: a lane takes 8 of them of one feature (lane % 32) from LDS, which are the 16-byte
        // piece of the value fragments with tokens 4 lh .. + 3 and 8 + 4 lh .. + 3; tokens beyond the last come out as zeros
        constexpr int VUPW = (TPR * 2 + W - 1) / W;
        float pt[VUPW][W][8];
        const int s2 = w & 1;
        auto tile_at = [&](int v, int& k) {
          k = min((W / 2) * v + (w >> 1), TPR - 1);
          return rd * TPR + (W / 2) * v + (w >> 1);
        };
#pragma unroll
        for (int v = 0; v < VUPW; v++) {
          int k;
          tile_at(v, k);
#pragma unroll
          for (int e = 0; e < 8; e++)
#pragma unroll
            for (int ww = 0; ww < W; ww++) pt[v][ww][e] = reinterpret_cast<const float*>(part(ww, k, lq >> 2, 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3)))[lq & 3];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int v = 0; v < VUPW; v++) {
          int k;
          const int tile = tile_at(v, k), tb = tile / NB, j = tile % NB, mt0 = m0 + tb * 32;
          if ((W / 2) * v + (w >> 1) >= TPR || tile >= TILES || nt0 + j >= p.n_tiles || mt0 >= p.M) continue;   // uniform
          const int col = j * 32 + lq, n = nt0 * 32 + col - p.q_cols - p.k_cols;
          const float bias = cols[col], cs = PRO == PRO_LN ? cols[NB * 32 + col] : 0.f;
          const int head = (int)(((float)n + 0.5f) * (1.0f / (float)p.head_dim)), dd = n - head * p.head_dim;   // exact: n < 2^16
          float rs_t = rs[0], mu_t = mu[0];   // of row lane % 32 of this token block
#pragma unroll
          for (int b = 1; b < MB; b++) {
            rs_t = tb == b ? rs[b] : rs_t;
            mu_t = tb == b ? mu[b] : mu_t;
          }
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const int row = 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3);
            float x = pt[v][0][e];
#pragma unroll
            for (int ww = 1; ww < W; ww++) x += pt[v][ww][e];
            if (PRO == PRO_RMS) x *= __shfl(rs_t, row, 64);
            if (PRO == PRO_LN) x = __shfl(rs_t, row, 64) * (x - __shfl(mu_t, row, 64) * cs);
            o[e] = (bf16)(x + bias);
          }
          if (mt0 + 32 > p.M) {   // uniform
#pragma unroll
            for (int e = 0; e < 8; e++) o[e] = mt0 + 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3) < p.M ? o[e] : (bf16)0.f;
          }
          if (head < p.kv_heads) {
            const unsigned off = (unsigned)(((head * p.kv_chunks + (mt0 >> 5)) * p.nvb + (dd >> 5)) * 2048 + s2 * 1024 + lh * 512 + (dd & 31) * 16);
            *reinterpret_cast<bf16x8*>(reinterpret_cast<char*>(p.vfrag) + off) = o;
          }
        }
      } else {
        // A unit is 8 features of a tile (features 8 q .. of it).  4 waves: wave w takes features 8 w of every tile, so token
        // block and column are constants; 8 waves: waves w and w + 4 share the tiles of a round.
        constexpr int UPW = (TPR * 4 + W - 1) / W, UG = W == 4 ? (TPR % 4 == 0 ? 4 : 3) : 2;   // units of a wave, of a group
        const int q = w & 3;
        // query / key stores: 8 features lie in one head if the head dimension is a multiple of 8; heads by a 32-bit reciprocal
        const bool whole = EPI == EPI_BF16 || ((nt0 + NB) * 32 <= p.q_cols + p.k_cols && (p.head_dim & 7) == 0);   // uniform
        const unsigned inv_head = EPI == EPI_QKV ? 0xffffffffu / (unsigned)p.head_dim + 1u : 0u;
        // where column j's units go: base, offset of token block 0 in bytes (the lane's part apart); bytes between token blocks
        const unsigned tb_step = EPI == EPI_BF16 ? (unsigned)(p.ldo >> 4) * 1024u : (unsigned)(p.dqk_pad >> 4) * 1024u;
        const unsigned lane_off = (unsigned)lq * 16u + (EPI == EPI_QKV && p.rope != nullptr ? (unsigned)lh * (8u * 1024u) : (unsigned)lh * 8u);
        auto column = [&](int j, char*& base, unsigned& off) {
          const int n8 = (nt0 + j) * 32 + 8 * q;
          if (EPI == EPI_BF16) {
            base = reinterpret_cast<char*>(p.out_bf16);
            off = (unsigned)(m0 >> 5) * tb_step + (unsigned)(n8 >> 4) * 1024u + (unsigned)((n8 >> 3) & 1) * 512u;
          } else {
            const bool is_q = n8 < p.q_cols;
            const int nl = is_q ? n8 : n8 - p.q_cols;
            const int head = p.rope != nullptr ? nl >> 8 : (int)(((unsigned long long)(unsigned)nl * inv_head) >> 32);
            const int dd = p.rope != nullptr ? (nl & 255) >> 1 : nl - head * p.head_dim;
            base = reinterpret_cast<char*>(is_q ? p.out_bf16 : p.kfrag);
            off = (unsigned)((is_q ? head * p.q_mbs : p.rope != nullptr ? 0 : head * p.kv_chunks) + (m0 >> 5)) * tb_step +
                  (unsigned)(dd >> 4) * 1024u + (unsigned)((dd >> 3) & 1) * 512u + (unsigned)(dd & 7) * 2u;
          }
        };
        if constexpr (EPI == EPI_QKV) {
          if (!whole) {   // a block with queries or keys and values, or heads that 8 features straddle: unit by unit
#pragma unroll 1
            for (int v = 0; v < UPW; v++) {
              const int k = W == 4 ? v : 2 * v + (w >> 2), tile = rd * TPR + k, tb = tile / NB, j = tile % NB, nt = nt0 + j, m = m0 + tb * 32 + lq;
              if (k >= TPR || tile >= TILES || nt >= p.n_tiles) continue;   // uniform
              f32x16 sum;
              f32x4 pt[W];
#pragma unroll
              for (int ww = 0; ww < W; ww++) pt[ww] = *part(ww, k, 2 * q + lh, lq);
              EpiOps ops;
              const float* const c4 = cols + (j * 32 + 8 * q + 4 * lh);
              ops.bias[0] = *reinterpret_cast<const f32x4*>(c4);
              if (PRO == PRO_LN) ops.colsum[0] = *reinterpret_cast<const f32x4*>(c4 + NB * 32);
              const int n4 = nt * 32 + 8 * q + 4 * lh;
              if (p.rope != nullptr && n4 < p.q_cols + p.k_cols)
                ops.aux[0] = *reinterpret_cast<const f32x4*>(p.rope + ((size_t)(p.pos0 + min(m, p.M - 1)) * 128 + (((n4 < p.q_cols ? n4 : n4 - p.q_cols) & 255) >> 1)) * 2);
#pragma unroll
              for (int jj = 0; jj < 4; jj++) {
                sum[jj] = pt[0][jj];
#pragma unroll
                for (int ww = 1; ww < W; ww++) sum[jj] += pt[ww][jj];
              }
              float ssum, ssq;
              stat_sums(tb * 32 + lq, ssum, ssq);
              if (m < p.M) epilogue_tile<PRO, EPI, 0, 1>(p, sum, nt, m, lh, ssum, ssq, 0, ops, LaunchCtx{}, q);
            }
            continue;   // next round
          }
        }
#pragma unroll
        for (int v0 = 0; v0 < UPW; v0 += UG) {
          f32x4 pt[UG][W], x[UG], rope[UG], bias[UG], cs[UG];
#pragma unroll
          for (int u = 0; u < UG; u++) {   // (beyond the last tile: a copy of it, not stored)
            const int k = min(W == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), TPR - 1), tile = min(rd * TPR + k, TILES - 1), tb = tile / NB, j = tile % NB;
            if (EPI == EPI_QKV && p.rope != nullptr)
              rope[u] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(p.rope) + (size_t)(p.pos0 + m0) * 1024 +
                                                        ((unsigned)min(tb * 32 + lq, p.M - 1 - m0) * 1024u + (unsigned)((nt0 * 32 + j * 32 + 8 * q) & 255) * 4u + (unsigned)lh * 16u));
#pragma unroll
            for (int ww = 0; ww < W; ww++) pt[u][ww] = *part(ww, k, 2 * q + lh, lq);
            const float* const c4 = cols + (j * 32 + 8 * q + 4 * lh);
            bias[u] = *reinterpret_cast<const f32x4*>(c4);
            if (PRO == PRO_LN) cs[u] = *reinterpret_cast<const f32x4*>(c4 + NB * 32);
          }
          __builtin_amdgcn_sched_barrier(0);   // every read in flight (left alone they are read and added one by one)
#pragma unroll
          for (int u = 0; u < UG; u++) {
            const int k = W == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), tb = min(rd * TPR + k, TILES - 1) / NB;
            float rs_t = rs[0], mu_t = mu[0];
#pragma unroll
            for (int b = 1; b < MB; b++) {
              rs_t = tb == b ? rs[b] : rs_t;
              mu_t = tb == b ? mu[b] : mu_t;
            }
            x[u] = pt[u][0];
#pragma unroll
            for (int ww = 1; ww < W; ww++) x[u] += pt[u][ww];
            if (PRO == PRO_RMS) x[u] *= rs_t;
            if (PRO == PRO_LN) x[u] = rs_t * (x[u] - mu_t * cs[u]);
            x[u] += bias[u];
          }
          if (EPI == EPI_BF16 && p.act == ACT_GELU) {
#pragma unroll
            for (int u = 0; u < UG; u++)
#pragma unroll
              for (int e = 0; e < 4; e++) x[u][e] = gelu_tanh_f(x[u][e]);
          }
#pragma unroll
          for (int u = 0; u < UG; u++) {
            const int k = W == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), tile = rd * TPR + k, tb = tile / NB, j = tile % NB;
            if (v0 + u >= UPW || k >= TPR || tile >= TILES) continue;   // uniform
            const int m = m0 + tb * 32 + lq, m_end = nt0 + j < p.n_tiles ? p.M : 0;
            char* base;
            unsigned off;
            column(j, base, off);
            uint2 o = __builtin_bit_cast(uint2, bf16x4{(bf16)x[u][0], (bf16)x[u][1], (bf16)x[u][2], (bf16)x[u][3]});
            if (EPI == EPI_QKV && p.rope != nullptr) {
              // rotated pairs: dimensions dd + 2 lh, + 1 and, 128 on, their partners; the lane halves swap, so that half 0
              // stores the four lower ones and half 1 the four upper ones
              const f32x4 r = rope[u];   // cos i0, sin i0, cos i0+1, sin i0+1
              const bf16x2 lo = {(bf16)(x[u][0] * r[0] - x[u][1] * r[1]), (bf16)(x[u][2] * r[2] - x[u][3] * r[3])};
              const bf16x2 hi = {(bf16)(x[u][1] * r[0] + x[u][0] * r[1]), (bf16)(x[u][3] * r[2] + x[u][2] * r[3])};
              const u32x2_t both = swap_halves(__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi));
              o = uint2{both[0], both[1]};
            }
            const bool column_ok = EPI == EPI_QKV || (nt0 + j) * 32 + 8 * q + 4 * lh < p.n_valid;
            if (m < m_end && column_ok) *reinterpret_cast<uint2*>(base + (off + (unsigned)tb * tb_step + lane_off)) = o;
          }
        }
      }
    }
  }
}

template <int MB, int NB, int W, int EPI>
constexpr int stream_smem_bytes() {
  return W * StreamRounds<MB, NB, W, EPI>::TPR * 4096 + 64 * W * 8 + 3 * NB * 32 * 4;
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
  int nb;   // feature tiles of a block
};
// value_tile: feature tile of QKV's output that the values start at, where the last 32-token chunk is incomplete, else 0.  Blocks of
// nothing but values then store the rest of the chunk as zeros (zero_values says why), so no block may straddle that boundary;
// the same stores in the blocks that straddle it would cost every QKV launch their code (3 views 9.704 -> 9.741 ms)
StreamChoice stream_choose(int pro, int epi, int M, int n_tiles, int kc16, int value_tile = 0) {
  StreamChoice best{nullptr, 0};
  float cost = 0.f;
#define X(MB, NB, W, D)                                                   \
  {                                                                       \
    const float c = stream_cost(MB, NB, M, n_tiles, kc16);                \
    if (value_tile % NB == 0 && (best.launch == nullptr || c < cost)) { cost = c; best = StreamChoice{&stream_launch<MB, NB, W, D, SPRO, SEPI>, NB}; } \
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
