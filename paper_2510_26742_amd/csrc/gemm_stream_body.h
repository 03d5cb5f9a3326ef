// Body of the stream GEMMs (gemm_stream.hip says what they are): one item, MB x NB tiles of 32 tokens x 32 features over the whole
// k range.  Written for an execution context (exec_ctx.h): the launches of gemm_stream.hip, and the vision tower as one persistent
// kernel (vision_persistent.hip), where the weights and column vectors are requested ahead of the wait for the inputs.
#pragma once
#include "pi0_internal.h"

#include "gemm_common.h"

constexpr int STREAM_RED_BYTES = 144 * 1024;   // partial tiles of one round: W waves x TPR tiles x 4 KiB, at most this much

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

// Which tiles a die takes: consecutive block ids go to different dies (an L2 each), and a die takes a contiguous eighth of the tiles, token
// tiles fastest: the tiles that share a weight panel meet in one L2, and no die has more than one tile more than another
// (whole panels dealt to dies in turn gave 18 panels x 12 token tiles as 36 blocks to two dies of 32 compute units).
__device__ __forceinline__ void stream_share(int die, int tiles, int& first, int& count) {
  first = die * (tiles >> 3) + min(die, tiles & 7);
  count = (tiles >> 3) + (die < (tiles & 7) ? 1 : 0);
}

// W: parts of the k range, added in order; V: parts that one wave accumulates (W / V waves in the block).  D: k steps in flight.
// SG: groups in which the planes of row statistics are added (group g: planes g, g + SG, ...; then the groups in order).
// PARTS: most planes.  NS: k steps of a wave if known, else 0.  LINES_SHARED: blocks of different dies wrote parts of one cache line
// of the row statistics, which are then read past the caches (exec_ctx.h, BULK_CACHED).  cx.bx: the item.
template <int MB, int NB, int W, int V, int D, int SG, int PARTS, int NS, int PRO, int EPI, bool LINES_SHARED = false, class Cx>
__device__ __forceinline__ void gemm_stream_body(const GemmParams& p, const Cx& cx, unsigned char* smem_raw) {
  constexpr int WR = W / V;   // waves
  static_assert(W % V == 0 && (WR == 4 || WR == 8), "four or eight waves");
  using Rounds = StreamRounds<MB, NB, W, EPI>;
  constexpr int TILES = MB * NB, ROUNDS = Rounds::ROUNDS, TPR = Rounds::TPR;
  float* red = reinterpret_cast<float*>(smem_raw);                        // [W][TPR][8 groups of 4 columns][32 rows, rotated by the group][4]
  float2* sstat = reinterpret_cast<float2*>(smem_raw + W * TPR * 4096);   // [groups][MB * 32]
  float* cols = reinterpret_cast<float*>(sstat + SG * MB * 32);                 // [bias, column sums, gain][NB * 32]

  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;

  int first, count;
  stream_share(cx.bx & 7, (p.n_tiles + NB - 1) / NB * p.m_tiles, first, count);
  if ((cx.bx >> 3) >= count) return;
  const int nb = (first + (cx.bx >> 3)) / p.m_tiles;
  const int mt = (first + (cx.bx >> 3)) - nb * p.m_tiles;
  const int nt0 = nb * NB;
  const int m0 = mt * MB * 32;
  const int mb_last = (p.M - 1) >> 5;
  const int KC16 = p.W.k_pad >> 4;
  const int XKC16 = p.ldx >> 4;
  const int per = NS > 0 ? NS : (KC16 + W - 1) / W;
  const int n = NS > 0 ? NS : V == 1 ? max(0, min(per, KC16 - w * per)) : per;   // this wave's k16 steps: w * per .. + n - 1 (several parts: of one size)

  const char* wb[NB];
  const char* xb[MB];
#pragma unroll
  for (int j = 0; j < NB; j++) wb[j] = reinterpret_cast<const char*>(p.W.w) + (size_t)min(nt0 + j, p.n_tiles - 1) * KC16 * 1024;
#pragma unroll
  for (int i = 0; i < MB; i++) xb[i] = reinterpret_cast<const char*>(p.X) + (size_t)min((m0 >> 5) + i, mb_last) * XKC16 * 1024;
  unsigned voff[V];
#pragma unroll
  for (int v = 0; v < V; v++) voff[v] = (unsigned)(min((w * V + v) * per, KC16 - 1) * 1024 + lane * 16);
  // Blocks and waves start at different steps of their range and wrap around: in step, the 32 compute units of a die ask
  // for addresses that are a power of two apart and meet in the same few cache channels (vision down at 512 tokens
  // 22.0 -> 18.5 us, prefix QKV at 256 tokens 12.4 -> 11.1 us).
  int rot[V];
#pragma unroll
  for (int v = 0; v < V; v++) rot[v] = (int)((unsigned)(nb * 3 + mt * 5 + (w * V + v) * 7) % (unsigned)max(n, 1));

  bf16x8 wr[D][V][NB], xr[D][V][MB];
  auto step_off = [&](int v, int i) {
    const int k = i + rot[v];
    return voff[v] + (unsigned)(k < n ? k : max(k - n, 0)) * 1024u;
  };
  auto issue_w = [&](int u, int i) {
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int j = 0; j < NB; j++) wr[u][v][j] = *reinterpret_cast<const bf16x8*>(wb[j] + step_off(v, i));
  };
  auto issue_x = [&](int u, int i) {
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int b = 0; b < MB; b++) xr[u][v][b] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(xb[b] + step_off(v, i)));
  };
  auto issue = [&](int u, int i) {
    issue_w(u, i);
    issue_x(u, i);
  };
  f32x16 acc[V][TILES];   // tile b * NB + j
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int k = 0; k < TILES; k++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[v][k][r] = 0.f;
  // The products of stage u, and between them, one by one, the requests of step i for stage nu.  All together behind the products,
  // the waves, which run in step, let the memory path idle while they multiply and the matrix cores while the path takes their requests
  // (64 bytes per clock: a step's operands take it as long as the products take): with everything in the first-level cache, up
  // at three views took 9.8 us behind its wait for 3.8 us of products and 3.8 us of requests.
  auto step = [&](int u, int nu, int i, bool more) {
    constexpr int TM = V * TILES, PV = NB + MB, TL = V * PV;
    unsigned off[V];
#pragma unroll
    for (int v = 0; v < V; v++) off[v] = more ? step_off(v, i) : 0u;
#pragma unroll
    for (int m = 0; m < TM; m++) {
      const int v = m / TILES, b = m % TILES / NB, j = m % NB;
      acc[v][b * NB + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[u][v][j], xr[u][v][b], acc[v][b * NB + j], 0, 0, 0);
#pragma unroll
      for (int q = m * TL / TM; q < (m + 1) * TL / TM; q++) {
        const int lv = q / PV, r = q % PV;
        if (!more) continue;
        if (r < NB) wr[nu][lv][r < NB ? r : 0] = *reinterpret_cast<const bf16x8*>(wb[r < NB ? r : 0] + off[lv]);
        else xr[nu][lv][r < NB ? 0 : r - NB] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(xb[r < NB ? 0 : r - NB] + off[lv]));
      }
    }
    if (more) {
#pragma unroll
      for (int m = 0; m < TM; m++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
        for (int q = m * TL / TM; q < (m + 1) * TL / TM; q++) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
    }
  };

  // column vectors of the epilogue (residual rows this early cost the small tiles more than the round trip they save at the
  // end: vision O at 256 tokens 6.0 -> 6.4 us)
  float col_bias = 0.f, col_sum = 0.f, col_gain = 1.f;
  auto load_cols = [&]() {
    if (t < NB * 32) {
      const int col = min(nt0 * 32 + t, p.W.n_pad - 1);
      if (p.bias != nullptr) col_bias = p.bias[col];
      if (PRO == PRO_LN) col_sum = p.colsum[col];
      if (EPI == EPI_RESID && p.gain != nullptr) col_gain = p.gain[min(col, p.n_valid - 1)];
    }
  };
  auto keep_cols = [&]() {
    if (t < NB * 32) {
      cols[t] = col_bias;
      if (PRO == PRO_LN) cols[NB * 32 + t] = col_sum;
      if (EPI == EPI_RESID) cols[2 * NB * 32 + t] = col_gain;
    }
  };
  if constexpr (Cx::kPersistent) {   // what is constant during the kernel, ahead of the wait
    load_cols();
#pragma unroll
    for (int u = 0; u < D - 1; u++) issue_w(u, max(0, min(u, n - 1)));
    keep_cols();
    cx.wait_inputs();
  } else {
#pragma unroll
    for (int u = 0; u < D - 1; u++) issue(u, max(0, min(u, n - 1)));
  }
  // Row statistics of the block's rows, as a launch behind the first stages, else ahead of them: whole-row sums, or partial sums in
  // planes, one per range of columns that a block of the producer owned (the groups are added in order in the epilogue)
  // A launch spreads a row's groups over threads; in the persistent kernel, where a row's planes come with the activations, one thread
  // takes a row and leaves what the epilogue wants, 1 / deviation and mean.
  constexpr int PPG = (PARTS + SG - 1) / SG;      // planes of a group, at most
  const bool stat_thread = PRO != PRO_NONE && t < (Cx::kPersistent ? 1 : SG) * MB * 32;
  const int stat_row = t % (MB * 32), stat_g = t / (MB * 32);
  const float inv_k = 1.0f / (float)p.k_true;
  auto scale_from = [&](float ssum, float ssq, float& rs, float& mu) {   // of the norm in front: 1 / deviation and mean of a row
    mu = PRO == PRO_LN ? ssum * inv_k : 0.f;
    rs = rsqrtf(PRO == PRO_LN ? fmaxf(ssq * inv_k - mu * mu, 0.f) + 1e-6f : ssq * inv_k + 1e-6f);
  };
  // Every plane's address is clamped and every load of a batch unconditional: with a branch around each, the first waited for the
  // stages in front of it.  A launch takes one load for whole-row sums, else batches of 36 planes.
  const int parts = Cx::kPersistent ? PARTS : p.rowstat_parts > 1 ? p.rowstat_parts : 1;
  const size_t stat_rowg = (size_t)min(m0 + stat_row, p.M - 1);
  auto plane = [&](int k) {
    const float2* const v = reinterpret_cast<const float2*>(p.rowstat + 2 * ((size_t)min(k, parts - 1) * p.stat_rows + stat_rowg));
    if constexpr (LINES_SHARED) return cx.ld(v);
    else return cx.ld_bulk(v);
  };
  float2 planes[Cx::kPersistent && PRO != PRO_NONE ? SG : 1][Cx::kPersistent && PRO != PRO_NONE ? PPG : 1];
  if (Cx::kPersistent && stat_thread) {
#pragma unroll
    for (int q = 0; q < (Cx::kPersistent ? SG : 0); q++)
#pragma unroll
      for (int jj = 0; jj < PPG; jj++) planes[q][jj] = plane(q + SG * jj);
  }
  if constexpr (Cx::kPersistent) {
#pragma unroll
    for (int u = 0; u < D - 1; u++) issue_x(u, max(0, min(u, n - 1)));
  }
  if (Cx::kPersistent && stat_thread) {
    float ssum = 0.f, ssq = 0.f, rs, mu;
#pragma unroll
    for (int q = 0; q < (Cx::kPersistent ? SG : 0); q++) {
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int jj = 0; jj < PPG; jj++) {
        a += q + SG * jj < parts ? planes[q][jj].x : 0.f;
        b += q + SG * jj < parts ? planes[q][jj].y : 0.f;
      }
      ssum += a;
      ssq += b;
    }
    scale_from(ssum, ssq, rs, mu);
    sstat[stat_row] = make_float2(rs, mu);
  }
  if (!Cx::kPersistent && stat_thread) {
    float a = 0.f, b = 0.f;
    if (parts == 1) {
      const float2 v = plane(0);
      a = stat_g == 0 ? v.x : 0.f;
      b = stat_g == 0 ? v.y : 0.f;
    } else {
      constexpr int B = (36 + SG - 1) / SG;
      for (int j0 = 0; j0 * SG < parts; j0 += B) {
        float2 v[B];
#pragma unroll
        for (int jj = 0; jj < B; jj++) v[jj] = plane(stat_g + SG * (j0 + jj));
#pragma unroll
        for (int jj = 0; jj < B; jj++) {
          a += stat_g + SG * (j0 + jj) < parts ? v[jj].x : 0.f;
          b += stat_g + SG * (j0 + jj) < parts ? v[jj].y : 0.f;
        }
      }
    }
    sstat[stat_g * (MB * 32) + stat_row] = make_float2(a, b);
  }
  if constexpr (!Cx::kPersistent) {
    load_cols();
    keep_cols();
  }
  // A block of nothing but value features: 16-byte stores into the value fragments (2-byte ones otherwise)
  const bool values = EPI == EPI_QKV && nt0 * 32 >= p.q_cols + p.k_cols;

  // stage u of a group of D steps asks for the step D - 1 ahead, which goes where the stage before was
  int i = 0;
  for (; i + 2 * D - 1 <= n; i += D) {
#pragma unroll
    for (int u = 0; u < D; u++) step(u, (u + D - 1) % D, i + u + D - 1, true);
  }
  // the last D - 1 .. 2 D - 2 steps (all of them if there are fewer); branches between products and requests where their number is
  // not a constant, which together as above would spill
#pragma unroll
  for (int u = 0; u < 2 * D - 2; u++) {
    if (NS > 0) {
      if (i + u < n) step(u % D, (u + D - 1) % D, i + u + D - 1, i + u + D - 1 < n);
    } else if (i + u < n) {
      step(u % D, 0, 0, false);
      if (i + u + D - 1 < n) issue((u + D - 1) % D, i + u + D - 1);
    }
  }

  cx.mark(1);
  // ---- partial tiles -> LDS, fixed-order sums, epilogue --------------------------------------------
  // A tile lies in LDS as 8 groups of 4 consecutive accumulator rows, each group's 32 lanes rotated by its number: lanes
  // that go through the columns of a row (residual epilogue) then meet different banks, like those that go through the rows.
  auto part = [&](int ww, int k, int c4, int r) {
    return reinterpret_cast<f32x4*>(red + (((size_t)ww * TPR + k) * 8 + c4) * 128 + (((r + c4) & 31) * 4));
  };
  auto stat_sums = [&](int row, float& ssum, float& ssq) {
    ssum = ssq = 0.f;
#pragma unroll
    for (int g = 0; g < SG; g++) {
      const float2 s2 = sstat[g * (MB * 32) + row];
      ssum += s2.x;
      ssq += s2.y;
    }
  };
  auto scale_of = [&](int row, float& rs, float& mu) {
    rs = 1.f;
    mu = 0.f;
    if (PRO == PRO_NONE) return;
    if (Cx::kPersistent) {
      const float2 s2 = sstat[row];
      rs = s2.x;
      mu = s2.y;
      return;
    }
    float ssum, ssq;
    stat_sums(row, ssum, ssq);
    scale_from(ssum, ssq, rs, mu);
  };
#pragma unroll
  for (int rd = 0; rd < ROUNDS; rd++) {
    // residual epilogue: a unit is 8 / NB rows x all of the block's columns, a lane 4 columns of one row, so that rows are
    // read and written in whole cache lines
    constexpr int RL = 8 * NB, RU = TPR / NB * 4 * NB, RUPW = EPI == EPI_RESID ? (RU + WR - 1) / WR : 1;
    f32x4 resid[RUPW];   // requested here: their round trip overlaps the sums through LDS
    auto resid_at = [&](int v, int& k, int& row, int& c4, int& n4) {
      const int unit = w + WR * v, bl = unit / (4 * NB), c = lane % RL;
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
        if (have && m < p.M && n4 < p.n_valid) resid[v] = cx.ld(reinterpret_cast<const f32x4*>(p.resid + (size_t)rr * p.ldo + n4));
      }
    }
    if (rd) __syncthreads();   // the readers of the round before are done
#pragma unroll
    for (int v = 0; v < V; v++) {
#pragma unroll
      for (int k = 0; k < TPR; k++) {
        if (rd * TPR + k < TILES) {
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const f32x16& a = acc[v][rd * TPR + k < TILES ? rd * TPR + k : 0];
            *part(w * V + v, k, 2 * q + lh, lq) = f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
          }
        }
      }
    }
    __syncthreads();
    if (rd == 0) cx.mark(2);
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
            cx.st(reinterpret_cast<f32x4*>(p.out_f32 + (size_t)mo * p.ldo + n4), x);
            cx.st(reinterpret_cast<bf16x4*>(p.out_bf16 + xf_index(mo, n4, p.ldo2 >> 4)), bf16x4{(bf16)y[0], (bf16)y[1], (bf16)y[2], (bf16)y[3]});
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
              cx.st(reinterpret_cast<float2*>(p.stat_out + ((size_t)nb * p.stat_rows + mo) * 2), make_float2(st_a, st_b));
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
        constexpr int VUPW = (TPR * 2 + WR - 1) / WR;
        float pt[VUPW][W][8];
        const int s2 = w & 1;
        auto tile_at = [&](int v, int& k) {
          k = min((WR / 2) * v + (w >> 1), TPR - 1);
          return rd * TPR + (WR / 2) * v + (w >> 1);
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
          if ((WR / 2) * v + (w >> 1) >= TPR || tile >= TILES || nt0 + j >= p.n_tiles || mt0 >= p.M) continue;   // uniform
          const int col = j * 32 + lq, n = nt0 * 32 + col - p.q_cols - p.k_cols;
          const float bias = cols[col], cs = PRO == PRO_LN ? cols[NB * 32 + col] : 0.f;
          const int head = (int)(((float)n + 0.5f) * (1.0f / (float)p.head_dim)), dd = n - head * p.head_dim;   // exact: n < 2^16
          float rs_t = rs[0], mu_t = mu[0];   // of row lane % 32 of this token block
          float rs_e[8], mu_e[8];             // of the lane's rows
          if (Cx::kPersistent && PRO != PRO_NONE) {   // (a shuffle each otherwise: a round trip through LDS for four bytes)
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              const f32x4 two = *reinterpret_cast<const f32x4*>(sstat + tb * 32 + 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3));
              rs_e[e] = two[0], mu_e[e] = two[1], rs_e[e + 1] = two[2], mu_e[e + 1] = two[3];
            }
          } else {
#pragma unroll
            for (int b = 1; b < MB; b++) {
              rs_t = tb == b ? rs[b] : rs_t;
              mu_t = tb == b ? mu[b] : mu_t;
            }
#pragma unroll
            for (int e = 0; e < 8; e++) {
              const int row = 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3);
              if (PRO != PRO_NONE) rs_e[e] = __shfl(rs_t, row, 64);
              if (PRO == PRO_LN) mu_e[e] = __shfl(mu_t, row, 64);
            }
          }
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; e++) {
            float x = pt[v][0][e];
#pragma unroll
            for (int ww = 1; ww < W; ww++) x += pt[v][ww][e];
            if (PRO == PRO_RMS) x *= rs_e[e];
            if (PRO == PRO_LN) x = rs_e[e] * (x - mu_e[e] * cs);
            o[e] = (bf16)(x + bias);
          }
          if (mt0 + 32 > p.M) {   // uniform
#pragma unroll
            for (int e = 0; e < 8; e++) o[e] = mt0 + 16 * s2 + 8 * (e >> 2) + 4 * lh + (e & 3) < p.M ? o[e] : (bf16)0.f;
          }
          if (head < p.kv_heads) {
            const unsigned off = (unsigned)(((head * p.kv_chunks + (mt0 >> 5)) * p.nvb + (dd >> 5)) * 2048 + s2 * 1024 + lh * 512 + (dd & 31) * 16);
            cx.st(reinterpret_cast<bf16x8*>(reinterpret_cast<char*>(p.vfrag) + off), o);
          }
        }
      } else {
        // A unit is 8 features of a tile (features 8 q .. of it).  4 waves: wave w takes features 8 w of every tile, so token
        // block and column are constants; 8 waves: waves w and w + 4 share the tiles of a round.
        constexpr int UPW = (TPR * 4 + WR - 1) / WR, UG = W == 4 ? (TPR % 4 == 0 ? 4 : 3) : 2;   // units of a wave, of a group
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
        if constexpr (EPI == EPI_QKV && !Cx::kPersistent) {   // (the persistent kernel takes shapes without such blocks)
          if (!whole) {   // a block with queries or keys and values, or heads that 8 features straddle: unit by unit
#pragma unroll 1
            for (int v = 0; v < UPW; v++) {
              const int k = WR == 4 ? v : 2 * v + (w >> 2), tile = rd * TPR + k, tb = tile / NB, j = tile % NB, nt = nt0 + j, m = m0 + tb * 32 + lq;
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
              if (m < p.M) epilogue_tile<PRO, EPI, 0, 1>(p, sum, nt, m, lh, ssum, ssq, 0, ops, cx, q);
            }
            continue;   // next round
          }
        }
        char* base_j[WR == 4 ? NB : 1];   // 4 waves: a wave's features are the same in every tile of a column
        unsigned off_j[WR == 4 ? NB : 1];
        if (WR == 4) {
#pragma unroll
          for (int j = 0; j < (WR == 4 ? NB : 0); j++) column(j, base_j[j], off_j[j]);
        }
#pragma unroll
        for (int v0 = 0; v0 < UPW; v0 += UG) {
          f32x4 pt[UG][W], x[UG], rope[UG], bias[UG], cs[UG];
#pragma unroll
          for (int u = 0; u < UG; u++) {   // (beyond the last tile: a copy of it, not stored)
            const int k = min(WR == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), TPR - 1), tile = min(rd * TPR + k, TILES - 1), tb = tile / NB, j = tile % NB;
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
            const int k = WR == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), tb = min(rd * TPR + k, TILES - 1) / NB;
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
            const int k = WR == 4 ? v0 + u : 2 * (v0 + u) + (w >> 2), tile = rd * TPR + k, tb = tile / NB, j = tile % NB;
            if (v0 + u >= UPW || k >= TPR || tile >= TILES) continue;   // uniform
            const int m = m0 + tb * 32 + lq, m_end = nt0 + j < p.n_tiles ? p.M : 0;
            char* base;
            unsigned off;
            if (WR == 4) {
              base = base_j[WR == 4 ? j : 0];
              off = off_j[WR == 4 ? j : 0];
            } else {
              column(j, base, off);
            }
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
            if (m < m_end && column_ok) cx.st(reinterpret_cast<uint2*>(base + (off + (unsigned)tb * tb_step + lane_off)), o);
          }
        }
      }
    }
  }
}

// shared memory of the body
template <int MB, int NB, int W, int SG, int EPI>
constexpr int stream_body_smem() {
  return W * StreamRounds<MB, NB, W, EPI>::TPR * 4096 + SG * MB * 32 * 8 + 3 * NB * 32 * 4;
}
