// Bodies of the attention kernels: attention_body (see attention.hip for the plan), and attention_suffix_body for the
// action expert, which also runs inside the persistent kernel of the denoise loop (exec_ctx.h).
#pragma once
#include "pi0_internal.h"
#include "exec_ctx.h"

#define NEG_BIG (-1.0e30f)
#define ATT_WAVES 8
#define ATT_SHARE 10   // most chunks of prefix keys in a share of the expert's attention

// MAXR: key rounds per wave over segment 0 (8 * MAXR chunks = 256 * MAXR keys); VRING: value
// chunks in flight per wave.
// CPW > 0 (needs MAXR == 1 and NVB == 8): phase 2 is shared out over all 8 waves instead of one wave per value slice.
// With nslice value slices in the block, the waves form G = 8 / nslice groups; wave (slice, group g) multiplies the
// chunks g, g + G, ... of [segment 0 ; segment 1] (at most CPW of them, held in registers: no ring, no second round
// trip), the G partial outputs of a slice meet in LDS and are added in group order.  The dependent chain of a wave
// drops from 2 x (all chunks) to 2 x CPW products.
template <int DQK, int NVB, int MAXR, int VRING, int CPW, class Cx>
__device__ __forceinline__ void attention_body(const AttnParams p, const Cx cx, unsigned char* smem_raw) {
  constexpr int S16 = DQK / 16;
  constexpr bool PVG = CPW > 0;
  static_assert(!PVG || (MAXR == 1 && NVB == ATT_WAVES), "chunk groups: one key round, 8 value slices");
  constexpr bool DUAL = MAXR == 1;             // second accumulators (register room permitting)
  constexpr int QB = (MAXR == 1 && S16 % 8 == 0) ? 8 : 1;   // Q fragments read from LDS per batch (register room permitting)
  constexpr int NPQ = 32 * DQK / 8;            // 16-byte pieces of the Q tile
  constexpr int QP = (NPQ + 511) / 512;        // pieces per thread
  constexpr int NPK1 = 2 * S16 * 64;           // 16-byte pieces of the two segment-1 key chunks
  constexpr int KP1 = (NPK1 + 511) / 512;
  bf16* qs = reinterpret_cast<bf16*>(smem_raw);                               // [S16][64][8]
  bf16* k1s = qs + S16 * 512;                                                 // [2][S16][64][8]
  float* mw = reinterpret_cast<float*>(k1s + 2 * S16 * 512);                  // [8][32]
  float* lw = mw + ATT_WAVES * 32;                                            // [8][32]
  bf16* pf = reinterpret_cast<bf16*>(lw + ATT_WAVES * 32);                    // [ntot][2][64][8]

  const int t = cx.tid();
  const int lane = t & 63;
  const int w = t >> 6;
  const int lq = lane & 31;
  const int lh = lane >> 5;
  if (cx.by >= p.heads) {   // warm-up block; rank = linear block index (mod 8)
    if (cx.bz == 0) prefetch_role(p.pf, cx.bx + (int)gridDim.x * (cx.by - p.heads));
    return;
  }
  // v_split > 1: the head dimension of the values (and of the output) is shared out over v_split blocks per
  // (query tile, head); each repeats phase 1 on all keys and runs phase 2 on its NVB / v_split slices only
  const int vs = p.v_split > 1 ? p.v_split : 1;
  const int tile = cx.bx / vs;
  const int vpart = cx.bx - tile * vs;
  const int nslice = NVB / vs;                 // value slices (waves of phase 2) of this block
  const int pv_groups = PVG ? ATT_WAVES / nslice : 1;   // G
  const int pv_g = PVG ? w / nslice : 0;                // this wave's group
  const int slice = vpart * nslice + (PVG ? w - pv_g * nslice : w);   // the slice this wave accumulates
  const int head = cx.by;
  const int row = tile * 32 + lq;
  const bool row_ok = row < p.Tq;

  int cbeg0 = 0, n0 = p.chunks0;
  if (p.view_tokens > 0) {
    const int view = (tile * 32) / p.view_tokens;
    cbeg0 = view * (p.view_tokens >> 5);
    n0 = p.view_tokens >> 5;
  }
  int n1 = p.chunks1;
  if (p.key_splits > 1) {   // this block's share of segment 0; the last share also takes segment 1
    cbeg0 = cx.bz * p.chunks_per_split;
    n0 = min(p.chunks_per_split, p.chunks0 - cbeg0);
    if (cx.bz != p.key_splits - 1) n1 = 0;
  }
  const bf16* kbase0 = p.k0 + ((size_t)head * p.kv_head_stride0 + (size_t)cbeg0 * S16 * 512) + lane * 8;
  const bf16* vbase0 = p.v0 + ((size_t)head * p.v_head_stride0 + (size_t)cbeg0 * NVB * 1024);
  const bf16* vslice0 = vbase0 + slice * 1024 + lane * 8;   // this wave's slice of the value fragments of segment 0

  // ---- issue every load of the first round (unconditional, clamped addresses) -----------------
  const bf16* qsrc = p.q + (size_t)head * p.q_head_stride + (size_t)tile * S16 * 512;
  bf16x8 qreg[QP];
  bf16x8 k1reg[KP1];
  bf16x8 kf[S16];
  bf16x8 vf[PVG ? CPW * 2 : VRING * 2];      // ring over the chunks of segment 0 (chunk groups: this wave's chunks)
  bf16x8 vs1[PVG ? 1 : 4];                   // the (at most two) chunks of segment 1 (chunk groups: they are in vf)
  const bool pv_wave = PVG ? true : w < nslice;
  auto load_seg0 = [&]() {
    const bf16* kp0 = kbase0 + (size_t)min(w, n0 - 1) * S16 * 512;
#pragma unroll
    for (int s = 0; s < S16; s++) kf[s] = *reinterpret_cast<const bf16x8*>(kp0 + (size_t)s * 512);
    if (PVG) {
#pragma unroll
      for (int j = 0; j < (PVG ? CPW : 0); j++) {   // chunks beyond segment 0: a valid address, replaced or unused later
        const bf16* vp = vslice0 + (size_t)min(pv_g + j * pv_groups, n0 - 1) * NVB * 1024;
        vf[2 * j] = *reinterpret_cast<const bf16x8*>(vp);
        vf[2 * j + 1] = *reinterpret_cast<const bf16x8*>(vp + 512);
      }
    } else if (pv_wave) {
#pragma unroll
      for (int c = 0; c < VRING; c++) {
        const bf16* vp = vslice0 + (size_t)min(c, n0 - 1) * NVB * 1024;
        vf[2 * c] = *reinterpret_cast<const bf16x8*>(vp);
        vf[2 * c + 1] = *reinterpret_cast<const bf16x8*>(vp + 512);
      }
    }
  };
#pragma unroll
  for (int i = 0; i < QP; i++) qreg[i] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(qsrc + (size_t)min(t + i * 512, NPQ - 1) * 8));
  if (n1 > 0) {
#pragma unroll
    for (int i = 0; i < KP1; i++)
      k1reg[i] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(p.k1 + (size_t)min(t + i * 512, n1 * S16 * 64 - 1) * 8));
    if (!PVG && pv_wave) {
#pragma unroll
      for (int c = 0; c < 2; c++) {
        const bf16* vp = p.v1 + (size_t)min(c, n1 - 1) * NVB * 1024 + slice * 1024 + lane * 8;
        vs1[2 * c] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(vp));
        vs1[2 * c + 1] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(vp + 512));
      }
    }
  }
  load_seg0();
  if (PVG && n1 > 0) {   // this wave's chunks that fall into segment 1 (after load_seg0, whose placeholders they replace)
#pragma unroll
    for (int j = 0; j < (PVG ? CPW : 0); j++) {
      const int c = pv_g + j * pv_groups - n0;
      if (c >= 0 && c < n1) {
        const bf16* vp = p.v1 + (size_t)c * NVB * 1024 + slice * 1024 + lane * 8;
        vf[2 * j] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(vp));
        vf[2 * j + 1] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(vp + 512));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < QP; i++) {
    const int pc = t + i * 512;
    if (pc < NPQ) *reinterpret_cast<bf16x8*>(qs + (size_t)pc * 8) = qreg[i];
  }
  if (n1 > 0) {
#pragma unroll
    for (int i = 0; i < KP1; i++) {
      const int pc = t + i * 512;
      if (pc < NPK1) *reinterpret_cast<bf16x8*>(k1s + (size_t)pc * 8) = k1reg[i];
    }
  }
  __syncthreads();

  // ---- phase 1: scores of this wave's chunks ------------------------------------------------
  float sv[MAXR][16];
  float sv1[16];
  float m_loc = NEG_BIG;
#pragma unroll
  for (int r = 0; r < MAXR; r++) {
    const int ci = w + ATT_WAVES * r;
    if (ci < n0) {
      const bool more = ci + ATT_WAVES < n0;
      const bf16* kn = kbase0 + (size_t)min(ci + ATT_WAVES, n0 - 1) * S16 * 512;
      f32x16 sacc, sacc1;      // two accumulators where registers allow: a dependent MFMA waits ~64 clocks
#pragma unroll
      for (int e = 0; e < 16; e++) sacc[e] = 0.f, sacc1[e] = 0.f;
      // the Q fragments come from LDS in batches of QB reads issued together: a read that is only
      // issued when its MFMA is next costs a full LDS round trip per step
#pragma unroll
      for (int s0 = 0; s0 < S16; s0 += QB) {
        bf16x8 qb[QB];
#pragma unroll
        for (int j = 0; j < QB; j++) qb[j] = *reinterpret_cast<const bf16x8*>(qs + ((size_t)(s0 + j) * 64 + lane) * 8);
#pragma unroll
        for (int j = 0; j < QB; j++) {
          const int s = s0 + j;
          const bf16x8 a = kf[s];
          if (r + 1 < MAXR && more) kf[s] = *reinterpret_cast<const bf16x8*>(kn + (size_t)s * 512);
          if (DUAL && (s & 1)) sacc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[j], sacc1, 0, 0, 0);
          else sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[j], sacc, 0, 0, 0);
        }
      }
      if (DUAL) {
#pragma unroll
        for (int e = 0; e < 16; e++) sacc[e] += sacc1[e];
      }
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int key = (cbeg0 + ci) * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
        sv[r][e] = key < p.valid0 ? sacc[e] * p.scale : NEG_BIG;
        m_loc = fmaxf(m_loc, sv[r][e]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; e++) sv[r][e] = NEG_BIG;
    }
  }
  const bool seg1_wave = w < n1;             // waves 0 and 1 score the second segment from LDS
  if (seg1_wave) {
    f32x16 sacc, sacc1;
#pragma unroll
    for (int e = 0; e < 16; e++) sacc[e] = 0.f, sacc1[e] = 0.f;
#pragma unroll
    for (int s0 = 0; s0 < S16; s0 += 4) {
      bf16x8 ka[4], qb[4];
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (s0 + j < S16) {
          ka[j] = *reinterpret_cast<const bf16x8*>(k1s + (((size_t)w * S16 + s0 + j) * 64 + lane) * 8);
          qb[j] = *reinterpret_cast<const bf16x8*>(qs + ((size_t)(s0 + j) * 64 + lane) * 8);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (s0 + j < S16) {
          if (DUAL && (j & 1)) sacc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[j], qb[j], sacc1, 0, 0, 0);
          else sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[j], qb[j], sacc, 0, 0, 0);
        }
      }
    }
    if (DUAL) {
#pragma unroll
      for (int e = 0; e < 16; e++) sacc[e] += sacc1[e];
    }
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int key = w * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
      const bool valid = p.suffix_mask ? (row == 0 ? key == 0 : true) : true;
      sv1[e] = valid ? sacc[e] * p.scale : NEG_BIG;
      m_loc = fmaxf(m_loc, sv1[e]);
    }
  }
  m_loc = max_xor32(m_loc);
  if (lh == 0) mw[w * 32 + lq] = m_loc;
  __syncthreads();
  float m_all = NEG_BIG;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) m_all = fmaxf(m_all, mw[i * 32 + lq]);
  float l_loc = 0.f;
  auto emit = [&](const float* svals, int slot) {   // probabilities -> B-operand fragments in LDS
    float pr[16];
#pragma unroll
    for (int e = 0; e < 16; e++) {
      pr[e] = svals[e] > 0.5f * NEG_BIG ? __expf(svals[e] - m_all) : 0.f;   // masked keys: exactly 0
      l_loc += pr[e];
    }
#pragma unroll
    for (int s2 = 0; s2 < 2; s2++) {
      bf16x8 pb;
#pragma unroll
      for (int j = 0; j < 8; j++) pb[j] = (bf16)pr[8 * s2 + j];
      *reinterpret_cast<bf16x8*>(pf + ((size_t)(slot * 2 + s2) * 64 + lane) * 8) = pb;
    }
  };
#pragma unroll
  for (int r = 0; r < MAXR; r++) {
    const int ci = w + ATT_WAVES * r;
    if (ci < n0) emit(sv[r], ci);
  }
  if (seg1_wave) emit(sv1, n0 + w);
  l_loc = add_xor32(l_loc);
  if (lh == 0) lw[w * 32 + lq] = l_loc;
  __syncthreads();
  if (!pv_wave) return;

  // ---- phase 2: this wave's 32-wide slice of the head dimension over all chunks --------------
  f32x16 o, o1;
#pragma unroll
  for (int e = 0; e < 16; e++) o[e] = 0.f, o1[e] = 0.f;
  // Segment 0: one ring of VRING chunks per round: the probability fragments of the whole round are read
  // from LDS up front (clamped, unconditional), chunks beyond the end multiply zeros; the value
  // fragments of the next round are requested (whole round, one uniform branch) as the registers
  // of this round are consumed.  Then the chunks of segment 1, whose value fragments came with Q.
  const bf16x8 zero8v = {(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
  if (PVG) {
    const int ntot = n0 + n1;
    bf16x8 bpg[PVG ? 2 * CPW : 1];   // the probability fragments of this wave's chunks, read together (clamped, unconditional)
#pragma unroll
    for (int j = 0; j < (PVG ? CPW : 0); j++) {
      const int c = min(pv_g + j * pv_groups, ntot - 1);
      bpg[2 * j] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c * 2) * 64 + lane) * 8);
      bpg[2 * j + 1] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c * 2 + 1) * 64 + lane) * 8);
    }
#pragma unroll
    for (int j = 0; j < (PVG ? CPW : 0); j++) {
      if (pv_g + j * pv_groups < ntot) {   // uniform per wave
        o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[2 * j], bpg[2 * j], o, 0, 0, 0);
        o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[2 * j + 1], bpg[2 * j + 1], o1, 0, 0, 0);
      }
    }
  } else {
    for (int c0 = 0; c0 < n0; c0 += VRING) {
      bf16x8 bp[2 * VRING];
  #pragma unroll
      for (int cc = 0; cc < VRING; cc++) {
        const int c = min(c0 + cc, n0 - 1);
  #pragma unroll
        for (int s2 = 0; s2 < 2; s2++)
          bp[2 * cc + s2] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c * 2 + s2) * 64 + lane) * 8);
      }
      const bool more_round = c0 + VRING < n0;
  #pragma unroll
      for (int cc = 0; cc < VRING; cc++) {
        const bool live = c0 + cc < n0;
  #pragma unroll
        for (int s2 = 0; s2 < 2; s2++) {
          const bf16x8 a = vf[2 * cc + s2];
          if (more_round) vf[2 * cc + s2] = *reinterpret_cast<const bf16x8*>(vslice0 + (size_t)min(c0 + cc + VRING, n0 - 1) * NVB * 1024 + (size_t)s2 * 512);
          if (DUAL && s2) o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, live ? bp[2 * cc + s2] : zero8v, o1, 0, 0, 0);
          else o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, live ? bp[2 * cc + s2] : zero8v, o, 0, 0, 0);
        }
      }
    }
    if (n1 > 0) {
  #pragma unroll
      for (int cc = 0; cc < 2; cc++) {
        const bool live = cc < n1;
        const int c = n0 + min(cc, n1 - 1);
  #pragma unroll
        for (int s2 = 0; s2 < 2; s2++) {
          const bf16x8 bpv = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c * 2 + s2) * 64 + lane) * 8);
          if (DUAL && s2) o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vs1[2 * cc + s2], live ? bpv : zero8v, o1, 0, 0, 0);
          else o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vs1[2 * cc + s2], live ? bpv : zero8v, o, 0, 0, 0);
        }
      }
    }
  }
  if (DUAL) {
#pragma unroll
    for (int e = 0; e < 16; e++) o[e] += o1[e];
  }
  float l_all = 0.f;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_all += lw[i * 32 + lq];
  const float inv = 1.0f / l_all;
  if (PVG && pv_groups > 1) {
    // the groups' partial outputs meet in LDS (over Q and the keys of segment 1, which phase 1 is done with):
    // [wave][4][64][4] floats; wave (slice, g) then finishes the pieces i = g, g + G, .. of its slice
    float* red = reinterpret_cast<float*>(smem_raw);
    static_assert(3 * S16 * 1024 >= ATT_WAVES * 4096 || !PVG, "partial outputs fit over Q and the keys of segment 1");
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const f32x4 v4 = {o[4 * i], o[4 * i + 1], o[4 * i + 2], o[4 * i + 3]};
      *reinterpret_cast<f32x4*>(red + (((size_t)w * 4 + i) * 64 + lane) * 4) = v4;
    }
    __syncthreads();
    const int sl = w - pv_g * nslice;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if ((i % pv_groups) == pv_g % 4 && pv_g < 4) {   // uniform per wave
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        for (int gg = 0; gg < pv_groups; gg++) {
          const f32x4 v4 = *reinterpret_cast<const f32x4*>(red + (((size_t)(gg * nslice + sl) * 4 + i) * 64 + lane) * 4);
          sum[0] += v4[0]; sum[1] += v4[1]; sum[2] += v4[2]; sum[3] += v4[3];
        }
        o[4 * i] = sum[0]; o[4 * i + 1] = sum[1]; o[4 * i + 2] = sum[2]; o[4 * i + 3] = sum[3];
      }
    }
  }
  if (!row_ok) return;
  if (p.ml_out != nullptr && w == 0 && lh == 0 && vpart == 0) {   // (row maximum, sum) of this share, for the consumer's merge
    float* dst = p.ml_out + ((((size_t)cx.bz * p.heads + head) * ((p.Tq + 31) >> 5) * 32) + row) * 2;
    cx.st(reinterpret_cast<float2*>(dst), make_float2(m_all, l_all));
  }
  bf16* outp = p.out + (size_t)cx.bz * p.out_split_stride;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (PVG && pv_groups > 1 && !((i % pv_groups) == pv_g % 4 && pv_g < 4)) continue;   // another wave's piece
    const int d = slice * 32 + 8 * i + 4 * lh;
    if (d < p.head_dim) {
      const bf16x4 ob = {(bf16)(o[4 * i] * inv), (bf16)(o[4 * i + 1] * inv), (bf16)(o[4 * i + 2] * inv),
                         (bf16)(o[4 * i + 3] * inv)};
      const int col = head * p.head_dim + d;
      cx.st(reinterpret_cast<bf16x4*>(outp + ((size_t)(row >> 5) * (p.out_ld >> 4) + (col >> 4)) * 512 +
                                      (((col & 15) >> 3) * 32 + (row & 31)) * 8 + (col & 7)), ob);
    }
  }
}


// ------------------------------------------------------------------------------------------------
// Attention inside a view of 256 tokens (head dimension 72 or 80 in 80 columns, three value slices) by WR waves, inside the
// persistent kernel of the vision tower: an item is QT tiles of 32 query rows of one head.  The sums of attention_body in their
// order, so the same bits: a chunk's scores as two interleaved products, its sum of exponentials on its own, the chunks' sums
// added in order, an output tile as two accumulators over the chunks.  Everything is requested at once behind the wait, Q straight into
// registers (5 KiB per tile that the compute unit's cache serves to all waves).
// ------------------------------------------------------------------------------------------------
constexpr int VIEW_CHUNKS = 8;
constexpr int attn_view_smem(int qt) { return qt * (2 * VIEW_CHUNKS * 32 * 4 + VIEW_CHUNKS * 2048); }

template <int WR, int QT, class Cx>
__device__ __forceinline__ void attention_view_body(const AttnParams& p, const Cx& cx, unsigned char* smem_raw) {
  constexpr int S16 = 5, NVB = 3, R = VIEW_CHUNKS / WR;
  float* mw = reinterpret_cast<float*>(smem_raw);                                                   // [QT][WR][32]
  float* lw = mw + QT * VIEW_CHUNKS * 32;                                                           // [QT][8 chunks][32]
  bf16* pf = reinterpret_cast<bf16*>(smem_raw + QT * 2 * VIEW_CHUNKS * 32 * 4);                     // [QT][8 chunks][2][64][8]
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;
  const int tile = cx.bx * QT, head = cx.by;
  const int cbeg = tile >> 3 << 3;   // the view's first chunk

  const bf16* qsrc = p.q + ((size_t)head * p.q_head_stride + (size_t)tile * S16 * 512);
  const bf16* kbase = p.k0 + ((size_t)head * p.kv_head_stride0 + (size_t)cbeg * S16 * 512);
  const bf16* vbase = p.v0 + ((size_t)head * p.v_head_stride0 + (size_t)cbeg * NVB * 1024 + (size_t)min(w, NVB - 1) * 1024);
  const unsigned l8 = (unsigned)lane * 8u;
  bf16x8 qf[QT][S16], kf[R][S16], vf[VIEW_CHUNKS][2];
#pragma unroll
  for (int q = 0; q < QT; q++)
#pragma unroll
    for (int s = 0; s < S16; s++) qf[q][s] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(qsrc + ((q * S16 + s) * 512 + l8)));
#pragma unroll
  for (int r = 0; r < R; r++)
#pragma unroll
    for (int s = 0; s < S16; s++) kf[r][s] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(kbase + ((unsigned)((w + WR * r) * S16 + s) * 512u + l8)));
  if (w < NVB) {
#pragma unroll
    for (int c = 0; c < VIEW_CHUNKS; c++)
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) vf[c][s2] = cx.ld_bulk(reinterpret_cast<const bf16x8*>(vbase + (unsigned)(c * NVB * 1024 + s2 * 512) + l8));
  }

  // The padding columns of queries and keys are nobody's: whatever is there counts as zero
  const bf16x8 zero8v = {(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
  const bool padding = (S16 - 1) * 16 + 8 * lh >= p.head_dim;   // a lane's 8 columns of the last fragment
#pragma unroll
  for (int q = 0; q < QT; q++) qf[q][S16 - 1] = padding ? zero8v : qf[q][S16 - 1];
#pragma unroll
  for (int r = 0; r < R; r++) kf[r][S16 - 1] = padding ? zero8v : kf[r][S16 - 1];

  // ---- scores ------------------------------------------------------------------------------------
  float sv[QT][R][16];
#pragma unroll
  for (int q = 0; q < QT; q++) {
    float m_loc = NEG_BIG;
#pragma unroll
    for (int r = 0; r < R; r++) {
      f32x16 sacc, sacc1;
#pragma unroll
      for (int e = 0; e < 16; e++) sacc[e] = 0.f, sacc1[e] = 0.f;
#pragma unroll
      for (int s = 0; s < S16; s++) {
        if (s & 1) sacc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[r][s], qf[q][s], sacc1, 0, 0, 0);
        else sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[r][s], qf[q][s], sacc, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 16; e++) {
        sv[q][r][e] = (sacc[e] + sacc1[e]) * p.scale;
        m_loc = fmaxf(m_loc, sv[q][r][e]);
      }
    }
    m_loc = max_xor32(m_loc);
    if (lh == 0) mw[(q * WR + w) * 32 + lq] = m_loc;
  }
  __syncthreads();
  // ---- probabilities -> B-operand fragments in LDS -----------------------------------------------
#pragma unroll
  for (int q = 0; q < QT; q++) {
    float m_all = NEG_BIG;
#pragma unroll
    for (int i = 0; i < WR; i++) m_all = fmaxf(m_all, mw[(q * WR + i) * 32 + lq]);
#pragma unroll
    for (int r = 0; r < R; r++) {
      float pr[16], l_loc = 0.f;
#pragma unroll
      for (int e = 0; e < 16; e++) {
        pr[e] = sv[q][r][e] > 0.5f * NEG_BIG ? __expf(sv[q][r][e] - m_all) : 0.f;
        l_loc += pr[e];
      }
      const int c = w + WR * r;
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) {
        bf16x8 pb;
#pragma unroll
        for (int j = 0; j < 8; j++) pb[j] = (bf16)pr[8 * s2 + j];
        *reinterpret_cast<bf16x8*>(pf + ((size_t)((q * VIEW_CHUNKS + c) * 2 + s2) * 64 + lane) * 8) = pb;
      }
      l_loc = add_xor32(l_loc);
      if (lh == 0) lw[(q * VIEW_CHUNKS + c) * 32 + lq] = l_loc;
    }
  }
  __syncthreads();
  if (w >= NVB) return;
  // ---- output: wave w the columns 32 w .. of the head --------------------------------------------
#pragma unroll 1
  for (int q = 0; q < QT; q++) {
    bf16x8 bp[VIEW_CHUNKS][2];
    float l_part[VIEW_CHUNKS];
#pragma unroll
    for (int c = 0; c < VIEW_CHUNKS; c++) {
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) bp[c][s2] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)((q * VIEW_CHUNKS + c) * 2 + s2) * 64 + lane) * 8);
      l_part[c] = lw[(q * VIEW_CHUNKS + c) * 32 + lq];
    }
    f32x16 o, o1;
#pragma unroll
    for (int e = 0; e < 16; e++) o[e] = 0.f, o1[e] = 0.f;
#pragma unroll
    for (int c = 0; c < VIEW_CHUNKS; c++) {
      o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c][0], bp[c][0], o, 0, 0, 0);
      o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c][1], bp[c][1], o1, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) o[e] += o1[e];
    float l_all = 0.f;
#pragma unroll
    for (int c = 0; c < VIEW_CHUNKS; c++) l_all += l_part[c];
    const float inv = 1.0f / l_all;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int d = w * 32 + 8 * i + 4 * lh;
      if (d < p.head_dim) {
        const bf16x4 ob = {(bf16)(o[4 * i] * inv), (bf16)(o[4 * i + 1] * inv), (bf16)(o[4 * i + 2] * inv), (bf16)(o[4 * i + 3] * inv)};
        const int col = head * p.head_dim + d;
        cx.st(reinterpret_cast<bf16x4*>(p.out + ((size_t)(tile + q) * (p.out_ld >> 4) + (col >> 4)) * 512 + (((col & 15) >> 3) * 32 + lq) * 8 + (col & 7)), ob);
      }
    }
  }
}

template <int DQK>
static constexpr int attn_smem_bytes(int ntot) { return 3 * (DQK / 16) * 1024 + 2 * ATT_WAVES * 32 * 4 + ntot * 2048; }

// ------------------------------------------------------------------------------------------------
// Attention of the action expert: 64 suffix rows over a share of the prefix cache (at most 10 chunks of 32 keys) and,
// in the last share, the suffix's own two chunks.  An item is 16 query rows of one head (and 1 / v_split of the head
// dimension of the output): mfma_f32_16x16x32 throughout.
// What bounds it in the persistent kernel is what follows the wait for the QKV projection, so everything that comes from
// the prefix cache is in registers before: wave w holds the keys of chunk w, waves 0 .. 3 one 16-key tile each of chunks 8 and
// 9 (a prompt of up to 48 tokens behind whole views takes no share of its own), and of the values its own 16 columns (two
// tiles of 16 with v_split 1) of every chunk.  After the wait each wave fetches one eighth of the 16 query rows (they
// meet in LDS: read by every wave from memory they were 64 of the 112 KB that the first-level cache, 64 bytes per clock,
// handed out behind the wait), waves 4 .. 7 one 16-key tile of the suffix each, and every wave its columns of the
// suffix's values; then scores, two LDS exchanges (row maximum, probabilities), and a wave accumulates its columns over
// all chunks: no sum over waves.  Chunks that a share does not have count as zero probabilities and values, so the
// products have no branches between them.
// Order of the keys inside a chunk: row i of 16-key tile t is key 16 (i / 8) + 8 t + i % 8 of the chunk.  The accumulator
// of S^T (lane = query lane % 16, rows 4 (lane / 16) + r of a tile) then gives each lane 8 keys that are one 16-byte piece
// of the value fragments, which makes them the B operand of the second product as they are.
// ------------------------------------------------------------------------------------------------
template <class Cx>
__device__ __forceinline__ void attention_suffix_body(const AttnParams p, const Cx cx, unsigned char* smem_raw) {
  constexpr int S16 = 16;                      // head dimension 256
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int qi = lane & 15;
  const int g = lane >> 4;
  if (!Cx::kPersistent) {
    if (cx.by >= p.heads) {   // warm-up block; rank = linear block index (mod 8)
      if (cx.bz == 0) prefetch_role(p.pf, cx.bx + (int)gridDim.x * (cx.by - p.heads));
      return;
    }
  }
  const int vs = p.v_split > 1 ? p.v_split : 1;
  const int qt = cx.bx / vs;                   // 16-row query tile
  const int vpart = cx.bx - qt * vs;
  const int head = cx.by;
  const int row = qt * 16 + qi;
  int cbeg0 = 0, n0 = p.chunks0, n1 = p.chunks1;
  if (p.key_splits > 1) {   // this block's share of the prefix; the last share also takes the suffix
    cbeg0 = cx.bz * p.chunks_per_split;
    n0 = min(p.chunks_per_split, p.chunks0 - cbeg0);
    if (cx.bz != p.key_splits - 1) n1 = 0;
  }
  const int nvb = 8 / vs;                      // 32-wide value slices of this item
  const int ntiles = 2 * nvb;                  // 16-column tiles of this item; this wave's are w and w + 8
  bf16* qlds = reinterpret_cast<bf16*>(smem_raw);                             // [8 steps of 32 k][64][8]
  bf16* pf = qlds + 8 * 512;                                                  // [8 + 2 of the suffix + 2 more][64][8]
  float* mw = reinterpret_cast<float*>(pf + (ATT_SHARE + 2) * 512);           // [8][16]
  float* lw = mw + ATT_WAVES * 16;                                            // [8][16]
  const bf16x8 zero8 = __builtin_bit_cast(bf16x8, u32x4_t{0u, 0u, 0u, 0u});
  // a 16-row operand of 32 k is half of two 32 x 16 fragments: lane (g, i) takes k = 8 g .. + 7 of row i (bytes; + 2 KiB per 32 k)
  const unsigned qpiece = (unsigned)((g >> 1) * 1024 + ((g & 1) * 32 + qi) * 16);                              // + 256 for the odd 16-row tile
  const unsigned kpiece = (unsigned)((g >> 1) * 1024 + ((g & 1) * 32 + (qi >> 3) * 16 + (qi & 7)) * 16);       // + 128 for tile 1
  const unsigned vpiece = (unsigned)((g >> 1) * 1024 + (g & 1) * 512 + qi * 16);                              // + 256 for the odd 16-column tile
  auto at = [](const char* base, unsigned off) { return reinterpret_cast<const bf16x8*>(base + off); };
  auto vtile = [&](const bf16* v, int dt) {    // values of chunk 0, 16-column tile dt of this item
    return reinterpret_cast<const char*>(v + (size_t)(vpart * nvb + (dt >> 1)) * 1024 + (dt & 1) * 128);
  };

  // ---- constants of the persistent kernel: keys and values of the prefix -------------------------------
  bf16x8 kf[2][8], k1f[8], vf[2][ATT_SHARE];
  const bool extra_wave = w < 4 && ATT_WAVES + (w >> 1) < n0;   // holds a 16-key tile of chunks 8 and 9
  auto load_prefix = [&]() {
    if (w < n0) {   // uniform
      const char* kp = reinterpret_cast<const char*>(p.k0 + (size_t)(cbeg0 + w) * S16 * 512);
#pragma unroll
      for (int j = 0; j < 8; j++)
#pragma unroll
        for (int h = 0; h < 2; h++) kf[h][j] = *at(kp, kpiece + h * 128 + j * 2048);
    } else {
#pragma unroll
      for (int j = 0; j < 8; j++) kf[0][j] = kf[1][j] = zero8;
    }
    if (extra_wave) {
      const char* kp = reinterpret_cast<const char*>(p.k0 + (size_t)(cbeg0 + ATT_WAVES + (w >> 1)) * S16 * 512 + (w & 1) * 64);
#pragma unroll
      for (int j = 0; j < 8; j++) k1f[j] = *at(kp, kpiece + j * 2048);
    }
#pragma unroll
    for (int a = 0; a < 2; a++) {
      const char* vp = vtile(p.v0 + (size_t)cbeg0 * 8 * 1024, w + ATT_WAVES * a);
#pragma unroll
      for (int c = 0; c < ATT_SHARE; c++) {
        if (c < n0 && w + ATT_WAVES * a < ntiles) vf[a][c] = *at(vp + (size_t)c * 16384, vpiece);   // uniform
        else vf[a][c] = zero8;
      }
    }
  };
  const bool seg1_wave = n1 > 0 && w >= 4;
  const int tile1 = w - 4;
  const char* qsrc = reinterpret_cast<const char*>(p.q + (size_t)head * p.q_head_stride + (size_t)(qt >> 1) * S16 * 512 + (qt & 1) * 128 + w * 1024);
  const char* k1src = reinterpret_cast<const char*>(p.k1 + (size_t)(max(tile1, 0) >> 1) * S16 * 512 + (tile1 & 1) * 64);
  const char* v1src[2] = {vtile(p.v1, min(w, ntiles - 1)), vtile(p.v1, min(w + ATT_WAVES, ntiles - 1))};
  // where the results go
  bf16* outp[2];
  unsigned off_out[2];
#pragma unroll
  for (int a = 0; a < 2; a++) {
    const int col = head * 256 + vpart * nvb * 32 + (w + ATT_WAVES * a) * 16 + 4 * g;
    outp[a] = p.out + (size_t)cx.bz * p.out_split_stride + ((size_t)(row >> 5) * (p.out_ld >> 4) + (col >> 4)) * 512 +
              (((col & 15) >> 3) * 32 + (row & 31)) * 8 + (col & 7);
    off_out[a] = cx.off(outp[a]);
  }
  if (Cx::kPersistent) {
    load_prefix();
    qsrc = computed_global(qsrc);
    k1src = computed_global(k1src);
    v1src[0] = computed_global(v1src[0]);
    v1src[1] = computed_global(v1src[1]);
    asm volatile("" : "+v"(off_out[0]), "+v"(off_out[1]));
    cx.wait_inputs();
  }
  // ---- inputs: query rows, suffix keys (waves 4 .. 7: 16-key tile w - 4), suffix values ---------------
  bf16x8 v1f[2][2];                            // [column tile][chunk]
  const bf16x8 qv = cx.ld_bulk(at(qsrc, qpiece));
  if (seg1_wave) {
#pragma unroll
    for (int j = 0; j < 8; j++) k1f[j] = cx.ld_bulk(at(k1src, kpiece + j * 2048));
  } else if (!extra_wave) {
#pragma unroll
    for (int j = 0; j < 8; j++) k1f[j] = zero8;
  }
  if (!Cx::kPersistent) load_prefix();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);   // all requested before the first one is waited for
  cx.mark(1);
  *reinterpret_cast<bf16x8*>(qlds + ((size_t)w * 64 + lane) * 8) = qv;
  __syncthreads();
  // the suffix's values come last: in front of the keys' requests they would delay the scores
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int c = 0; c < 2; c++) {
      if (n1 > 0 && (a == 0 || vs == 1)) v1f[a][c] = cx.ld_bulk(at(v1src[a] + c * 16384, vpiece));
      else v1f[a][c] = zero8;
    }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);

  // ---- scores ---------------------------------------------------------------------------------------
  bf16x8 qf[8];
#pragma unroll
  for (int j = 0; j < 8; j++) qf[j] = *reinterpret_cast<const bf16x8*>(qlds + ((size_t)j * 64 + lane) * 8);
  f32x4 sv[2], sv1, sodd[2], sodd1;   // even and odd k steps apart: half the dependent chain
#pragma unroll
  for (int h = 0; h < 2; h++) sv[h] = sodd[h] = f32x4{0.f, 0.f, 0.f, 0.f};
  sv1 = sodd1 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      sv[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[h][j], qf[j], sv[h], 0, 0, 0);
      sodd[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[h][j + 1], qf[j + 1], sodd[h], 0, 0, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);   // the suffix keys are not waited for above
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    sv1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1f[j], qf[j], sv1, 0, 0, 0);
    sodd1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1f[j + 1], qf[j + 1], sodd1, 0, 0, 0);
  }
#pragma unroll
  for (int h = 0; h < 2; h++) sv[h] = (sv[h] + sodd[h]) * p.scale;
  sv1 = (sv1 + sodd1) * p.scale;
  const int kg = 16 * (g >> 1) + 4 * (g & 1);   // first of this lane's keys in a chunk; + 8 for tile 1
  if (w >= n0 || (cbeg0 + w + 1) * 32 > p.valid0) {   // uniform: no chunk, or one with keys beyond the last
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int e = 0; e < 4; e++) sv[h][e] = w < n0 && (cbeg0 + w) * 32 + kg + 8 * h + e < p.valid0 ? sv[h][e] : NEG_BIG;
  }
  if (extra_wave) {   // uniform
#pragma unroll
    for (int e = 0; e < 4; e++) sv1[e] = (cbeg0 + ATT_WAVES + (w >> 1)) * 32 + kg + 8 * (w & 1) + e < p.valid0 ? sv1[e] : NEG_BIG;
  } else if (!seg1_wave) {
    sv1 = f32x4{NEG_BIG, NEG_BIG, NEG_BIG, NEG_BIG};
  } else if (p.suffix_mask) {
#pragma unroll
    for (int e = 0; e < 4; e++) sv1[e] = row != 0 || (tile1 >> 1) * 32 + kg + 8 * (tile1 & 1) + e == 0 ? sv1[e] : NEG_BIG;
  }
  float m_loc = fmaxf(fmaxf(fmaxf(sv1[0], sv1[1]), fmaxf(sv1[2], sv1[3])), NEG_BIG);
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int e = 0; e < 4; e++) m_loc = fmaxf(m_loc, sv[h][e]);
  m_loc = max_xor32(max_xor16(m_loc));
  if (g == 0) mw[w * 16 + qi] = m_loc;
  __syncthreads();
  cx.mark(2);   // scores done
  float m_part[ATT_WAVES];
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) m_part[i] = mw[i * 16 + qi];
  __builtin_amdgcn_sched_barrier(0);
  float m_all = NEG_BIG;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) m_all = fmaxf(m_all, m_part[i]);

  // ---- probabilities -> B operand of the second product, in LDS ---------------------------------------
  // Masked keys come out as exactly 0: far below any maximum, or (a row without a key) below half of the mask value
  const float m_sub = fmaxf(m_all, 0.5f * NEG_BIG);
  float l_loc = 0.f;
  auto prob = [&](float v) {
    const float e = __expf(v - m_sub);
    l_loc += e;
    return e;
  };
  {
    bf16x8 pb;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int e = 0; e < 4; e++) pb[4 * h + e] = (bf16)prob(sv[h][e]);
    *reinterpret_cast<bf16x8*>(pf + ((size_t)w * 64 + lane) * 8) = pb;
  }
  if (w >= 4 || n0 > ATT_WAVES) {   // uniform: the suffix's from waves 4 .. 7, then chunks 8 and 9 from waves 0 .. 3
    bf16x4 pb;
#pragma unroll
    for (int e = 0; e < 4; e++) pb[e] = (bf16)prob(sv1[e]);
    *reinterpret_cast<bf16x4*>(pf + ((size_t)(ATT_WAVES + ((w ^ 4) >> 1)) * 64 + lane) * 8 + (w & 1) * 4) = pb;
  }
  l_loc = add_xor32(add_xor16(l_loc));
  if (g == 0) lw[w * 16 + qi] = l_loc;
  __syncthreads();
  cx.mark(3);   // probabilities in LDS
  if (w >= ntiles) return;

  // ---- output columns: O^T tile = V^T P^T over all chunks, two chains per tile ------------------------
  bf16x8 b[ATT_WAVES + 2];
#pragma unroll
  for (int c = 0; c < ATT_WAVES + 2; c++) b[c] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)c * 64 + lane) * 8);
  float l_part[ATT_WAVES];
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_part[i] = lw[i * 16 + qi];
  __builtin_amdgcn_sched_barrier(0);   // every read in flight
  f32x4 o[2][2];
#pragma unroll
  for (int a = 0; a < 2; a++)
#pragma unroll
    for (int c = 0; c < 2; c++) o[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < ATT_WAVES + 2; c++)
#pragma unroll
    for (int a = 0; a < 2; a++)
      o[a][c & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c < ATT_WAVES ? vf[a][c] : v1f[a][c - ATT_WAVES], b[c], o[a][c & 1], 0, 0, 0);
  if (n0 > ATT_WAVES) {   // uniform; without the branch these two chunks cost the shares that have none 0.15 us
#pragma unroll
    for (int c = ATT_WAVES; c < ATT_SHARE; c++) {
      const bf16x8 bc = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c + 2) * 64 + lane) * 8);
#pragma unroll
      for (int a = 0; a < 2; a++) o[a][c & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[a][c], bc, o[a][c & 1], 0, 0, 0);
    }
  }
  cx.mark(4);   // P V done
  float l_all = 0.f;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_all += l_part[i];
  const float inv = 1.0f / l_all;
  if (row >= p.Tq) return;
  if (p.ml_out != nullptr && w == 0 && g == 0 && vpart == 0) {   // (row maximum, sum) of this share, for the consumer's merge
    float* dst = p.ml_out + ((((size_t)cx.bz * p.heads + head) * ((p.Tq + 31) >> 5) * 32) + row) * 2;
    cx.st(reinterpret_cast<float2*>(dst), make_float2(m_all, l_all));
  }
#pragma unroll
  for (int a = 0; a < 2; a++) {
    if (a == 0 || vs == 1) {
      bf16x4 ob;
#pragma unroll
      for (int e = 0; e < 4; e++) ob[e] = (bf16)((o[a][0][e] + o[a][1][e]) * inv);
      if (Cx::kPersistent) cx.st_off(off_out[a], ob);
      else cx.st(reinterpret_cast<bf16x4*>(outp[a]), ob);
    }
  }
}

// query rows, probabilities, row maxima and sums
static constexpr int ATTN_SUFFIX_SMEM = 8 * 1024 + (ATT_SHARE + 2) * 1024 + 2 * ATT_WAVES * 16 * 4;
// shapes attention_suffix_body covers: n0 = prefix chunks per share; the expert's rows with their own two chunks, or any number
// of rows without
static inline bool attn_suffix_ok(const AttnParams& p, int n0) {
  const int vs = p.v_split > 1 ? p.v_split : 1;
  return p.head_dim == 256 && (p.chunks1 == 0 || (p.chunks1 == 2 && p.Tq == 64)) && p.view_tokens == 0 && p.kv_head_stride0 == 0 && p.v_head_stride0 == 0 &&
         n0 >= 1 && n0 <= ATT_SHARE && (vs == 1 || vs == 2 || vs == 4 || vs == 8);
}

// ------------------------------------------------------------------------------------------------
// Attention of the prefix inside its persistent kernel, by four waves.  An item is 16 query rows of one head over at most 10 chunks of
// keys (attention_prefix16_body: the sums of attention_suffix_body without a suffix) or 32 query rows over more
// (attention_prefix32_body: those of attention_body with several key rounds), in the same order, so the same bits: a wave does what
// waves w and w + 4 of those do.  512 registers per wave hold all keys and values of the former; the latter keeps two chunks of
// keys and a ring of values on their way.
// ------------------------------------------------------------------------------------------------
constexpr int PREFIX_WAVES = 4;
constexpr int ATTN_PREFIX16_SMEM = 8 * 1024 + ATT_SHARE * 1024 + 2 * ATT_WAVES * 16 * 4;
template <class Cx>
__device__ __forceinline__ void attention_prefix16_body(const AttnParams p, const Cx cx, unsigned char* smem_raw) {
  constexpr int S16 = 16, V = ATT_WAVES / PREFIX_WAVES;   // head dimension 256
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int qi = lane & 15;
  const int g = lane >> 4;
  const int qt = cx.bx, head = cx.by, n0 = p.chunks0;
  const int row = qt * 16 + qi;
  bf16* qlds = reinterpret_cast<bf16*>(smem_raw);                             // [8 steps of 32 k][64][8]
  bf16* pf = qlds + 8 * 512;                                                  // [10 chunks][64][8]
  float* mw = reinterpret_cast<float*>(pf + ATT_SHARE * 512);                 // [8][16]
  float* lw = mw + ATT_WAVES * 16;                                            // [8][16]
  const bf16x8 zero8 = __builtin_bit_cast(bf16x8, u32x4_t{0u, 0u, 0u, 0u});
  const unsigned qpiece = (unsigned)((g >> 1) * 1024 + ((g & 1) * 32 + qi) * 16);                              // + 256 for the odd 16-row tile
  const unsigned kpiece = (unsigned)((g >> 1) * 1024 + ((g & 1) * 32 + (qi >> 3) * 16 + (qi & 7)) * 16);       // + 128 for tile 1
  const unsigned vpiece = (unsigned)((g >> 1) * 1024 + (g & 1) * 512 + qi * 16);                              // + 256 for the odd 16-column tile
  auto ld = [&](const char* base, unsigned off) { return cx.ld_bulk(reinterpret_cast<const bf16x8*>(base + off)); };

  bf16x8 qv[V], kf[V][2][8], k1f[8], vf[V][2][ATT_SHARE];
  const char* const qsrc = reinterpret_cast<const char*>(p.q + (size_t)head * p.q_head_stride + (size_t)(qt >> 1) * S16 * 512 + (qt & 1) * 128);
#pragma unroll
  for (int v = 0; v < V; v++) qv[v] = ld(qsrc, qpiece + (unsigned)(w + PREFIX_WAVES * v) * 2048u);
#pragma unroll
  for (int v = 0; v < V; v++) {
    const int c = w + PREFIX_WAVES * v;
    const char* const kp = reinterpret_cast<const char*>(p.k0 + (size_t)c * S16 * 512);
    if (c < n0) {   // uniform
#pragma unroll
      for (int j = 0; j < 8; j++)
#pragma unroll
        for (int h = 0; h < 2; h++) kf[v][h][j] = ld(kp, kpiece + h * 128 + j * 2048);
    } else {
#pragma unroll
      for (int j = 0; j < 8; j++) kf[v][0][j] = kf[v][1][j] = zero8;
    }
  }
  const bool extra = ATT_WAVES + (w >> 1) < n0;   // this wave also has a 16-key tile of chunks 8 and 9
  if (extra) {
    const char* const kp = reinterpret_cast<const char*>(p.k0 + (size_t)(ATT_WAVES + (w >> 1)) * S16 * 512 + (w & 1) * 64);
#pragma unroll
    for (int j = 0; j < 8; j++) k1f[j] = ld(kp, kpiece + j * 2048);
  } else {
#pragma unroll
    for (int j = 0; j < 8; j++) k1f[j] = zero8;
  }
  // 16-column tiles w, w + 4, w + 8, w + 12 of the values
#pragma unroll
  for (int c = 0; c < ATT_SHARE; c++)
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int a = 0; a < 2; a++) {
        const int dt = w + PREFIX_WAVES * v + ATT_WAVES * a;
        if (c < n0) vf[v][a][c] = ld(reinterpret_cast<const char*>(p.v0 + (size_t)(dt >> 1) * 1024 + (dt & 1) * 128) + (size_t)c * 16384, vpiece);   // uniform
        else vf[v][a][c] = zero8;
      }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);   // all requested before the first one is waited for
#pragma unroll
  for (int v = 0; v < V; v++) *reinterpret_cast<bf16x8*>(qlds + ((size_t)(w + PREFIX_WAVES * v) * 64 + lane) * 8) = qv[v];
  __syncthreads();

  // ---- scores ---------------------------------------------------------------------------------------
  bf16x8 qf[8];
#pragma unroll
  for (int j = 0; j < 8; j++) qf[j] = *reinterpret_cast<const bf16x8*>(qlds + ((size_t)j * 64 + lane) * 8);
  f32x4 sv[V][2], sodd[V][2], sv1 = {0.f, 0.f, 0.f, 0.f}, sodd1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int h = 0; h < 2; h++) sv[v][h] = sodd[v][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < 8; j += 2)
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        sv[v][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[v][h][j], qf[j], sv[v][h], 0, 0, 0);
        sodd[v][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[v][h][j + 1], qf[j + 1], sodd[v][h], 0, 0, 0);
      }
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    sv1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1f[j], qf[j], sv1, 0, 0, 0);
    sodd1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k1f[j + 1], qf[j + 1], sodd1, 0, 0, 0);
  }
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int h = 0; h < 2; h++) sv[v][h] = (sv[v][h] + sodd[v][h]) * p.scale;
  sv1 = (sv1 + sodd1) * p.scale;
  const int kg = 16 * (g >> 1) + 4 * (g & 1);   // first of this lane's keys in a chunk; + 8 for tile 1
#pragma unroll
  for (int v = 0; v < V; v++) {
    const int c = w + PREFIX_WAVES * v;
    float m_loc = NEG_BIG;
    if (c >= n0 || (c + 1) * 32 > p.valid0) {   // uniform: no chunk, or one with keys beyond the last
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int e = 0; e < 4; e++) sv[v][h][e] = c < n0 && c * 32 + kg + 8 * h + e < p.valid0 ? sv[v][h][e] : NEG_BIG;
    }
    if (v == 0) {
#pragma unroll
      for (int e = 0; e < 4; e++) {
        sv1[e] = extra && (ATT_WAVES + (w >> 1)) * 32 + kg + 8 * (w & 1) + e < p.valid0 ? sv1[e] : NEG_BIG;
        m_loc = fmaxf(m_loc, sv1[e]);
      }
    }
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int e = 0; e < 4; e++) m_loc = fmaxf(m_loc, sv[v][h][e]);
    m_loc = max_xor32(max_xor16(m_loc));
    if (g == 0) mw[c * 16 + qi] = m_loc;
  }
  __syncthreads();
  float m_part[ATT_WAVES];
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) m_part[i] = mw[i * 16 + qi];
  __builtin_amdgcn_sched_barrier(0);
  float m_all = NEG_BIG;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) m_all = fmaxf(m_all, m_part[i]);

  // ---- probabilities -> B operand of the second product, in LDS ---------------------------------------
  const float m_sub = fmaxf(m_all, 0.5f * NEG_BIG);
#pragma unroll
  for (int v = 0; v < V; v++) {
    float l_loc = 0.f;
    auto prob = [&](float x) {
      const float e = __expf(x - m_sub);
      l_loc += e;
      return e;
    };
    bf16x8 pb;
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
      for (int e = 0; e < 4; e++) pb[4 * h + e] = (bf16)prob(sv[v][h][e]);
    *reinterpret_cast<bf16x8*>(pf + ((size_t)(w + PREFIX_WAVES * v) * 64 + lane) * 8) = pb;
    if (v == 0 && n0 > ATT_WAVES) {   // uniform
      bf16x4 p1;
#pragma unroll
      for (int e = 0; e < 4; e++) p1[e] = (bf16)prob(sv1[e]);
      *reinterpret_cast<bf16x4*>(pf + ((size_t)(ATT_WAVES + (w >> 1)) * 64 + lane) * 8 + (w & 1) * 4) = p1;
    }
    l_loc = add_xor32(add_xor16(l_loc));
    if (g == 0) lw[(w + PREFIX_WAVES * v) * 16 + qi] = l_loc;
  }
  __syncthreads();

  // ---- output columns: O^T tile = V^T P^T over all chunks, two chains per tile ------------------------
  float l_part[ATT_WAVES];
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_part[i] = lw[i * 16 + qi];
  bf16x8 b[ATT_WAVES];
#pragma unroll
  for (int c = 0; c < ATT_WAVES; c++) b[c] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)c * 64 + lane) * 8);
  __builtin_amdgcn_sched_barrier(0);   // every read in flight
  f32x4 o[V][2][2];
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int a = 0; a < 2; a++) o[v][a][0] = o[v][a][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < ATT_WAVES; c++)
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int a = 0; a < 2; a++) o[v][a][c & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[v][a][c], b[c], o[v][a][c & 1], 0, 0, 0);
  if (n0 > ATT_WAVES) {   // uniform
#pragma unroll
    for (int c = ATT_WAVES; c < ATT_SHARE; c++) {
      const bf16x8 bc = *reinterpret_cast<const bf16x8*>(pf + ((size_t)c * 64 + lane) * 8);
#pragma unroll
      for (int v = 0; v < V; v++)
#pragma unroll
        for (int a = 0; a < 2; a++) o[v][a][c & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[v][a][c], bc, o[v][a][c & 1], 0, 0, 0);
    }
  }
  float l_all = 0.f;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_all += l_part[i];
  const float inv = 1.0f / l_all;
  if (row >= p.Tq) return;
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int a = 0; a < 2; a++) {
      const int col = head * 256 + (w + PREFIX_WAVES * v + ATT_WAVES * a) * 16 + 4 * g;
      bf16x4 ob;
#pragma unroll
      for (int e = 0; e < 4; e++) ob[e] = (bf16)((o[v][a][0][e] + o[v][a][1][e]) * inv);
      cx.st(reinterpret_cast<bf16x4*>(p.out + ((size_t)(row >> 5) * (p.out_ld >> 4) + (col >> 4)) * 512 + (((col & 15) >> 3) * 32 + (row & 31)) * 8 + (col & 7)), ob);
    }
}

// CM: most chunks of a wave (4 CM in all); RING: chunks of values in flight, EARLY of them from the start
constexpr int attn_prefix32_smem(int cm) { return 16 * 1024 + 2 * ATT_WAVES * 32 * 4 + 4 * cm * 2048; }
template <int CM, int EARLY, int RING, class Cx>
__device__ __forceinline__ void attention_prefix32_body(const AttnParams& p, const Cx& cx, unsigned char* smem_raw) {
  constexpr int S16 = 16, NVB = 8, V = 2;
  bf16* qs = reinterpret_cast<bf16*>(smem_raw);                               // [16][64][8]
  float* mw = reinterpret_cast<float*>(qs + S16 * 512);                       // [4][32]
  float* lw = mw + ATT_WAVES * 32;                                            // [8][32]
  bf16* pf = reinterpret_cast<bf16*>(lw + ATT_WAVES * 32);                    // [chunks][2][64][8]
  const int t = cx.tid();
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lq = lane & 31;
  const int lh = lane >> 5;
  const int tile = cx.bx, head = cx.by, n0 = p.chunks0;
  const int row = tile * 32 + lq;
  const unsigned l16 = (unsigned)lane * 16u;
  auto ld = [&](const char* base, unsigned off) { return cx.ld_bulk(reinterpret_cast<const bf16x8*>(base + off)); };
  const char* const qsrc = reinterpret_cast<const char*>(p.q + (size_t)head * p.q_head_stride + (size_t)tile * S16 * 512);
  const char* const kbase = reinterpret_cast<const char*>(p.k0);
  const char* const vbase = reinterpret_cast<const char*>(p.v0) + w * 2048;   // slice w; slice w + 4: + 8 KiB

  bf16x8 qreg[4], kf[2][S16], vf[RING][V][2];
#pragma unroll
  for (int i = 0; i < 4; i++) qreg[i] = ld(qsrc, (unsigned)(w * 4 + i) * 1024u + l16);
  auto kchunk = [&](int i) { return kbase + (size_t)min(w + PREFIX_WAVES * i, n0 - 1) * (S16 * 1024); };   // the wave's chunk i, clamped
#pragma unroll
  for (int u = 0; u < 2; u++)
#pragma unroll
    for (int s = 0; s < S16; s++) kf[u][s] = ld(kchunk(u), (unsigned)s * 1024u + l16);
  auto load_v = [&](int r, int c) {
    const char* const vp = vbase + (size_t)min(c, n0 - 1) * (NVB * 2048);
#pragma unroll
    for (int v = 0; v < V; v++)
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) vf[r][v][s2] = ld(vp, (unsigned)(v * 8192 + s2 * 1024) + l16);
  };
#pragma unroll
  for (int r = 0; r < EARLY; r++) load_v(r, r);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 4; i++) *reinterpret_cast<bf16x8*>(qs + ((size_t)(w * 4 + i) * 64 + lane) * 8) = qreg[i];
  __syncthreads();

  // ---- scores of chunks w, w + 4, ..., two at a time --------------------------------------------------
  float sv[CM][16], m_loc = NEG_BIG;
#pragma unroll
  for (int i = 0; i < CM; i += 2) {
    if (w + PREFIX_WAVES * i < n0) {   // uniform
      const bool more = i + 2 < CM && w + PREFIX_WAVES * (i + 2) < n0;
      f32x16 acc[2];
#pragma unroll
      for (int e = 0; e < 16; e++) acc[0][e] = acc[1][e] = 0.f;
#pragma unroll
      for (int s0 = 0; s0 < S16; s0 += 4) {
        bf16x8 qb[4];
#pragma unroll
        for (int j = 0; j < 4; j++) qb[j] = *reinterpret_cast<const bf16x8*>(qs + ((size_t)(s0 + j) * 64 + lane) * 8);
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
          for (int u = 0; u < 2; u++) {
            const bf16x8 a = kf[u][s0 + j];
            if (more) kf[u][s0 + j] = ld(kchunk(i + 2 + u), (unsigned)(s0 + j) * 1024u + l16);
            acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qb[j], acc[u], 0, 0, 0);
          }
      }
#pragma unroll
      for (int u = 0; u < 2; u++) {
        if (i + u >= CM) continue;
        const int c = w + PREFIX_WAVES * (i + u);
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int key = c * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
          sv[i + u < CM ? i + u : 0][e] = c < n0 && key < p.valid0 ? acc[u][e] * p.scale : NEG_BIG;
          m_loc = fmaxf(m_loc, sv[i + u < CM ? i + u : 0][e]);
        }
      }
    }
  }
#pragma unroll
  for (int r = EARLY; r < RING; r++) load_v(r, r);   // in the keys' registers
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  m_loc = max_xor32(m_loc);
  if (lh == 0) mw[w * 32 + lq] = m_loc;
  __syncthreads();
  float m_all = NEG_BIG;
#pragma unroll
  for (int i = 0; i < PREFIX_WAVES; i++) m_all = fmaxf(m_all, mw[i * 32 + lq]);
  float l_loc[V] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < CM; i++) {
    const int c = w + PREFIX_WAVES * i;
    if (c < n0) {   // uniform
      float pr[16];
#pragma unroll
      for (int e = 0; e < 16; e++) {
        pr[e] = sv[i][e] > 0.5f * NEG_BIG ? __expf(sv[i][e] - m_all) : 0.f;   // masked keys: exactly 0
        l_loc[i & 1] += pr[e];
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) {
        bf16x8 pb;
#pragma unroll
        for (int j = 0; j < 8; j++) pb[j] = (bf16)pr[8 * s2 + j];
        *reinterpret_cast<bf16x8*>(pf + ((size_t)(c * 2 + s2) * 64 + lane) * 8) = pb;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < V; v++) {
    l_loc[v] = add_xor32(l_loc[v]);
    if (lh == 0) lw[(w + PREFIX_WAVES * v) * 32 + lq] = l_loc[v];
  }
  __syncthreads();

  // ---- output: slices w and w + 4 of the head over all chunks -------------------------------------------
  f32x16 o[V];
#pragma unroll
  for (int e = 0; e < 16; e++) o[0][e] = o[1][e] = 0.f;
  for (int c0 = 0; c0 < n0; c0 += RING) {
#pragma unroll
    for (int r = 0; r < RING; r++) {
      const int c = c0 + r;
      if (c >= n0) break;   // uniform
      bf16x8 bp[2];
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++) bp[s2] = *reinterpret_cast<const bf16x8*>(pf + ((size_t)(c * 2 + s2) * 64 + lane) * 8);
#pragma unroll
      for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
        for (int v = 0; v < V; v++) o[v] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[r][v][s2], bp[s2], o[v], 0, 0, 0);
      if (c + RING < n0) load_v(r, c + RING);
    }
  }
  float l_all = 0.f;
#pragma unroll
  for (int i = 0; i < ATT_WAVES; i++) l_all += lw[i * 32 + lq];
  const float inv = 1.0f / l_all;
  if (row >= p.Tq) return;
#pragma unroll
  for (int v = 0; v < V; v++)
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int col = head * 256 + (w + PREFIX_WAVES * v) * 32 + 8 * i + 4 * lh;
      const bf16x4 ob = {(bf16)(o[v][4 * i] * inv), (bf16)(o[v][4 * i + 1] * inv), (bf16)(o[v][4 * i + 2] * inv), (bf16)(o[v][4 * i + 3] * inv)};
      cx.st(reinterpret_cast<bf16x4*>(p.out + ((size_t)(row >> 5) * (p.out_ld >> 4) + (col >> 4)) * 512 + (((col & 15) >> 3) * 32 + (row & 31)) * 8 + (col & 7)), ob);
    }
}
