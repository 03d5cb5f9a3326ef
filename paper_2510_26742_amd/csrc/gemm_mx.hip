// Reduced-precision variant of the prefix feed-forward GEMMs (gate||up with the GeGLU epilogue, down as
// split-K partials) on MXFP8 operands: FP8 E4M3 elements with one power-of-two scale per 32 consecutive
// k, multiplied by mfma_scale_f32_32x32x64_f8f6f4, which applies the block scales in hardware.  The
// paper only names 8-bit multiplication as a direction (Section 9.1); the format and where the rounding
// happens are choices of this library.
//
// Same plan as the bf16 kernel of gemm_tile.hip: a block of 4 waves owns 2 MT * 32 tokens x 2 NT * 32 features, one wave per SIMD, both
// operands requested straight into LDS.  A fragment of 32 rows x 64 k is two pieces of 1 KiB, and a product of 64 k takes as long as two of the bf16
// loop's: in pieces and cycles a step of 64 k is a stage of that loop, and such a GEMM is the bf16 one with half the contraction.  Tile and
// number of k ranges are therefore what gemm_tile.hip chooses for half the contraction.  The scales of four steps are one dword per
// lane and 32 rows; they go to LDS ahead of the operands of the first of them, and to registers a step ahead.
// What bounds it: at 256 tokens the weights' way from memory (67 MB of gate||up: 14 of 24.5 us), beyond that the clock that the matrix cores'
// power leaves (768 tokens: 49 thousand cycles of products and 19 thousand of the epilogue's instructions per compute unit, in 53 us).  us per launch in traced passes
// at 256 / 512 / 533 / 768 / 816 tokens, 128 x 256 tiles with the weights straight to registers (two blocks on a compute unit from 512 tokens on) -> this:
// gate||up 27.0 / 39.0 / 53.6 / 58.2 / 66.1 -> 24.5 / 35.2 / 53.3 / 53.3 / 66.4, down with its reduction 26.3 / 34.4 / 36.6 / 43.6 / 48.0 -> 20.9 / 31.4 / 34.3 / 41.0 / 44.6.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pi0_internal.h"

#include "gemm_tile_body.h"

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ i32x8 cat(const i32x4& lo, const i32x4& hi) {
  i32x8 r;
  r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
  r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
  return r;
}

__device__ __forceinline__ float gelu_tanh_mx(float x) {
  // 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3); the exponent as in gelu_tanh_f
  const float e = x * __builtin_fmaf(x * x, -2.3022081984f * 0.044715f, -2.3022081984f);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(e));
}

// steps of 64 k in LDS: eight with the smallest tile, as in gemm_tile.hip, four otherwise (eight of 3 x 2 leave no room for the scales)
constexpr int mx_stages(int MT, int NT) { return MT * NT <= 4 ? 8 : 4; }
constexpr int mx_smem(int MT, int NT) { return mx_stages(MT, NT) * 4 * (MT + NT) * 1024 + 2 * 2 * (MT + NT) * 256; }
static_assert(mx_stages(2, 2) * 64 == 2 * lds_tile_group(2, 2), "gemm_lds_tile knows what a turn of the loop is");

// range_per_die: partial sums, blocks in order and a k range for each die, as in gemm_lds_body.  WALK: a block takes its tiles one after the
// other, and the next one's first stages are on their way during the epilogue.
template <int MT, int NT, int EPI, bool WALK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_mx_kernel(MxGemmParams p, int range_per_die) {
  constexpr int W = 4, S = mx_stages(MT, NT);
  constexpr int XB = 2 * MT, WB = 2 * NT, NB = XB + WB;   // 32-row blocks of the two operands
  constexpr int NF = 2 * NB, L = NF / W;                  // pieces of a stage, of a wave's share of it
  constexpr int SL = (NB + W - 1) / W;                    // scale requests of a wave, for a group of four steps
  static_assert(NF % W == 0 && S % 4 == 0 && NT % 2 == 0 && 8 % WB == 0, "even shares, whole groups, pairs of feature tiles, features are a multiple of 256");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [stage][block][2][1 KiB], then scales [group % 2][block][256]
  unsigned char* const scales = smem + S * NF * 1024;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = w & 1, wn = w >> 1;
  const int lq = lane & 31;
  const int lh = lane >> 5;

  const int n_tiles = p.n_pad >> 5;
  const int total = n_tiles / WB * p.m_tiles;
  const int bx = range_per_die ? (int)blockIdx.x >> 3 : (int)blockIdx.x, by = range_per_die ? (int)blockIdx.x & 7 : (int)blockIdx.y;
  int first = 0, of_die = total, rank = bx;
  if (!range_per_die) {   // consecutive ids on different dies, a die takes a contiguous eighth, token tiles fastest
    lds_tile_share(bx & 7, total, first, of_die);
    rank = bx >> 3;
  }
  if (rank >= of_die) return;
  int nb = (first + rank) / p.m_tiles;
  int m0 = ((first + rank) - nb * p.m_tiles) * (XB * 32);
  const int mb_last = (p.M - 1) >> 5;
  const int KC64 = p.k_pad >> 6, XKC64 = p.ldx >> 6;
  const int kbeg = by * (p.k_per_split >> 6);
  const int turns = (min(kbeg + (p.k_per_split >> 6), KC64) - kbeg) / S;

  // the wave's piece i of a stage is piece w + 4 i of the block's: operand block f / 2 (tokens first), half f % 2; blocks beyond the
  // rows repeat the last one and are not stored (features: a multiple of every tile)
  const unsigned char *src[L], *ssrc[SL];
  unsigned sdst[SL];
  auto set_sources = [&]() {
#pragma unroll
    for (int i = 0; i < L; i++) {
      const int f = w + W * i, b = f >> 1;
      const unsigned char* const base = b < XB ? p.X8 + (size_t)min((m0 >> 5) + b, mb_last) * XKC64 * 2048 : p.W8 + (size_t)(nb * WB + (b - XB)) * KC64 * 2048;
      src[i] = base + (size_t)kbeg * 2048 + (f & 1) * 1024;
    }
#pragma unroll
    for (int i = 0; i < SL; i++) {
      const int b = min(w + W * i, NB - 1);
      const unsigned char* const base = b < XB ? p.XS + (size_t)min((m0 >> 5) + b, mb_last) * (XKC64 >> 2) * 256 : p.WS + (size_t)(nb * WB + (b - XB)) * (KC64 >> 2) * 256;
      ssrc[i] = base + (size_t)(kbeg >> 2) * 256;
      sdst[i] = lds_address(scales) + (unsigned)b * 256u;
    }
  };
  set_sources();
  const unsigned lds0 = lds_address(smem) + (unsigned)w * 1024u;
  // blocks start at different places of their range and go round it where gemm_lds_body's do
  int turn = p.m_tiles == 1 || (EPI == MX_EPI_PARTIAL && p.M <= 320) ? (int)((unsigned)nb % (unsigned)turns) : 0;
  const unsigned vfirst = (unsigned)lane * 16u + 4096u;
  unsigned voff = vfirst + (unsigned)turn * (S * 2048u);   // of the current turn: stages 0 .. 3 are at 2048 q - 4096, a 13-bit constant
  unsigned par = 0;                                        // four stages: half of the scales' place that the current turn's are in
  auto issue = [&](auto Q, auto I, unsigned v) {
    constexpr int q = decltype(Q)::value, i = decltype(I)::value, off = q % 4 * 2048 - 4096;
    const unsigned l0 = lds0;
    const unsigned char* const s = src[i];
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%4" ::"s"(l0), "v"(v + (unsigned)(q / 4) * 8192u), "s"(s),
                 "n"((q * NF + W * i) * 1024 - off), "n"(off)
                 : "memory", "scc");
  };
  // scales of the group that starts with stage q, into half `half` of their place; turn: the stage's
  auto issue_scales = [&](int q, unsigned half, int turn) {
    const unsigned v = (unsigned)lane * 4u + (unsigned)(turn * (S / 4) + q / 4) * 256u;
#pragma unroll
    for (int i = 0; i < SL; i++) {
      const unsigned to = sdst[i] + half * (NB * 256u);
      const unsigned char* const s = ssrc[i];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(to), "v"(v), "s"(s) : "memory");
    }
  };
  // row statistics, of which RMS wants the sum of squares: in front of everything
  float ssq[MT];
  auto load_stats = [&](float (&to)[MT]) {
#pragma unroll
    for (int i = 0; i < MT; i++) to[i] = EPI == MX_EPI_GEGLU ? p.rowstat[2 * (size_t)min(m0 + (wm * MT + i) * 32 + lq, p.M - 1) + 1] : 0.f;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  load_stats(ssq);
  auto issue_first = [&]() {
    for_each<S - 1>([&](auto Q) {
      constexpr int q = decltype(Q)::value;
      if constexpr (q % 4 == 0) issue_scales(q, (q / 4) & 1, turn);
      for_each<L>([&](auto I) { issue(Q, I, voff); });
    });
  };
  issue_first();

  for (int next = rank + WALK_BLOCKS / 8;; next += WALK_BLOCKS / 8) {
    f32x16 acc[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; j++)
#pragma unroll
      for (int i = 0; i < MT; i++) zero_accumulator(acc[j][i]);
    i32x4 xf[2][MT][2], wf[2][NT][2];
    int sx[2][MT], sw[2][NT];
    constexpr int R = 2 * (MT + NT), P = MT * NT;   // reads and products of a step
    const unsigned char* const xs = smem + lane * 16 + wm * MT * 2048;
    const unsigned char* const ws = smem + lane * 16 + (XB + wn * NT) * 2048;
    const unsigned char* const sxs = scales + lane * 4 + wm * MT * 256;
    const unsigned char* const sws = scales + lane * 4 + (XB + wn * NT) * 256;
    // read r of stage q, in the order in which the products need them: x0, w0 .. , x1 ..
    auto read = [&](int u, int q, int r) {
      const int f = r >> 1, h = r & 1, o = q * NF * 1024 + h * 1024;
      if (f == 0) xf[u][0][h] = *reinterpret_cast<const i32x4*>(xs + o);
      else if (f <= NT) wf[u][f - 1][h] = *reinterpret_cast<const i32x4*>(ws + o + (f - 1) * 2048);
      else xf[u][f - NT][h] = *reinterpret_cast<const i32x4*>(xs + o + (f - NT) * 2048);
    };
    auto read_scales = [&](int set, unsigned half) {
#pragma unroll
      for (int i = 0; i < MT; i++) sx[set][i] = *reinterpret_cast<const int*>(sxs + half * (NB * 256u) + i * 256);
#pragma unroll
      for (int j = 0; j < NT; j++) sw[set][j] = *reinterpret_cast<const int*>(sws + half * (NB * 256u) + j * 256);
    };
    // requests of stages a .. b of a turn and the next
    constexpr auto requests = [](int a, int b) constexpr {
      int n = 0;
      for (int q = a; q <= b; q++) n += L + (q % 4 == 0 ? SL : 0);
      return n;
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(requests(1, S - 2)) : "memory");   // stage 0 is complete for everybody
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_scales(0, 0);
#pragma unroll
    for (int r = 0; r < R; r++) read(0, 0, r);

    // One turn of S steps; LAST: nothing beyond it is requested.  Step s multiplies the fragments of set s % 2 and reads those of the next step
    // into the other one: the next stage must be complete for everybody (those up to S - 2 on may be on their way).  Everybody is then through with
    // stage s - 1, whose place stage s + S - 1 takes.
    auto group = [&](auto last_turn) {
      constexpr bool LAST = decltype(last_turn)::value != 0;
      const int turn_now = turn;
      turn = turn + 1 == turns ? 0 : turn + 1;
      const unsigned vnext = vfirst + (unsigned)turn * (S * 2048u);
      for_each<S>([&](auto SS) {
        constexpr int s = decltype(SS)::value, u = s & 1, q = (s + S - 1) % S;   // q: the stage requested
        constexpr bool more = !(LAST && s == S - 1), request = !LAST || s == 0;
        constexpr int set = S == 8 ? (s >> 2) & 1 : 0;
        if constexpr (more) {
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(requests(s + 2, LAST ? S - 1 < s + S - 2 ? S - 1 : s + S - 2 : s + S - 2)) : "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
        }
        if constexpr (request && q % 4 == 0) {
          issue_scales(q, S == 8 ? (unsigned)(q >> 2) & 1u : par ^ 1u, s == 0 ? turn_now : turn);
        }
        for_each<P>([&](auto MM) {
          constexpr int m = decltype(MM)::value;
          if constexpr (more) {
#pragma unroll
            for (int r = 0; r < R; r++)
              if (r * P / R == m) read(u ^ 1, (s + 1) % S, r);
            if constexpr (s % 4 == 3 && m == 0) read_scales(S == 8 ? set ^ 1 : 1, S == 8 ? (unsigned)((s + 1) >> 2) & 1u : par ^ 1u);
          }
          if constexpr (request) {
            for_each<L>([&](auto I) {
              if constexpr ((2 * decltype(I)::value + 1) * P / (2 * L) == m) issue(Int<q>{}, I, s == 0 ? voff : vnext);
            });
          }
          constexpr int i = m / NT, j = m % NT;
          acc[j][i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cat(wf[u][j][0], wf[u][j][1]), cat(xf[u][i][0], xf[u][i][1]), acc[j][i], 0, 0, s & 3, sw[set][j], s & 3, sx[set][i]);
          __builtin_amdgcn_sched_barrier(0);   // this order
        });
      });
      voff = vnext;
      if constexpr (S == 4 && !LAST) {
        par ^= 1u;
#pragma unroll
        for (int i = 0; i < MT; i++) sx[0][i] = sx[1][i];
#pragma unroll
        for (int j = 0; j < NT; j++) sw[0][j] = sw[1][j];
      }
    };
    for (int g = 0; g + 1 < turns; g++) group(Int<0>{});
    group(Int<1>{});
    // every product is done here: left alone, the compiler moves a tile's last ones behind the conditions of its stores, one chain each, with
    // their operands spilled
#pragma unroll
    for (int i = 0; i < MT; i++)
#pragma unroll
      for (int j = 0; j < NT; j++) asm volatile("" ::"v"(acc[j][i][0]));

    const int nt0 = nb * WB + wn * NT, mb0 = (m0 >> 5) + wm * MT;
    int nb_next = 0, m0_next = 0;
    float ssq_next[MT] = {};
    if (WALK && next < of_die) {
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();   // everybody has read the last stage
      const int nb_now = nb, m0_now = m0;
      nb = nb_next = (first + next) / p.m_tiles;
      m0 = m0_next = ((first + next) - nb * p.m_tiles) * (XB * 32);
      set_sources();
      load_stats(ssq_next);
      voff = vfirst;
      par = 0;
      issue_first();
      nb = nb_now;
      m0 = m0_now;
    }

    // ---- epilogue: lane -> token lq of each 32-token block, features nt * 32 + 8 * (r / 4) + 4 * lh + r % 4 ----
    if constexpr (EPI == MX_EPI_PARTIAL) {   // whole tiles, see partial_tile_at; rows beyond the last are never read
      const int mbs = (p.M + 31) >> 5;
#pragma unroll
      for (int i = 0; i < MT; i++) {
        if (mb0 + i >= mbs) break;   // uniform
#pragma unroll
        for (int j = 0; j < NT; j++) {
          float* const dst = p.out_f32 + (((size_t)by * mbs + mb0 + i) * n_tiles + nt0 + j) * 1024 + lane * 4;
#pragma unroll
          for (int q = 0; q < 4; q++) *reinterpret_cast<f32x4*>(dst + q * 256) = f32x4{acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
        }
      }
    } else {
      // 1 / rms of the row, then gelu(gate) * up of neighbouring accumulator pairs: two feature tiles
      // give 32 consecutive product columns = one scale block of the down projection's input
      const float inv_k = 1.0f / (float)p.k_true;
      const int OKC64 = p.ldo8 >> 6;
#pragma unroll
      for (int i = 0; i < MT; i++) {
        const int mbg = mb0 + i, m = mbg * 32 + lq;
        const float rs = rsqrtf(ssq[i] * inv_k + 1e-6f);
#pragma unroll
        for (int jp = 0; jp < NT; jp += 2) {
          float pr[2][8];        // products 4 q + 2 lh + {0, 1} of tile jp + j at [j][2 q + {0, 1}]
          float amax = 0.f;
#pragma unroll
          for (int j = 0; j < 2; j++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
              const f32x16& a = acc[jp + j][i];
              const float g0 = a[4 * q] * rs, u0 = a[4 * q + 1] * rs;
              const float g1 = a[4 * q + 2] * rs, u1 = a[4 * q + 3] * rs;
              pr[j][2 * q] = gelu_tanh_mx(g0) * u0;
              pr[j][2 * q + 1] = gelu_tanh_mx(g1) * u1;
              amax = fmaxf(amax, fmaxf(fabsf(pr[j][2 * q]), fabsf(pr[j][2 * q + 1])));
            }
          amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
          const int code = mx_scale_code(amax);
          const float inv = mx_inv_scale(code);
#pragma unroll
          for (int j = 0; j < 2; j++) {
            const int col0 = (nt0 + jp + j) * 16;                 // first of the tile's 16 product columns
            unsigned char* frag = p.out8 + ((size_t)mbg * OKC64 + (col0 >> 6)) * 2048 + ((size_t)((col0 & 63) >> 4) * 32 + lq) * 16;
#pragma unroll
            for (int ip = 0; ip < 2; ip++) {
              // steps 2 ip and 2 ip + 1: half 0 ends up with the four columns of step 2 ip, half 1 with those of step 2 ip + 1
              const unsigned e_even = mx_encode2(pr[j][4 * ip], pr[j][4 * ip + 1], inv);
              const unsigned e_odd = mx_encode2(pr[j][4 * ip + 2], pr[j][4 * ip + 3], inv);
              const unsigned give = lh ? e_even : e_odd;
              const unsigned got = (unsigned)__shfl_xor((int)give, 32, 64);
              const unsigned word = lh ? (got | (e_odd << 16)) : (e_even | (got << 16));
              if (m < p.M) *reinterpret_cast<unsigned*>(frag + 8 * ip + 4 * lh) = word;
            }
          }
          if (lh == 0 && m < p.M) {
            const int chunk = ((nt0 + jp) * 16) >> 6, b = (((nt0 + jp) * 16) & 63) >> 5;
            p.out_scales[(((size_t)mbg * (OKC64 >> 2) + (chunk >> 2)) * 64 + b * 32 + lq) * 4 + (chunk & 3)] = (unsigned char)code;
          }
        }
      }
    }
    if (!WALK || next >= of_die) return;
    nb = nb_next;
    m0 = m0_next;
#pragma unroll
    for (int i = 0; i < MT; i++) ssq[i] = ssq_next[i];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the counts above take no stores
  }
}

// tiles (MT, NT) as gemm_lds_tile has them: of gate||up, and, of partial sums only, of a range per die
#define MX_TILES(X) X(4, 2) X(5, 2) X(3, 4) X(4, 4)
#define MX_RANGE_TILES(X) X(2, 2) X(3, 2)

template <int MT, int NT, int EPI>
hipError_t mx_launch(hipStream_t s, MxGemmParams p, int z) {
  p.m_tiles = ceil_div(p.M, 64 * MT);
  const int total = (p.n_pad >> 5) / (2 * NT) * p.m_tiles;
  if constexpr (EPI == MX_EPI_GEGLU && MT * NT <= 12) {   // (as in gemm_tile.hip; tiles of 256 x 256 spill)
    if (total > 256 && p.m_tiles > 1) {
      gemm_mx_kernel<MT, NT, EPI, true><<<dim3(WALK_BLOCKS), dim3(256), mx_smem(MT, NT), s>>>(p, 0);
      return hipGetLastError();
    }
  }
  const bool ranges = EPI == MX_EPI_PARTIAL && z == LDS_DIES;
  gemm_mx_kernel<MT, NT, EPI, false><<<ranges ? dim3(8 * total) : dim3(8 * ceil_div(total, 8), z), dim3(256), mx_smem(MT, NT), s>>>(p, ranges);
  return hipGetLastError();
}
template <int MT, int NT, int EPI>
hipError_t mx_init(hipError_t before) {
  constexpr bool WALK = EPI == MX_EPI_GEGLU && MT * NT <= 12;
  if (before == hipSuccess && WALK) before = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mx_kernel<MT, NT, EPI, WALK>), hipFuncAttributeMaxDynamicSharedMemorySize, mx_smem(MT, NT));
  return before != hipSuccess ? before : hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_mx_kernel<MT, NT, EPI, false>), hipFuncAttributeMaxDynamicSharedMemorySize, mx_smem(MT, NT));
}

}  // namespace

// (the cost's own choice: eight ranges are no better at 768 tokens, down and reduction 40.9 us as against 41.0 with five, and worse at 816, 48.0 as against 44.6 with six)
int gemm_mx_k_per_split(int M, int n_pad, int k_pad) {
  return 2 * round_up(ceil_div(k_pad / 2, gemm_lds_splits(M, n_pad / 32, k_pad / 2, LDS_DIES, false)), 128);
}

hipError_t gemm_mx_init_attributes() {
  hipError_t e = hipSuccess;
#define X(MT, NT) e = mx_init<MT, NT, MX_EPI_PARTIAL>(e);
  MX_TILES(X) MX_RANGE_TILES(X)
#undef X
#define X(MT, NT) e = mx_init<MT, NT, MX_EPI_GEGLU>(e);
  MX_TILES(X)
#undef X
  return e;
}

hipError_t launch_gemm_mx(hipStream_t s, int epi, const MxGemmParams& p, int z_splits) {
  // everything the kernel's indexing assumes
  if (p.X8 == nullptr || p.XS == nullptr || p.W8 == nullptr || p.WS == nullptr || p.M <= 0 || z_splits < 1) return hipErrorInvalidValue;
  if (p.n_pad % 256 != 0 || p.k_pad % 256 != 0 || p.ldx % 256 != 0 || p.ldx < p.k_pad) return hipErrorInvalidValue;
  if (p.k_per_split <= 0 || p.k_per_split % 256 != 0 || (long)p.k_per_split * z_splits < p.k_pad) return hipErrorInvalidValue;
  if ((long)p.k_per_split * (z_splits - 1) >= p.k_pad) return hipErrorInvalidValue;     // no empty slice
  if ((size_t)p.k_pad * 32 > 0x7fffffffu) return hipErrorInvalidValue;                  // a row of fragments is addressed with 32 bits
  if (epi == MX_EPI_PARTIAL) {
    if (p.out_f32 == nullptr) return hipErrorInvalidValue;
  } else if (epi == MX_EPI_GEGLU) {
    if (z_splits != 1 || p.rowstat == nullptr || p.out8 == nullptr || p.out_scales == nullptr || p.k_true <= 0 || p.k_per_split != p.k_pad) return hipErrorInvalidValue;
    if (p.ldo8 % 256 != 0 || p.ldo8 < p.n_pad / 2) return hipErrorInvalidValue;
  } else {
    return hipErrorInvalidValue;
  }
  int mt = 0, nt = 0;
  gemm_lds_tile(p.M, p.n_pad / 32, p.k_pad / 2, p.k_per_split / 2, z_splits, epi == MX_EPI_PARTIAL, &mt, &nt);
#define X(MT, NT) if (epi == MX_EPI_PARTIAL && mt == MT && nt == NT) return mx_launch<MT, NT, MX_EPI_PARTIAL>(s, p, z_splits);
  MX_TILES(X) MX_RANGE_TILES(X)
#undef X
#define X(MT, NT) if (epi == MX_EPI_GEGLU && mt == MT && nt == NT) return mx_launch<MT, NT, MX_EPI_GEGLU>(s, p, z_splits);
  MX_TILES(X)
#undef X
  return hipErrorInvalidValue;
}
