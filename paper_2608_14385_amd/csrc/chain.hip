// Down projections fused with the weighted combine of Eq. 3, for batches of
// at most 32 tokens (one or two token tiles of 16).
//
// For every active unit u (department, expert, shared expert) the gate/up
// stage has stored a_{t,u} = SiLU(G_u x_t) * (U_u x_t) for the unit's tokens,
// one row per member token in ascending token order.  The layer output is
//
//   y_t = sum_u p_{t,u} W_u a_{t,u}
//
// (P_{t,j} for a department, Sec. 3.2), one product over the concatenated K
// steps of all units in which token t's column carries the weight p_{t,u}
// and zero for units it does not use.  A workgroup owns 32 rows of y (two
// 16-row halves sharing the token operand; 16 or 8 rows on narrow layers) and
// splits the concatenated K steps into KSC contiguous ranges, one per wave,
// so that every wave streams one long run of weight rows; each K step's
// product is added to the
// accumulator with the lane's token weight (times the fp8 block scale), and
// the partial tiles are summed through LDS in wave order and rounded once.
// No fp32 partial rows and no combine launch.  The FACTORED department down
// projections (W_d^T Z) are the same product over the departments, with the
// routing weights already inside Z and unit weights here.
#include "gemm_tile.h"
#include "launch.h"

namespace deamoe {

// One K step of every half: the step's products start from zero and are
// added, on the lanes whose token is a member, with the per-lane factor f (the
// token's weight, times the fp8 scale).
template <int WT, int NW, int NTT>
__device__ inline void chain_mma(const u32x4 (&a)[NW][4], const u32x4 (&b)[4], bool member, float f,
                                 f32x4 (&acc)[NW][NTT], int tt) {
#pragma unroll
  for (int n = 0; n < NW; ++n) {
    f32x4 t = {0.f, 0.f, 0.f, 0.f};
    if constexpr (WT == WT_F32) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          t = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[n][m][e]),
                                                   __uint_as_float(b[m][e]), t, 0, 0, 0);
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const bf16x8 w = WT == WT_FP8 ? fp8x8_to_bf16(a[n][m][0], a[n][m][1]) : as_bf16x8(a[n][m]);
        t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, as_bf16x8(b[m]), t, 0, 0, 0);
      }
    }
    const f32x4 nx = acc[n][tt] + f * t;
    acc[n][tt] = member ? nx : acc[n][tt];
  }
}

// NW: 16-row halves of y per workgroup (1 or 2; two share the token operand).
// Bound by the read rate on wide layers (224 workgroups at 7168: 6.7 TB/s at
// 16 tokens), on narrow ones by the token operand beside few rows (4.1 TB/s
// on the 7B-class layer at 16) and the prologue.  A CU holds one workgroup of
// pairs (142 registers, two waves per SIMD; a second needs 128), two of single
// halves with one token tile.  Scalar step addresses, the unit fields through
// scalar loads instead of LDS and one loop exit saved the pair kernel 28
// registers, at the same occupancy; kernel time by trace, us, before -> after:
// the DeepSeek-V3 shape 174.9 -> 171.9 at 16
// tokens, 214.5 -> 212.4 at 32, fp8 142.1 -> 135.3 at 32 and 20.5 -> 19.7 at
// one token, the 256-wide fp32 layer 7.4 -> 5.7 at 4.
// P: with NW == 1, a load group is P K steps of 16 / P rows instead of one
// step of 16 rows: the same 16-row segments in flight, in P times the
// workgroups.  A matrix-core tile then holds the rows P times over.
template <int WT, int NW, int P, int NTT, int KSC>
__global__ __launch_bounds__(KSC * kWave) void chain_down_kernel(ChainArgs a) {
  static_assert(P == 1 || NW == 1, "K steps side by side only in one half");
  using Tr = WTraits<WT>;
  using LD = WLoad<WT>;
  static_assert(LD::NQ % P == 0, "a K step is a whole number of load instructions");
  constexpr int SR = kTile / P;    // rows of a K step
  constexpr int TR = NW * SR;      // rows of y per workgroup
  constexpr int QS = LD::NQ / P;   // load instructions of a K step and half
  constexpr int ASEG = Tr::K_STEP * Tr::A_BYTES;
  constexpr int STAGE = NW * LD::REGION;
  constexpr int RED = NW * NTT * kWave * 16;
  constexpr int WB = STAGE > RED ? STAGE : RED;
  __shared__ __attribute__((aligned(16))) char s_buf[KSC][WB];
  const int wave = uniform(threadIdx.x / kWave), lane = lane_id();
  const int g = lane >> 4, j = lane & 15;
  const int T = a.T, R = a.h, rt = blockIdx.x;
  const int lrow = lane / LD::LPR, lchunk = lane % LD::LPR;
  // Where the wave's range starts: every lane counts the units that begin at
  // or before it.  As many entries are read as the batch can have units, not
  // as it has, so that the table's loads don't wait for the counts'.
  int step0[kMaxChainUnits / kWave];
#pragma unroll
  for (int i = 0; i < kMaxChainUnits / kWave; ++i) {
    step0[i] = 0;
    if (i * kWave < a.max_units)
      step0[i] = glob(a.units)[min(i * kWave + lane, a.max_units - 1)].step0;
  }
  const int n_units = uniform(a.counts[0]), S = uniform(a.counts[1]);
  const int s_lo = uniform((int)((int64_t)S * wave / KSC));
  const int total = uniform((int)((int64_t)S * (wave + 1) / KSC)) - s_lo;
  char *lds = s_buf[wave];
  // acc[n][tt]: rows of half n, tokens 16 * tt + (lane % 16)
  f32x4 acc[NW][NTT];
#pragma unroll
  for (int n = 0; n < NW; ++n)
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) acc[n][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (total > 0) {
    int cu = -1;   // the unit holding step s_lo: the last one that begins by then
#pragma unroll
    for (int i = 0; i < kMaxChainUnits / kWave; ++i)
      if (i * kWave < a.max_units)
        cu += __popcll(__ballot(i * kWave + lane < n_units && step0[i] <= s_lo));
    // issue cursor: K step ck of nk of unit cu.  Every address is a scalar
    // base, moved per step, plus a 32-bit lane offset, set per unit: a step's
    // loads cost one scalar addition each.  The next unit's fields are loaded
    // while this one streams.
    const auto *units = reinterpret_cast<const __attribute__((address_space(4))) ChainUnit *>(
        reinterpret_cast<uintptr_t>(a.units));
    ChainUnit nu;
    auto fetch = [&](int u) {
      const auto *p = units + min(u, n_units - 1);
      nu.w = p->w; nu.s = p->s; nu.in = p->in; nu.pw = p->pw; nu.K = p->K; nu.mask = p->mask;
      nu.step0 = p->step0;
    };
    fetch(cu);
    int ck = s_lo - nu.step0 - 1, nk = 0;
    const char *wb = nullptr, *in = nullptr;   // this tile's rows; the unit's token rows
    const float *sp = nullptr, *pw = nullptr;
    uint32_t wq = 0, wvo = 0, bvo[NTT];        // wq: bytes from one load instruction's rows to the next
    uint32_t m32 = 0;
    const uint32_t tmask = T >= 32 ? 0xffffffffu : (1u << T) - 1u;
    auto next_unit = [&]() {
      const int K = nu.K;
      nk = K / Tr::K_STEP;
      wb = static_cast<const char *>(nu.w) + (size_t)(rt * TR) * K * Tr::W_BYTES;
      wq = (uint32_t)LD::RPI * K * Tr::W_BYTES;
      wvo = (uint32_t)lrow * K * Tr::W_BYTES + lchunk * 16;
      m32 = nu.mask & tmask;
      in = static_cast<const char *>(nu.in);
      pw = nu.pw;
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) {
        // a member's row is its rank among the members; other lanes read the
        // first member's row, so each load touches only the unit's rows
        const int tok = kTile * tt + j;
        const int rank = (m32 >> tok) & 1 ? __popc(m32 & ((1u << tok) - 1u)) : 0;
        bvo[tt] = (uint32_t)rank * K * Tr::A_BYTES + b_chunk_offset(g, 0);
      }
      if constexpr (WT == WT_FP8)   // the tile's rows lie in one scale row
        sp = nu.s + (size_t)((rt * TR) / 128) * (K / 128);
      fetch(++cu);
    };
    next_unit();
    u32x4 G[2][NW][LD::NQ];   // one load group in flight, one multiplied
    u32x4 B[2][P][NTT][4];
    uint32_t MM[2][P];        // the step's member tokens, none past the wave's range
    float SC[2][P], PW[2][P][NTT];
    // the loads of the wave's steps v .. v + P - 1 (past the range a cached
    // token row in the weights' place, and no members)
    auto issue = [&](int q, int v) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        if (v + p < total) {
          if (++ck == nk) {
            ck = 0;
            next_unit();
          }
          MM[q][p] = m32;
        } else {
          MM[q][p] = 0;
        }
        const bool ok = v + p < total;
        const char *base = ok ? wb + (size_t)ck * LD::WSEG : in;
        const uint32_t rows = ok ? wq : 0u;
        lane_offset(wvo);
        const uint32_t vo = ok ? wvo : (lane & 15) * 16;
#pragma unroll
        for (int i = 0; i < QS; ++i) {
          G[q][0][p * QS + i] =
              __builtin_nontemporal_load(gptr(scalar_base(base + (size_t)i * rows) + vo));
          if constexpr (NW == 2)
            G[q][1][i] =
                __builtin_nontemporal_load(gptr(scalar_base(base + (size_t)(QS + i) * rows) + vo));
        }
        const char *bb = scalar_base(in + (size_t)ck * ASEG);
#pragma unroll
        for (int tt = 0; tt < NTT; ++tt) lane_offset(bvo[tt]);
        // two steps of one unit load the same token weights: kept two loads,
        // as one would be copied, and so waited for, where they are issued
        const float *pws = pw;
        asm("" : "+s"(pws));
#pragma unroll
        for (int tt = 0; tt < NTT; ++tt) {
#pragma unroll
          for (int i = 0; i < 4; ++i) B[q][p][tt][i] = *gptr(bb + bvo[tt] + b_chunk_offset(0, i));
          PW[q][p][tt] = *gfptr(pws + (uint32_t)(kTile * tt + j));
        }
        if constexpr (WT == WT_FP8) SC[q][p] = *gfptr(sp + ck);
      }
    };
    auto multiply = [&](int q) {
      __builtin_amdgcn_sched_barrier(0);
      u32x4 w[P][NW][4];
      stage_weights<WT, NW, P>(lds, G[q], w);
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int tt = 0; tt < NTT; ++tt) {
          // other tokens' lanes hold a member's row, or no weights at all
          // past the range: whatever their product is, it is dropped
          const bool member = (MM[q][p] >> (kTile * tt + j)) & 1;
          const float f = WT == WT_FP8 ? PW[q][p][tt] * SC[q][p] : PW[q][p][tt];
          chain_mma<WT, NW>(w[p], B[q][p][tt], member, f, acc, tt);
        }
      __builtin_amdgcn_sched_barrier(0);
    };
    // one exit, in the middle: with more, the compiler peels a first round
    // and waits for its loads to copy their registers
    issue(0, 0);
    for (int v = 0;; v += 2 * P) {
      issue(1, v + P);
      multiply(0);
      if (v + 2 * P >= total) break;
      issue(0, v + 2 * P);
      multiply(1);
    }
    multiply(1);
  }
  // partial tiles summed in wave order; wave 0 rounds and stores
  __syncthreads();   // every wave is done with its staging region
  f32x4 *red = reinterpret_cast<f32x4 *>(s_buf[wave]);
  if (wave > 0) {
#pragma unroll
    for (int n = 0; n < NW; ++n)
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) red[(n * NTT + tt) * kWave + lane] = acc[n][tt];
  }
  __syncthreads();
  if (wave == 0) {
    for (int q = 1; q < KSC; ++q) {
      const f32x4 *r = reinterpret_cast<const f32x4 *>(s_buf[q]);
#pragma unroll
      for (int n = 0; n < NW; ++n)
#pragma unroll
        for (int tt = 0; tt < NTT; ++tt) acc[n][tt] += r[(n * NTT + tt) * kWave + lane];
    }
    if (4 * g >= SR) return;   // the rows' copies
    const int row0 = rt * TR + 4 * g, row1 = row0 + kTile;
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) {
      const int tok = kTile * tt + j;
      if (tok < T) {
        const size_t off = (size_t)tok * R + row0;
        if (row0 < R) store4(a.y, a.act_f32, off, acc[0][tt], row0 + 3 < R, R - row0);
        if (NW == 2 && row1 < R)
          store4(a.y, a.act_f32, off + kTile, acc[NW - 1][tt], row1 + 3 < R, R - row1);
      }
    }
  }
}

// 8 waves per workgroup, each streaming one contiguous range of the
// concatenated K steps, one load group in flight while one is multiplied.
constexpr int kChainWaves = 8;

template <int WT, int NW, int P, int NTT>
static hipError_t launch_chain_wt(const ChainArgs &a, hipStream_t s) {
  constexpr int TR = NW * kTile / P, KSC = kChainWaves;
  hipLaunchKernelGGL((chain_down_kernel<WT, NW, P, NTT, KSC>), dim3((a.h + TR - 1) / TR),
                     dim3(KSC * kWave), 0, s, a);
  return hipGetLastError();
}

// Layers narrower than 5120 take one 16-row half per workgroup: twice the
// workgroups (two per CU, four waves per SIMD with one token tile) where row
// pairs leave most CUs idle.  Same-process A/B on the 2048-wide 7B-class
// layer: 36.7 -> 33.9 us per step at one token, 54.4 -> 49.3 at four; on
// the 4096-wide Qwen3 FACTORED layer 79.2 -> 76.9 at one token, 312.3 ->
// 305.1 at 16.  At 5120 (DeepSeek-V2 FACTORED: 86.6 -> 88.1 at one token,
// 389.0 -> 393.5 at 16) and at the 7168-wide DeepSeek-V3 shape (108.3 ->
// 110.4 us at one token, 525.4 -> 546.7 at 16) single halves were slower.
constexpr int kChainPairMinH = 5120;
// Up to 2048, where 16-row blocks leave half the CUs idle, a workgroup takes
// 8 rows, two K steps side by side in a load group (at most 256 workgroups of
// one a CU); 12 or 16 waves on 128 CUs instead were no faster.  The price is
// the token operand, 4 KB per token tile and K step beside 2 KB of weights.
// Kernel time by trace, us, 16 rows -> 8: the 7B-class layer 10.0 -> 8.4 at one
// token, 16.4 -> 13.7
// at 5, 22.2 -> 18.6 at 16, 29.5 -> 26.9 at 24; Baseline-7B (1024 wide) 6.3
// -> 5.5 at 16.  At 4096 (Qwen3, 512 workgroups in two rounds) 8 rows lost:
// 18.9 -> 25.2 at 16, and 4 rows lost at 2048 too.
// A step of fewer than kChainSplitSteps K steps keeps 16 rows: a wave then has
// three steps at most, a 16-row wave requests two of them at once, and the
// pairs only double the matrix products and the prologue's work.  Step times,
// us, 8 rows -> 16: Baseline-7B FACTORED at one token (at most 12 steps) 33.7
// -> 33.3; 1024-wide layers of 8 steps at one token 14.9 -> 14.4 (bf16) and
// 14.7 -> 14.3 (fp8), of 16 (fp32) 17.8 -> 16.3; 8 steps, 2048 wide, 30.6 ->
// 27.9 at 20 tokens.  From 24 steps on 8 rows gain: the Baseline-7B vanilla
// layer at one token (24) 18.3 -> 17.7, the 7B-class layer (at most 82) 33.6
// -> 32.4.
constexpr int kChainSplitMaxH = 2048, kChainSplitSteps = 3 * kChainWaves;

template <int WT>
static hipError_t launch_chain_ntt(const ChainArgs &a, hipStream_t s) {
  const bool one = a.T <= kTile;
  if (a.h <= kChainSplitMaxH && a.max_steps >= kChainSplitSteps)
    return one ? launch_chain_wt<WT, 1, 2, 1>(a, s) : launch_chain_wt<WT, 1, 2, 2>(a, s);
  if (a.h < kChainPairMinH)
    return one ? launch_chain_wt<WT, 1, 1, 1>(a, s) : launch_chain_wt<WT, 1, 1, 2>(a, s);
  return one ? launch_chain_wt<WT, 2, 1, 1>(a, s) : launch_chain_wt<WT, 2, 1, 2>(a, s);
}

hipError_t launch_chain(const ChainArgs &a, int wtype, hipStream_t s) {
  switch (wtype) {
    case WT_F32: return launch_chain_ntt<WT_F32>(a, s);
    case WT_BF16: return launch_chain_ntt<WT_BF16>(a, s);
    default: return launch_chain_ntt<WT_FP8>(a, s);
  }
}

}  // namespace deamoe
