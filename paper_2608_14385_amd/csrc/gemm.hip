// Grouped skinny GEMM over a device-built list of units (one launch per
// stage).  The number of units and row tiles is only known on the device, so
// the grid is fixed on the host and every workgroup walks tiles
// blockIdx.x * TPB, + gridDim.x * TPB, ...; tiles past the end do nothing.
#include "gemm_tile.h"
#include "launch.h"

namespace deamoe {

// The unit a work item belongs to: the last one whose first item is <= item.
// Every lane of the wave compares one entry of the prefix per 64 units.  A
// work item starts with a chain of dependent reads (counts, prefix, unit,
// weights), so finding its unit is one round trip after the counts, which say
// whether the workgroup has an item at all: no copy to LDS, no barrier, no
// search over dependent LDS reads.
__device__ inline int find_unit(const GemmStage &st, int n_units, int item) {
  constexpr int U = 8;
  const gmem<const int32_t> *begin = glob(st.begin);
  const int lane = lane_id();
  int u = -1;
  for (int u0 = 0; u0 < st.max_units; u0 += U * kWave) {
    int b[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      b[i] = 0;
      if (u0 + i * kWave < st.max_units)
        b[i] = begin[min(u0 + i * kWave + lane, st.max_units - 1)];
    }
#pragma unroll
    for (int i = 0; i < U; ++i)
      if (u0 + i * kWave < st.max_units)
        u += __popcll(__ballot(u0 + i * kWave + lane < n_units && b[i] <= item));
  }
  return u;
}

template <int WT, int NW, int NTT, int KS, bool SPLIT, bool PAIR, bool B1>
__device__ __attribute__((always_inline)) void grouped_gemm_body(const GemmStage &st) {
  using Run = TileRunner<WT, NW, NTT, KS, SPLIT, PAIR, B1>;
  __shared__ typename Run::Smem sm;
  const int wave = uniform(threadIdx.x / kWave);
  // the grid is sized for the most work a step can have; the prefix is read as
  // far as the batch can have units, entries past the step's units not counted
  const int n_units = uniform(st.counts[0]), n_tiles = uniform(st.counts[1]);
  for (int base = blockIdx.x * Run::TPB; base < n_tiles; base += gridDim.x * Run::TPB) {
    const int tile = base + wave / KS;
    const bool active = tile < n_tiles;
    const int u = uniform(max(0, find_unit(st, n_units, min(tile, n_tiles - 1))));
    const GemmUnit U = load_unit(st.units + u);
    Run::run(sm, &U, active ? tile - uniform(st.begin[u]) : 0, active, st.sigma);
  }
}

template <int WT, int NW, int NTT, int KS, bool SPLIT, bool PAIR>
__global__ __launch_bounds__(256) void grouped_gemm_kernel(GemmStage st) {
  grouped_gemm_body<WT, NW, NTT, KS, SPLIT, PAIR, false>(st);
}

// The same at three waves per SIMD (at most 168 registers), for the
// instantiations that fit them without spilling:
//  - the split-operand stage with one token tile (the FACTORED private
//    gate/up), its two token operands requested per step (B1).  With both
//    operands double-buffered the stage's earlier per-lane addresses took 166
//    registers at two waves per SIMD, or 168 and a 24-byte spill at three;
//    with scalar bases three waves hold them, even or within 1 % either way
//    (Baseline-7B 66.4 -> 67.4 us at 16 tokens, DeepSeek-V2 375.8 -> 373.5).
//    Same-process A/B of B1 against the spilling form (outputs bit-identical): 745.6 -> 704.4 us per step
//    at 16 tokens on the DeepSeek-V3 FACTORED layer (the stage 405.0 ->
//    364.3), 2071.8 -> 1977.4 at 64, 148.4 -> 145.3 at one token; Kimi-K2
//    879.6 -> 839.6, DeepSeek-V2 406.2 -> 391.6, Qwen3 330.8 -> 319.5 at 16;
//  - fp8 stages with two token tiles: with the token operand requested per
//    step (B1) and loaded as whole row segments for row pairs and for gate/up
//    pairs with a K split over 2 waves (above 32 tokens; same-process A/B at
//    the DeepSeek-V3 shape, us per step: 477.6 -> 458.4 at 64 tokens, 631.0
//    -> 569.1 at 128), double-buffered at 17-32 tokens (348.5 -> 351.4 at 24
//    with B1);
//  - bf16 and fp32 stages with two token tiles whose token operand is
//    requested per step (B1): row pairs (same-process A/B at the DeepSeek-V3
//    shape, down stage at 128 tokens 378.3 -> 370.0 us, skewed 178.9 ->
//    172.8), the FACTORED department gate/up (dept_ntt_of), and gate/up
//    pairs of SLICE layers narrower than 4096 (the 7B-class
//    layer 48.5 -> 44.9 us at 32 tokens, 52.3 -> 48.5 at 64; at the
//    DeepSeek-V3 shape they were 0-2 % slower, so two waves stay there).
template <int WT, int NW, int NTT, int KS, bool SPLIT, bool PAIR, bool B1>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
void grouped_gemm_occ3_kernel(GemmStage st) {
  grouped_gemm_body<WT, NW, NTT, KS, SPLIT, PAIR, B1>(st);
}

// Four token tiles per wave (64 tokens), for the gate/up stage of wide
// layers above 64 tokens (fp8: above 96), the row pairs of the bf16 and fp32
// down stages there, and the FACTORED department gate/up (dept_ntt_of: from 49
// tokens on layers at least 5120 wide): a unit with many tokens streams its
// rows once per 64 tokens instead of once per 32.  The token operand is
// requested per step (B1); two waves per SIMD.
template <int WT, int NW, int NTT, int KS, bool PAIR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void grouped_gemm_wide_kernel(GemmStage st) {
  grouped_gemm_body<WT, NW, NTT, KS, false, PAIR, true>(st);
}

// Launch of the stage's kernel, for the forms the host's rules pick (any other
// combination is an error).  three: two-token-tile gate/up pairs run at three
// waves per SIMD.
template <int WT, int NTT, int KS>
static hipError_t launch_gemm(const GemmStage &st, int mode, int max_tiles, int grid_cap,
                              bool three, hipStream_t s) {
  constexpr int TPB = 4 / KS;
  int grid = (max_tiles + TPB - 1) / TPB;
  grid = grid < 1 ? 1 : (grid > grid_cap ? grid_cap : grid);
  auto run = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, s, st);
    return hipGetLastError();
  };
  if (mode == GEMM_SPLIT) {
    if constexpr (NTT == 1 && KS <= 2)
      return run(grouped_gemm_occ3_kernel<WT, 2, NTT, KS, true, false, true>);
  } else if (mode == GEMM_PAIR) {
    if constexpr (NTT == 1)
      return run(grouped_gemm_kernel<WT, 2, NTT, KS, false, true>);
    else if constexpr (NTT == 2 && KS <= 2)
      return run(grouped_gemm_occ3_kernel<WT, 2, NTT, KS, false, true, true>);
    else if constexpr (NTT == 4 && KS == 1 && WT != WT_FP8)
      return run(grouped_gemm_wide_kernel<WT, 2, NTT, KS, true>);
  } else {
    if constexpr (NTT == 1 && KS == 4) {
      return run(grouped_gemm_kernel<WT, 2, NTT, KS, false, false>);
    } else if constexpr (NTT == 2 && KS >= 2) {
      if constexpr (WT == WT_FP8)
        return run(grouped_gemm_occ3_kernel<WT, 2, NTT, KS, false, false, KS == 2>);
      else if (three)
        return run(grouped_gemm_occ3_kernel<WT, 2, NTT, KS, false, false, true>);
      else
        return run(grouped_gemm_kernel<WT, 2, NTT, KS, false, false>);
    } else if constexpr (NTT == 4 && KS == 2) {
      return run(grouped_gemm_wide_kernel<WT, 2, NTT, KS, false>);
    }
  }
  return hipErrorInvalidValue;
}

// Token tiles per wave (larger token sets are split into groups) and K split.
template <int WT, int KS>
static hipError_t dispatch_ntt(const GemmStage &st, int mode, int ntt, int max_tiles, int cap,
                               bool three, hipStream_t s) {
  switch (ntt) {
    case 1: return launch_gemm<WT, 1, KS>(st, mode, max_tiles, cap, three, s);
    case 2: return launch_gemm<WT, 2, KS>(st, mode, max_tiles, cap, three, s);
    case 4: return launch_gemm<WT, 4, KS>(st, mode, max_tiles, cap, three, s);
    default: return hipErrorInvalidValue;
  }
}

template <int WT>
static hipError_t dispatch_ks(const GemmStage &st, int mode, int ntt, int ks, int max_tiles,
                              int cap, bool three, hipStream_t s) {
  switch (ks) {
    case 1: return dispatch_ntt<WT, 1>(st, mode, ntt, max_tiles, cap, three, s);
    case 2: return dispatch_ntt<WT, 2>(st, mode, ntt, max_tiles, cap, three, s);
    default: return dispatch_ntt<WT, 4>(st, mode, ntt, max_tiles, cap, three, s);
  }
}

hipError_t launch_grouped_gemm(const GemmStage &st, int wtype, int nw, int mode, int ntt,
                               int ks, int max_tiles, int grid_cap, hipStream_t s, bool three) {
  if (nw != 2) return hipErrorInvalidValue;   // every stage streams two matrices or a row pair
  switch (wtype) {
    case WT_F32: return dispatch_ks<WT_F32>(st, mode, ntt, ks, max_tiles, grid_cap, three, s);
    case WT_BF16: return dispatch_ks<WT_BF16>(st, mode, ntt, ks, max_tiles, grid_cap, three, s);
    default: return dispatch_ks<WT_FP8>(st, mode, ntt, ks, max_tiles, grid_cap, three, s);
  }
}

}  // namespace deamoe
