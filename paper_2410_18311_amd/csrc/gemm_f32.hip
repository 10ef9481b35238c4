// Dense prefill FFN (Def. 1 of arXiv 2410.18311) for the fp32 element type, on
// the fp32 matrix instructions: same contraction, arguments and epilogues as
// the 16-bit kernels of gemm_mfma.hip.
//
// Both kernels feed the matrix cores straight from global memory.  An fp32 MFMA
// takes 32 (16x16x4) or 64 (32x32x2) cycles for 256 + 256 bytes of operands, so
// the L1 keeps up without a detour through LDS, and a wave runs its own loads
// ahead without any barrier.  The order of k inside an instruction is free as
// long as both operands agree: a lane loads four consecutive k of its row in
// one 16-byte load and hands them to four instructions one after the other.
//
//   gemm_f32_split_kernel : 16x16 outputs per workgroup, the waves split k and
//                           are added up through LDS.  For the small layers of
//                           the fp32 configuration, where a launch is a chain of
//                           load and MFMA latencies and the chip has work for a
//                           few hundred waves only: both projections of 32 tokens,
//                           d = 256, N = 1024 took 132 us with the 64x64 FMA tiles
//                           this replaces (a workgroup per tile walking all of k
//                           behind two barriers per 16 k) and take 9.5 us; 128
//                           tokens, d = 1024, N = 4096: 574 -> 67 us.
//   gemm_f32_tile_kernel  : 128x128 outputs per workgroup, 2x2 waves of 64x64,
//                           for grids that fill the chip (512 tokens, d = 4096,
//                           N = 16384: 4.62 -> 2.59 ms, 53 TFLOP/s; the loads touch
//                           32 rows each and bound it, not the matrix cores).
#include "gemm_common.hpp"

namespace ci {

namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int EPI>
__device__ __forceinline__ void store_f32(const GemmArgs& g, int row, int col, float c0, float c1) {
  const float* bias = reinterpret_cast<const float*>(g.bias);
  const float bv = bias ? bias[col] : 0.f;
  float h, score;
  if (EPI == EPI_SWIGLU) {
    h = silu(c0) * c1;
    score = fabsf(h);
  } else if (EPI == EPI_RELU) {
    h = fmaxf(c0 + bv, 0.f);
    score = h;
  } else {
    h = c0 + bv;
    score = h;
  }
  const size_t o = (size_t)row * g.ldo + col;
  if (g.out_f) g.out_f[o] = score;
  if (g.out_e) reinterpret_cast<float*>(g.out_e)[o] = h;
}

// Four consecutive k (k .. k+3) of one operand row / column; zeros past the end.  Kk is a multiple
// of 4 (rows are whole 16-byte vectors), so a quad is inside or outside as a whole.
template <bool KMAJOR>
__device__ __forceinline__ f32x4_t load_quad(const float* __restrict__ p, int64_t ld, int idx, int k, int Kk) {
  const bool in = k < Kk;
  const int kc = in ? k : 0;
  f32x4_t v;
  if (!KMAJOR) {
    v = *reinterpret_cast<const f32x4_t*>(p + (size_t)idx * ld + kc);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = p[(size_t)(kc + e) * ld + idx];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = in ? v[e] : 0.f;
  return v;
}

constexpr int kMaxSplitWaves = 16;

template <int EPI, bool BNN>
__global__ __launch_bounds__(64 * kMaxSplitWaves) void gemm_f32_split_kernel(GemmArgs g) {
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int NB = DUAL ? 2 : 1;
  constexpr int U = 4;  // groups of 16 k whose loads are in flight together
  __shared__ float red[kMaxSplitWaves][NB][256];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int tiles_m = (g.M + 15) / 16;
  const int m0 = (blockIdx.x % tiles_m) * 16, n0 = (blockIdx.x / tiles_m) * 16;
  const float* A = reinterpret_cast<const float*>(g.A);
  const float* Bp[2] = {reinterpret_cast<const float*>(g.B0), reinterpret_cast<const float*>(g.B1)};
  const int l15 = lane & 15, kq = (lane >> 4) * 4;
  const int row = min(m0 + l15, g.M - 1), col = min(n0 + l15, g.Nn - 1);
  // k range of this wave, whole groups of 16
  const int groups = (g.Kk + 15) / 16;
  const int g0 = (int)((int64_t)wave * groups / nw), g1 = (int)((int64_t)(wave + 1) * groups / nw);

  f32x4_t acc[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) acc[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int t = g0; t < g1; t += U) {
    f32x4_t a[U], b[NB][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = t + u < g1 ? (t + u) * 16 + kq : g.Kk;  // past this wave's range: zeros
      a[u] = load_quad<false>(A, g.lda, row, k, g.Kk);
#pragma unroll
      for (int q = 0; q < NB; ++q) b[q][u] = load_quad<BNN>(Bp[q], g.ldb, col, k, g.Kk);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < NB; ++q)
          acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[q][u][e], acc[q], 0, 0, 0);
  }
  // element v of lane l is C[4 (l / 16) + v][l % 16]
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave][q][((lane >> 4) * 4 + v) * 16 + l15] = acc[q][v];
  __syncthreads();
  for (int o = tid; o < 256; o += blockDim.x) {
    const int r = m0 + (o >> 4), c = n0 + (o & 15);
    if (r >= g.M || c >= g.Nn) continue;
    float c0 = 0.f, c1 = 0.f;
    for (int w = 0; w < nw; ++w) {
      c0 += red[w][0][o];
      if (DUAL) c1 += red[w][NB - 1][o];
    }
    store_f32<EPI>(g, r, c, c0, c1);
  }
}

template <int EPI, bool BNN>
__global__ __launch_bounds__(256) void gemm_f32_tile_kernel(GemmArgs g) {
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  constexpr int NB = DUAL ? 2 : 1;
  constexpr int U = 2;  // groups of 8 k per register stage
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_m = (g.M + 127) / 128;
  const int t = xcd_swizzle(blockIdx.x, gridDim.x);
  const int m0 = (t % tiles_m) * 128 + (wave >> 1) * 64, n0 = (t / tiles_m) * 128 + (wave & 1) * 64;
  const float* A = reinterpret_cast<const float*>(g.A);
  const float* Bp[2] = {reinterpret_cast<const float*>(g.B0), reinterpret_cast<const float*>(g.B1)};
  const int l31 = lane & 31, kq = (lane >> 5) * 4;
  int row[2], col[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    row[i] = min(m0 + 32 * i + l31, g.M - 1);
    col[i] = min(n0 + 32 * i + l31, g.Nn - 1);
  }
  f32x16_t acc[NB][2][2];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[q][i][j][v] = 0.f;

  f32x4_t a[2][U][2], b[2][NB][U][2];
  auto load = [&](int st, int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[st][u][i] = load_quad<false>(A, g.lda, row[i], k0 + 8 * u + kq, g.Kk);
#pragma unroll
        for (int q = 0; q < NB; ++q) b[st][q][u][i] = load_quad<BNN>(Bp[q], g.ldb, col[i], k0 + 8 * u + kq, g.Kk);
      }
  };
  auto multiply = [&](int st) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[q][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[st][u][i][e], b[st][q][u][j][e], acc[q][i][j], 0, 0, 0);
  };
  load(0, 0);
  for (int k0 = 0; k0 < g.Kk; k0 += 16 * U) {
    load(1, k0 + 8 * U);
    multiply(0);
    load(0, k0 + 16 * U);
    multiply(1);  // zeros when the reduction ends before it
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = n0 + 32 * j + l31;
    if (c >= g.Nn) continue;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = m0 + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (r < g.M) store_f32<EPI>(g, r, c, acc[0][i][j][v], acc[NB - 1][i][j][v]);
      }
  }
}

// From this many 128x128 tiles on the tile kernel is used: 128 tiles keep half of the compute units
// busy with one workgroup each, and it reads an eighth of what the 16x16 tiles read from L2 (256
// tokens, 2048 -> 8192: 128 tiles, 468 us for both projections, 1235 us with the former kernel).
constexpr int kMinTiles = 128;

template <int EPI, bool BNN>
int launch_typed(const GemmArgs& g, hipStream_t s) {
  const int64_t big = (int64_t)((g.M + 127) / 128) * ((g.Nn + 127) / 128);
  if (big >= kMinTiles) {
    hipLaunchKernelGGL((gemm_f32_tile_kernel<EPI, BNN>), dim3((unsigned)big), dim3(256), 0, s, g);
  } else {
    const int64_t tiles = (int64_t)((g.M + 15) / 16) * ((g.Nn + 15) / 16);
    // one register stage (64 k) per wave and step at least; four waves per workgroup once the grid
    // alone fills the chip
    int nw = g.Kk / 64;
    nw = nw < 1 ? 1 : (nw > kMaxSplitWaves ? kMaxSplitWaves : nw);
    if (tiles > 1024 && nw > 4) nw = 4;
    hipLaunchKernelGGL((gemm_f32_split_kernel<EPI, BNN>), dim3((unsigned)tiles), dim3(64 * nw), 0, s, g);
  }
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

}  // namespace

int launch_gemm_f32(int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  switch (epi) {
    case EPI_RELU: return launch_typed<EPI_RELU, false>(g, s);
    case EPI_SWIGLU: return launch_typed<EPI_SWIGLU, false>(g, s);
    case EPI_LINEAR: return b_kmajor ? launch_typed<EPI_LINEAR, true>(g, s) : launch_typed<EPI_LINEAR, false>(g, s);
  }
  return CI_ERR_INVALID_ARG;
}

}  // namespace ci
