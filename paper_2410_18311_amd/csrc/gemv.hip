// Dense FFN for a handful of tokens (M <= 4): the dense decode baseline that
// the sparse path of arXiv 2410.18311 (Sec. 4.2) is compared against, and the
// activation vector A(x) of Def. 1 for single tokens.  Bandwidth bound: every
// weight is read once, whatever M, and meets all tokens in registers.
//   up_rows_kernel   : H[m, n] = act(<w_up[n, :], X[m, :]> [+ b_up[n]]), fp32
//   down_rows_kernel : Y[m, j] = <w_down[j, :], H[m, :]> [+ b_down[j]], w_down [d, N]
//   down_cols_kernel : the same from w_down [N, d]: partial sums by slices of the neurons,
//                      which decode_reduce_kernel adds up
// Measured, scores and output, before (a pass over the weights per token) and now: 4096 x 16384 fp16, 2 tokens 81 ->
// 55 us, 4 tokens 155 -> 73; neuron-major 94 -> 48 and 173 -> 54 (the read alone 43); 5120 x 13824 gated bf16, 4 tokens
// 249 -> 93 (67).
// Weights that a cache holds many times over are read once per token instead, by workgroups of its own (grid.y): with
// so few rows a call is a chain of latencies, and several tokens' reductions in one workgroup make it longer (see
// kPerTokenBytes).
// The row kernels: a workgroup owns a contiguous slice of groups of output rows; its threads
// split the reduction dimension with 16-byte loads, reduce by wave shuffles and then
// across waves through LDS (two buffers: one barrier per group).
#include "common.hpp"
#include "decode_common.hpp"

namespace ci {

namespace {

constexpr int RC = 4;  // weight rows in flight per thread; down_rows_kernel with several tokens: 8, as it
                       // reads the tokens' fp32 hidden values once per group of rows

// EACH: the MT tokens of blockIdx.y (an instantiation of its own: the offsets cost the others 0.3 of 4.3 us)
template <class D, bool SWIGLU, int MT, bool EACH>
__global__ __launch_bounds__(256) void up_rows_kernel(const void* __restrict__ X,
                                                      const void* __restrict__ w_up,
                                                      const void* __restrict__ w_gate,
                                                      const void* __restrict__ b_up, float* H,
                                                      float* A, int d, int N) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  constexpr int NM = SWIGLU ? 2 : 1;
  __shared__ float red[2][NM][4][MT * RC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_grp = (N + RC - 1) / RC;
  const int g0 = (int)(((int64_t)blockIdx.x * n_grp) / gridDim.x);
  const int g1 = (int)(((int64_t)(blockIdx.x + 1) * n_grp) / gridDim.x);
  const T* x = reinterpret_cast<const T*>(X);
  if constexpr (EACH) {
    x += (size_t)blockIdx.y * MT * d;
    if (H) H += (size_t)blockIdx.y * MT * N;
    if (A) A += (size_t)blockIdx.y * MT * N;
  }
  const T* wu = reinterpret_cast<const T*>(w_up);
  const T* wg = reinterpret_cast<const T*>(w_gate);

  for (int g = g0; g < g1; ++g) {
    const int rb = g * RC;
    float s[NM][MT][RC];
#pragma unroll
    for (int q = 0; q < NM; ++q)
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < RC; ++j) s[q][m][j] = 0.f;
    for (int c = tid * VEC; c < d; c += 256 * VEC) {
      uint4 xv[MT], v[NM][RC];
#pragma unroll
      for (int m = 0; m < MT; ++m) xv[m] = ld16(x + (size_t)m * d + c);
#pragma unroll
      for (int j = 0; j < RC; ++j) {
        const int r = min(rb + j, N - 1);
        v[0][j] = ld16(wu + (size_t)r * d + c);
        if (SWIGLU) v[NM - 1][j] = ld16(wg + (size_t)r * d + c);
      }
      float xf[MT][VEC];
#pragma unroll
      for (int m = 0; m < MT; ++m) unpack<D>(xv[m], xf[m]);
#pragma unroll
      for (int j = 0; j < RC; ++j)
#pragma unroll
        for (int q = 0; q < NM; ++q) {
          float f[VEC];
          unpack<D>(v[q][j], f);
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int e = 0; e < VEC; ++e) s[q][m][j] = fmaf(f[e], xf[m][e], s[q][m][j]);
        }
    }
    const int buf = g & 1;
#pragma unroll
    for (int q = 0; q < NM; ++q)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        halve_rows<RC, 32>(s[q][m], lane);  // lanes 16 j .. 16 j + 15: the sum of row j
        if ((lane & 15) == 0) red[buf][q][wave][m * RC + (lane >> 4)] = s[q][m][0];
      }
    __syncthreads();  // the other buffer was read before it: no second barrier
    if (tid < MT * RC && rb + tid % RC < N) {
      const int m = tid / RC, r = rb + tid % RC;
      float zu = red[buf][0][0][tid] + red[buf][0][1][tid] + red[buf][0][2][tid] + red[buf][0][3][tid];
      float h;
      if (SWIGLU) {
        constexpr int G = NM - 1;
        const float zg = red[buf][G][0][tid] + red[buf][G][1][tid] + red[buf][G][2][tid] + red[buf][G][3][tid];
        h = silu(zg) * zu;
      } else {
        if (b_up) zu += to_float<D>(reinterpret_cast<const T*>(b_up)[r]);
        h = fmaxf(zu, 0.f);
      }
      if (H) H[(size_t)m * N + r] = h;
      if (A) A[(size_t)m * N + r] = fabsf(h);
    }
  }
}

template <class D, int MT, int RD, bool EACH>
__global__ __launch_bounds__(256) void down_rows_kernel(const float* __restrict__ H,
                                                        const void* __restrict__ w_down,
                                                        const void* __restrict__ b_down, void* Y,
                                                        int d, int N) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  __shared__ float red[2][4][MT * RD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_grp = (d + RD - 1) / RD;
  const int g0 = (int)(((int64_t)blockIdx.x * n_grp) / gridDim.x);
  const int g1 = (int)(((int64_t)(blockIdx.x + 1) * n_grp) / gridDim.x);
  const T* w = reinterpret_cast<const T*>(w_down);
  T* y_out = reinterpret_cast<T*>(Y);
  if constexpr (EACH) {
    H += (size_t)blockIdx.y * MT * N;
    y_out += (size_t)blockIdx.y * MT * d;
  }

  for (int g = g0; g < g1; ++g) {
    const int rb = g * RD;
    float s[MT][RD];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int j = 0; j < RD; ++j) s[m][j] = 0.f;
    for (int c = tid * VEC; c < N; c += 256 * VEC) {
      uint4 vw[RD];
#pragma unroll
      for (int j = 0; j < RD; ++j) vw[j] = ld16(w + (size_t)min(rb + j, d - 1) * N + c);
      float hf[MT][VEC];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int e = 0; e < VEC; e += 4) {
          const float4 t = *reinterpret_cast<const float4*>(H + (size_t)m * N + c + e);
          hf[m][e] = t.x; hf[m][e + 1] = t.y; hf[m][e + 2] = t.z; hf[m][e + 3] = t.w;
        }
#pragma unroll
      for (int j = 0; j < RD; ++j) {
        float f[VEC];
        unpack<D>(vw[j], f);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int e = 0; e < VEC; ++e) s[m][j] = fmaf(f[e], hf[m][e], s[m][j]);
      }
    }
    const int buf = g & 1;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      halve_rows<RD, 32>(s[m], lane);
      constexpr int W = 64 / RD;  // lanes that hold the same row
      if (lane % W == 0) red[buf][wave][m * RD + lane / W] = s[m][0];
    }
    __syncthreads();
    if (tid < MT * RD && rb + tid % RD < d) {
      const int m = tid / RD, r = rb + tid % RD;
      float y = red[buf][0][tid] + red[buf][1][tid] + red[buf][2][tid] + red[buf][3][tid];
      if (b_down) y += to_float<D>(reinterpret_cast<const T*>(b_down)[r]);
      y_out[(size_t)m * d + r] = from_float<D>(y);
    }
  }
}

// Neuron-major down matrix [N, d].  A workgroup owns 64 16-byte columns and a slice of the neurons; its waves split
// the slice, stream the rows (two batches of RB in flight), take a row's hidden values from the lane that loaded
// them, and add their sums up through LDS at the end, so that the partial sums stay few.
constexpr int kColWaves = 8;
template <class D, int MT>
__global__ __launch_bounds__(64 * kColWaves) void down_cols_kernel(const float* __restrict__ H,
                                                                   const void* __restrict__ w_down,
                                                                   float* __restrict__ partial, int d, int N) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  constexpr int RB = 16;
  __shared__ float red[kColWaves][64 * VEC];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = (blockIdx.x * 64 + lane) * VEC;
  const int pieces = gridDim.y * kColWaves;
  const int piece = blockIdx.y * kColWaves + wave;
  const int k0 = (int)((int64_t)piece * N / pieces), k1 = (int)((int64_t)(piece + 1) * N / pieces);
  const T* w = reinterpret_cast<const T*>(w_down) + min(col, d - VEC);  // d is a multiple of VEC
  float acc[MT][VEC];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[m][e] = 0.f;

  // Loads are issued on every path (rows past the end: the last one again), so that the waits are exact.
  uint4 v[2][RB];
  float hl[MT], hn[MT];
  auto request = [&](uint4* q, int k) {
#pragma unroll
    for (int j = 0; j < RB; ++j) q[j] = ld16_stream(w + (size_t)min(k + j, k1 - 1) * d);
  };
  auto consume = [&](const uint4* q, int k, int first) {
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      if (k + j < k1) {  // uniform; a row that is not there must not be multiplied by zero (it may hold an infinity)
        float f[VEC];
        unpack<D>(q[j], f);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const float h = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(hl[m]), first + j));
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[m][e] = fmaf(f[e], h, acc[m][e]);
        }
      }
    }
  };
  if (k0 < k1) {
#pragma unroll
    for (int m = 0; m < MT; ++m) hl[m] = H[(size_t)m * N + min(k0 + lane, k1 - 1)];
    request(v[0], k0);
    for (int k = k0; k < k1; k += 2 * RB) {
      request(v[1], k + RB);
#pragma unroll
      for (int m = 0; m < MT; ++m) hn[m] = H[(size_t)m * N + min(k + 2 * RB + lane, k1 - 1)];
      consume(v[0], k, 0);
      request(v[0], k + 2 * RB);
      consume(v[1], k + RB, RB);
#pragma unroll
      for (int m = 0; m < MT; ++m) hl[m] = hn[m];
    }
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (m) __syncthreads();
#pragma unroll
    for (int e = 0; e < VEC; ++e) red[wave][e * 64 + lane] = acc[m][e];
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * VEC; i += 64 * kColWaves) {
      float t = red[0][(i % VEC) * 64 + i / VEC];
#pragma unroll
      for (int q = 1; q < kColWaves; ++q) t += red[q][(i % VEC) * 64 + i / VEC];
      const int c = blockIdx.x * 64 * VEC + i;
      if (c < d) partial[((size_t)m * gridDim.y + blockIdx.y) * d + c] = t;
    }
  }
}

int chip_cus() {
  DeviceInfo di;
  return device_info(&di) == CI_OK ? di.cus : 256;
}

// Workgroups for `rows` output rows in groups of `rc`: at most gemv_wgs_per_cu per compute unit, with the same
// number of groups each (rounded up; one token, 5120 x 13824 gated: 85 us with uneven slices, 75 us).
int row_grid(int64_t rows, int rc) {
  const int64_t groups = (rows + rc - 1) / rc;
  const int64_t most = (int64_t)chip_cus() * params().gemv_wgs_per_cu;
  const int64_t rounds = (groups + most - 1) / most;
  return (int)((groups + rounds - 1) / rounds);
}

template <class D, int MT, bool EACH = false>
int up_tokens(const void* X, const void* w_up, const void* w_gate, const void* b_up, int act, int d, int N, float* H,
              float* A, hipStream_t s, int groups = 1) {
  dim3 grid(row_grid(N, RC), groups), block(256);
  if (act == CI_ACT_SWIGLU)
    hipLaunchKernelGGL((up_rows_kernel<D, true, MT, EACH>), grid, block, 0, s, X, w_up, w_gate, b_up, H, A, d, N);
  else
    hipLaunchKernelGGL((up_rows_kernel<D, false, MT, EACH>), grid, block, 0, s, X, w_up, w_gate, b_up, H, A, d, N);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

// Weights of one launch up to which every token has workgroups of its own.  Tokens together / one by one (us): 4 tokens,
// both projections of 128 x 512 gated fp32 (0.5 + 0.3 MB) 8.6 / 6.7, of 256 x 1024 fp32 (1 MB each) 7.5 / 6.7; the up
// projection of 512 x 2048 fp16 (2.1 MB) 4.2 / 4.5, of 384 x 1536 fp32 (2.4 MB) 4.2 / 4.4, of 256 x 1024 gated fp32
// (2.1 MB in two matrices) 5.4 / 5.1.
constexpr double kPerTokenBytes = 1.6e6, kPerTokenGatedBytes = 2.2e6;

template <class D>
int up_typed(const void* X, int M, const void* w_up, const void* w_gate, const void* b_up, int act,
             int d, int N, float* H, float* A, hipStream_t s) {
  if (M > 1 && (double)d * N * D::BYTES * (act == CI_ACT_SWIGLU ? 2 : 1) <= (act == CI_ACT_SWIGLU ? kPerTokenGatedBytes : kPerTokenBytes))
    return up_tokens<D, 1, true>(X, w_up, w_gate, b_up, act, d, N, H, A, s, M);
  switch (M) {
    case 1: return up_tokens<D, 1>(X, w_up, w_gate, b_up, act, d, N, H, A, s);
    case 2: return up_tokens<D, 2>(X, w_up, w_gate, b_up, act, d, N, H, A, s);
    case 3: return up_tokens<D, 3>(X, w_up, w_gate, b_up, act, d, N, H, A, s);
    case 4: return up_tokens<D, 4>(X, w_up, w_gate, b_up, act, d, N, H, A, s);
  }
  return CI_ERR_UNSUPPORTED;
}

template <class D, int MT, int RD, bool EACH = false>
int down_tokens(const float* H, const void* w_down, const void* b_down, int d, int N, void* Y, hipStream_t s,
                int groups = 1) {
  hipLaunchKernelGGL((down_rows_kernel<D, MT, RD, EACH>), dim3(row_grid(d, RD), groups), dim3(256), 0, s, H, w_down, b_down, Y, d, N);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

// Several tokens: groups of 8 rows halve the reads of the fp32 hidden values, which bound this kernel from three
// tokens on (4 tokens, 4096 x 16384 fp16: 49 us for down against 23 for up; groups of 16 60), where that leaves a
// group per compute unit (4 tokens, 1024 x 4096: 13.3 us with 8, 10.8 with 4).
template <class D, int MT>
int down_group(const float* H, const void* w_down, const void* b_down, int d, int N, void* Y, hipStream_t s) {
  if (MT > 1 && d >= 2 * RC * chip_cus()) return down_tokens<D, MT, 2 * RC>(H, w_down, b_down, d, N, Y, s);
  return down_tokens<D, MT, RC>(H, w_down, b_down, d, N, Y, s);
}

template <class D>
int down_typed(const float* H, int M, const void* w_down, const void* b_down, int d, int N, void* Y,
               hipStream_t s) {
  if (M > 1 && (double)d * N * D::BYTES <= kPerTokenBytes) return down_tokens<D, 1, RC, true>(H, w_down, b_down, d, N, Y, s, M);
  switch (M) {
    case 1: return down_group<D, 1>(H, w_down, b_down, d, N, Y, s);
    case 2: return down_group<D, 2>(H, w_down, b_down, d, N, Y, s);
    case 3: return down_group<D, 3>(H, w_down, b_down, d, N, Y, s);
    case 4: return down_group<D, 4>(H, w_down, b_down, d, N, Y, s);
  }
  return CI_ERR_UNSUPPORTED;
}

template <class D>
int down_cols_typed(const float* H, int M, const void* w_down, int d, int N, float* partial, int slices,
                    hipStream_t s) {
  const dim3 grid((d / D::VEC + 63) / 64, slices), block(64 * kColWaves);
  switch (M) {
    case 1: hipLaunchKernelGGL((down_cols_kernel<D, 1>), grid, block, 0, s, H, w_down, partial, d, N); break;
    case 2: hipLaunchKernelGGL((down_cols_kernel<D, 2>), grid, block, 0, s, H, w_down, partial, d, N); break;
    case 3: hipLaunchKernelGGL((down_cols_kernel<D, 3>), grid, block, 0, s, H, w_down, partial, d, N); break;
    case 4: hipLaunchKernelGGL((down_cols_kernel<D, 4>), grid, block, 0, s, H, w_down, partial, d, N); break;
    default: return CI_ERR_UNSUPPORTED;
  }
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

}  // namespace

// partial: fp32 [M, slices, d], slices <= min(N, 1024)
int launch_down_cols(const float* H, int64_t M, const void* w_down, const void* b_down, int dtype,
                     int64_t d, int64_t N, void* Y, float* partial, hipStream_t s) {
  const int64_t chunks = (d * (dtype == CI_F32 ? 4 : 2) / 16 + 63) / 64;
  int64_t slices = (int64_t)chip_cus() * params().gemv_cols_wgs_per_cu / chunks;
  if (slices > (N + kColWaves - 1) / kColWaves) slices = (N + kColWaves - 1) / kColWaves;
  if (slices > 1024) slices = 1024;
  if (slices < 1) slices = 1;
  int rc = CI_ERR_BAD_DTYPE;
  switch (dtype) {
    case CI_F32: rc = down_cols_typed<F32>(H, (int)M, w_down, (int)d, (int)N, partial, (int)slices, s); break;
    case CI_F16: rc = down_cols_typed<F16>(H, (int)M, w_down, (int)d, (int)N, partial, (int)slices, s); break;
    case CI_BF16: rc = down_cols_typed<BF16>(H, (int)M, w_down, (int)d, (int)N, partial, (int)slices, s); break;
  }
  if (rc != CI_OK) return rc;
  return launch_decode_reduce(partial, b_down, Y, (int)slices, (int)d, (int)M, dtype, s);
}

int launch_up_rows(const void* X, int64_t M, const void* w_up, const void* w_gate, const void* b_up,
                   int dtype, int act, int64_t d, int64_t N, float* H, float* A, hipStream_t s) {
  switch (dtype) {
    case CI_F32: return up_typed<F32>(X, (int)M, w_up, w_gate, b_up, act, (int)d, (int)N, H, A, s);
    case CI_F16: return up_typed<F16>(X, (int)M, w_up, w_gate, b_up, act, (int)d, (int)N, H, A, s);
    case CI_BF16: return up_typed<BF16>(X, (int)M, w_up, w_gate, b_up, act, (int)d, (int)N, H, A, s);
  }
  return CI_ERR_BAD_DTYPE;
}

int launch_down_rows(const float* H, int64_t M, const void* w_down, const void* b_down, int dtype,
                     int64_t d, int64_t N, void* Y, hipStream_t s) {
  switch (dtype) {
    case CI_F32: return down_typed<F32>(H, (int)M, w_down, b_down, (int)d, (int)N, Y, s);
    case CI_F16: return down_typed<F16>(H, (int)M, w_down, b_down, (int)d, (int)N, Y, s);
    case CI_BF16: return down_typed<BF16>(H, (int)M, w_down, b_down, (int)d, (int)N, Y, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
