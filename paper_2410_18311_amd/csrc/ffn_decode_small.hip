// Decode-stage FFN of small layers in one launch without an exchange between workgroups (neuron-major compact weights):
//   y = W_down_c^T act(W_up_c x [+ b]) [+ b_down]
// The two launches of ffn_decode.hip cost the host about 3.9 us each, more than the GPU needs for both where the weights
// are a few hundred kilobytes.  So every workgroup here computes ALL hidden values, from weights that lie in its L2, keeps
// them in LDS and sums its own columns of y over all neurons: no partial sums, no second launch, nothing to agree on.
// What bounds it is the fill of a compute unit's L1 with the up (and gate) rows: by the slope of its time over their size 124 GB/s
// in fp32 and 85 in 16 bits, with twice the products a byte (256 x 96 to 256 x 512).  The down rows of the workgroup's columns
// are requested ahead of them and wait in registers.
// A call gives the same bits whichever way it goes (launched or captured, apart or in place; finite weights): dot products are
// added up over the lanes as there, down rows slice by slice, and the slices in the order of decode_reduce_kernel.  That costs
// nothing measurable: 256 x 424 fp32 from a graph 6.91 us, and 6.89 with the rows spread over all threads.
#include "common.hpp"
#include "decode_common.hpp"

namespace ci {

namespace {

struct SmallArgs {
  const void* x;
  const void* w_up;
  const void* w_gate;
  const void* b_up;
  const void* w_down;
  const void* b_down;
  void* y;
  int K, d;
  int n_wg;           // slices of the neurons
  uint32_t inv_n_wg;  // 2^32 / n_wg rounded up: a product below 2^20 times it, 32 bits up, is the product over n_wg
  int most_rows;      // at least the rows of any slice
};

constexpr int kSmallThreads = 512, kSmallWaves = 8;
constexpr int kSmallQuads = 4;   // 16-byte vectors of columns of a workgroup
constexpr int kSmallRows = 8;    // rows in flight per group of lanes
constexpr int kSmallDown = 4;    // down rows a thread holds at a time
constexpr int kSmallMaxK = 4096; // hidden values in LDS
constexpr int kReduceGroups = 32;  // groups of slices in decode_reduce_kernel: 256 threads, eight column quads
constexpr int kSmallSlices = 8 * kReduceGroups;  // most slices of the neurons, two a thread

// The value L lanes further on in the same sixteen (past them: zero).
template <int L>
__device__ __forceinline__ float lane_behind(float v) {
  return u2f((uint32_t)__builtin_amdgcn_mov_dpp((int)f2u(v), 0x100 + L, 0xf, 0xf, true));
}

// G lanes share a row of d elements, NI vectors each.
template <class D, int G, int NI, bool SWIGLU>
__global__ __launch_bounds__(kSmallThreads) void ffn_decode_small_kernel(SmallArgs a) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  constexpr int GPW = 64 / G, STEP = kSmallWaves * GPW;  // rows side by side
  __shared__ float h[kSmallMaxK];
  __shared__ float sums[kSmallWaves][kSmallQuads * VEC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y;
  const size_t rowbytes = (size_t)a.d * sizeof(T);
  const int vecs = a.d / VEC;
  const char* x = reinterpret_cast<const char*>(a.x) + (size_t)b * rowbytes;
  const char* up = reinterpret_cast<const char*>(a.w_up);
  const char* gate = reinterpret_cast<const char*>(a.w_gate);

  const int gl = lane % G, row0 = wave * GPW + lane / G;
  uint32_t off[NI];
  float xr[NI][VEC];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int v = i * G + gl;
    off[i] = v < vecs ? (uint32_t)v * 16u : 0u;  // a vector past the end re-reads the first; its x is zero
    unpack<D>(ld16(x + off[i]), xr[i]);
    if (v >= vecs) {
#pragma unroll
      for (int c = 0; c < VEC; ++c) xr[i][c] = 0.f;
    }
  }
  // Columns of y: 16 bytes of them a thread, and one slice of the neurons or, of more than 128, two: rows from a0 to a1 and
  // from b0 to b1.  Lanes: two bits of the columns (neighbours, as they lie), two of the slice, two of the reduction's group.  The
  // first rows, which need no hidden value to be requested:
  const int q = lane & 3, group = wave * 4 + (lane >> 4), first = group + kReduceGroups * (lane >> 2 & 3);
  const bool two = a.n_wg > kSmallSlices / 2;  // uniform
  auto slice = [&](int w) { return w < a.n_wg ? (int)__umulhi((uint32_t)w * (uint32_t)a.K, a.inv_n_wg) : a.K; };
  const int a0 = slice(first), a1 = slice(first + 1);
  const int b0 = two ? slice(first + kSmallSlices / 2) : 0, b1 = two ? slice(first + kSmallSlices / 2 + 1) : 0;
  const int vec = blockIdx.x * kSmallQuads + q;
  const char* down = reinterpret_cast<const char*>(a.w_down) + (size_t)(vec < vecs ? vec : 0) * 16;
  // of the rows that a thread holds at a time, the second half is of its second slice, if it has one
  auto row_of = [&](int i, int r) { return two ? (i < kSmallDown / 2 ? a0 + r + i : b0 + r + i - kSmallDown / 2) : a0 + r + i; };
  auto end_of = [&](int i) { return two && i >= kSmallDown / 2 ? b1 : a1; };
  const int step = two ? kSmallDown / 2 : kSmallDown;  // rows of a slice at a time
  uint4 dn[2][kSmallDown];
  auto request_down = [&](uint4 (&to)[kSmallDown], int r) {
#pragma unroll
    for (int i = 0; i < kSmallDown; ++i) to[i] = ld16(down + (size_t)min(row_of(i, r), a.K - 1) * rowbytes);
  };
  request_down(dn[0], 0);

  constexpr int SH = G / kSmallRows;  // lanes that end with the same row's sum
  for (int r0 = row0; r0 - row0 < a.K; r0 += kSmallRows * STEP) {
    const int mine = r0 + gl / SH * STEP;  // the row whose sum ends in this lane
    float bias = 0.f;
    if (!SWIGLU && a.b_up) bias = to_float<D>(reinterpret_cast<const T*>(a.b_up)[min(mine, a.K - 1)]);
    uint4 u[kSmallRows][NI], g[SWIGLU ? kSmallRows : 1][NI];
#pragma unroll
    for (int s = 0; s < kSmallRows; ++s) {
      const size_t row = (size_t)min(r0 + s * STEP, a.K - 1) * rowbytes;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (SWIGLU) g[s][i] = ld16(gate + row + off[i]);
        u[s][i] = ld16(up + row + off[i]);
      }
    }
    float zu[kSmallRows], zg[kSmallRows];
#pragma unroll
    for (int s = 0; s < kSmallRows; ++s) {
      zu[s] = zg[s] = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        float f[VEC];
        unpack<D>(u[s][i], f);
#pragma unroll
        for (int c = 0; c < VEC; ++c) zu[s] = fmaf(f[c], xr[i][c], zu[s]);
        if (SWIGLU) {
          unpack<D>(g[s][i], f);
#pragma unroll
          for (int c = 0; c < VEC; ++c) zg[s] = fmaf(f[c], xr[i][c], zg[s]);
        }
      }
    }
    halve_rows<kSmallRows, G / 2>(zu, lane);
    if (SWIGLU) halve_rows<kSmallRows, G / 2>(zg, lane);
    if (gl % SH == 0 && mine < a.K) h[mine] = SWIGLU ? silu(zg[0]) * zu[0] : fmaxf(zu[0] + bias, 0.f);
  }
  if (a.most_rows > step) request_down(dn[1], step);  // uniform
  __syncthreads();

  // the slices' sums, row by row
  float acc[2][VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) acc[0][c] = acc[1][c] = 0.f;
  auto add_row = [&](const uint4& from, float hk, bool valid, float (&to)[VEC]) {
    if (valid) {
      float f[VEC];
      unpack<D>(from, f);
#pragma unroll
      for (int c = 0; c < VEC; ++c) to[c] = fmaf(hk, f[c], to[c]);
    }
  };
  auto rows = [&](const uint4 (&from)[kSmallDown], int r) {
    float hk[kSmallDown];
#pragma unroll
    for (int i = 0; i < kSmallDown; ++i) hk[i] = h[min(row_of(i, r), a.K - 1)];
#pragma unroll
    for (int i = 0; i < kSmallDown / 2; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[0]);
    if (two) {
#pragma unroll
      for (int i = kSmallDown / 2; i < kSmallDown; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[1]);
    } else {
#pragma unroll
      for (int i = kSmallDown / 2; i < kSmallDown; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[0]);
    }
  };
  for (int r = 0; r < a.most_rows; r += 2 * step) {
    rows(dn[0], r);
    if (r + 2 * step < a.most_rows) request_down(dn[0], r + 2 * step);
    if (r + step < a.most_rows) {
      rows(dn[1], r + step);
      if (r + 3 * step < a.most_rows) request_down(dn[1], r + 3 * step);
    }
  }
  // The sums of the slices, in the order of decode_reduce_kernel: slices of a group (32 apart) one after the other, groups of
  // eight pairwise, the eights one after the other.  A slice that there is not adds zero.
#pragma unroll
  for (int c = 0; c < VEC; ++c) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (i == 0 || two) {
        t += acc[i][c];
        t += lane_behind<4>(acc[i][c]);
        t += lane_behind<8>(acc[i][c]);
        t += lane_behind<12>(acc[i][c]);
      }
    }
    const auto s16 = __builtin_amdgcn_permlane16_swap(f2u(t), f2u(t), false, false);
    t = u2f(s16[0]) + u2f(s16[1]);  // lanes 16 apart, then 32
    const auto s32 = __builtin_amdgcn_permlane32_swap(f2u(t), f2u(t), false, false);
    t = u2f(s32[0]) + u2f(s32[1]);
    if ((lane & 0x3c) == 0) sums[wave][q * VEC + c] = t;
  }
  __syncthreads();
  const int col = blockIdx.x * kSmallQuads * VEC + tid;
  if (tid < kSmallQuads * VEC && col < a.d) {
    float t = sums[0][tid] + sums[1][tid];
#pragma unroll
    for (int w = 2; w < kSmallWaves; w += 2) t += sums[w][tid] + sums[w + 1][tid];
    const float bias = a.b_down ? to_float<D>(reinterpret_cast<const T*>(a.b_down)[col]) : 0.f;
    reinterpret_cast<T*>(a.y)[(size_t)b * a.d + col] = from_float<D>(t + bias);
  }
}

template <class D, bool SWIGLU>
int launch_typed(const SmallArgs& a, int B, hipStream_t s) {
  const int vecs = a.d / D::VEC;
  const dim3 grid((vecs + kSmallQuads - 1) / kSmallQuads, B), block(kSmallThreads);
  if (vecs <= 16) hipLaunchKernelGGL((ffn_decode_small_kernel<D, 16, 1, SWIGLU>), grid, block, 0, s, a);
  else if (vecs <= 32) hipLaunchKernelGGL((ffn_decode_small_kernel<D, 32, 1, SWIGLU>), grid, block, 0, s, a);
  else if (vecs <= 64) hipLaunchKernelGGL((ffn_decode_small_kernel<D, 64, 1, SWIGLU>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((ffn_decode_small_kernel<D, 64, 2, SWIGLU>), grid, block, 0, s, a);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D>
int launch_dtype(const SmallArgs& a, int B, int act, hipStream_t s) {
  return act == CI_ACT_SWIGLU ? launch_typed<D, true>(a, B, s) : launch_typed<D, false>(a, B, s);
}

}  // namespace

// Where one launch beats two, by elements of the up and gate matrices with rows rounded up to what the lanes of their loads hold.
// Launched call by call, two launches are bound by the host and one is faster up to kSmallElements, over one to four tokens,
// both activations and all types; replayed from a graph two cost no host time, and one is faster up to kSmallElementsGraph only (us,
// two launches / one; call by call, then from a graph):
//   one token     fp32  256 x 256   7.7 / 5.2, 5.7 / 5.3     256 x 288  7.8 / 5.7, 5.7 / 5.9   256 x 424 7.8 / 6.9, 5.8 / 6.9
//                       128 x 1024  7.7 / 7.6, 5.7 / 7.6     gated 512 x 72  7.8 / 6.6, 6.2 / 6.7
//                 fp16  256 x 256   7.6 / 4.8, 5.8 / 4.9     256 x 512  7.6 / 6.4, 5.9 / 6.5   gated 256 x 256 7.7 / 5.8, 6.1 / 5.8
//                 bf16  256 x 424   7.8 / 6.4, 6.0 / 6.5     gated 256 x 256 7.8 / 6.0, 6.2 / 6.0
//   four tokens   fp32  256 x 256   7.9 / 5.2, 5.9 / 5.2     256 x 512  7.8 / 7.8, 6.7 / 8.1   gated 512 x 72 7.8 / 6.9, 6.3 / 7.0
//                 fp16  256 x 512   7.9 / 6.8, 6.9 / 6.9     gated 256 x 256  7.8 / 5.6, 6.6 / 5.7
// (of 208 such layers none of up to 64 K elements was slower in either way).  Both ways give the same bits.
constexpr int64_t kSmallElements = 128 * 1024, kSmallElementsGraph = 64 * 1024;
bool decode_small_pays(int64_t B, int64_t K, int64_t d, int dtype, int act, int n_wg, hipStream_t s) {
  const int mode = params().decode_small;
  const int64_t vec = 16 / elem_bytes(dtype), vecs = d / vec;
  if (mode == 0 || K < 1 || K > kSmallMaxK || vecs > 128 || B > 4 || n_wg > kSmallSlices) return false;
  const int64_t held = vecs <= 16 ? 16 : vecs <= 32 ? 32 : (vecs + 63) / 64 * 64;
  const int64_t elements = (act == CI_ACT_SWIGLU ? 2 : 1) * K * held * vec;
  if (mode == 2 || elements <= kSmallElementsGraph) return true;
  if (elements > kSmallElements) return false;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;  // the null stream is never captured
  return !s || (hipStreamIsCapturing(s, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone);
}

int launch_ffn_decode_small(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act, void* y, int n_wg, hipStream_t s) {
  const int K = (int)w->K;
  const SmallArgs a{x, w->w_up, w->w_gate, w->b_up, w->w_down, w->b_down, y, K, (int)w->d, n_wg,
                    (uint32_t)(((1ull << 32) + n_wg - 1) / n_wg), (K + n_wg - 1) / n_wg};
  switch (dtype) {
    case CI_F32: return launch_dtype<F32>(a, (int)B, act, s);
    case CI_F16: return launch_dtype<F16>(a, (int)B, act, s);
    case CI_BF16: return launch_dtype<BF16>(a, (int)B, act, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
