// Decode-stage FFN of small layers in one launch without an exchange between workgroups (neuron-major compact weights):
//   y = W_down_c^T act(W_up_c x [+ b]) [+ b_down]
// The two launches of ffn_decode.hip cost the host about 3.9 us each, more than the GPU needs for both where the weights
// are a few hundred kilobytes.  So every workgroup here computes ALL hidden values, from weights that lie in its L2, keeps
// them in LDS and sums its own columns of y over all neurons: no partial sums, no second launch, nothing to agree on.
// What bounds it is the fill of a compute unit's L1 with the up (and gate) rows, about 130 GB/s (fp32; 80 in 16 bits,
// with twice the products a byte); the down rows of the workgroup's
// columns are requested first and wait in registers.  Eight waves with eight rows in flight each: with sixteen 7.5, with four rows
// 8.4 and with the next rows requested ahead 6.9 instead of 6.7 us (256 x 410 fp32, from a graph).
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
};

constexpr int kSmallThreads = 512, kSmallWaves = 8;
constexpr int kSmallQuads = 4;   // 16-byte vectors of columns of a workgroup
constexpr int kSmallRows = 8;    // rows in flight per group of lanes
constexpr int kSmallDown = 4;    // down rows a thread holds at a time
constexpr int kSmallMaxK = 4096; // hidden values in LDS

// G lanes share a row of d elements, NI vectors each.
template <class D, int G, int NI, bool SWIGLU>
__global__ __launch_bounds__(kSmallThreads) void ffn_decode_small_kernel(SmallArgs a) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  constexpr int GPW = 64 / G, STEP = kSmallWaves * GPW;  // rows side by side
  constexpr int KG = kSmallThreads / kSmallQuads;        // down rows side by side
  __shared__ float h[kSmallMaxK];
  __shared__ float sums[kSmallWaves][kSmallQuads * VEC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y;
  const size_t rowbytes = (size_t)a.d * sizeof(T);
  const int vecs = a.d / VEC;
  const char* x = reinterpret_cast<const char*>(a.x) + (size_t)b * rowbytes;
  const char* up = reinterpret_cast<const char*>(a.w_up);
  const char* gate = reinterpret_cast<const char*>(a.w_gate);

  // columns of y: the first down rows, which need no hidden value to be requested
  const int q = blockIdx.x * kSmallQuads + tid % kSmallQuads, kg = tid / kSmallQuads;
  const bool qv = q < vecs;
  const char* down = reinterpret_cast<const char*>(a.w_down) + (size_t)(qv ? q : 0) * 16;
  uint4 dn[kSmallDown];
  auto request_down = [&](int k0) {
#pragma unroll
    for (int s = 0; s < kSmallDown; ++s) dn[s] = ld16(down + (size_t)min(k0 + s * KG, a.K - 1) * rowbytes);
  };
  request_down(kg);

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
  __syncthreads();

  float acc[VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) acc[c] = 0.f;
  for (int k0 = kg; k0 < a.K; k0 += kSmallDown * KG) {
#pragma unroll
    for (int s = 0; s < kSmallDown; ++s) {
      const int k = k0 + s * KG;
      float f[VEC];
      unpack<D>(dn[s], f);
      if (k < a.K) {
        const float hk = h[k];
#pragma unroll
        for (int c = 0; c < VEC; ++c) acc[c] = fmaf(hk, f[c], acc[c]);
      }
    }
    if (k0 + kSmallDown * KG < a.K) request_down(k0 + kSmallDown * KG);
  }
  // lanes of the same columns, then the waves in order
#pragma unroll
  for (int m = kSmallQuads; m < 64; m <<= 1)
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] += __shfl_xor(acc[c], m, kWave);
  if (lane < kSmallQuads) {
#pragma unroll
    for (int c = 0; c < VEC; ++c) sums[wave][lane * VEC + c] = acc[c];
  }
  __syncthreads();
  const int col = blockIdx.x * kSmallQuads * VEC + tid;
  if (tid < kSmallQuads * VEC && col < a.d) {
    float t = sums[0][tid];
#pragma unroll
    for (int w = 1; w < kSmallWaves; ++w) t += sums[w][tid];
    if (a.b_down) t += to_float<D>(reinterpret_cast<const T*>(a.b_down)[col]);
    reinterpret_cast<T*>(a.y)[(size_t)b * a.d + col] = from_float<D>(t);
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

// Where one launch beats two by the time of the whole call, host included: up to kSmallElements of the up and gate matrices, rows
// rounded up to what the lanes of their loads hold.  fp32, one token, launched call by call / replayed from a graph (us, two
// launches -> one): 26 K elements 8.6 / 7.0 -> 4.8 / 3.8; 52 K 8.9 / 7.1 -> 5.2 / 5.0; 105 K (256 x 410) 8.6 / 5.6 -> 6.8 / 6.7; 210 K
// 8.5 / 5.7 -> 9.7 / 9.6; fp16 8 K 8.7 / 5.4 -> 4.8 / 3.6, 210 K 8.7 / 5.9 -> 8.8 / 8.6.  A sentence of 16 tokens of the 105 K layer, prompt
// to last token, 192 -> 155.  From about 70 K elements on a graph would be faster with two launches; the line is drawn for calls that
// are launched, since a program that replays a graph has layers of millions.
constexpr int64_t kSmallElements = 128 * 1024;
bool decode_small_pays(int64_t B, int64_t K, int64_t d, int dtype, int act) {
  const int mode = params().decode_small;
  const int64_t vec = 16 / elem_bytes(dtype), vecs = d / vec;
  if (mode == 0 || K < 1 || K > kSmallMaxK || vecs > 128 || B > 4) return false;
  const int64_t held = vecs <= 16 ? 16 : vecs <= 32 ? 32 : (vecs + 63) / 64 * 64;
  return mode == 2 || (act == CI_ACT_SWIGLU ? 2 : 1) * K * held * vec <= kSmallElements;
}

int launch_ffn_decode_small(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act, void* y, hipStream_t s) {
  const SmallArgs a{x, w->w_up, w->w_gate, w->b_up, w->w_down, w->b_down, y, (int)w->K, (int)w->d};
  switch (dtype) {
    case CI_F32: return launch_dtype<F32>(a, (int)B, act, s);
    case CI_F16: return launch_dtype<F16>(a, (int)B, act, s);
    case CI_BF16: return launch_dtype<BF16>(a, (int)B, act, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
