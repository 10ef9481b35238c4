// Dense prefill FFN (Def. 1 of arXiv 2410.18311: the activation vector A(x)
// of every prompt token) -- the one real dense contraction of the path, so it
// runs on the matrix cores.
//
//   C[M, Nn] = A[M, Kk] * B^T   with B given as [Nn, Kk] (both operands
//   k-contiguous, the nn.Linear layout) or, for a neuron-major down matrix, as
//   [Kk, Nn].
//
// This file plans a product (which tile shape, whether the last round of tiles is
// split along k) for the kernels of gemm_wide.hip and gemm_mid.hip, and adds up
// split sums.
// The fp32 element type has its own kernels (gemm_f32.hip).
#include "gemm_common.hpp"

namespace ci {

namespace {

// Y[m, n] = sum_s partial[s][tile][m, n] + bias[n], converted to the element type, over the `tail` tiles that were
// split (bm x bn, from place `first` in the order of tile_of).  A workgroup takes the rows of a tile that give each
// thread four columns of one row; all splits' loads of it are in flight together.  (16 rows, several turns a thread, left
// half of the compute units without work where one row of tiles is split: 256 tokens, 4096 x 16384, both products 105.8 -> 105.0 us.)
constexpr int reduce_rows(int bn) { return 1024 / bn; }
template <class D>
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ partial, const void* __restrict__ bias,
                                                           void* __restrict__ out, int splits, int M, int Nn, int bm,
                                                           int bn, int first, int tail) {
  using T = typename D::T;
  const int strips = bm * bn / 1024;
  int tm, tn;
  const int tile = blockIdx.x / strips, quads = bn / 4;
  const int r = blockIdx.x % strips * reduce_rows(bn) + threadIdx.x / quads, c = threadIdx.x % quads * 4;
  const size_t stride = (size_t)tail * sums_pitch(bm, bn);  // a split's tiles
  tile_of(first + tile, (M + bm - 1) / bm, (Nn + bn - 1) / bn, &tm, &tn);
  const int row = tm * bm + r, col = tn * bn + c;
  if (row >= M || col >= Nn) return;
  const float* p = partial + (size_t)tile * sums_pitch(bm, bn) + r * bn + c;
  float4 a = *reinterpret_cast<const float4*>(p);
#pragma unroll 4
  for (int s = 1; s < splits; ++s) {
    const float4 v = *reinterpret_cast<const float4*>(p + s * stride);
    a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
  }
  const float o[4] = {a.x, a.y, a.z, a.w};
  T e[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    e[k] = from_float<D>(o[k] + (bias ? to_float<D>(reinterpret_cast<const T*>(bias)[col + k]) : 0.f));
  uint2 pack;
  __builtin_memcpy(&pack, e, 8);
  *reinterpret_cast<uint2*>(reinterpret_cast<T*>(out) + (size_t)row * Nn + col) = pack;
}

// ---- which tiles, and how they are spread over the chip ------------------------
struct TileShape {
  int shape;        // kMid..., or kWide
  int bm, bn;       // rows of A, rows of B (SwiGLU: half of them gate, half up)
  double rate;      // flop/s of one compute unit inside a tile (measured: rounds of full tiles at 512 to 4096 rows)
};
constexpr int kWide = 4;
constexpr int kTileK = 64;       // k of a tile
constexpr int kFullChip = 256;  // compute units of an MI355X
constexpr TileShape kShapes[] = {{kMid128x128, 128, 128, 3.6e12},
                                 {kMid128x256, 128, 256, 4.4e12},
                                 {kMid256x64, 256, 64, 3.2e12},
                                 {kMid128x64, 128, 64, 2.7e12},
                                 {kWide, 256, 256, 5.5e12}};

// Every workgroup takes all of a compute unit's LDS, so tiles run in rounds of 256.  Tiles of the last, partly
// filled round can be split along k into `splits` parts each, whose fp32 sums are written, read back and
// added by another launch (about 4.5 TB/s and 5 us).  The shape and split of the least estimated time whose sums fit
// `room` bytes are taken; out_bytes: written per output.  Examples (both projections, former kernels -> these): 77 tokens, 4096 x 11008
// gated 97 -> 71 us; 700 tokens, 4096 x 16384, neuron-major down 708 -> 207 us; 1000 tokens, 7168 x 28672,
// neuron-major 2446 -> 715 us; 8 x 512 tokens, 9216 x 36864 4.9 -> 4.2 ms (its down projection: 576 tiles =
// two rounds and 64 tiles in four parts, where the former plan split all 576).
GemmPlan plan_gemm(int64_t M, int64_t Nn, int64_t Kk, bool dual, int out_bytes, size_t room) {
  GemmPlan best{};
  double best_t = 1e30;
  const int force = params().gemm_tile, force_splits = params().gemm_splits;
  for (const TileShape& ts : kShapes) {
    if (force >= 0 && ts.shape != force) continue;
    const int bn = dual ? ts.bn / 2 : ts.bn;
    const int64_t tiles = ((M + ts.bm - 1) / ts.bm) * ((Nn + bn - 1) / bn);
    const double t_tile = 2.0 * ts.bm * ts.bn * (double)Kk / ts.rate;
    // first loads; results of a round, which nothing overlaps
    const double t_fixed = 3e-6 + (double)ts.bm * bn * out_bytes * kFullChip / 4.5e12;
    for (int sp = 1; sp <= 8; ++sp) {
      if (sp > 1 && Kk / ((int64_t)sp * kTileK) < 4) break;  // at least four k tiles per split
      const int64_t full = sp == 1 ? tiles : tiles / kFullChip * kFullChip, tail = tiles - full;
      if (sp > 1 && (tail == 0 || (size_t)sp * (size_t)tail * sums_pitch(ts.bm, bn) * sizeof(float) > room)) break;
      const double t_full = (double)((full + kFullChip - 1) / kFullChip) * (t_tile + t_fixed);
      const double t_tail = (double)((tail * sp + kFullChip - 1) / kFullChip) * (t_tile / sp + t_fixed);
      const double t_sum = tail == 0 ? 0.0 : 2.0 * sp * (double)tail * ts.bm * bn * 4.0 / 4.5e12 + 5e-6;
      const double t = t_full + t_tail + t_sum;
      if (force_splits > 0 && room > 0 ? sp == force_splits : t < best_t) {
        best_t = t;
        best = GemmPlan{ts.shape, ts.bm, bn, (int)full, (int)tail, sp, (int)Kk};
        if (sp > 1) best.k_chunk = (int)(((Kk + sp - 1) / sp + kTileK - 1) / kTileK * kTileK);
      }
    }
    if (best_t > 1e29 && force_splits > 0) best = GemmPlan{ts.shape, ts.bm, bn, (int)tiles, 0, 1, (int)Kk};
  }
  if (best.splits > 1) best.splits = (int)((Kk + best.k_chunk - 1) / best.k_chunk);  // rounding the chunk up can empty the last one
  return best;
}

template <class D, int EPI, bool BNN>
int launch_mfma(GemmArgs& g, const GemmPlan& p, hipStream_t s) {
  g.full = p.full;
  g.tail = p.tail;
  g.splits = p.splits;
  g.k_chunk = p.k_chunk;
  constexpr int dtype = __is_same(D, F16) ? CI_F16 : CI_BF16;
  const int rc = p.shape == kWide ? launch_gemm_wide(dtype, EPI, BNN, g, s) : launch_gemm_mid(p.shape, dtype, EPI, BNN, g, s);
  if (rc != CI_OK || p.tail == 0) return rc;
  hipLaunchKernelGGL((split_reduce_kernel<D>), dim3((unsigned)(p.tail * (p.bm / reduce_rows(p.bn)))), dim3(256), 0, s, g.partial, g.bias,
                     g.out_e, p.splits, g.M, g.Nn, p.bm, p.bn, p.full, p.tail);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <int EPI, bool BNN>
int launch_any(int dtype, GemmArgs& g, const GemmPlan& p, hipStream_t s) {
  switch (dtype) {
    case CI_F32: return launch_gemm_f32(EPI, BNN, g, s);
    case CI_F16: return launch_mfma<F16, EPI, BNN>(g, p, s);
    case CI_BF16: return launch_mfma<BF16, EPI, BNN>(g, p, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace

int launch_gemm_up(const void* X, int64_t M, const void* w_up, const void* w_gate, const void* b_up,
                   int dtype, int act, int64_t d, int64_t N, void* H, float* A, hipStream_t s) {
  GemmArgs g;
  g.A = X;
  g.lda = d;
  g.ldb = d;
  g.ldo = N;
  g.M = (int)M;
  g.Nn = (int)N;
  g.Kk = (int)d;
  g.out_e = H;
  g.out_f = A;
  g.k_chunk = (int)d;
  g.partial = nullptr;
  const GemmPlan p = dtype == CI_F32 ? GemmPlan{} : plan_gemm(M, N, d, act == CI_ACT_SWIGLU, 6, 0);
  if (act == CI_ACT_SWIGLU) {
    g.B0 = w_gate;
    g.B1 = w_up;
    g.bias = nullptr;
    return launch_any<EPI_SWIGLU, false>(dtype, g, p, s);
  }
  g.B0 = w_up;
  g.B1 = nullptr;
  g.bias = b_up;
  return launch_any<EPI_RELU, false>(dtype, g, p, s);
}

// The down projection's plan, made once per call: the size check, the place of the sums and the launches all go by it.
GemmPlan gemm_down_plan(int64_t M, int64_t d, int64_t N, int dtype, size_t room) {
  return dtype == CI_F32 ? GemmPlan{} : plan_gemm(M, d, N, false, 2, room);
}

size_t gemm_plan_bytes(const GemmPlan& p) {
  return p.tail > 0 ? (size_t)p.splits * (size_t)p.tail * sums_pitch(p.bm, p.bn) * sizeof(float) : 0;
}

int launch_gemm_down(const void* H, int64_t M, const void* w_down, const void* b_down,
                     int down_layout, int dtype, int64_t d, int64_t N, void* Y, float* partial,
                     const GemmPlan& p, hipStream_t s) {
  GemmArgs g;
  g.A = H;
  g.lda = N;
  g.B0 = w_down;
  g.B1 = nullptr;
  g.bias = b_down;
  g.out_e = Y;
  g.out_f = nullptr;
  g.ldo = d;
  g.M = (int)M;
  g.Nn = (int)d;
  g.Kk = (int)N;
  g.k_chunk = (int)N;
  g.partial = partial;
  if (down_layout == CI_DOWN_OUT_MAJOR) {
    g.ldb = N;
    return launch_any<EPI_LINEAR, false>(dtype, g, p, s);
  }
  g.ldb = d;
  return launch_any<EPI_LINEAR, true>(dtype, g, p, s);
}

}  // namespace ci
