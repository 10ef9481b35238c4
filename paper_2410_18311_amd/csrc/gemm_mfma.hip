// Dense prefill FFN (Def. 1 of arXiv 2410.18311: the activation vector A(x)
// of every prompt token) -- the one real dense contraction of the path, so it
// runs on the matrix cores.
//
//   C[M, Nn] = A[M, Kk] * B^T   with B given as [Nn, Kk] (both operands
//   k-contiguous, the nn.Linear layout) or, for a neuron-major down matrix, as
//   [Kk, Nn].
//
// This file plans a product (which tile shape, whether the last round of tiles is
// split along k) for the kernels of gemm_wide.hip, gemm_mid.hip and gemm_slim.hpp,
// and adds up split sums.
// The fp32 element type has its own kernels (gemm_f32.hip).
#include "gemm_common.hpp"

namespace ci {

namespace {

// Y[m, n] = sum_s partial[s][tile][m, n] + bias[n], converted to the element type, over the `tail` tiles that were
// split (bm x bn, from place `first` in the order of tile_of).  A thread has four columns of one row; all splits' loads
// of it are in flight together.  (16 rows a workgroup, several turns a thread, left half of the compute units without work
// where one row of tiles is split: 256 tokens, 4096 x 16384, both products 105.8 -> 105.0 us.)
constexpr int kReduceQuads = 256;
template <class D>
__global__ __launch_bounds__(kReduceQuads) void split_reduce_kernel(const float* __restrict__ partial, const void* __restrict__ bias,
                                                           void* __restrict__ out, int splits, int M, int Nn, int bm,
                                                           int bn, int first, int tail) {
  using T = typename D::T;
  const int strips = (bm * bn / 4 + kReduceQuads - 1) / kReduceQuads;
  int tm, tn;
  const int tile = blockIdx.x / strips, quads = bn / 4;
  const int quad = blockIdx.x % strips * kReduceQuads + threadIdx.x;
  const int r = quad / quads, c = quad % quads * 4;
  const size_t stride = (size_t)tail * sums_pitch(bm, bn);  // a split's tiles
  tile_of(first + tile, (M + bm - 1) / bm, (Nn + bn - 1) / bn, &tm, &tn);
  const int row = tm * bm + r, col = tn * bn + c;
  if (r >= bm || row >= M || col >= Nn) return;
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
// Every workgroup takes all of a compute unit's LDS, so tiles run in rounds of 256.  Three estimates, each for the products it was
// fitted to.
constexpr int kTileK = 64;      // k of a tile
constexpr int kFullChip = 256;  // compute units of an MI355X
constexpr int kSlimRows = 128;

struct Product {
  int M, Nn, Kk;
  bool up, dual;  // the up projection, whose k is not split; with a gate matrix
  bool b_kmajor;
  int out_bytes;  // written per output
  // 16-bit elements: what share of the 128-byte pieces of a row lie in two cache lines
  double two_lines() const {
    const int odd = Kk * 2 % 128;
    return odd == 0 ? 0.0 : odd % 64 == 0 ? 0.5 : odd % 32 == 0 ? 0.75 : 0.875;
  }
};

// More than 128 rows.  A round of n tiles takes their multiplications, faster the fewer run side by side (they share the chip's
// power and caches), a fixed part (first loads, results) and the stores; the sums of split tiles are written, read back
// and added by another launch.  The constants are those that came closest to 4900 measured products of 129 to 4096 rows, d
// 1024 to 9216 and N 2048 to 36864, odd lengths among them, all shapes and splits (7.6 % off on average), the last four shapes' to 394 more
// up projections.  The tiles of 128 rows were measured with an earlier kernel, 4 to 8 % slower than gemm_mid.hip's.  That costs
// little: over 222 other products of 129 to 2048 rows on the present kernels, layers in turn, the up plans are on average 0.9 % behind the fastest
// of all shapes and the down plans 0.9 % behind the fastest of all shapes and splits (one in ten by more than 2 and 3.5 %, at most by 21 and 17 %),
// both projections together 1.4 %.  A quarter of the up plans take one of the last four, and 15 % less time than the fastest other shape,
// one of 55 more than it (3.4 %).
struct ManyShape {
  int shape;
  int bm, bn;        // rows of A, rows of B (SwiGLU: half of them gate, half up)
  double rate;       // flop/s of one compute unit inside a tile, all of them busy
  double fixed;      // s of a round
  double alone;      // a tile's time with nothing beside it, as a share of that
  double two_lines;  // what share more it takes when every 128 bytes of a row lie in two lines
};
constexpr ManyShape kManyShapes[] = {{kMid128x128, 128, 128, 3.54e12, 2.8e-6, 0.58, 0.37}, {kMid128x256, 128, 256, 4.41e12, 3.9e-6, 0.61, 0.41},
                                     {kMid128x64, 128, 64, 2.72e12, 2.1e-6, 0.70, 0.42},   {kWide, 256, 256, 6.12e12, 8.0e-6, 0.72, 0.13},
                                     {kWide224, 256, 224, 5.85e12, 6.3e-6, 0.73, 0.16},    {kWide192, 256, 192, 5.51e12, 4.9e-6, 0.71, 0.19},
                                     {kWide160, 256, 160, 4.94e12, 3.0e-6, 0.69, 0.24},    {kMid192x128, 192, 128, 4.35e12, 2.3e-6, 0.90, 0.25},
                                     {kMid128x96, 128, 96, 3.17e12, 2.5e-6, 0.56, 0.30},   {kMid128x160, 128, 160, 3.83e12, 3.7e-6, 0.61, 0.36},
                                     {kMid128x192, 128, 192, 4.08e12, 3.5e-6, 0.69, 0.38}};
struct ManyRowsTime {
  double t_k, alone, fixed, store, t_sums, doubt;
  int out_bytes;
  ManyRowsTime(const ManyShape& ts, const Product& p) {
    const int bn = p.dual ? ts.bn / 2 : ts.bn;
    t_k = 2.0 * ts.bm * ts.bn * (double)p.Kk / ts.rate * (1.0 + ts.two_lines * p.two_lines() * (p.b_kmajor ? 0.5 : 1.0));
    alone = ts.alone;
    fixed = ts.fixed;
    store = (double)ts.bm * bn / 16e12;
    t_sums = (double)ts.bm * bn / 5e12;
    // An up projection whose rows are shorter than those of the fit is mostly results, and takes longer than estimated on tiles that are not
    // powers of two in both directions: those are taken where they promise 8 % (of 120 drawn products of 200 to 4096 rows, d 128 to 1100, the
    // shapes are so on average 0.5 % behind the fastest, seven by more than 3 % and at most by 13; 1.4 %, 15 and 33 without it, e.g.
    // gated 2908 x 144 x 2400 23.4 us on 256 x 160 and 17.6 on 256 x 256; 0.7 % at a promise of 5 and 0.9 % at 15).
    doubt = p.up && p.Kk < 1024 && ((ts.bm & (ts.bm - 1)) != 0 || (ts.bn & (ts.bn - 1)) != 0) ? 1.08 : 1.0;
    out_bytes = p.out_bytes;
  }
  double round(int n, double t, int bytes) const { return t * (alone + (1.0 - alone) / kFullChip * n) + fixed + n * store * bytes; }
  double rounds(int wgs, double t, int bytes) const {
    const int whole = wgs / kFullChip, rest = wgs % kFullChip;
    return (whole > 0 ? whole * round(kFullChip, t, bytes) : 0.0) + (rest > 0 ? round(rest, t, bytes) : 0.0);
  }
  double operator()(int full, int tail, int sp) const {
    return doubt * (rounds(full, t_k, out_bytes) + (tail == 0 ? 0.0 : rounds(tail * sp, t_k / sp, 4) + (double)tail * (4 * sp + 2) * t_sums + 3e-6));
  }
};

// Up to 128 rows.  The first estimate counts whole rounds of the larger tiles (about 4.5 TB/s and 5 us for split sums).
struct FewShape {
  int shape;
  int bm, bn;
  double rate;  // flop/s of one compute unit inside a tile
  // FewRowsTime: bytes/s and flop/s of one compute unit, s of a round, and what share more of its time a
  // fill takes when every 128 bytes of a row lie in two lines
  double fill, flops, fixed, two_lines;
};
constexpr FewShape kFewShapes[] = {{kMid128x128, 128, 128, 3.6e12, 144e9, 10.1e12, 4.3e-6, 0.85},
                                   {kMid128x256, 128, 256, 4.4e12, 114e9, 16.6e12, 4.0e-6, 1.0},
                                   {kMid128x64, 128, 64, 2.7e12, 212e9, 6.5e12, 4.5e-6, 1.8},
                                   {kWide, 256, 256, 5.5e12, 1e15, 8.1e12, 4.2e-6, 0}};
constexpr FewShape slim_shape(int tm, int tn) {
  return FewShape{kSlim + 16 * tm + tn, 16 * tm, 16 * tn, 2.7e12, 165e9, 7.3e12, 5.3e-6, 2.6};
}
struct WholeRoundsTime {
  double t_tile, t_fixed, t_sums;
  WholeRoundsTime(const FewShape& ts, const Product& p) {
    const int bn = p.dual ? ts.bn / 2 : ts.bn;
    t_tile = 2.0 * ts.bm * ts.bn * (double)p.Kk / ts.rate;
    // first loads; results of a round, which nothing overlaps
    t_fixed = 3e-6 + (double)ts.bm * bn * p.out_bytes * kFullChip / 4.5e12;
    t_sums = 2.0 * ts.bm * bn * 4.0 / 4.5e12;
  }
  double operator()(int full, int tail, int sp) const {
    return (double)((full + kFullChip - 1) / kFullChip) * (t_tile + t_fixed) +
           (double)((tail * sp + kFullChip - 1) / kFullChip) * (t_tile / sp + t_fixed) +
           (tail == 0 ? 0.0 : (double)sp * tail * t_sums + 5e-6);
  }
};

// The second is a sum rather than a maximum of three parts: what an L1 is filled with, the multiplications, and the weights that a
// round reads from memory (a maximum, or a power mean of any higher order, fits worse).  It is a fit, not a model of the chip: the
// constants of kFewShapes are those that come closest to 26000 measured products of 5 to 512 rows, d 1024 to 9216 and N 2816 to
// 36864, odd lengths among them, all shapes and splits, those of 128 rows with the same earlier kernel.  On the present ones the plans for 299 other
// products of 5 to 128 rows are on average 1.6 % (up) and 4.1 % (down) behind the fastest of all, one in ten by more than 4 and 14 %, at
// most by 50 and 28 %.  (For tiles of 256 x 256 a fill that costs nothing came closest, with
// fewer flop/s.  Only down projections of layers much wider than their N take those: none of 600000 drawn plans with N of 2.6 to 4 d, three
// of 600000 of any proportions, e.g. 128 x 21752 x 4744.)
struct FewRowsTime {
  int tiles_m, out_bytes;
  double k, fill, columns_fill, inv_tiles_m, fixed, store, t_sums;
  FewRowsTime(const FewShape& ts, const Product& p) {
    const int bn = p.dual ? ts.bn / 2 : ts.bn, rows = p.M < ts.bm ? p.M : ts.bm;
    tiles_m = (p.M + ts.bm - 1) / ts.bm;
    out_bytes = p.out_bytes;
    k = p.Kk;
    fill = 2.0 * ((rows + ts.bn) * (1.0 + ts.two_lines * p.two_lines()) / ts.fill + (double)ts.bm * ts.bn / ts.flops);
    columns_fill = 2.0 * ts.bn / 9.9e12;
    inv_tiles_m = 1.0 / tiles_m;
    fixed = ts.fixed;
    store = (double)rows * bn / 4.5e12;
    t_sums = (double)rows * bn * 4.0 / 7.9e12;
  }
  double round(int n, double k_n, int bytes) const {
    const double columns = n > tiles_m ? n * inv_tiles_m : 1.0;  // tiles whose weights differ
    return k_n * (fill + columns * columns_fill) + fixed + n * store * bytes;
  }
  double rounds(int wgs, double k_n, int bytes) const {
    const int whole = wgs / kFullChip, rest = wgs % kFullChip;
    return (whole > 0 ? whole * round(kFullChip, k_n, bytes) : 0.0) + (rest > 0 ? round(rest, k_n, bytes) : 0.0);
  }
  double operator()(int full, int tail, int sp) const {
    return rounds(full, k, out_bytes) + (tail == 0 ? 0.0 : rounds(tail * sp, k / sp, 4) + (double)sp * tail * t_sums + 2.5e-6);
  }
};

// Adds a shape, whole and with its last round in 2 .. 8 parts, to the best plan so far by the estimate Time.
template <class Time, class Shape>
void consider(const Shape& ts, const Product& p, size_t room, GemmPlan& best, double& best_t) {
  const Time time(ts, p);
  const int force_splits = params().gemm_splits;
  const int bn = p.dual ? ts.bn / 2 : ts.bn;
  const int tiles = ((p.M + ts.bm - 1) / ts.bm) * ((p.Nn + bn - 1) / bn);
  for (int sp = 1; sp <= 8; ++sp) {
    if (sp > 1 && p.Kk < 4 * kTileK * sp) break;  // at least four k tiles per split
    const int full = sp == 1 ? tiles : tiles / kFullChip * kFullChip, tail = tiles - full;
    // rounding the chunk up can leave the last split without work: it then needs no room either (or a workspace of just what
    // the plan needs would lead to another plan than a larger one)
    const int k_chunk = sp == 1 ? p.Kk : ((p.Kk + sp - 1) / sp + kTileK - 1) / kTileK * kTileK;
    const int parts = (p.Kk + k_chunk - 1) / k_chunk;
    if (sp > 1 && (tail == 0 || (size_t)parts * (size_t)tail * sums_pitch(ts.bm, bn) * sizeof(float) > room)) break;
    const double t = time(full, tail, sp);
    if (force_splits > 0 && !p.up ? sp == force_splits : t < best_t) {
      best_t = t;
      best = GemmPlan{ts.shape, ts.bm, bn, full, tail, sp, k_chunk};
    }
  }
  if (best_t > 1e29 && force_splits > 0) best = GemmPlan{ts.shape, ts.bm, bn, tiles, 0, 1, p.Kk};
}

// The shape and split of the least estimated time whose sums fit `room` bytes.  Examples (both projections, former
// kernels -> these): 77 tokens, 4096 x 11008 gated 97 -> 66 us; 700 tokens, 4096 x 16384, neuron-major down 708 -> 207 us; 1000
// tokens, 7168 x 28672, neuron-major 2446 -> 715 us; 8 x 512 tokens, 9216 x 36864 4.9 -> 4.0 ms (its down projection: 576 tiles =
// two rounds and 64 tiles in four parts, where the former plan split all 576).
// Up to 128 rows the plan is made again by FewRowsTime, for a k-contiguous B with the tiles of 16 tm x 16 tn too, and taken if
// that estimate promises 6 % or more (a line drawn with that earlier kernel of the 128-row tiles): over 578 measured products 7 % faster on average, one in a hundred by more than 5 % (at
// most 14 %) slower; without the line at 6 % 8 % and three in a hundred, up to 32 %.  (The line was drawn on these products.  164
// others, both projections together, layers of 120 to 330 MB in turn: 13 % faster on average, at most 2.5 % slower.)  From 129 rows on the slim tiles are 3 to
// 50 % slower than the others (their rows of B are read by several workgroups), and a k-major B, whose rows would be pieces of 32
// to 256 bytes, ran on them from 23 % faster to 25 % slower.
GemmPlan plan_gemm(int64_t M, int64_t Nn, int64_t Kk, bool up, bool dual, bool b_kmajor, int out_bytes, size_t room) {
  const Product p{(int)M, (int)Nn, (int)Kk, up, dual, b_kmajor, out_bytes};
  GemmPlan best{};
  double best_t = 1e30;
  const int force = params().gemm_tile;
  if (force >= kSlim && !b_kmajor) {
    consider<WholeRoundsTime>(slim_shape((force - kSlim) / 16, (force - kSlim) % 16), p, room, best, best_t);
  } else if (M > kSlimRows || (force >= 0 && force < kSlim)) {
    for (const ManyShape& ts : kManyShapes)
      if ((force < 0 || force >= kSlim || ts.shape == force) && (up || !only_up(ts.shape)))
        consider<ManyRowsTime>(ts, p, room, best, best_t);
    if (best.bm == 0) consider<ManyRowsTime>(kManyShapes[0], p, room, best, best_t);  // a forced shape that is not for down projections
  } else {
    for (const FewShape& ts : kFewShapes) consider<WholeRoundsTime>(ts, p, room, best, best_t);
    if (force < 0 && params().gemm_splits == 0) {
      double few_t = 0.0;
      for (const FewShape& ts : kFewShapes)
        if (ts.shape == best.shape) few_t = 0.94 * FewRowsTime(ts, p)(best.full, best.tail, best.splits);
      for (const FewShape& ts : kFewShapes) consider<FewRowsTime>(ts, p, room, best, few_t);
      if (!b_kmajor)
        for (int tn = 2; tn <= 8; ++tn)
          if (slim_built((p.M + 15) / 16, tn)) consider<FewRowsTime>(slim_shape((p.M + 15) / 16, tn), p, room, best, few_t);
    }
  }
  if (best.splits > 1) best.splits = ((int)Kk + best.k_chunk - 1) / best.k_chunk;
  return best;
}

// Whether the rows of B go through the caches as data that is not read again, which leaves the caches to the rows of A: products
// of one row of tiles over 80 MB of weights and more, whose layer does not fit the memory-side cache (256 MB), or of up to 32
// rows.  us, ordinary loads -> these, both projections, for one layer again and again / layers in turn that fit no cache:
//   larger than it   67 x 4288 x 15616 (268 MB) 60.1 -> 61.1 / 68.5 -> 67.4; 91 x 4928 x 15424 (304 MB) 81.5 -> 70.3 / 83.6 -> 79.4;
//                    7 x 4928 x 16640 (328 MB) 63.3 -> 57.8 / 64.7 -> 59.5; 81 x 4096 x 14720 gated (362 MB) 85.5 -> 78.4 / 85.6 -> 79.2
//   smaller          16 x 3264 x 10304 gated (202 MB) 37.2 -> 40.3 / 44.7 -> 43.4; 5 x 4224 x 13632 (230 MB) 42.1 -> 43.6 / 48.6 -> 45.3;
//                    54 x 3968 x 13504 (214 MB) 46.6 -> 54.4 / 56.1 -> 55.3; 120 x 3584 x 11456 (164 MB) 44.7 -> 60.4 / 59.2 -> 60.3
// (of 190 such layers).  Of the smaller ones a single layer is slower with them, in a model of several it is 2 to 8 % faster
// up to 32 rows and 0 to 3 % above.  Two layers of 81 MB in turn: 74 x 2944 x 9152 36 -> 45.  Pieces that lie in two lines each need both
// lines to stay for the next k-tile (9 x 5912 x 21232 gated 165 -> 192).  Two rows of tiles read B twice: 256 x 4096 x 16384
// 104.7 -> 102.8, but 145 x 2816 x 9728 gated 71 -> 77.6.
bool read_once(const GemmPlan& p, int64_t M, int64_t Nn, int64_t Kk, bool dual, bool b_kmajor, bool gated) {
  const int mode = params().gemm_once;
  if (mode == 0 || b_kmajor || is_wide(p.shape) || only_up(p.shape)) return false;
  const int64_t one = Nn * Kk * 2;  // bytes of a matrix of the layer
  return mode == 2 || (M <= 128 && (dual ? 2 : 1) * one >= 80000000 && Kk % 64 == 0 &&
                       (M <= 32 || (gated ? 3 : 2) * one > (int64_t)256 << 20));
}

template <class D>
int launch_sums(const GemmArgs& g, const GemmPlan& p, hipStream_t s) {
  const int strips = (p.bm * p.bn / 4 + kReduceQuads - 1) / kReduceQuads;
  hipLaunchKernelGGL((split_reduce_kernel<D>), dim3((unsigned)(p.tail * strips)), dim3(kReduceQuads), 0, s, g.partial, g.bias,
                     g.out_e, p.splits, g.M, g.Nn, p.bm, p.bn, p.full, p.tail);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, int EPI, bool BNN>
int launch_mfma(GemmArgs& g, const GemmPlan& p, hipStream_t s) {
  g.full = p.full;
  g.tail = p.tail;
  g.splits = p.splits;
  g.k_chunk = p.k_chunk;
  g.once = p.once;
  constexpr int dtype = __is_same(D, F16) ? CI_F16 : CI_BF16;
  int rc = CI_ERR_UNSUPPORTED;
  if (p.shape >= kSlim) {
    const int tm = (p.shape - kSlim) / 16, tn = (p.shape - kSlim) % 16;
    if (!BNN) rc = __is_same(D, F16) ? launch_gemm_slim_f16(tm, tn, EPI, g, s) : launch_gemm_slim_bf16(tm, tn, EPI, g, s);
  } else {
    rc = is_wide(p.shape) ? launch_gemm_wide(p.shape, dtype, EPI, BNN, g, s) : launch_gemm_mid(p.shape, dtype, EPI, BNN, g, s);
  }
  if (rc != CI_OK || p.tail == 0) return rc;
  return launch_sums<D>(g, p, s);
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
  const GemmPlan p = gemm_up_plan(M, d, N, dtype, act);
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

GemmPlan gemm_up_plan(int64_t M, int64_t d, int64_t N, int dtype, int act) {
  // one plan whichever outputs are asked for: another tile adds up in another order, and their bits are the same in every call
  if (dtype == CI_F32) return GemmPlan{};
  const bool gated = act == CI_ACT_SWIGLU;
  GemmPlan p = plan_gemm(M, N, d, true, gated, false, 6, 0);
  p.once = read_once(p, M, N, d, gated, false, gated);
  return p;
}

// The down projection's plan, made once per call: the size check, the place of the sums and the launches all go by it.
GemmPlan gemm_down_plan(int64_t M, int64_t d, int64_t N, int down_layout, int dtype, bool gated, size_t room) {
  if (dtype == CI_F32) return GemmPlan{};
  const bool b_kmajor = down_layout == CI_DOWN_NEURON_MAJOR;
  GemmPlan p = plan_gemm(M, d, N, false, false, b_kmajor, 2, room);
  p.once = read_once(p, M, d, N, false, b_kmajor, gated);
  return p;
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
