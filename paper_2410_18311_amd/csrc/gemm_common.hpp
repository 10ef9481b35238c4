// What the dense GEMM kernels share: their arguments, the epilogue kinds and the order of the tiles.
#pragma once

#include "common.hpp"

namespace ci {

enum { EPI_RELU = 0, EPI_SWIGLU = 1, EPI_LINEAR = 2 };

struct GemmArgs {
  const void* A;
  const void* B0;  // EPI_SWIGLU: gate
  const void* B1;  // EPI_SWIGLU: up
  const void* bias;
  void* out_e;     // [M, Nn] element type, may be null
  float* out_f;    // [M, Nn] fp32, may be null
  int64_t lda, ldb, ldo;
  int M, Nn, Kk;
  float* partial;  // where the k of a product is split: [splits][tail] tiles of fp32 partial products, sums_pitch apart
  // tiles computed whole, tiles computed by `splits` workgroups of k_chunk each (a multiple of the k tile)
  int full, tail, splits, k_chunk;
  bool once;  // B is loaded as data that is not read again
};

// Floats from one tile of sums to the next.  Most tiles are powers of two and their workgroups store in step: 256 bytes in
// between keep them off the same memory channels (256 tokens, gated 8192 x 28672: 380 us with tiles end to end or
// 1 KB apart in one run of two, 370 to 373 with 256 bytes and in rows of the whole product).
__host__ __device__ constexpr int64_t sums_pitch(int bm, int bn) { return (int64_t)bm * bn + 64; }

// Spreads consecutive tiles over one XCD (workgroup ids go round-robin over the
// 8 XCDs, each with its own L2), so that tiles sharing a B panel share an L2.
__device__ __forceinline__ int xcd_swizzle(int id, int n) {
  if (n % 8 != 0) return id;
  return (id % 8) * (n / 8) + id / 8;
}

// The same for any n (workgroup id -> place in an order of which each XCD walks one stretch).
__device__ __forceinline__ int xcd_spread(int id, int n) {
  const int x = id & 7, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + (id >> 3);
}

// Place t in the order of the tiles -> tile, such that tiles that run at the same time are close to square:
// groups of eight tile rows, columns outermost.  The 32 compute units of an XCD then read eight row panels and
// four column panels through their L2 at a time (all 16 row panels of a 4096-row product first would make
// that 18 panels).
__device__ __forceinline__ void tile_of(int t, int tiles_m, int tiles_n, int* tm, int* tn) {
  constexpr int G = 8;
  const int per_group = G * tiles_n;
  const int grp = t / per_group, in = t % per_group;
  const int rows = tiles_m - grp * G < G ? tiles_m - grp * G : G;
  *tm = grp * G + in % rows;
  *tn = in / rows;
}

// Tile shapes for 16-bit types, rows of A x rows of B per workgroup: 128 x 64 .. 256 and 192 x 128 (gemm_mid.hip), 256 x 160 .. 256
// (gemm_wide.hip).  The last four are for up projections, whose k is not split: a down projection's splits fill the chip as well.  (Without
// them the best of the other shapes is on average 5.2 % behind the best of all for an up projection, and 1.3 % for a down projection.)
enum { kMid128x128 = 0, kMid128x256 = 1, kWide192 = 2, kMid128x64 = 3, kWide = 4, kWide224 = 5, kWide160 = 6, kMid192x128 = 7,
       kMid128x96 = 8, kMid128x160 = 9, kMid128x192 = 10, kShapes };
constexpr bool only_up(int shape) { return shape >= kMid192x128 && shape < kShapes; }
constexpr bool is_wide(int shape) { return shape == kWide || shape == kWide224 || shape == kWide192 || shape == kWide160; }
int launch_gemm_wide(int shape, int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s);
int launch_gemm_mid(int shape, int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s);
// Tiles of 16 tm rows of A x 16 tn rows of B (gemm_slim.hpp), B k-contiguous.
constexpr int kSlim = 16;  // a tile shape's number: kSlim + 16 tm + tn
// Three shapes are not built: of 24 million plans (d up to 32768, N up to 200000, workspaces of any size) three took one of them.
// The other large ones are rare too (one plan in 1700 to 500000, and only where d is far from a third of N or the workspace small),
// but the next best shape is 6 % slower there and more.
constexpr bool slim_built(int tm, int tn) {
  return tm >= 1 && tm <= 8 && tn >= 2 && tn <= 8 && !(tm == 8 && (tn == 4 || tn == 7 || tn == 8));
}
int launch_gemm_slim_f16(int tm, int tn, int epi, const GemmArgs& g, hipStream_t s);
int launch_gemm_slim_bf16(int tm, int tn, int epi, const GemmArgs& g, hipStream_t s);
// fp32 kernels (gemm_f32.hip); epi: EPI_*, b_kmajor: B given as [Kk, Nn].
int launch_gemm_f32(int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s);

}  // namespace ci
