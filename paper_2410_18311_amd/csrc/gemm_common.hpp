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
  int k_chunk;     // k range handled by one workgroup along blockIdx.y (a multiple of the k tile)
  float* partial;  // split-K only: [gridDim.y][M][Nn] fp32 partial products (epilogue skipped)
};

// Spreads consecutive tiles over one XCD (workgroup ids go round-robin over the
// 8 XCDs, each with its own L2), so that tiles sharing a B panel share an L2.
__device__ __forceinline__ int xcd_swizzle(int id, int n) {
  if (n % 8 != 0) return id;
  return (id % 8) * (n / 8) + id / 8;
}

// fp32 kernels (gemm_f32.hip); epi: EPI_*, b_kmajor: B given as [Kk, Nn].
int launch_gemm_f32(int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s);

}  // namespace ci
