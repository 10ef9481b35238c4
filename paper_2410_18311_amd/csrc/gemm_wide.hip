// Dense prefill FFN (Def. 1 of arXiv 2410.18311): the 256x256-tile GEMM for
// 16-bit element types, C[M, Nn] = A[M, Kk] * B^T with the fused epilogues of
// gemm_mfma.hip.
//
// What bounds a tiled MFMA kernel here is LDS traffic next to the matrix cores:
// per 64-k tile the fragments of 2x2 waves of 128x128 outputs take 131 KB of
// LDS reads and the two operand tiles 64 KB of writes, 1536 clocks at 128 bytes
// per clock against 2048 clocks of MFMAs (eight waves of 128x64 would read half
// as much again and come out level).  So four waves, one per SIMD, with the
// accumulators in 256 registers each; and since a wave then has nobody to hide
// its waits behind, nothing in its instruction stream may wait:
//   - the operand tiles go from global memory straight into LDS, as buffer loads
//     with a 32-bit offset per lane (with 64-bit addresses an issuing wave stood
//     still for longer: 1325 against 1374 TFLOP/s at 4096 x 36864 x 9216), in rows
//     of 128 bytes (rows of 64 bytes cost twice the tag look-ups of the L1:
//     1156 TFLOP/s);
//   - fragments are read TWO k-steps (of 16) before they are multiplied, so that
//     the last fragment of a k-tile is read in its second step, and the one
//     barrier per k-tile sits there;
//   - LDS holds five operand tiles of 32 KB: A and B of the k-tile that is
//     multiplied and of the next one, and room for A of the one after, so that
//     four loads go out in every k-step and have a k-tile's time to arrive;
//   - between two MFMAs at most one LDS read and one load are issued, in the order
//     written.
// Measured at 4096 x 9216 x 36864 in bf16: 1559 TFLOP/s without the stores of the
// results (torch's library: 1341 to 1532 for the same two products); in fp16 the
// matrix pipes are busy 81 % (up) and 89 % (down) of the cycles in which a compute unit
// has work, at 1.5 and 1.3 GHz under the profiler: the clock is the limit then.
//
// LDS layout: the destination of such a load cannot be padded, so the 16-byte
// chunks are permuted instead, on the global side.  k-contiguous operand: rows of
// 128 bytes, chunk j of row r at j ^ ((r / 2) & 7) (any 16 rows of one chunk then
// touch every bank once).  k-major B (a neuron-major down matrix): rows of 512
// bytes (one k, 256 columns), chunk j of row k at j ^ 4 (k & 3), read through
// ds_read_b64_tr_b16, whose 32 lanes then cover four rows x 64 bytes in 256
// different bytes of the banks.
#include "gemm_tile.hpp"

namespace ci {

namespace {

constexpr int WT = 256;                // output rows and B rows (k-major: columns) of a workgroup
constexpr int kOperand = WT * WK * 2;  // bytes of one operand tile
constexpr int kUnits = 5;              // operand tiles in LDS: all of its 160 KB

// TAIL: the last k-tile is not full; chunks past the end of k are read from the start of the row instead and
// zeroed, in both operands, before they are multiplied.
template <class D, int EPI, bool BNN, bool TAIL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_wide_kernel(GemmArgs g) {
  using T = typename D::T;
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  static_assert(!(BNN && DUAL), "k-major B is only needed for the down projection");
  constexpr int BNO = DUAL ? WT / 2 : WT;  // output columns of a workgroup
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kUnits * kOperand];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const TileWork w = tile_work(g, WT, BNO);
  const int m0 = w.tm * WT, n0 = w.tn * BNO;
  const int k_begin = w.k_begin, k_end = w.k_end;
  const int nk = (k_end - k_begin + WK - 1) / WK;
  const int tail_chunks = TAIL ? ((k_end - k_begin) - (nk - 1) * WK) / 8 : 8;  // valid 16-byte chunks of the last k-tile
  (void)tail_chunks;

  // Loads: piece p of a k-contiguous operand is rows 32 p + 8 wave + lane / 8 (rows past the edge are
  // clamped: they only feed outputs that are not stored); of a k-major B it is k rows 8 p + 2 wave +
  // lane / 32.  Uniform bases plus 32-bit byte offsets (256 rows of an operand span less than 4 GB).
  const char* Ab = reinterpret_cast<const char*>(g.A) + ((size_t)m0 * g.lda + k_begin) * sizeof(T);
  const char* Bb = BNN ? reinterpret_cast<const char*>(g.B0) + ((size_t)k_begin * g.ldb + n0) * sizeof(T)
                       : reinterpret_cast<const char*>(g.B0) + ((size_t)n0 * g.ldb + k_begin) * sizeof(T);
  const char* Ub = DUAL ? reinterpret_cast<const char*>(g.B1) + ((size_t)n0 * g.ldb + k_begin) * sizeof(T) : Bb;
  uint32_t offA[8], offB[8];
  const int lrow = 8 * wave + (lane >> 3);
  const int chunk = (lane & 7) ^ ((lrow >> 1) & 7);  // the same in all pieces: 32 p does not reach bits 1 .. 3
  const int bchunk = (lane & 31) ^ ((2 * (wave & 1) + (lane >> 5)) << 2);  // k-major: k & 3 of row 8 p + 2 wave + lane / 32
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    offA[p] = (uint32_t)(((size_t)min(32 * p + lrow, g.M - 1 - m0) * g.lda + chunk * 8) * sizeof(T));
    if (BNN) {
      const int col = min(n0 + bchunk * 8, g.Nn - 8) - n0;  // Nn is a multiple of 8
      offB[p] = (uint32_t)(((size_t)(8 * p + 2 * wave + (lane >> 5)) * g.ldb + col) * sizeof(T));
    } else {
      const int r = DUAL ? 32 * (p & 3) + lrow : 32 * p + lrow;
      offB[p] = (uint32_t)(((size_t)min(r, g.Nn - 1 - n0) * g.ldb + chunk * 8) * sizeof(T));
    }
  }
  const size_t stepB = BNN ? (size_t)WK * g.ldb * sizeof(T) : (size_t)WK * sizeof(T);

  // piece p of operand A / B of k-tile kt into LDS unit `unit`: 1 KB per wave, 8 rows of 128 bytes, k-major 2
  // rows of 512
  auto load_a = [&](int unit, int kt, int p) {
    const int t = min(kt, nk - 1);
    uint32_t off = offA[p];
    if (TAIL && t == nk - 1 && chunk >= tail_chunks) off -= (uint32_t)(chunk * 8 * sizeof(T));
    load_to_lds(smem + unit * kOperand + (4 * p + wave) * 1024, off, rsrc_at(Ab + (size_t)t * (WK * sizeof(T))));
  };
  auto load_b = [&](int unit, int kt, int p) {
    const int t = min(kt, nk - 1);
    uint32_t off = offB[p];
    if (TAIL && t == nk - 1) {
      if (BNN) {
        const int kr = 8 * p + 2 * wave + (lane >> 5);
        if (kr >= tail_chunks * 8) off -= (uint32_t)((size_t)kr * g.ldb * sizeof(T));
      } else if (chunk >= tail_chunks) {
        off -= (uint32_t)(chunk * 8 * sizeof(T));
      }
    }
    load_to_lds(smem + unit * kOperand + (4 * p + wave) * 1024, off,
                rsrc_at(((DUAL && p >= 4) ? Ub : Bb) + (size_t)t * stepB));
  };

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Fragments of k-step s: A rows 128 wm + 32 i + l31; B rows 128 wn + 32 j + l31, SwiGLU: gate rows
  // 64 wn + 32 j (j < 2) and up rows 128 + 64 wn + 32 (j - 2); chunk 2 s + lane / 32.
  const int l31 = lane & 31, hi = lane >> 5;
  const int trow = 8 * hi + ((lane & 15) >> 2);  // k-major: k row of this lane's transposing read, upper half + 4
  uint4 fa[4][4], fb[4][4];
  auto read_frag = [&](const unsigned char* sa, const unsigned char* sb, int s, int f) {  // f: 0 .. 3 A, 4 .. 7 B
    const int sw = ((2 * s + hi) ^ ((l31 >> 1) & 7)) << 4;
    const int j = f & 3;
    if (f < 4) {
      fa[s][j] = *reinterpret_cast<const uint4*>(sa + (wm * 128 + l31) * 128 + sw + j * 4096);
    } else if (!BNN) {
      const int r = DUAL ? (j >> 1) * 128 + wn * 64 + (j & 1) * 32 : wn * 128 + j * 32;
      fb[s][j] = *reinterpret_cast<const uint4*>(sb + l31 * 128 + sw + r * 128);
    } else {
      const int c = (wn * 16 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) + ((j ^ ((lane & 15) >> 2)) << 2);
      const unsigned char* p = sb + (16 * s + trow) * 512 + c * 16 + (lane & 1) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * 512));
      fb[s][j] = __builtin_bit_cast(uint4, __builtin_shufflevector(lo, h4, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // prologue: k-tiles 0 and 1 on their way, the first two k-steps' fragments read
#pragma unroll
  for (int t = 0; t < 2; ++t) {
#pragma unroll
    for (int p = 0; p < 8; ++p) load_a(2 * t, t, p);
#pragma unroll
    for (int p = 0; p < 8; ++p) load_b(2 * t + 1, t, p);
  }
  __builtin_amdgcn_s_waitcnt(0x4F70);  // vmcnt(16): k-tile 0 has landed
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < 16; ++f) read_frag(smem, smem + kOperand, f >> 3, f & 7);

  // K-tile kt lies in units ua, ua + 1 (modulo 5), k-tile kt + 1 in the two after them, the fifth is free.
  // Steps 0 and 1 read the fragments of steps 2 and 3 and send A of k-tile kt + 2 into the free unit; then
  // everybody has read all of k-tile kt and k-tile kt + 1 has landed (all but the 8 newest loads), so steps 2
  // and 3 read from k-tile kt + 1 and send B of k-tile kt + 2 into unit ua.
  int ua = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const int ub = ua + 1 >= kUnits ? ua + 1 - kUnits : ua + 1;
    const int na = ua + 2 >= kUnits ? ua + 2 - kUnits : ua + 2;
    const int nb = ua + 3 >= kUnits ? ua + 3 - kUnits : ua + 3;
    const int uf = ua + 4 >= kUnits ? ua + 4 - kUnits : ua + 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const unsigned char* sa = smem + (s < 2 ? ua : na) * kOperand;
      const unsigned char* sb = smem + (s < 2 ? ub : nb) * kOperand;
      if (TAIL && kt == nk - 1 && 2 * s + hi >= tail_chunks) {
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[s][i] = fb[s][i] = make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        acc[m >> 2][m & 3] = mfma<D>(fa[s][m >> 2], fb[s][m & 3], acc[m >> 2][m & 3]);
        if ((m & 1) == 0) read_frag(sa, sb, (s + 2) & 3, m >> 1);
        if ((m & 3) == 1) {
          if (s < 2) load_a(uf, kt + 2, 4 * s + (m >> 2));
          else load_b(ua, kt + 2, 4 * (s - 2) + (m >> 2));
        }
        __builtin_amdgcn_sched_barrier(0);  // this order: one LDS read or one load between two MFMAs
      }
      if (s == 1) {
        __builtin_amdgcn_s_waitcnt(0x0078);  // vmcnt(8), lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    ua = na;
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // nothing of mine is still on its way into LDS
  __syncthreads();  // the units are free: each wave turns its outputs to rows in one of its own
  store_wave<D, EPI, 4, 4>(g, acc, reinterpret_cast<float*>(smem + wave * kOperand), m0 + wm * 128,
                           n0 + wn * (DUAL ? 64 : 128), w.sums, BNO, lane);
}

template <class D, int EPI, bool BNN>
int launch_typed(const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)(g.full + g.tail * g.splits));
  if (g.Kk % WK == 0) hipLaunchKernelGGL((gemm_wide_kernel<D, EPI, BNN, false>), grid, dim3(256), 0, s, g);
  else hipLaunchKernelGGL((gemm_wide_kernel<D, EPI, BNN, true>), grid, dim3(256), 0, s, g);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D>
int launch_epi(int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  switch (epi) {
    case EPI_RELU: return launch_typed<D, EPI_RELU, false>(g, s);
    case EPI_SWIGLU: return launch_typed<D, EPI_SWIGLU, false>(g, s);
    case EPI_LINEAR:
      return b_kmajor ? launch_typed<D, EPI_LINEAR, true>(g, s) : launch_typed<D, EPI_LINEAR, false>(g, s);
  }
  return CI_ERR_INVALID_ARG;
}

}  // namespace

int launch_gemm_wide(int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  switch (dtype) {
    case CI_F16: return launch_epi<F16>(epi, b_kmajor, g, s);
    case CI_BF16: return launch_epi<BF16>(epi, b_kmajor, g, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
