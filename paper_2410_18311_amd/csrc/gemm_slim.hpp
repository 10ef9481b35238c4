// Dense prefill FFN (Def. 1 of arXiv 2410.18311): the GEMM for 16-bit element types where few rows of tokens meet
// many weights (up to 128 tokens), with the operand layouts in LDS, the loads and the epilogues of gemm_wide.hip.
//
// What bounds such a product is the fill of a compute unit's L1: it keeps about 110 lines of 128 bytes outstanding, whatever the
// ring in LDS holds, and one that misses the L2 in part takes 700 cycles (77 x 4096 x 11008 gated: 10.4 thousand lines in 66
// thousand cycles, 20 bytes per clock, where a stream of hits alone comes at 50).  So a tile should have no
// row of padding, and there should be as many tiles as compute units: tiles are any multiple of 16 in both directions.
// To make that possible the four waves of a workgroup share no rows or columns but the k-tiles: wave w multiplies the
// whole tile for k-tiles w, w + 4, ..., with loads and an LDS ring of its own (18 to 40 KB), so there is no barrier in the
// loop, every fragment is read from LDS once (waves of 64x64 of a 128x128 tile read each twice), and blocks need not
// divide by four.  The four sums are added at the end, in the order of the waves, on the way to the outputs.
// Measured (gated up projection of 4096 x 11008 in bf16, 180 MB of weights; gemm_mid.hip -> here): 16 tokens 36.8 -> 29.8 us
// (6.0 TB/s), 77 tokens 44.8 -> 36.6 us (4.9 TB/s, 230 tiles of 80 x 96 where 172 of 128 x 128 left a third of the chip idle).
#pragma once

#include "gemm_tile.hpp"

namespace ci {

namespace {

constexpr int kLds = 163840;

// TM x TN blocks of 16x16: 16 TM rows of A, 16 TN rows of B.  SwiGLU: a block of B rows is eight gate and eight up rows of
// the same columns.  epi: EPI_*.  ONCE: B's lines are the first to leave the caches.
template <class D, int TM, int TN, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_slim_kernel(GemmArgs g, int epi) {
  using T = typename D::T;
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr int PA = 2 * TM, PB = 2 * TN, NP = PA + PB;  // pieces of 1 KB (8 rows of 128 bytes) of a k-tile
  constexpr int STAGE = NP * 1024;
  constexpr int S = kLds / 4 / STAGE < 3 ? kLds / 4 / STAGE : 3;  // k-tiles in a wave's ring
  static_assert(S >= 1 && S * NP < 64, "ring depth against the load counter");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool dual = epi == EPI_SWIGLU;
  const int bno = dual ? BN / 2 : BN;  // output columns of a workgroup
  const TileWork w = tile_work(g, BM, bno);
  const int m0 = w.tm * BM, n0 = w.tn * bno;
  const int nk = (w.k_end - w.k_begin + WK - 1) / WK;
  const int tail_chunks = ((w.k_end - w.k_begin) - (nk - 1) * WK) / 8;  // valid 16-byte chunks of the last k-tile

  // Loads.  Piece p of a k-contiguous operand is rows 8 p + lane / 8 (clamped at the edge: those outputs are not stored),
  // 16-byte chunk j of row r at j ^ ((r / 2) & 7).  Chunks past the end of k are read from the start of the row and zeroed
  // later.
  const char* Ab = reinterpret_cast<const char*>(g.A) + ((size_t)m0 * g.lda + w.k_begin) * sizeof(T);
  const char* Bb = reinterpret_cast<const char*>(g.B0) + ((size_t)n0 * g.ldb + w.k_begin) * sizeof(T);
  const char* Ub = dual ? reinterpret_cast<const char*>(g.B1) + ((size_t)n0 * g.ldb + w.k_begin) * sizeof(T) : Bb;
  uint32_t offA[PA], offB[PB];
  const int lrow = lane >> 3;
  auto chunk_of = [&](int p) { return (lane & 7) ^ ((4 * p + (lrow >> 1)) & 7); };  // of row 8 p + lrow
#pragma unroll
  for (int p = 0; p < PA; ++p)
    offA[p] = (uint32_t)(((size_t)min(8 * p + lrow, g.M - 1 - m0) * g.lda + chunk_of(p) * 8) * sizeof(T));
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    const int r = dual ? 8 * (p / 2) + lrow : 8 * p + lrow;
    offB[p] = (uint32_t)(((size_t)min(r, g.Nn - 1 - n0) * g.ldb + chunk_of(p) * 8) * sizeof(T));
  }
  // Column tiles start at different places of k, as in gemm_mid.hip.
  const int rot = (int)((int64_t)w.tn * nk / ((g.Nn + bno - 1) / bno));
  auto place = [&](int n) {  // the k-tile that is this wave's number n
    const int t = min(wave + 4 * n, nk - 1) + rot;
    return t >= nk ? t - nk : t;
  };
  unsigned char* ring = smem + wave * (S * STAGE);
  // the way back to the start of the row for a chunk past the end, by the parity of the piece
  const uint32_t back[2] = {chunk_of(0) >= tail_chunks ? (uint32_t)(chunk_of(0) * 8 * sizeof(T)) : 0u,
                            chunk_of(1) >= tail_chunks ? (uint32_t)(chunk_of(1) * 8 * sizeof(T)) : 0u};
  auto load_piece = [&](unsigned char* st, int t, int p) {  // p < PA: A, else B
    const uint32_t past = t == nk - 1 ? back[p & 1] : 0u;  // the parities of p and p - PA are the same
    const size_t k = (size_t)t * (WK * sizeof(T));
    if (p < PA) load_to_lds<false>(st + p * 1024, offA[p] - past, rsrc_at(Ab + k));
    else load_to_lds<ONCE>(st + p * 1024, offB[p - PA] - past, rsrc_at((dual && (p & 1) ? Ub : Bb) + k));
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int l15 = lane & 15, quarter = lane >> 4;
  // fragments of a whole k-tile, or of half of one where 256 registers of sums leave no room
  constexpr int SETS = TM * TN > 56 ? 1 : 2;
  uint4 fa[SETS][TM], fb[SETS][TN];
  auto read_frags = [&](const unsigned char* st, int s, int f) {
    const unsigned char* sb = st + BM * 128;
    const int sw = ((4 * s + quarter) ^ (l15 >> 1)) << 4;
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[f][j] = *reinterpret_cast<const uint4*>(sb + (16 * j + l15) * 128 + sw);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[f][i] = *reinterpret_cast<const uint4*>(st + (16 * i + l15) * 128 + sw);
  };

#pragma unroll
  for (int n = 0; n < S; ++n)
#pragma unroll
    for (int p = 0; p < NP; ++p) load_piece(ring + n * STAGE, place(n), p);

  const int mine = (nk - wave + 3) >> 2;  // k-tiles of this wave
  int slot = 0;
  for (int n = 0; n < mine; ++n) {
    unsigned char* st = ring + slot * STAGE;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * NP) : "memory");  // all but the k-tiles behind it
    const bool ragged = tail_chunks < 8 && place(n) == nk - 1;
    auto clear = [&](int f, int s) {
      if (ragged && 4 * s + quarter >= tail_chunks) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[f][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[f][j] = make_uint4(0, 0, 0, 0);
      }
    };
    const int t = place(n + S);
    constexpr int HF = TM * TN;  // products of half a k-tile
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      constexpr int both = SETS == 2;
      if (s == 0 || !both) {
        read_frags(st, s, s & (SETS - 1));
        if (both) read_frags(st, 1, 1);
        clear(s & (SETS - 1), s);
        if (both) clear(1, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read whole, the stage takes k-tile n + S
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int m = 0; m < HF; ++m) {
        const int f = s & (SETS - 1), i = m / TN, j = m % TN;
        acc[i][j] = mfma16<D>(fb[f][j], fa[f][i], acc[i][j]);
        if (s == SETS % 2) {  // the loads go out between the first products after that
          const int p0 = m * NP / HF, p1 = (m + 1) * NP / HF;
#pragma unroll
          for (int p = p0; p < p1; ++p) load_piece(st, t, p);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    slot = slot + 1 == S ? 0 : slot + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of mine is still on its way into LDS
  __syncthreads();

  // Sums of the waves, RC rows at a time: element v of lane l is row l % 16, column 4 (l / 16) + v of a block (B's
  // fragment is the first operand).  PITCH: eight neighbouring rows lie in different banks.
  constexpr int PITCH = BN + 4;
  constexpr int FIT = kLds / (4 * PITCH * 4) / 16;
  constexpr int IC = FIT < TM ? FIT : TM;  // blocks of rows at a time
  float* part = reinterpret_cast<float*>(smem);
  const int quads = bno / 4;
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += IC) {
    if (i0 > 0) __syncthreads();
#pragma unroll
    for (int i = i0; i < (i0 + IC < TM ? i0 + IC : TM); ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        *reinterpret_cast<f32x4*>(part + ((wave * IC + i - i0) * 16 + l15) * PITCH + 16 * j + 4 * quarter) = acc[i][j];
    __syncthreads();
    const int rows = min(16 * (TM - i0 < IC ? TM - i0 : IC), g.M - m0 - 16 * i0);
    for (int e = tid; e < rows * quads; e += 256) {
      const int r = e / quads, q = e % quads, col = n0 + 4 * q;
      if (col >= g.Nn) continue;  // Nn is a multiple of 8: a quad is inside or outside as a whole
      // SwiGLU: columns 8 b .. 8 b + 7 are gate rows 16 b .. and up rows 16 b + 8 .. of the tile
      const int c = dual ? 16 * (q >> 1) + 4 * (q & 1) : 4 * q;
      const float* src = part + r * PITCH + c;
      f32x4 z = *reinterpret_cast<const f32x4*>(src), u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 1; v < 4; ++v) z += *reinterpret_cast<const f32x4*>(src + v * IC * 16 * PITCH);
      if (dual) {
        u = *reinterpret_cast<const f32x4*>(src + 8);
#pragma unroll
        for (int v = 1; v < 4; ++v) u += *reinterpret_cast<const f32x4*>(src + v * IC * 16 * PITCH + 8);
      }
      const int row = m0 + 16 * i0 + r;
      if (w.sums) {
        *reinterpret_cast<f32x4*>(w.sums + (ptrdiff_t)row * bno + col) = z;
        continue;
      }
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (g.bias) {
#pragma unroll
        for (int k = 0; k < 4; ++k) bv[k] = to_float<D>(reinterpret_cast<const T*>(g.bias)[col + k]);
      }
      const size_t o = (size_t)row * g.ldo + col;
      if (dual) store_quad<D, EPI_SWIGLU>(g, z, u, bv, o);
      else if (epi == EPI_RELU) store_quad<D, EPI_RELU>(g, z, u, bv, o);
      else store_quad<D, EPI_LINEAR>(g, z, u, bv, o);
    }
  }
}

template <class D, int TM, int TN>
int launch_shape(int epi, const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)(g.full + g.tail * g.splits));
  if (g.once) hipLaunchKernelGGL((gemm_slim_kernel<D, TM, TN, true>), grid, dim3(256), 0, s, g, epi);
  else hipLaunchKernelGGL((gemm_slim_kernel<D, TM, TN, false>), grid, dim3(256), 0, s, g, epi);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, int TM, int TN>
int launch_built(int epi, const GemmArgs& g, hipStream_t s) {
  if constexpr (slim_built(TM, TN)) return launch_shape<D, TM, TN>(epi, g, s);
  else return CI_ERR_UNSUPPORTED;
}

template <class D, int TM>
int launch_tn(int tn, int epi, const GemmArgs& g, hipStream_t s) {
  switch (tn) {
    case 2: return launch_built<D, TM, 2>(epi, g, s);
    case 3: return launch_built<D, TM, 3>(epi, g, s);
    case 4: return launch_built<D, TM, 4>(epi, g, s);
    case 5: return launch_built<D, TM, 5>(epi, g, s);
    case 6: return launch_built<D, TM, 6>(epi, g, s);
    case 7: return launch_built<D, TM, 7>(epi, g, s);
    case 8: return launch_built<D, TM, 8>(epi, g, s);
  }
  return CI_ERR_UNSUPPORTED;
}

template <class D>
int launch_tm(int tm, int tn, int epi, const GemmArgs& g, hipStream_t s) {
  switch (tm) {
    case 1: return launch_tn<D, 1>(tn, epi, g, s);
    case 2: return launch_tn<D, 2>(tn, epi, g, s);
    case 3: return launch_tn<D, 3>(tn, epi, g, s);
    case 4: return launch_tn<D, 4>(tn, epi, g, s);
    case 5: return launch_tn<D, 5>(tn, epi, g, s);
    case 6: return launch_tn<D, 6>(tn, epi, g, s);
    case 7: return launch_tn<D, 7>(tn, epi, g, s);
    case 8: return launch_tn<D, 8>(tn, epi, g, s);
  }
  return CI_ERR_UNSUPPORTED;
}

}  // namespace

}  // namespace ci
