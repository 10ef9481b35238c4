// Dense prefill FFN (Def. 1 of arXiv 2410.18311): the GEMM of gemm_wide.hip for
// products that are too small for tiles of 256 rows, with the same operand
// layouts in LDS, loads, fragment reads, products and results.
//
// A workgroup is again four waves, one per SIMD.  With 64x64 outputs a wave has 32 products (512 clocks) per 64-k tile, so a
// wait for an LDS read or a load in front of them would be a large share: the fragments of a whole k-tile are
// read one k-tile ahead (two register sets), and the loads run S k-tiles ahead
// through a ring of S stages that takes all of LDS.  One barrier per k-tile.
// What bounds it where the weights come from memory is the load stream, about 117 lines in flight in a compute unit's L1 times their
// latency: 256 x 4096 x 16384, up projection with layers in turn, 46.2 us, 44.4 without products and LDS reads, 30 without
// loads.  What a wave does beside its products counts where the weights are in a cache: with 160 instructions a k-tile, addresses and
// descriptors made for each load, that took 43.4 us, with 100 it takes 39.9 (layers in turn 49.2 -> 47.3; 500 x 4096 x 11008
// gated 109 -> 100 and 126 -> 122.6).
// Tiles of 192 x 128 and 128 x 96, 160 and 192 fill a round where those of powers of two leave a third of the chip idle: up projections
// of 129 to 1536 rows 4 % faster on average over all, 16 % over those that take them.
#include "gemm_tile.hpp"

namespace ci {

namespace {

// 2 x 2 waves of TI x TJ blocks of 16x16: 32 TI rows of A, 32 TJ rows of B.  SwiGLU: a block of B rows is eight gate and eight up
// rows of the same columns.  ONCE: B's lines are the first to leave the caches.
template <class D, bool BNN, int TI, int TJ, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_mid_kernel(GemmArgs g, int epi) {
  using T = typename D::T;
  constexpr int BM = 32 * TI, BN = 32 * TJ;
  static_assert(!BNN || TJ == 2 || TJ == 4 || TJ == 8, "whole k rows in a piece of a k-major B");
  constexpr int STAGE = (BM + BN) * WK * 2;
  constexpr int S = 163840 / STAGE < 8 ? 163840 / STAGE : 8;
  constexpr int NP = TI + TJ;  // 1 KB pieces per wave and k-tile
  static_assert(S >= 3 && (S - 2) * NP < 64, "ring depth against the load counter");
  const bool dual = !BNN && epi == EPI_SWIGLU;
  const int bno = dual ? BN / 2 : BN;  // output columns of a workgroup
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const TileWork w = tile_work(g, BM, bno);
  const int m0 = w.tm * BM, n0 = w.tn * bno;
  const int nk = (w.k_end - w.k_begin + WK - 1) / WK;
  const int tail_chunks = ((w.k_end - w.k_begin) - (nk - 1) * WK) / 8;  // valid 16-byte chunks of the last k-tile

  // Loads as in gemm_wide.hip; a piece of a k-major B is 512 / BN rows of k.
  constexpr int KPP = 512 / BN > 0 ? 512 / BN : 1, CPR = BN / 8;
  const char* Ab = reinterpret_cast<const char*>(g.A) + ((size_t)m0 * g.lda + w.k_begin) * sizeof(T) - 3072;
  const size_t b0 = (BNN ? (size_t)w.k_begin * g.ldb + n0 : (size_t)n0 * g.ldb + w.k_begin) * sizeof(T);
  const bool swap = dual && (TJ * wave & 1);
  const void* Bm[2] = {swap ? g.B1 : g.B0, dual && !swap ? g.B1 : g.B0};  // of the pieces of even and of odd number
  const char* B[2] = {reinterpret_cast<const char*>(Bm[0]) + b0 - 3072, reinterpret_cast<const char*>(Bm[1]) + b0 - 3072};
  uint32_t offA[TI], offB[TJ];
#pragma unroll
  for (int p = 0; p < TI; ++p) {
    const int r = 8 * (TI * wave + p) + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
    offA[p] = (uint32_t)(((size_t)min(r, g.M - 1 - m0) * g.lda + chunk * 8) * sizeof(T)) + (3 - (p & 3)) * 1024;
  }
#pragma unroll
  for (int p = 0; p < TJ; ++p) {
    if (BNN) {
      const int kr = KPP * (TJ * wave + p) + lane / CPR;
      const int col = min(n0 + ((lane % CPR) ^ kmajor_swizzle<BN>(kr)) * 8, g.Nn - 8) - n0;  // Nn is a multiple of 8
      offB[p] = (uint32_t)(((size_t)kr * g.ldb + col) * sizeof(T)) + (3 - (p & 3)) * 1024;
    } else {
      const int r = 8 * (TJ * wave + p) + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
      const int row = dual ? 8 * ((TJ * wave + p) >> 1) + (lane >> 3) : r;
      offB[p] = (uint32_t)(((size_t)min(row, g.Nn - 1 - n0) * g.ldb + chunk * 8) * sizeof(T)) + (3 - (p & 3)) * 1024;
    }
  }
  const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t myA = lds + wave * (TI * 1024), myB = lds + BM * 128 + wave * (TJ * 1024);
  const size_t bytesB = (size_t)(BNN ? g.Kk : g.Nn) * g.ldb * sizeof(T);
  const i32x4 rsrcA = rsrc_until(Ab, reinterpret_cast<const char*>(g.A) + (size_t)g.M * g.lda * sizeof(T));
  const i32x4 rsrcB[2] = {rsrc_until(B[0], reinterpret_cast<const char*>(Bm[0]) + bytesB),
                          rsrc_until(B[1], reinterpret_cast<const char*>(Bm[1]) + bytesB)};
  // k-major: bytes from the last k-tile's first row to the end of the matrix
  const int last_rows = BNN ? (int)((size_t)tail_chunks * 8 * g.ldb * sizeof(T) - (size_t)n0 * sizeof(T)) + 3072 : 0;
  int rangeA = rsrcA[2], rangeB[2] = {rsrcB[0][2], rsrcB[1][2]};
  const uint32_t stepB = (uint32_t)g.ldb * (WK * sizeof(T));  // k-major: from one k-tile to the next
  uint64_t atB = reinterpret_cast<uint64_t>(B[0]);            // k-major: of the k-tile that is loaded
  // The tiles start at different places of k and go round: with all of them at the same one, the rows of B that
  // are on their way lie a power of two apart and use a fraction of the memory channels (16 tokens, 4096 x 16384,
  // down projection 53 -> 33 us; 77 tokens, up 35 -> 31).  Neighbouring column tiles, which share an L2, start
  // next to each other, so that rows of A are read there at about the same time.  A k-major B is read in whole
  // rows by neighbouring tiles in step, and slower (34 -> 44 us) out of step.
  const int rot = BNN ? 0 : (int)((int64_t)w.tn * nk / ((g.Nn + bno - 1) / bno));
  const uint32_t k_bytes = (uint32_t)nk * (WK * sizeof(T));
  uint32_t kofs = (uint32_t)rot * (WK * sizeof(T));           // of the k-tile that is loaded
  auto with_range = [](i32x4 rsrc, int bytes) { return i32x4{rsrc[0], rsrc[1], bytes, rsrc[3]}; };
  auto load = [&](uint32_t place, int p) {  // p < TI: A, else B
    if (p < TI) {
      load_to_lds_at(p & 3, place, offA[p], with_range(rsrcA, rangeA), kofs);
    } else {
      const int q = p - TI;
      const i32x4 r = BNN ? i32x4{(int)(uint32_t)atB, (int)(uint32_t)(atB >> 32), rangeB[0], rsrcB[0][3]} : with_range(rsrcB[q & 1], rangeB[q & 1]);
      load_to_lds_at<ONCE>(q & 3, place, offB[q], r, BNN ? 0u : kofs);
    }
  };
  // On to the next k-tile, behind which there are `behind` more; past the last one nothing is in range and loads read nothing.
  auto step = [&](int behind) {
    asm volatile("s_add_u32 %0, %0, %3\n\ts_cmp_eq_u32 %0, %5\n\ts_cselect_b32 %0, 0, %0\n\ts_cmp_lt_i32 %4, 0\n\t"
                 "s_cselect_b32 %0, 0, %0\n\ts_cselect_b32 %1, 0, %1\n\ts_cselect_b32 %2, 0, %2"
                 : "+s"(kofs), "+s"(rangeA), "+s"(rangeB[1])
                 : "n"(WK * sizeof(T)), "s"(behind), "s"(k_bytes)
                 : "scc");
    if (BNN) {
      atB += stepB;
      asm volatile("s_cmp_eq_u32 %1, 0\n\ts_cselect_b32 %0, %2, -1\n\ts_cmp_lt_i32 %1, 0\n\ts_cselect_b32 %0, 0, %0"
                   : "=&s"(rangeB[0])
                   : "s"(behind), "s"(last_rows)
                   : "scc");
    } else {
      asm volatile("s_cmp_lt_i32 %1, 0\n\ts_cselect_b32 %0, 0, %0" : "+s"(rangeB[0]) : "s"(behind) : "scc");
    }
  };

  f32x4 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Fragments of a whole k-tile, one k-tile ahead; half s: A rows 16 (TI wm + i) + lane % 16, B rows 16 (TJ wn + j) + lane % 16,
  // chunk 4 s + lane / 16.
  const int l15 = lane & 15, quarter = lane >> 4;
  const uint32_t in_row = (uint32_t)((quarter ^ (l15 >> 1)) << 4);
  const uint32_t laneA = (uint32_t)(wm * TI * 16 + l15) * 128 + in_row;
  uint32_t laneB[BNN ? TJ : 1];
  if constexpr (BNN) {
    const int k = 8 * quarter + (l15 >> 2);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      laneB[j] = (uint32_t)(BM * 128 + k * (BN * 2) + (((2 * (wn * TJ + j) + ((lane & 3) >> 1)) ^ kmajor_swizzle<BN>(k)) << 4) + (lane & 1) * 8);
  } else {
    laneB[0] = (uint32_t)(BM + wn * TJ * 16 + l15) * 128 + in_row;
  }
  constexpr int FR = TI + TJ;
  uint4 fa[2][2][TI], fb[2][2][TJ];
  auto read_frag = [&](uint32_t st, int set, int f) {  // f / FR: half, f % FR < TJ: B, else A
    const int s = f / FR, q = f % FR;
    if (q >= TJ) {
      fa[set][s][q - TJ] = *reinterpret_cast<const uint4*>(smem + ((laneA ^ (s << 6)) + st) + (q - TJ) * 2048);
    } else if (!BNN) {
      fb[set][s][q] = *reinterpret_cast<const uint4*>(smem + ((laneB[0] ^ (s << 6)) + st) + q * 2048);
    } else {
      const unsigned char* p = smem + (laneB[BNN ? q : 0] + st) + 32 * s * (BN * 2);
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * (BN * 2)));
      fb[set][s][q] = __builtin_bit_cast(uint4, __builtin_shufflevector(lo, h4, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // K-tile kt is multiplied from registers; its stage is free (everybody read it before the last barrier) and
  // takes k-tile kt + S; the fragments of k-tile kt + 1 are read, and k-tile kt + 2 has to have landed at the end.
  constexpr int MF = 2 * TI * TJ;
  auto tile = [&](auto set_, uint32_t cur, uint32_t nxt, bool ragged) {
    constexpr int set = set_.value;
    constexpr Places<MF, 2 * FR, NP, TI> places;
    if (ragged) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
        if (4 * s + quarter >= tail_chunks) {
#pragma unroll
          for (int i = 0; i < TI; ++i) fa[set][s][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
          for (int j = 0; j < TJ; ++j) fb[set][s][j] = make_uint4(0, 0, 0, 0);
        }
      asm volatile("s_nop 1");  // between such a zero and its product
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t place = 0;
#pragma unroll
    for (int m = 0; m < MF; ++m) {
      const int s = m / (TI * TJ), i = m % (TI * TJ) / TJ, j = m % TJ;
      mfma16_in_place<D>(fb[set][s][j], fa[set][s][i], acc[i][j]);
      if (places.read[m] >= 0) read_frag(nxt, set ^ 1, places.read[m]);
      if (places.place[m] >= 0) place = lds_place(cur + (places.place[m] < TI ? myA + places.place[m] * 1024 : myB + (places.place[m] - TI) * 1024));
      if (places.load[m] >= 0) load(place, places.load[m]);
      __builtin_amdgcn_sched_barrier(0);  // this order
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * NP) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int t = 0; t < S; ++t) {
    uint32_t place = 0;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p < TI ? p % 4 == 0 : (p - TI) % 4 == 0) place = lds_place(t * STAGE + (p < TI ? myA + p * 1024 : myB + (p - TI) * 1024), true);
      load(place, p);
    }
    step(nk - t - 2);
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * NP) : "memory");  // k-tiles 0 and 1
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < 2 * FR; ++f) read_frag(0, 0, f);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);

  const int ragged_at = tail_chunks < 8 ? rot + 1 : 0;
  uint32_t cur = 0;  // stage of the k-tile that is multiplied
  auto after = [](uint32_t stage) { return stage + STAGE == S * STAGE ? 0u : stage + STAGE; };
  int left = nk;
  for (;;) {
    uint32_t nxt = after(cur);
    tile(Const<0>{}, cur, nxt, left == ragged_at);
    if (left == 1) break;
    step(left - S - 2);
    cur = after(nxt);
    tile(Const<1>{}, nxt, cur, left - 1 == ragged_at);
    left -= 2;
    if (left == 0) break;
    step(left - S - 1);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // nothing of mine is still on its way into LDS
  store_blocks<D, TI, TJ>(g, epi, dual, acc, m0 + wm * TI * 16, n0, wn, w.sums, bno, lane);
}

// ONCE: with a build for weights that are not read again
template <class D, bool BNN, int TI, int TJ, bool ONCE = !BNN>
int launch_shape(int epi, const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)(g.full + g.tail * g.splits));
  if (ONCE && g.once) hipLaunchKernelGGL((gemm_mid_kernel<D, BNN, TI, TJ, ONCE>), grid, dim3(256), 0, s, g, epi);
  else hipLaunchKernelGGL((gemm_mid_kernel<D, BNN, TI, TJ, false>), grid, dim3(256), 0, s, g, epi);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, bool BNN>
int launch_typed(int shape, int epi, const GemmArgs& g, hipStream_t s) {
  switch (shape) {
    case kMid128x128: return launch_shape<D, BNN, 4, 4>(epi, g, s);
    case kMid128x256: return launch_shape<D, BNN, 4, 8>(epi, g, s);
    case kMid128x64: return launch_shape<D, BNN, 4, 2>(epi, g, s);
  }
  if constexpr (!BNN) {
    switch (shape) {  // of more than 128 rows only, which read_once() leaves out
      case kMid192x128: return launch_shape<D, BNN, 6, 4, false>(epi, g, s);
      case kMid128x96: return launch_shape<D, BNN, 4, 3, false>(epi, g, s);
      case kMid128x160: return launch_shape<D, BNN, 4, 5, false>(epi, g, s);
      case kMid128x192: return launch_shape<D, BNN, 4, 6, false>(epi, g, s);
    }
  }
  return CI_ERR_UNSUPPORTED;
}

}  // namespace

int launch_gemm_mid(int shape, int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  if (dtype == CI_F16) return b_kmajor ? launch_typed<F16, true>(shape, epi, g, s) : launch_typed<F16, false>(shape, epi, g, s);
  if (dtype == CI_BF16) return b_kmajor ? launch_typed<BF16, true>(shape, epi, g, s) : launch_typed<BF16, false>(shape, epi, g, s);
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
