// Dense prefill FFN (Def. 1 of arXiv 2410.18311): the GEMM of gemm_wide.hip for
// products that are too small for its 256x256 tiles, with the same operand
// layouts in LDS, loads, fragment reads and epilogue.
//
// A workgroup is again four waves, one per SIMD.  With 64x64 outputs a wave has
// only 16 MFMAs (512 clocks) per 64-k tile, so a wait for an LDS read or a load
// in front of them would be a large share: the fragments of a whole k-tile are
// read one k-tile ahead (two register sets), and the loads run S k-tiles ahead
// through a ring of S stages that takes all of LDS.  One barrier per k-tile.
#include "gemm_tile.hpp"

namespace ci {

namespace {

// WM x WN waves of TI x TJ blocks of 32x32.  ONCE: B's lines are the first to leave the caches.
template <class D, int EPI, bool BNN, int WM, int WN, int TI, int TJ, bool ONCE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_mid_kernel(GemmArgs g) {
  using T = typename D::T;
  constexpr bool DUAL = (EPI == EPI_SWIGLU);
  static_assert(!(BNN && DUAL), "k-major B is only needed for the down projection");
  static_assert(WM * WN == 4 && (!DUAL || TJ % 2 == 0), "four waves; gate and up blocks in one wave");
  constexpr int BM = WM * TI * 32, BN = WN * TJ * 32;  // rows of the A and B images
  constexpr int BNO = DUAL ? BN / 2 : BN;              // output columns of a workgroup
  constexpr int STAGE = (BM + BN) * WK * 2;
  constexpr int S = 163840 / STAGE < 8 ? 163840 / STAGE : 8;
  constexpr int PA = BM / 32, PB = BN / 32, NP = PA + PB;  // 1 KB pieces per wave and k-tile
  static_assert(S >= 3 && (S - 2) * NP < 64, "ring depth against the load counter");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * STAGE];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const TileWork w = tile_work(g, BM, BNO);
  const int m0 = w.tm * BM, n0 = w.tn * BNO;
  const int nk = (w.k_end - w.k_begin + WK - 1) / WK;
  const int tail_chunks = ((w.k_end - w.k_begin) - (nk - 1) * WK) / 8;  // valid 16-byte chunks of the last k-tile

  // Loads: piece p of a k-contiguous operand is rows 32 p + 8 wave + lane / 8 (clamped at the edge: those
  // outputs are not stored); of a k-major B it is 512 / BN rows of k.  Chunks past the end of k are read from
  // the start of the row and zeroed later.
  const char* Ab = reinterpret_cast<const char*>(g.A) + ((size_t)m0 * g.lda + w.k_begin) * sizeof(T);
  const char* Bb = BNN ? reinterpret_cast<const char*>(g.B0) + ((size_t)w.k_begin * g.ldb + n0) * sizeof(T)
                       : reinterpret_cast<const char*>(g.B0) + ((size_t)n0 * g.ldb + w.k_begin) * sizeof(T);
  const char* Ub = DUAL ? reinterpret_cast<const char*>(g.B1) + ((size_t)n0 * g.ldb + w.k_begin) * sizeof(T) : Bb;
  constexpr int CPR = BN / 8;        // k-major: 16-byte chunks of a row of k
  constexpr int RPP = 64 / CPR;      // k-major: rows of k per piece
  auto swz = [](int k) { return BN >= 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; };  // k-major: four rows x 64 bytes in all banks
  uint32_t offA[PA], offB[PB];
  const int lrow = 8 * wave + (lane >> 3);
  const int chunk = (lane & 7) ^ ((lrow >> 1) & 7);
  const int krow = wave * RPP + lane / CPR;
#pragma unroll
  for (int p = 0; p < PA; ++p)
    offA[p] = (uint32_t)(((size_t)min(32 * p + lrow, g.M - 1 - m0) * g.lda + chunk * 8) * sizeof(T));
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    if (BNN) {
      const int col = min(n0 + ((lane % CPR) ^ swz(krow)) * 8, g.Nn - 8) - n0;  // Nn is a multiple of 8
      offB[p] = (uint32_t)(((size_t)(4 * p * RPP + krow) * g.ldb + col) * sizeof(T));
    } else {
      const int r = DUAL ? 32 * (p % (PB / 2 > 0 ? PB / 2 : 1)) + lrow : 32 * p + lrow;
      offB[p] = (uint32_t)(((size_t)min(r, g.Nn - 1 - n0) * g.ldb + chunk * 8) * sizeof(T));
    }
  }
  // The tiles start at different places of k and go round: with all of them at the same one, the rows of B that
  // are on their way lie a power of two apart and use a fraction of the memory channels (16 tokens, 4096 x 16384,
  // down projection 53 -> 33 us; 77 tokens, up 35 -> 31).  Neighbouring column tiles, which share an L2, start
  // next to each other, so that rows of A are read there at about the same time.  A k-major B is read in whole
  // rows by neighbouring tiles in step, and slower (34 -> 44 us) out of step.
  const int rot = BNN ? 0 : (int)((int64_t)w.tn * nk / ((g.Nn + BNO - 1) / BNO));
  auto place = [&](int kt) {  // the k-tile that is taken as number kt
    const int t = min(kt, nk - 1) + rot;
    return t >= nk ? t - nk : t;
  };
  const size_t stepB = BNN ? (size_t)WK * g.ldb * sizeof(T) : (size_t)WK * sizeof(T);
  const uint32_t tail_back = chunk >= tail_chunks ? (uint32_t)(chunk * 8 * sizeof(T)) : 0u;
  auto load_piece = [&](unsigned char* st, int kt, int p) {  // p < PA: A, else B
    const int t = place(kt);
    uint32_t off;
    const char* base;
    if (p < PA) {
      off = offA[p] - (t == nk - 1 ? tail_back : 0u);
      base = Ab + (size_t)t * (WK * sizeof(T));
    } else {
      const int q = p - PA;
      off = offB[q];
      if (BNN) {
        const int kr = 4 * q * RPP + krow;
        if (t == nk - 1 && kr >= tail_chunks * 8) off -= (uint32_t)((size_t)kr * g.ldb * sizeof(T));
      } else {
        off -= t == nk - 1 ? tail_back : 0u;
      }
      base = ((DUAL && q >= PB / 2) ? Ub : Bb) + (size_t)t * stepB;
    }
    if (p < PA) load_to_lds(st + (4 * p + wave) * 1024, off, rsrc_at(base));
    else load_to_lds<ONCE>(st + (BM / 8 + 4 * (p - PA) + wave) * 1024, off, rsrc_at(base));
  };

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int l31 = lane & 31, hi = lane >> 5;
  const int trow = 8 * hi + ((lane & 15) >> 2);
  uint4 fa[2][4][TI], fb[2][4][TJ];
  auto read_frag = [&](const unsigned char* st, int set, int s, int f) {  // f < TI: A, else B
    const int sw = ((2 * s + hi) ^ ((l31 >> 1) & 7)) << 4;
    const unsigned char* sb = st + BM * 128;
    const int j = f - TI;
    if (f < TI) {
      fa[set][s][f] = *reinterpret_cast<const uint4*>(st + (wm * TI * 32 + l31) * 128 + sw + f * 4096);
    } else if (!BNN) {
      const int r = DUAL ? (j / (TJ / 2 > 0 ? TJ / 2 : 1)) * (BN / 2) + (wn * (TJ / 2) + j % (TJ / 2 > 0 ? TJ / 2 : 1)) * 32
                         : (wn * TJ + j) * 32;
      fb[set][s][j] = *reinterpret_cast<const uint4*>(sb + l31 * 128 + sw + r * 128);
    } else {
      const int c = ((wn * TJ + j) * 4 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ swz((lane & 15) >> 2);
      const unsigned char* p = sb + (16 * s + trow) * (BN * 2) + c * 16 + (lane & 1) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * (BN * 2)));
      fb[set][s][j] = __builtin_bit_cast(uint4, __builtin_shufflevector(lo, h4, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // waits: all but the newest (S - 2) k-tiles' loads have landed, all of my LDS reads are done
  constexpr int kNewest = (S - 2) * NP;
  constexpr int kWait = 0x0070 | (kNewest & 15) | ((kNewest >> 4) << 14);
#pragma unroll
  for (int t = 0; t < S; ++t)
#pragma unroll
    for (int p = 0; p < NP; ++p) load_piece(smem + t * STAGE, t, p);
  __builtin_amdgcn_s_waitcnt(kWait);  // k-tiles 0 and 1
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int f = 0; f < TI + TJ; ++f) read_frag(smem, 0, s, f);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);

  // K-tile kt is multiplied from registers; its stage is free (everybody read it before the last barrier) and
  // takes k-tile kt + S; the fragments of k-tile kt + 1 are read, in the first three of the four k-steps, so
  // that they have arrived at the end, where k-tile kt + 2 has to have landed.
  constexpr int MF = TI * TJ, RD = 4 * (TI + TJ);
  constexpr int kMost = (RD + 3 * MF - 1) / (3 * MF) > (NP + 4 * MF - 1) / (4 * MF) ? (RD + 3 * MF - 1) / (3 * MF) : (NP + 4 * MF - 1) / (4 * MF);
  int cur = 0;  // stage of k-tile kt
  for (int kt0 = 0; kt0 < nk; kt0 += 2) {
#pragma unroll
    for (int set = 0; set < 2; ++set) {
      const int kt = kt0 + set;
      const int nxt = cur + 1 == S ? 0 : cur + 1;
      unsigned char* sc = smem + cur * STAGE;
      const unsigned char* sn = smem + nxt * STAGE;
      if (kt >= nk || (tail_chunks < 8 && place(kt) == nk - 1)) {  // a padding k-tile is all zeros, the last may not be full
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (2 * s + hi >= tail_chunks || kt >= nk) {
#pragma unroll
            for (int i = 0; i < TI; ++i) fa[set][s][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < TJ; ++j) fb[set][s][j] = make_uint4(0, 0, 0, 0);
          }
      }
#pragma unroll
      for (int m = 0; m < 4 * MF; ++m) {
        const int s = m / MF, i = (m % MF) / TJ, j = m % TJ;
        acc[i][j] = mfma<D>(fa[set][s][i], fb[set][s][j], acc[i][j]);
        // reads spread over the first three quarters, loads over all of it
        const int r0 = (m * RD + 3 * MF - 1) / (3 * MF), r1 = ((m + 1) * RD + 3 * MF - 1) / (3 * MF);
        const int p0 = (m * NP + 4 * MF - 1) / (4 * MF), p1 = ((m + 1) * NP + 4 * MF - 1) / (4 * MF);
#pragma unroll
        for (int q = 0; q < kMost; ++q) {
          if (r0 + q < r1 && r0 + q < RD) read_frag(sn, set ^ 1, (r0 + q) / (TI + TJ), (r0 + q) % (TI + TJ));
          if (p0 + q < p1) load_piece(sc, kt + S, p0 + q);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(kWait);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      cur = nxt;
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // nothing of mine is still on its way into LDS
  __syncthreads();
  constexpr int PITCH = TJ * 32 + 8;
  store_wave<D, EPI, TI, TJ>(g, acc, reinterpret_cast<float*>(smem) + wave * 32 * PITCH, m0 + wm * TI * 32,
                             n0 + wn * (DUAL ? TJ * 16 : TJ * 32), w.sums, BNO, lane);
}

template <class D, int EPI, bool BNN, int WM, int WN, int TI, int TJ>
int launch_shape(const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)(g.full + g.tail * g.splits));
  if (!BNN && g.once)
    hipLaunchKernelGGL((gemm_mid_kernel<D, EPI, BNN, WM, WN, TI, TJ, !BNN>), grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL((gemm_mid_kernel<D, EPI, BNN, WM, WN, TI, TJ, false>), grid, dim3(256), 0, s, g);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, int EPI, bool BNN>
int launch_typed(int shape, const GemmArgs& g, hipStream_t s) {
  switch (shape) {
    case kMid128x128: return launch_shape<D, EPI, BNN, 2, 2, 2, 2>(g, s);
    case kMid128x256: return launch_shape<D, EPI, BNN, 2, 2, 2, 4>(g, s);
    case kMid128x64: return launch_shape<D, EPI, BNN, 4, 1, 1, 2>(g, s);
  }
  return CI_ERR_UNSUPPORTED;
}

template <class D>
int launch_epi(int shape, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  switch (epi) {
    case EPI_RELU: return launch_typed<D, EPI_RELU, false>(shape, g, s);
    case EPI_SWIGLU: return launch_typed<D, EPI_SWIGLU, false>(shape, g, s);
    case EPI_LINEAR:
      return b_kmajor ? launch_typed<D, EPI_LINEAR, true>(shape, g, s) : launch_typed<D, EPI_LINEAR, false>(shape, g, s);
  }
  return CI_ERR_INVALID_ARG;
}

}  // namespace

int launch_gemm_mid(int shape, int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  switch (dtype) {
    case CI_F16: return launch_epi<F16>(shape, epi, b_kmajor, g, s);
    case CI_BF16: return launch_epi<BF16>(shape, epi, b_kmajor, g, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
