// Dense prefill FFN (Def. 1 of arXiv 2410.18311): the GEMM for 16-bit element types
// with tiles of 256 rows, C[M, Nn] = A[M, Kk] * B^T with the fused epilogues of gemm_mfma.hip.
//
// What bounds a tiled MFMA kernel here is LDS traffic next to the matrix cores, and the power of both:
// per 64-k tile the fragments of 2x2 waves of 128x128 outputs take 131 KB of
// LDS reads and the two operand tiles 64 KB of writes, 1536 clocks at 128 bytes
// per clock against 2048 clocks of MFMAs (eight waves of 128x64 would read half
// as much again and come out level).  So four waves, one per SIMD, with the
// accumulators in 256 registers each; and since a wave then has nobody to hide
// its waits behind, nothing in its instruction stream may wait:
//   - products of 16x16x32: per multiplication they read and write half as many sums as those of 32x32x16, and the chip then
//     holds 1.5 to 1.7 GHz at 4096 x 9216 x 36864 where it held 1.3 to 1.5 (all of that layer 4210 -> 3955 us, 1024 x 5120 x 13824
//     gated 383 -> 365; with shapes of 160 to 224 columns for its rounds 352);
//   - they are written out, sums in place: the compiler gives a product's result other registers than its
//     sum has and moves them back, up to one move a product (the build looks for what it then no longer does, isa_check.py);
//   - the operand tiles go from global memory straight into LDS, as buffer loads
//     with a 32-bit offset per lane (with 64-bit addresses an issuing wave stands
//     still for longer), in rows of 128 bytes (rows of 64 bytes cost twice the tag
//     look-ups of the L1), a constant offset apart for one place in LDS.  Both were
//     measured with 32x32x16 products, at 4096 x 36864 x 9216: 1374 TFLOP/s, 1325 with
//     64-bit addresses, 1156 with rows of 64 bytes;
//   - fragments are read half a k-tile before they are multiplied, and the one barrier per k-tile sits in its middle;
//   - LDS holds five operand tiles of 32 KB: A and B of the k-tile that is
//     multiplied and of the next one, and room for B of the one after;
//   - loads go out evenly, eight in half a k-tile: in bursts of one to two products, for more time to arrive, 1970 -> 2100 us for the
//     larger layer's up projection, and at places of its own for each wave, by branches, 2310.
// What is left of a k-tile of 256 x 256 at 4096 x 9216 x 36864, 1.37 us: 1.0 us the products with nothing beside them, 0.14 the
// LDS reads, 0.25 the loads, mostly as lower clock (the same k-tile again and again takes as long, one of zeros 0.95).
// A tile of fewer columns takes its share of the time: 256, 224, 192 and 160 columns 126, 112, 98 and 84 us in one round of 5120 k.
//
// LDS layout: the destination of such a load cannot be padded, so the 16-byte
// chunks are permuted instead, on the global side.  k-contiguous operand: rows of
// 128 bytes, chunk j of row r at j ^ ((r / 2) & 7) (any 16 rows of one chunk then
// touch every bank once).  k-major B (a neuron-major down matrix): rows of 512
// bytes (one k, 256 columns or fewer), chunk j of row k at j ^ 4 (k & 3) ^ 2 (k / 8 & 1), read through
// ds_read_b64_tr_b16, whose 32 lanes then cover eight rows x 32 bytes in 256
// different bytes of the banks.
#include "gemm_tile.hpp"

namespace ci {

namespace {

constexpr int WT = 256;                // output rows of a workgroup
constexpr int kOperand = WT * WK * 2;  // bytes of LDS for one operand tile
constexpr int kUnits = 5;              // operand tiles in LDS: all of its 160 KB

// 2 x 2 waves of 8 x TJ blocks of 16x16: 256 rows of A, 32 TJ rows of B.  SwiGLU: a block of B rows is eight gate and eight up
// rows of the same columns.
template <class D, bool BNN, int TJ>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gemm_wide_kernel(GemmArgs g, int epi) {
  using T = typename D::T;
  constexpr int TI = 8;
  constexpr int BN = 32 * TJ;
  constexpr int PB = BNN ? 8 : TJ;  // 1 KB pieces of B per wave and k-tile (k-major: rows of 512 bytes, whatever BN)
  const bool dual = !BNN && epi == EPI_SWIGLU;
  const int bno = dual ? BN / 2 : BN;  // output columns of a workgroup
  __shared__ __attribute__((aligned(1024))) unsigned char smem[kUnits * kOperand];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const TileWork w = tile_work(g, WT, bno);
  const int m0 = w.tm * WT, n0 = w.tn * bno;
  const int nk = (w.k_end - w.k_begin + WK - 1) / WK;
  const int tail_chunks = ((w.k_end - w.k_begin) - (nk - 1) * WK) / 8;  // valid 16-byte chunks of the last k-tile

  // Loads: piece p of a k-contiguous operand is eight rows, 8 (8 wave + p) + lane / 8 of A and 8 (TJ wave + p) + lane / 8 of B
  // (rows past the edge are clamped: they only feed outputs that are not stored); of a k-major B it is k rows 16 wave + 2 p +
  // lane / 32.  A load adds its constant offset, 1 KB for a piece, to both of its addresses, so that four pieces go by one place
  // in LDS; the lanes' offsets take it back, and 3 KB that the bases lie ahead keep them positive (256 rows of an operand span less
  // than 4 GB).  Chunks past the end of k are whatever follows the row, zero behind the matrix, and are zeroed before
  // they are multiplied.
  const char* Ab = reinterpret_cast<const char*>(g.A) + ((size_t)m0 * g.lda + w.k_begin) * sizeof(T) - 3072;
  const size_t b0 = (BNN ? (size_t)w.k_begin * g.ldb + n0 : (size_t)n0 * g.ldb + w.k_begin) * sizeof(T);
  // SwiGLU: pieces of even rows of eight are the gate's, of odd ones the up matrix's
  const bool swap = dual && (TJ * wave & 1);
  const char* B[2] = {reinterpret_cast<const char*>(swap ? g.B1 : g.B0) + b0 - 3072,
                      reinterpret_cast<const char*>(dual && !swap ? g.B1 : g.B0) + b0 - 3072};
  uint32_t offA[8], offB[PB];
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    const int r = 64 * wave + 8 * p + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
    offA[p] = (uint32_t)(((size_t)min(r, g.M - 1 - m0) * g.lda + chunk * 8) * sizeof(T)) + (3 - (p & 3)) * 1024;
  }
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    if (BNN) {
      const int kr = 16 * wave + 2 * p + (lane >> 5);
      int c = (lane & 31) ^ kmajor_swizzle<256>(kr);
      if (c >= BN / 8) c = 0;                        // no such columns: a chunk that is loaded anyway
      const int col = min(n0 + c * 8, g.Nn - 8) - n0;  // Nn is a multiple of 8
      offB[p] = (uint32_t)(((size_t)kr * g.ldb + col) * sizeof(T)) + (3 - (p & 3)) * 1024;
    } else {
      const int r = 8 * (TJ * wave + p) + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
      const int row = dual ? 8 * ((TJ * wave + p) >> 1) + (lane >> 3) : r;
      offB[p] = (uint32_t)(((size_t)min(row, g.Nn - 1 - n0) * g.ldb + chunk * 8) * sizeof(T)) + (3 - (p & 3)) * 1024;
    }
  }
  const uint32_t lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t myA = lds + wave * 8192, myB = lds + wave * (PB * 1024);
  const char* endA = reinterpret_cast<const char*>(g.A) + (size_t)g.M * g.lda * sizeof(T);
  const size_t bytesB = (size_t)(BNN ? g.Kk : g.Nn) * g.ldb * sizeof(T);
  const i32x4 rsrcA = rsrc_until(Ab, endA);
  // k-major: bytes from the last k-tile's first row to the end of the matrix
  const int last_rows = BNN ? (int)((size_t)tail_chunks * 8 * g.ldb * sizeof(T) - (size_t)n0 * sizeof(T)) + 3072 : 0;
  const i32x4 rsrcB[2] = {rsrc_until(B[0], reinterpret_cast<const char*>(swap ? g.B1 : g.B0) + bytesB),
                    rsrc_until(B[1], reinterpret_cast<const char*>(dual && !swap ? g.B1 : g.B0) + bytesB)};
  int rangeA = rsrcA[2], rangeB[2] = {rsrcB[0][2], rsrcB[1][2]};
  const uint32_t stepB = (uint32_t)g.ldb * (WK * sizeof(T));  // k-major: from one k-tile to the next
  uint32_t kofs = 0;                                          // of the k-tile that is loaded

  uint64_t atB = reinterpret_cast<uint64_t>(B[0]);           // k-major: of the k-tile that is loaded
  auto with_range = [](i32x4 rsrc, int bytes) { return i32x4{rsrc[0], rsrc[1], bytes, rsrc[3]}; };
  auto load_a = [&](uint32_t place, int p) { load_to_lds_at(p & 3, place, offA[p], with_range(rsrcA, rangeA), kofs); };
  auto load_b = [&](uint32_t place, int p) {
    const i32x4 r = BNN ? i32x4{(int)(uint32_t)atB, (int)(uint32_t)(atB >> 32), rangeB[0], rsrcB[0][3]} : with_range(rsrcB[p & 1], rangeB[p & 1]);
    load_to_lds_at(p & 3, place, offB[p], r, BNN ? 0u : kofs);
  };
  // On to the next k-tile, behind which there are `behind` more; past the last one nothing is in range and loads read nothing.
  // (Written out, so that the loop is not taken apart at its last turns: every copy of it would have its own sums' registers.)
  auto step = [&](int behind) {
    asm volatile("s_add_u32 %0, %0, %3\n\ts_cmp_lt_i32 %4, 0\n\ts_cselect_b32 %0, 0, %0\n\ts_cselect_b32 %1, 0, %1\n\ts_cselect_b32 %2, 0, %2"
                 : "+s"(kofs), "+s"(rangeA), "+s"(rangeB[1])
                 : "n"(WK * sizeof(T)), "s"(behind)
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

  // Fragments of half s of a k-tile (32 k): A rows 128 wm + 16 i + lane % 16, B rows 16 (TJ wn + j) + lane % 16, chunk
  // 4 s + lane / 16.
  const int l15 = lane & 15, quarter = lane >> 4;
  const uint32_t in_row = (uint32_t)((quarter ^ (l15 >> 1)) << 4);
  const uint32_t laneA = (uint32_t)(wm * 128 + l15) * 128 + in_row;
  uint32_t laneB[BNN ? TJ : 1];
  if constexpr (BNN) {
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      laneB[j] = (uint32_t)((8 * quarter + (l15 >> 2)) * 512 + (((2 * (wn * TJ + j) + ((lane & 3) >> 1)) ^ kmajor_swizzle<256>(8 * quarter + (l15 >> 2))) << 4) + (lane & 1) * 8);
  } else {
    laneB[0] = (uint32_t)(wn * TJ * 16 + l15) * 128 + in_row;
  }
  uint4 fa[2][TI], fb[2][TJ];
  auto read_frag = [&](uint32_t ua, uint32_t ub, int s, int f) {  // f < TJ: B, else A
    if (f >= TJ) {
      fa[s][f - TJ] = *reinterpret_cast<const uint4*>(smem + ((laneA ^ (s << 6)) + ua) + (f - TJ) * 2048);
    } else if (!BNN) {
      fb[s][f] = *reinterpret_cast<const uint4*>(smem + ((laneB[0] ^ (s << 6)) + ub) + f * 2048);
    } else {
      const unsigned char* p = smem + (laneB[BNN ? f : 0] + ub) + 32 * s * 512;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 h4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * 512));
      fb[s][f] = __builtin_bit_cast(uint4, __builtin_shufflevector(lo, h4, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // K-tile kt lies in units ua and ub, k-tile kt + 1 in na and nb, `spare` is free.  The first half reads the fragments of the
  // second and sends B of k-tile kt + 2, weights that come from memory, into the spare unit; then everybody has read all of
  // k-tile kt and k-tile kt + 1 has landed (all but the newest B), so the second half reads from k-tile kt + 1 and sends A of
  // k-tile kt + 2 into unit ua.
  uint32_t ua = 0, ub = kOperand, na = 2 * kOperand, nb = 3 * kOperand, spare = 4 * kOperand;
  constexpr int MF = TI * TJ;
  auto half = [&](auto s_, bool ragged) {
    constexpr int s = s_.value;
    constexpr Places<MF, TI + TJ, s == 0 ? PB : 8> places;
    if (ragged) {
      if (4 * s + quarter >= tail_chunks) {
#pragma unroll
        for (int i = 0; i < TI; ++i) fa[s][i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < TJ; ++j) fb[s][j] = make_uint4(0, 0, 0, 0);
      }
      asm volatile("s_nop 1");  // between such a zero and its product
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t place = 0;
#pragma unroll
    for (int m = 0; m < MF; ++m) {
      mfma16_in_place<D>(fb[s][m % TJ], fa[s][m / TJ], acc[m / TJ][m % TJ]);
      if (places.read[m] >= 0) read_frag(s == 0 ? ua : na, s == 0 ? ub : nb, s ^ 1, places.read[m]);
      if (places.place[m] >= 0) place = lds_place((s == 0 ? spare + myB : ua + myA) + places.place[m] * 1024);
      if (places.load[m] >= 0) {
        if (s == 0) load_b(place, places.load[m]);
        else load_a(place, places.load[m]);
      }
      __builtin_amdgcn_sched_barrier(0);  // this order
    }
  };

  // prologue: k-tiles 0 and 1 on their way, the first half's fragments read
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    uint32_t place = 0;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      if (p % 4 == 0) place = lds_place(myA + 2 * t * kOperand + p * 1024, true);
      load_a(place, p);
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      if (p % 4 == 0) place = lds_place(myB + (2 * t + 1) * kOperand + p * 1024, true);
      load_b(place, p);
    }
    step(nk - t - 2);
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 + PB) : "memory");  // k-tile 0 has landed
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < TI + TJ; ++f) read_frag(ua, ub, 0, f);
  const int ragged_at = tail_chunks < 8 ? 1 : 0;
  for (int left = nk; left > 0; --left) {
    const bool ragged = left == ragged_at;
    half(Const<0>{}, ragged);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(PB) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    half(Const<1>{}, ragged);
    step(left - 4);
    const uint32_t a = ua, b = ub;
    ua = na; ub = nb; na = a; nb = spare; spare = b;
  }
  __builtin_amdgcn_s_waitcnt(0x0070);  // nothing of mine is still on its way into LDS
  store_blocks<D, TI, TJ>(g, epi, dual, acc, m0 + wm * 16 * TI, n0, wn, w.sums, bno, lane);
}

template <class D, bool BNN, int TJ>
int launch_width(int epi, const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)(g.full + g.tail * g.splits));
  hipLaunchKernelGGL((gemm_wide_kernel<D, BNN, TJ>), grid, dim3(256), 0, s, g, epi);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, bool BNN>
int launch_typed(int shape, int epi, const GemmArgs& g, hipStream_t s) {
  switch (shape) {
    case kWide: return launch_width<D, BNN, 8>(epi, g, s);
    case kWide224: return launch_width<D, BNN, 7>(epi, g, s);
    case kWide192: return launch_width<D, BNN, 6>(epi, g, s);
    case kWide160: return launch_width<D, BNN, 5>(epi, g, s);
  }
  return CI_ERR_UNSUPPORTED;
}

}  // namespace

int launch_gemm_wide(int shape, int dtype, int epi, bool b_kmajor, const GemmArgs& g, hipStream_t s) {
  if (dtype == CI_F16) return b_kmajor ? launch_typed<F16, true>(shape, epi, g, s) : launch_typed<F16, false>(shape, epi, g, s);
  if (dtype == CI_BF16) return b_kmajor ? launch_typed<BF16, true>(shape, epi, g, s) : launch_typed<BF16, false>(shape, epi, g, s);
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
