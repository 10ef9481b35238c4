// Device code that the LDS-tiled GEMM kernels for 16-bit types share (gemm_wide.hip, gemm_mid.hip, gemm_slim.hpp).
#pragma once

#include "gemm_common.hpp"

namespace ci {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int WK = 64;             // k per tile

template <int V>
struct Const {
  static constexpr int value = V;
};

template <class D>
__device__ __forceinline__ f32x4 mfma16(const uint4& a, const uint4& b, f32x4 c) {
  if constexpr (__is_same(D, F16))
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The same, c = a * b + c, written out: the sum stays where it is.  The compiler does not see a matrix product in it: two wait
// states after a vector instruction that writes an operand, and 18 before anything else touches the sum, are the caller's.
template <class D>
__device__ __forceinline__ void mfma16_in_place(const uint4& a, const uint4& b, f32x4& c) {
  if constexpr (__is_same(D, F16))
    asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(__builtin_bit_cast(f16x8, a)), "v"(__builtin_bit_cast(f16x8, b)));
  else
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(__builtin_bit_cast(bf16x8, a)), "v"(__builtin_bit_cast(bf16x8, b)));
}

// Four consecutive columns of one output row: the score and the element type's bits of each.
struct Quad {
  f32x4 score;
  uint2 bits;
};
template <class D, int EPI>
__device__ __forceinline__ Quad epilogue_quad(f32x4 z, f32x4 u, const float (&bv)[4]) {
  using T = typename D::T;
  Quad q;
  T e[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float h = EPI == EPI_SWIGLU ? silu(z[k]) * u[k] : EPI == EPI_RELU ? fmaxf(z[k] + bv[k], 0.f) : z[k] + bv[k];
    // opaque: else the compiler makes a product and its conversion to fp16 one instruction with one rounding, and the bits are no longer
    // those of the score, rounded
    asm("" : "+v"(h));
    q.score[k] = EPI == EPI_SWIGLU ? fabsf(h) : h;
    e[k] = from_float<D>(h);
  }
  __builtin_memcpy(&q.bits, e, 8);
  return q;
}

// One 16-byte and / or one 8-byte store of them.
template <class D, int EPI>
__device__ __forceinline__ void store_quad(const GemmArgs& g, f32x4 z, f32x4 u, const float (&bv)[4], size_t o) {
  const Quad q = epilogue_quad<D, EPI>(z, u, bv);
  if (g.out_f) *reinterpret_cast<f32x4*>(g.out_f + o) = q.score;
  if (g.out_e) *reinterpret_cast<uint2*>(reinterpret_cast<typename D::T*>(g.out_e) + o) = q.bits;
}

// Buffer descriptor over everything from a uniform address on: a load then takes one 32-bit offset per lane.
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 rsrc_at(const char* p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return i32x4{(int)a, (int)((a >> 32) & 0xffffu), -1, 0x00020000};
}

// 16 bytes per lane from `rsrc` + `off` to LDS at `lds` + 16 * lane.  Written out, because the compiler
// orders transposing LDS reads behind every such load it knows of; nothing is returned to a register, and
// the waits for its arrival are the kernel's own (s_waitcnt vmcnt ahead of a barrier).  The compiler does not
// look for hazards inside: five wait states have to lie between a vector instruction that writes a scalar register (a
// lane read that makes a descriptor uniform or fetches a spilled one) and a load that reads it.  The moves that make the
// descriptors here are scalar, which need none; the build looks at every such load of the library and fails where the
// compiler has come to something else (isa_check.py).  Waiting here instead, whatever stands before, costs the 40
// loads that a small product starts with 0.35 us (four idle states: both products of 5 x 256 x 1024 13.2 -> 13.8 us; a copy
// of the descriptor by scalar moves 13.6).  ONCE: the lines are the first to leave the caches.
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds(const unsigned char* lds, uint32_t off, i32x4 rsrc) {
  const uint32_t m = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)lds;
  uint32_t m0;  // says that m0 is written (as a clobber it is refused with a warning)
  if constexpr (ONCE)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen nt lds"
                 : "={m0}"(m0)
                 : "s"(m), "v"(off), "s"(rsrc)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds"
                 : "={m0}"(m0)
                 : "s"(m), "v"(off), "s"(rsrc)
                 : "memory");
}

// The same from an address up to an end: reads at or past it return zero.
__device__ __forceinline__ i32x4 rsrc_until(const char* p, const char* end) {
  i32x4 r = rsrc_at(p);
  const size_t n = (size_t)(end - p);
  r[2] = n < 0xffffffffu ? (int)n : -1;
  return r;
}

// A load into LDS in two instructions: the place, written at least one instruction ahead (at_once: a load may follow immediately),
// and loads that go by it, to 1 KB `piece` behind the place, from as far behind `off` + `scalar_off`.
__device__ __forceinline__ uint32_t lds_place(uint32_t place, bool at_once = false) {
  uint32_t m0;
  if (at_once) asm volatile("s_mov_b32 m0, %1\n\ts_nop 0" : "={m0}"(m0) : "s"(place));
  else asm volatile("s_mov_b32 m0, %1" : "={m0}"(m0) : "s"(place));
  return m0;
}
template <bool ONCE = false>
__device__ __forceinline__ void load_to_lds_at(int piece, uint32_t place, uint32_t off, i32x4 rsrc, uint32_t scalar_off) {
  if constexpr (ONCE)
    asm volatile("buffer_load_dwordx4 %1, %2, %3 offen offset:%4 nt lds"
                 :: "{m0}"(place), "v"(off), "s"(rsrc), "s"(scalar_off), "n"(piece * 1024)
                 : "memory");
  else
    asm volatile("buffer_load_dwordx4 %1, %2, %3 offen offset:%4 lds"
                 :: "{m0}"(place), "v"(off), "s"(rsrc), "s"(scalar_off), "n"(piece * 1024)
                 : "memory");
}

// k-major B in LDS, rows of BN columns (of one k): chunk j of row k lies at j ^ this.  Transposing reads of 32 lanes cover eight rows
// (k % 4 and k / 8 % 2) x 32 bytes in 256 different bytes of the banks.
template <int BN>
__device__ __forceinline__ int kmajor_swizzle(int k) {
  return BN >= 128 ? (k & 3) << 2 | (k >> 3 & 1) << 1 : (k >> 1 & 1) << 2 | (k >> 3 & 1) << 1;
}

// What goes out behind which of MF products: at most one LDS read (of a fragment) and one load, and mostly not both; the
// scalar register that a load takes its place in LDS from is written one product ahead, for every four pieces of an operand (the first
// FIRST loads are one operand's, the others another's).
template <int MF, int READS, int LOADS, int FIRST = LOADS>
struct Places {
  int read[MF] = {}, load[MF] = {}, place[MF] = {};  // number, -1: none; place: of the load it is for
  constexpr Places() {
    for (int m = 0; m < MF; ++m) read[m] = load[m] = place[m] = -1;
    for (int r = 0; r < READS; ++r) read[r * MF * 3 / (4 * READS)] = r;  // in the first three quarters
    for (int p = 0; p < LOADS; ++p) {
      int m = (2 * p + 1) * MF / (2 * LOADS);
      if (m + 1 < MF && read[m] >= 0 && read[m + 1] < 0) ++m;
      load[m] = p;
      if (p < FIRST ? p % 4 == 0 : (p - FIRST) % 4 == 0) place[m - 1] = p;
    }
  }
};

// Results of 2 x 2 waves of TI x TJ blocks of 16x16, sums of mfma16_in_place with B's fragment first: element v of lane l is row
// l % 16, column 4 (l / 16) + v of a block, so that four neighbouring columns go out as they are.  SwiGLU (dual): a block is eight
// gate and eight up columns.  row0: the wave's first row, n0: the tile's first output column, wn: the wave's half of its columns; sums:
// not null where raw sums are stored instead of outputs, by row and column of the product `bno` apart.
template <class D, int TI, int TJ>
__device__ __forceinline__ void store_blocks(const GemmArgs& g, int epi, bool dual, f32x4 (&acc)[TI][TJ], int row0, int n0, int wn,
                                             float* sums, int bno, int lane) {
  using T = typename D::T;
  // the last products' sums are in their registers 18 wait states later
  asm volatile("s_nop 15\n\ts_nop 3");
  auto settled = [&](int i) {
#pragma unroll
    for (int j = 0; j < TJ; ++j) asm volatile("" : "+a"(acc[i][j]));
  };

  const int l15 = lane & 15, quarter = lane >> 4;
  if (sums) {
    const int col0 = n0 + wn * 16 * TJ + 4 * quarter;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const int row = row0 + l15 + 16 * i;
      settled(i);
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int col = col0 + 16 * j;
        if (row < g.M && col < g.Nn) *reinterpret_cast<f32x4*>(sums + (ptrdiff_t)row * bno + col) = acc[i][j];
      }
    }
    return;
  }
  // Outputs go through descriptors: an output that is not wanted has none of its bytes in range, and rows and columns past the edge get
  // an offset that is in range of neither, so that nothing branches between one quad and the next.  With a test of the kind, of each
  // output and of the edge at every quad, and 16-bit values in pieces of 32 bytes, 248 x 128 x 384 ReLU fp16 with both outputs took 11.8 us
  // and bf16 13.3 (two kernels with the kind built in, rows through LDS: 11.1 and 12.9); so 11.0 and 12.2, 256 x 4096 x 16384 101.1 for
  // 102.0, and 1024 x 5120 x 13824 gated bf16 345.1 for 352.8 (with offsets that the compiler chose by branches 356).  Blocks of 16 rows behind the last one are left out, or a prompt of a few tokens works out and drops as many quads as one of 128
  // (14 x 128 x 144 gated bf16 10.6 us, 8.8 without them).  128 rows of 2^20 columns at most: elements below 2^27.  A row or a column past the
  // edge is 2^28 elements off and both 2^29: outside the ranges, and far from 2^32 bytes, where the last words of a store would come
  // round to the first of the range.
  constexpr uint32_t kNowhere = 1u << 28;
  constexpr int kRange = 1 << 29;  // bytes, of either output
  const size_t origin = (size_t)row0 * g.ldo + n0;
  auto output = [&](const void* p, size_t bytes) {  // integers: a null pointer is not added to
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(reinterpret_cast<uintptr_t>(p) + origin * bytes), 0, p ? kRange : 0, 0x00020000);
  };
  const auto to_f = output(g.out_f, sizeof(float)), to_e = output(g.out_e, sizeof(T));
  auto row_at = [&](int i) {  // element offset of this lane's row of block i
    const uint32_t r = l15 + 16 * i, o = r * (uint32_t)g.ldo;
    return row0 + (int)r < g.M ? o : kNowhere;
  };
  auto column_at = [&](int c, bool there) { return there & (n0 + c < g.Nn) ? (uint32_t)c : kNowhere; };
  auto put_scores = [&](const Quad& q, uint32_t o) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, q.score), to_f, (int)(o * 4u), 0, 0);
  };
  // Two neighbouring sixteens of columns from c on, four a lane, of which there are `n`: they go out eight a lane, so that a row's
  // piece is 64 bytes.
  auto put_bits = [&](uint2 a, uint2 b, uint32_t row, int c, int n) {
    const auto x = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false), y = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false), hi = __builtin_amdgcn_permlane16_swap(y[0], y[1], false, false);
    const u32x4 v = {lo[0], hi[0], lo[1], hi[1]};
    __builtin_amdgcn_raw_buffer_store_b128(v, to_e, (int)((row + column_at(c + 8 * quarter, 8 * quarter < n)) * 2u), 0, 0);
  };
  if (dual) {
    // lanes 0 .. 31 hold the gate, 32 .. 63 the up values of a block's eight columns: two blocks change halves
    const int c0 = wn * 8 * TJ;
    if (n0 + c0 >= g.Nn) return;
    const float none[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if (row0 + 16 * i >= g.M) break;
      settled(i);
      const uint32_t row = row_at(i);
      uint2 bits[2];
#pragma unroll
      for (int j = 0; j < TJ; j += 2) {
        const bool pair = j + 1 < TJ;
        f32x4 z, u;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const auto sw = __builtin_amdgcn_permlane32_swap(f2u(acc[i][j][v]), f2u(acc[i][pair ? j + 1 : j][v]), false, false);
          z[v] = u2f(sw[0]);
          u[v] = u2f(sw[1]);
        }
        const Quad q = epilogue_quad<D, EPI_SWIGLU>(z, u, none);
        put_scores(q, row + column_at(c0 + 8 * j + 4 * quarter, pair | (quarter < 2)));
        bits[j >> 1 & 1] = q.bits;
        if (j & 2) put_bits(bits[0], bits[1], row, c0 + 8 * (j - 2), pair ? 32 : 24);
        else if (j + 2 >= TJ) put_bits(bits[0], bits[0], row, c0 + 8 * j, pair ? 16 : 8);
      }
    }
    return;
  }
  const int c0 = wn * 16 * TJ;
  if (row0 >= g.M || n0 + c0 >= g.Nn) return;
  float bv[TJ][4];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int col = n0 + c0 + 16 * j + 4 * quarter;
      bv[j][k] = g.bias && col < g.Nn ? to_float<D>(reinterpret_cast<const T*>(g.bias)[col + k]) : 0.f;
    }
  auto all = [&](auto kind) {
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if (row0 + 16 * i >= g.M) break;
      settled(i);
      const uint32_t row = row_at(i);
      uint2 bits[2];
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const Quad q = epilogue_quad<D, kind.value>(acc[i][j], acc[i][j], bv[j]);
        if (kind.value == EPI_RELU) put_scores(q, row + column_at(c0 + 16 * j + 4 * quarter, true));
        bits[j & 1] = q.bits;
        if (j & 1) put_bits(bits[0], bits[1], row, c0 + 16 * (j - 1), 32);
        else if (j + 1 == TJ) put_bits(bits[0], bits[0], row, c0 + 16 * j, 16);
      }
    }
  };
  if (epi == EPI_RELU) all(Const<EPI_RELU>{});
  else all(Const<EPI_LINEAR>{});  // a down projection, which has no scores
}

// Which tile and which part of k a workgroup has: the first g.full tiles are computed whole, each of the
// g.tail tiles behind them by g.splits workgroups.
struct TileWork {
  int tm, tn;
  int k_begin, k_end;
  float* sums;  // null, or where store_blocks finds row 0, column 0 of the product for this workgroup's tile of sums
};
__device__ __forceinline__ TileWork tile_work(const GemmArgs& g, int bm, int bn) {
  const int tiles_m = (g.M + bm - 1) / bm, tiles_n = (g.Nn + bn - 1) / bn;
  const int id = blockIdx.x;
  TileWork w;
  int t, local = 0;
  if (id < g.full) {
    t = xcd_spread(id, g.full);
    w.sums = nullptr;
    w.k_begin = 0;
    w.k_end = g.Kk;
  } else {
    local = xcd_spread(id - g.full, g.tail * g.splits);
    t = g.full + local % g.tail;
    w.k_begin = local / g.tail * g.k_chunk;
    w.k_end = min(g.Kk, w.k_begin + g.k_chunk);
  }
  tile_of(t, tiles_m, tiles_n, &w.tm, &w.tn);
  if (id >= g.full)  // `local` is split * tail + tile: the place of this workgroup's sums
    w.sums = g.partial + (ptrdiff_t)local * sums_pitch(bm, bn) - ((ptrdiff_t)w.tm * bm * bn + (ptrdiff_t)w.tn * bn);
  return w;
}

}  // namespace

}  // namespace ci
