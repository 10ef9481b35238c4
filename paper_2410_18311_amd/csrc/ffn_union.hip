// Union-batched decode: several sentences, each with its own frozen core set,
// decode one token each against the same resident weights (the large-model
// scenario of Sec. 5.3 of arXiv 2410.18311, extended to a batch).  Instead of
// fetching every sentence's rows separately, each row of the union of the core
// sets is read ONCE and applied to the sentences that own it (a bit mask per
// row).  The result per sentence is exactly its own sparse FFN (Sec. 4.2).
//
//   union_scatter / union_place : owner masks [N] -> ascending row list + masks + count
//   union_up_kernel   : dots of the up (and gate) rows with every owner's x, then the
//                       hidden values h[row][sentence] (rows wider than 2048 vectors:
//                       partial dots per column chunk, union_act_kernel adds them up)
//   union_down_kernel : y_s += h[row][s] * W_down[row, :] -> partial[s][slice][d]
//   (decode_reduce_kernel of the single-sentence path sums the slices.)
// The gathered decode (core_idx = [B, K]) of several sentences runs the same way
// where that is the faster order (gathered_union_bytes): sentences that share
// resident weights share most of their rows.
//
// The number of union rows lives in device memory: the kernels slice the rows
// themselves, so no host synchronisation separates building the union from
// using it.
#include "common.hpp"
#include "decode_common.hpp"

namespace ci {

namespace {

constexpr int SB = 8;  // sentences per batch (bits of the owner mask that the kernels look at)
constexpr int kSuperMax = 256;  // up phase: most rows of a slice between two drains of the load ring

struct UnionArgs {
  const void* x;
  const void* w_up;
  const void* w_gate;
  const void* b_up;
  const void* w_down;
  const int32_t* uidx;
  const uint32_t* umask;
  const int32_t* ucount;
  const uint32_t* dup;  // NULL, or: dup[0] != 0 if a list names a neuron more than once, dup[1 + SB n + s] how often
                        // beyond the first time sentence s does (gathered lists: every time counts)
  float* hp;       // [cap][SB] hidden values; c_up > 1: partial dots [c_up][NDOT][cap][SB] first
  float* partial;  // [B][n_down][d]
  int B, d, N, cap, vecs;
  int vc;  // up phase: 16-byte vectors of a row per column chunk
  int n_up, c_up, n_down, c_down;
  int ks_up;  // up phase: most rows of a slice handled between two drains of the load ring
};

__global__ void union_zero_kernel(uint32_t* owners, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) owners[i] = 0u;
}

// owners[n] |= 1 << s for every valid member n of sentence s's list; dup as in UnionArgs
__global__ void union_scatter_kernel(const int32_t* __restrict__ core_idx, int64_t n_idx, int64_t K,
                                     int64_t N, uint32_t* __restrict__ owners, uint32_t* __restrict__ dup) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_idx) return;
  const int n = core_idx[i];
  if (n < 0 || n >= N) return;
  const uint32_t t = (uint32_t)(i / K), bit = 1u << t;
  if (!dup) {
    atomicOr(&owners[n], bit);  // nothing to wait for
  } else if (atomicOr(&owners[n], bit) & bit) {
    dup[0] = 1u;
    atomicAdd(&dup[1 + (size_t)n * SB + t], 1u);
  }
}

// Ordered compaction of the neurons with a non-empty owner mask over blocks of 1024 neurons: every block adds
// up the owned neurons of the blocks before it and places its own behind them (ascending, so the result does
// not depend on the scheduling).  Up to kUnionRecount blocks a block counts those before it itself (36 blocks: 10.0 us
// for the whole build, 8.4 with the launch that counts; 11 blocks: 8.1 either way); above that, union_count_kernel has done so.
constexpr int kUnionBlock = 1024;
constexpr int kUnionRecount = 8;

__global__ __launch_bounds__(kUnionBlock) void union_count_kernel(const uint32_t* __restrict__ owners, int N,
                                                                  uint32_t* __restrict__ blkcnt) {
  __shared__ int wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = blockIdx.x * kUnionBlock + tid;
  const uint32_t m = i < N ? owners[i] : 0u;
  const uint64_t bal = __ballot(m != 0u);
  if (lane == 0) wsum[wave] = __popcll(bal);
  __syncthreads();
  if (tid == 0) {
    int t = 0;
    for (int w = 0; w < 16; ++w) t += wsum[w];
    blkcnt[blockIdx.x] = (uint32_t)t;
  }
}

__global__ __launch_bounds__(kUnionBlock) void union_place_kernel(const uint32_t* __restrict__ owners, int N,
                                                                  int cap, const uint32_t* __restrict__ blkcnt,
                                                                  int32_t* __restrict__ uidx,
                                                                  uint32_t* __restrict__ umask,
                                                                  int32_t* __restrict__ ucount) {
  __shared__ int wsum[16];
  __shared__ int bsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int blk = blockIdx.x;
  const int i = blk * kUnionBlock + tid;
  const uint32_t m = i < N ? owners[i] : 0u;
  const uint64_t bal = __ballot(m != 0u);
  const int before = __popcll(bal & lanemask_lt());
  if (lane == 0) wsum[wave] = __popcll(bal);
  // owned neurons in the blocks before mine (at most 1024 blocks: one per thread)
  int c = 0;
  if (blkcnt) {
    c = tid < blk ? (int)blkcnt[tid] : 0;
  } else {
#pragma unroll 8
    for (int q = 0; q < blk; ++q) c += owners[q * kUnionBlock + tid] != 0u ? 1 : 0;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off);
  if (lane == 0) bsum[wave] = c;
  __syncthreads();
  int base = 0, own = 0;
  for (int w = 0; w < 16; ++w) {
    base += bsum[w];
    own += wsum[w];
  }
  int off = base;
  for (int w = 0; w < wave; ++w) off += wsum[w];
  const int pos = off + before;
  if (m != 0u && pos < cap) {
    uidx[pos] = i;
    umask[pos] = m;
  }
  if (blk == (int)gridDim.x - 1 && tid == 0) {
    const int total = base + own;
    ucount[0] = total < cap ? total : cap;
  }
}

__device__ __forceinline__ int union_rows_clamped(const UnionArgs& a) {
  const int k = *a.ucount;
  return k < 0 ? 0 : (k > a.cap ? a.cap : k);
}

// Stages the weight row and owner mask of each row of a super-chunk in LDS.
// Rows whose index is out of range get mask 0 and read row 0.
__device__ __forceinline__ void union_stage(const UnionArgs& a, int row0, int Rs, int* sidx,
                                            uint32_t* smask) {
  for (int r = threadIdx.x; r < Rs; r += blockDim.x) {
    const int n = a.uidx[row0 + r];
    const bool ok = n >= 0 && n < a.N;
    sidx[r] = ok ? n : 0;
    smask[r] = ok ? (a.umask[row0 + r] & ((1u << a.B) - 1u)) : 0u;
  }
}

// ---- up phase ----------------------------------------------------------------
// dot of one 16-byte vector of weights with the matching 16 bytes of x, both in
// the element type: two-element dot instructions with fp32 accumulation for the
// 16-bit types (no conversions), plain FMAs for fp32.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

template <class D>
__device__ __forceinline__ float dot16(const uint4& w, const uint4& x, float acc);
template <>
__device__ __forceinline__ float dot16<F32>(const uint4& w, const uint4& x, float acc) {
  acc = fmaf(u2f(w.x), u2f(x.x), acc);
  acc = fmaf(u2f(w.y), u2f(x.y), acc);
  acc = fmaf(u2f(w.z), u2f(x.z), acc);
  return fmaf(u2f(w.w), u2f(x.w), acc);
}
template <>
__device__ __forceinline__ float dot16<F16>(const uint4& w, const uint4& x, float acc) {
  acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, w.x), __builtin_bit_cast(half2_t, x.x), acc, false);
  acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, w.y), __builtin_bit_cast(half2_t, x.y), acc, false);
  acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, w.z), __builtin_bit_cast(half2_t, x.z), acc, false);
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2_t, w.w), __builtin_bit_cast(half2_t, x.w), acc, false);
}
template <>
__device__ __forceinline__ float dot16<BF16>(const uint4& w, const uint4& x, float acc) {
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.x), __builtin_bit_cast(bf16x2_t, x.x), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.y), __builtin_bit_cast(bf16x2_t, x.y), acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.z), __builtin_bit_cast(bf16x2_t, x.z), acc, false);
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, w.w), __builtin_bit_cast(bf16x2_t, x.w), acc, false);
}

// Hidden value of (row n, sentence t) from its dots (SwiGLU: z0 gate, z1 up); 0 where t does not own the row.
template <class D, bool SWIGLU>
__device__ __forceinline__ float union_hidden(const UnionArgs& a, int n, bool owns, int t, float z0, float z1) {
  using T = typename D::T;
  float h;
  if (SWIGLU) h = silu(z0) * z1;
  else h = fmaxf(z0 + (a.b_up ? to_float<D>(reinterpret_cast<const T*>(a.b_up)[n]) : 0.f), 0.f);
  if (a.dup && a.dup[0]) h *= (float)(1u + a.dup[1 + (size_t)n * SB + t]);
  return owns ? h : 0.f;
}

// One thread owns NI 16-byte column vectors of its chunk and keeps the matching
// x values of all sentences in registers (element type, 4 registers per vector).
// DEPTH rows are in flight per thread; every ring position issues its loads
// (filler positions from x), so the outstanding-load count is the same on
// every path.  One cross-lane reduction per row serves all NI vectors.
template <class T, int NI, bool SWIGLU>
__device__ __forceinline__ void union_up_issue(int pos, int Rs, int QB, const char* __restrict__ gate,
                                               const char* __restrict__ up,
                                               const char* __restrict__ filler, size_t rowbytes,
                                               const int* sidx, const uint32_t (&coff)[NI],
                                               uint4 (&dst)[NI]) {
  const bool valid = pos < QB;
  const bool second = SWIGLU && pos >= Rs;  // gate rows first, then up rows
  int r = second ? pos - Rs : pos;
  r = r > Rs - 1 ? Rs - 1 : r;
  const char* base = (SWIGLU && !second) ? gate : up;
  const char* prow = base + (size_t)sidx[r] * rowbytes;
  prow = valid ? prow : filler;
#pragma unroll
  for (int i = 0; i < NI; ++i) dst[i] = ld16_stream(prow + coff[i]);
}

template <class D, int NI, bool SWIGLU, int DEPTH>
__global__ __launch_bounds__(512) void union_up_kernel(UnionArgs a) {
  using T = typename D::T;
  constexpr int NDOT = SWIGLU ? 2 : 1;

  extern __shared__ float smem[];
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
  const int slice = blockIdx.x, chunk = blockIdx.y;
  const int Ku = union_rows_clamped(a);
  const int r0 = (int)(((int64_t)slice * Ku) / a.n_up);
  const int r1 = (int)(((int64_t)(slice + 1) * Ku) / a.n_up);
  const int R = r1 - r0;

  const int ks = a.ks_up;
  float* red = smem;                                              // [nw][NDOT * ks][SB]
  int* sidx = reinterpret_cast<int*>(red + nw * NDOT * ks * SB);  // [ks]
  uint32_t* smask = reinterpret_cast<uint32_t*>(sidx + ks);       // [ks]

  const size_t rowbytes = (size_t)a.d * sizeof(T);
  const char* up = reinterpret_cast<const char*>(a.w_up);
  const char* gate = reinterpret_cast<const char*>(a.w_gate);
  const char* xbase = reinterpret_cast<const char*>(a.x);

  // vectors [chunk * vc, (chunk + 1) * vc) of a row belong to this chunk
  uint32_t coff[NI];
  uint4 xq[SB][NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int local = i * nt + tid;
    const int vec = chunk * a.vc + local;
    const bool cv = local < a.vc && vec < a.vecs;
    // a column past the end re-reads column 0 with x = 0, so every load is unconditional
    coff[i] = cv ? (uint32_t)vec * 16u : 0u;
#pragma unroll
    for (int t = 0; t < SB; ++t) {
      xq[t][i] = (t < a.B && cv) ? ld16(xbase + (size_t)t * rowbytes + coff[i]) : make_uint4(0u, 0u, 0u, 0u);
    }
  }

  // super-chunks of equal size (a short last one would pay a full drain and refill of the ring)
  const int nsc = (R + ks - 1) / ks;
  const int step = nsc > 0 ? (R + nsc - 1) / nsc : 1;
  for (int s0 = 0; s0 < R; s0 += step) {
    const int Rs = min(step, R - s0);
    const int QB = NDOT * Rs;
    const int QBp = (QB + DEPTH - 1) / DEPTH * DEPTH;
    __syncthreads();  // previous super-chunk done with sidx / smask / red
    union_stage(a, r0 + s0, Rs, sidx, smask);
    __syncthreads();

    uint4 buf[DEPTH][NI];
#define CI_UISSUE(pos, slot) \
  union_up_issue<T, NI, SWIGLU>((pos), Rs, QB, gate, up, xbase, rowbytes, sidx, coff, buf[slot])
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      CI_UISSUE(s, s);
      __builtin_amdgcn_sched_barrier(0);
    }

    for (int g0 = 0; g0 < QBp; g0 += DEPTH) {
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        const int pos = g0 + s;
        int r = (SWIGLU && pos >= Rs) ? pos - Rs : pos;
        r = r > Rs - 1 ? Rs - 1 : r;
        const uint32_t m = __builtin_amdgcn_readfirstlane(pos < QB ? smask[r] : 0u);
        float p[SB];
#pragma unroll
        for (int t = 0; t < SB; ++t) {
          float sum = 0.f;
          if (m & (1u << t)) {  // uniform: only the owners' dots are computed
#pragma unroll
            for (int i = 0; i < NI; ++i) sum = dot16<D>(buf[s][i], xq[t][i], sum);
          }
          p[t] = sum;
        }
        // refill the slot as soon as it has been consumed
        __builtin_amdgcn_sched_barrier(0);
        CI_UISSUE(pos + DEPTH, s);
        __builtin_amdgcn_sched_barrier(0);
        halve_rows<SB, 32>(p, lane);  // lanes 8t .. 8t+7 now hold sentence t's wave sum
        if ((lane & 7) == 0 && pos < QB) red[((wave * NDOT * ks) + pos) * SB + (lane >> 3)] = p[0];
      }
    }
    // filler loads issued past the end are still outstanding
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
#undef CI_UISSUE
    // sum over the waves; gate rows are matrix 0, up rows matrix 1 (SwiGLU), else matrix 0
    for (int o = tid; o < Rs * SB; o += nt) {
      const int r = o / SB, t = o % SB;
      float z[NDOT];
#pragma unroll
      for (int m = 0; m < NDOT; ++m) {
        z[m] = 0.f;
        for (int w = 0; w < nw; ++w) z[m] += red[((w * NDOT * ks) + m * Rs + r) * SB + t];
      }
      const size_t u = (size_t)(r0 + s0 + r);
      if (a.c_up == 1) {
        a.hp[u * SB + t] = union_hidden<D, SWIGLU>(a, sidx[r], (smask[r] >> t) & 1u, t, z[0], z[NDOT - 1]);
      } else {
#pragma unroll
        for (int m = 0; m < NDOT; ++m) a.hp[(((size_t)chunk * NDOT + m) * a.cap + u) * SB + t] = z[m];
      }
    }
  }
}

// c_up > 1: hidden values from the column chunks' partial dots, over the first of them in place.
template <class D, bool SWIGLU>
__global__ __launch_bounds__(256) void union_act_kernel(UnionArgs a) {
  constexpr int NDOT = SWIGLU ? 2 : 1;
  const int Ku = union_rows_clamped(a);
  const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= (int64_t)Ku * SB) return;
  const size_t u = (size_t)(o / SB);
  const int t = (int)(o % SB), n = a.uidx[u];
  const bool ok = n >= 0 && n < a.N;
  float z[NDOT];
#pragma unroll
  for (int m = 0; m < NDOT; ++m) {
    z[m] = 0.f;
    for (int c = 0; c < a.c_up; ++c) z[m] += a.hp[(((size_t)c * NDOT + m) * a.cap + u) * SB + t];
  }
  a.hp[o] = union_hidden<D, SWIGLU>(a, ok ? n : 0, ok && t < a.B && ((a.umask[u] >> t) & 1u), t, z[0], z[NDOT - 1]);
}

// ---- down phase ----------------------------------------------------------------
// A workgroup has 64 column vectors (1 KB of a row) and a slice of the rows; its waves split the slice, each
// lane holding one vector for all eight sentences, and are added up through LDS at the end, so that a slice
// leaves one partial sum per column: with 384 vectors per workgroup and six times as many slices, 50 MB of them
// were written and read back per step at 36864 x 9216 and 8 sentences (13 us to add them up; now 8 MB, 4.5 us).
// What a wave needs to know of a group of eight rows -- indices, owners, 8 x 8 hidden values, one per lane --
// are three small loads that run ahead in the same in-order queue as the rows, and reach scalar registers by
// lane reads: nothing is staged ahead of the stream and no barrier interrupts it.  (Scalar loads instead cost
// a wait per owner: 173 us for the phase at 8 sentences and a keep fraction of 0.6.)
template <class D, int DEPTH>
__global__ __launch_bounds__(512) void union_down_kernel(UnionArgs a) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  __shared__ float red[2][8][64 * VEC];
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = blockIdx.x, chunk = blockIdx.y;
  const int Ku = __builtin_amdgcn_readfirstlane(union_rows_clamped(a));
  // the slice's rows [.., r1) go to the waves in groups of DEPTH, turn by turn
  const int step = nw * DEPTH;
  const int r0 = (int)((int64_t)slice * Ku / a.n_down) + wave * DEPTH, r1 = (int)((int64_t)(slice + 1) * Ku / a.n_down);

  const size_t rowbytes = (size_t)a.d * sizeof(T);
  const char* down = reinterpret_cast<const char*>(a.w_down);
  const int vec = chunk * 64 + lane;
  const bool cv = vec < a.vecs;
  const uint32_t coff = cv ? (uint32_t)vec * 16u : 0u;
  float acc[SB][VEC];
#pragma unroll
  for (int t = 0; t < SB; ++t)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[t][v] = 0.f;

  if (r0 < r1) {
    const uint32_t all = (1u << a.B) - 1u;
    // indices and owners of the rows from `g` on, one per lane (DEPTH <= 64); rows past the end belong to nobody
    auto load_idx = [&](int g) { return a.uidx[min(g + (lane & (DEPTH - 1)), r1 - 1)]; };
    auto load_mask = [&](int g) { return a.umask[min(g + (lane & (DEPTH - 1)), r1 - 1)]; };
    // hidden values of the rows from `g` on: lane 8 i + t holds row i, sentence t
    auto load_h = [&](int g, float (&h)[DEPTH / 8]) {
#pragma unroll
      for (int q = 0; q < DEPTH / 8; ++q) h[q] = a.hp[(size_t)min(g + 8 * q + (lane >> 3), r1 - 1) * SB + (lane & 7)];
    };
    // row s of the group whose indices are in `idx`; past the end: x, which is in cache
    auto row_ptr = [&](int idx, int g, int s) {
      const int n = __builtin_amdgcn_readlane(idx, s);
      return g + s < r1 ? down + (size_t)((n >= 0 && n < a.N) ? n : 0) * rowbytes : reinterpret_cast<const char*>(a.x);
    };
    int idx0 = load_idx(r0), idx1 = load_idx(r0 + step);
    uint32_t mask = load_mask(r0);
    float h[DEPTH / 8];
    load_h(r0, h);
    uint4 buf[DEPTH];
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      buf[s] = ld16_stream(row_ptr(idx0, r0, s) + coff);
      __builtin_amdgcn_sched_barrier(0);
    }
    for (int g0 = r0; g0 < r1; g0 += step) {
      const int idx2 = load_idx(g0 + 2 * step);
      const uint32_t mask_next = load_mask(g0 + step);
      float h_next[DEPTH / 8];
      load_h(g0 + step, h_next);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < DEPTH; ++s) {
        float f[VEC];
        unpack<D>(buf[s], f);
        __builtin_amdgcn_sched_barrier(0);
        buf[s] = ld16_stream(row_ptr(idx1, g0 + step, s) + coff);
        __builtin_amdgcn_sched_barrier(0);
        const int n = __builtin_amdgcn_readlane(idx0, s);
        const uint32_t own = (uint32_t)__builtin_amdgcn_readlane((int)mask, s) & all;
        const uint32_t m = (g0 + s < r1 && n >= 0 && n < a.N) ? own : 0u;
#pragma unroll
        for (int t = 0; t < SB; ++t) {
          if (m & (1u << t)) {  // uniform
            const float ht = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(h[s >> 3]), 8 * (s & 7) + t));
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[t][v] = fmaf(ht, f[v], acc[t][v]);
          }
        }
      }
      idx0 = idx1;
      idx1 = idx2;
      mask = mask_next;
#pragma unroll
      for (int q = 0; q < DEPTH / 8; ++q) h[q] = h_next[q];
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }

  // sum over the waves, in wave order, one sentence after the other; thread -> columns.  Sentences alternate between
  // two tables: one is written again behind the barrier of the other, which everybody reaches with its sums done.
#pragma unroll
  for (int t = 0; t < SB; ++t) {
    if (t < a.B) {  // uniform
#pragma unroll
      for (int v = 0; v < VEC; ++v) red[t & 1][wave][v * 64 + lane] = acc[t][v];
      __syncthreads();
      for (int o = tid; o < 64 * VEC; o += blockDim.x) {
        float z = 0.f;
        for (int w = 0; w < nw; ++w) z += red[t & 1][w][o];
        const int col = (chunk * 64 + (o & 63)) * VEC + (o >> 6);
        if (chunk * 64 + (o & 63) < a.vecs) a.partial[((size_t)t * a.n_down + slice) * a.d + col] = z;
      }
    }
  }
}

inline size_t union_up_lds(int t_up, int ndot, int ks) {
  return (size_t)(t_up / 64) * ndot * ks * SB * sizeof(float) + 2 * (size_t)ks * sizeof(int);
}

template <class D, int NI, bool SWIGLU>
void launch_union_up(const UnionArgs& a, int t_up, hipStream_t s) {
  constexpr int NDOT = SWIGLU ? 2 : 1;
  const size_t lds = union_up_lds(t_up, NDOT, a.ks_up);
  const dim3 g(a.n_up, a.c_up);
  // about 16 loads in flight per thread
  if constexpr (NI >= 3) hipLaunchKernelGGL((union_up_kernel<D, NI, SWIGLU, 4>), g, dim3(t_up), lds, s, a);
  else if constexpr (NI == 2) hipLaunchKernelGGL((union_up_kernel<D, NI, SWIGLU, 8>), g, dim3(t_up), lds, s, a);
  else hipLaunchKernelGGL((union_up_kernel<D, NI, SWIGLU, 16>), g, dim3(t_up), lds, s, a);
}

template <class D, bool SWIGLU>
int launch_union_typed(const UnionArgs& a, int ni, int t_up, int t_down, hipStream_t s) {
  switch (ni) {
    case 1: launch_union_up<D, 1, SWIGLU>(a, t_up, s); break;
    case 2: launch_union_up<D, 2, SWIGLU>(a, t_up, s); break;
    case 3: launch_union_up<D, 3, SWIGLU>(a, t_up, s); break;
    case 4: launch_union_up<D, 4, SWIGLU>(a, t_up, s); break;
    default: return CI_ERR_UNSUPPORTED;
  }
  if (a.c_up > 1)
    hipLaunchKernelGGL((union_act_kernel<D, SWIGLU>), dim3((unsigned)(((int64_t)a.cap * SB + 255) / 256)), dim3(256), 0, s, a);
  const dim3 gd(a.n_down, a.c_down);
  if (params().union_depth == 16) hipLaunchKernelGGL((union_down_kernel<D, 16>), gd, dim3(t_down), 0, s, a);
  else hipLaunchKernelGGL((union_down_kernel<D, 8>), gd, dim3(t_down), 0, s, a);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

}  // namespace

// Column chunks of the up phase for a row of `vecs` 16-byte vectors (a
// workgroup covers at most 512 threads x 4 vectors); part of the workspace layout.
int union_up_chunks(int64_t vecs) { return (int)((vecs + 2047) / 2048); }

int launch_union_build(const int32_t* core_idx, int64_t B, int64_t K, int64_t N, int64_t cap,
                       int32_t* uidx, uint32_t* umask, int32_t* ucount, uint32_t* owners, uint32_t* dup,
                       hipStream_t s) {
  // owner masks, and behind them dup if there is one (gathered_union_layout keeps the two adjacent)
  const int64_t n_zero = dup ? (dup - owners) + 1 + N * SB : N;
  hipLaunchKernelGGL(union_zero_kernel, dim3((unsigned)((n_zero + 255) / 256)), dim3(256), 0, s, owners, n_zero);
  const int64_t n_idx = B * K;
  if (n_idx > 0)
    hipLaunchKernelGGL(union_scatter_kernel, dim3((unsigned)((n_idx + 255) / 256)), dim3(256), 0, s,
                       core_idx, n_idx, K, N, owners, dup);
  const unsigned nblk = (unsigned)((N + kUnionBlock - 1) / kUnionBlock);  // <= 1024: N <= CI_MAX_NEURONS
  uint32_t* blkcnt = nullptr;
  if (nblk > kUnionRecount) {
    blkcnt = owners + (N + 63) / 64 * 64;
    hipLaunchKernelGGL(union_count_kernel, dim3(nblk), dim3(kUnionBlock), 0, s, owners, (int)N, blkcnt);
  }
  hipLaunchKernelGGL(union_place_kernel, dim3(nblk), dim3(kUnionBlock), 0, s, owners, (int)N, (int)cap, blkcnt, uidx,
                     umask, ucount);
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

namespace {

// Slices of the down phase: one workgroup of eight waves per compute unit over all column chunks, at most 256 (what the
// workspace holds), and at least 32 rows each: below that the end of a workgroup, which adds up its waves, is most of
// it.  (With 128 rows at least, small unions left compute units without work: 8 sentences of 256 x 1024 fp32 24.8 us
// against 21.9, 819 rows of 4096 in 16 bits 17.9 against 15.4; with 16 rows 22.2 and 15.4.)
int down_slices(int64_t vecs, int64_t cap, int cus) {
  const int64_t chunks = (vecs + 63) / 64;
  int64_t n = (int64_t)cus * params().union_down_wgs_per_cu / chunks;
  const int64_t most = (cap + 31) / 32;
  if (n > 256) n = 256;
  if (n > most) n = most;
  return n < 1 ? 1 : (int)n;
}

int chip_cus() {
  DeviceInfo di;
  return device_info(&di) == CI_OK ? di.cus : 256;
}

GatheredUnion gathered_union_layout(int64_t B, int64_t K, int64_t N, int64_t d, int dtype, int act) {
  GatheredUnion g;
  auto up64 = [](size_t n) { return (n + 63) / 64 * 64; };
  const int64_t vecs = d / (dtype == CI_F32 ? 4 : 8);
  g.cap = B * K < N ? B * K : N;
  g.partial = up64((size_t)union_up_chunks(vecs) * (act == CI_ACT_SWIGLU ? 2 : 1) * (size_t)g.cap * SB);
  g.n_down = down_slices(vecs, g.cap, chip_cus());
  g.owners = g.partial + up64((size_t)B * g.n_down * (size_t)d);
  g.dup = g.owners + up64((size_t)N) + 1024;  // 1024: counts per block of union_place_kernel
  g.uidx = g.dup + up64(1 + (size_t)N * SB);
  g.umask = g.uidx + up64((size_t)g.cap);
  g.ucount = g.umask + up64((size_t)g.cap);
  g.total = g.ucount + 64;
  return g;
}

}  // namespace

// Whether a gathered decode of B lists goes through their union.  Reading every list's rows separately runs at
// about 7 TB/s (sentences in flight together find shared rows in the caches), the union at 5.6 TB/s (gated layers
// 5.0) and 23 us for building it, two more dependent launches and the ends of the kernels.  Lists are taken to
// overlap as random ones do -- core sets of one model overlap more -- and the union has to win by a tenth.
// Measured, separate / union (us): 36864 x 9216 ReLU: 8 lists at a keep fraction of 0.4 573 / 241, 4 at 0.4
// 304 / 217, 3 at 0.4 236 / 194, 4 at 0.2 163 / 153 (stays separate); 13824 x 5120 gated: 8 at 0.3 134 / 109,
// 8 at 0.2 95 / 100, 4 at 0.4 94 / 98 (stay separate); 16384 x 4096 ReLU: 8 at 0.3 87 / 67, 8 at 0.2 60 / 63 (stays);
// 3840 x 1280: separate throughout (15 / 28).  Its scratch has to fit what both gathered entry points offer for any
// such call: the workspace by its published size, and the 16 MiB of library scratch.
bool gathered_union_pays(int64_t B, int64_t K, int64_t N, int64_t d, int dtype, int act, GatheredUnion* plan) {
  if (params().gathered_union == 0 || B < 2 || B > SB || K < 1 || K > N) return false;
  if (d / (dtype == CI_F32 ? 4 : 8) > 4096) return false;  // wider rows are turned down by the gathered kernel, and stay so
  *plan = gathered_union_layout(B, K, N, d, dtype, act);
  const size_t bytes = plan->total * 4;
  const size_t ws = (size_t)B * (size_t)(K < 1024 ? K : 1024) * (size_t)d * sizeof(float);
  if (bytes > ws || bytes > ((size_t)16 << 20)) return false;
  if (params().gathered_union == 2) return true;
  const double row = (double)d * elem_bytes(dtype) * (act == CI_ACT_SWIGLU ? 3 : 2);
  double miss = 1.0;
  for (int64_t b = 0; b < B; ++b) miss *= 1.0 - (double)K / (double)N;
  const double t_lists = (double)(B * K) * row / 7.0e12 + 4e-6;
  const double t_union = (double)N * (1.0 - miss) * row / (act == CI_ACT_SWIGLU ? 5.0e12 : 5.6e12) + 23e-6;
  return t_union * 1.1 < t_lists;
}

int launch_gathered_union(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act, void* y, float* ws,
                          const GatheredUnion& g, hipStream_t s) {
  uint32_t* base = reinterpret_cast<uint32_t*>(ws);
  int32_t* uidx = reinterpret_cast<int32_t*>(base + g.uidx);
  int32_t* ucount = reinterpret_cast<int32_t*>(base + g.ucount);
  const int rc = launch_union_build(w->core_idx, B, w->K, w->N, g.cap, uidx, base + g.umask, ucount, base + g.owners,
                                    base + g.dup, s);
  if (rc != CI_OK) return rc;
  return launch_ffn_decode_union(x, B, w, uidx, base + g.umask, ucount, g.cap, dtype, act, y, ws, s, base + g.dup, g.n_down);
}

int launch_ffn_decode_union(const void* x, int64_t B, const ci_ffn_weights* w, const int32_t* uidx,
                            const uint32_t* umask, const int32_t* ucount, int64_t cap, int dtype,
                            int act, void* y, float* ws, hipStream_t s, const uint32_t* dup, int n_down) {
  UnionArgs a;
  a.dup = dup;
  a.x = x;
  a.w_up = w->w_up;
  a.w_gate = w->w_gate;
  a.b_up = w->b_up;
  a.w_down = w->w_down;
  a.uidx = uidx;
  a.umask = umask;
  a.ucount = ucount;
  a.B = (int)B;
  a.d = (int)w->d;
  a.N = (int)w->N;
  a.cap = (int)cap;
  a.vecs = (int)(w->d / (dtype == CI_F32 ? 4 : 8));
  const int ndot = act == CI_ACT_SWIGLU ? 2 : 1;

  const int cus = chip_cus();
  a.c_up = union_up_chunks(a.vecs);
  a.vc = (a.vecs + a.c_up - 1) / a.c_up;
  // vectors per thread: the choice that pads the chunk least, the larger one on ties (one
  // cross-lane reduction per row serves all of a thread's vectors)
  int ni = 1, t_up = 512, waste = 1 << 30;
  for (int n = 4; n >= 1; --n) {
    const int t = ((a.vc + n - 1) / n + 63) / 64 * 64;
    if (t > 512) continue;
    if (t * n - a.vc < waste) { waste = t * n - a.vc; ni = n; t_up = t; }
  }
  int t_down = params().union_down_threads / 64 * 64;
  if (t_down < 64) t_down = 64;
  if (t_down > 512) t_down = 512;
  a.c_down = (a.vecs + 63) / 64;
  a.n_down = n_down > 0 ? n_down : down_slices(a.vecs, a.cap, cus);
  // up phase: about 384 threads per compute unit (at d = 4096 the two waves of four vectors per lane that a
  // workgroup has were alone on theirs: 36 us for 13650 rows, now 25)
  a.n_up = cus * params().union_up_wgs_per_cu * ((384 + t_up / 2) / t_up > 1 ? (384 + t_up / 2) / t_up : 1) / a.c_up;
  if (a.n_up > 1024) a.n_up = 1024;
  if (a.n_up > a.cap) a.n_up = a.cap;
  if (a.n_up < 1) a.n_up = 1;

  // rows between two drains: as many as 64 KB of LDS hold (wave sums of the up phase)
  a.ks_up = kSuperMax;
  while (a.ks_up > 64 && union_up_lds(t_up, ndot, a.ks_up) > 65536) a.ks_up >>= 1;
  const int ks_cap = params().union_super;
  if (ks_cap > 0 && a.ks_up > ks_cap) a.ks_up = ks_cap;

  a.hp = ws;
  const size_t hp_floats = ((size_t)a.c_up * ndot * (size_t)a.cap * SB + 63) / 64 * 64;
  a.partial = ws + hp_floats;

  int rc;
  const bool sw = act == CI_ACT_SWIGLU;
  switch (dtype) {
    case CI_F32: rc = sw ? launch_union_typed<F32, true>(a, ni, t_up, t_down, s) : launch_union_typed<F32, false>(a, ni, t_up, t_down, s); break;
    case CI_F16: rc = sw ? launch_union_typed<F16, true>(a, ni, t_up, t_down, s) : launch_union_typed<F16, false>(a, ni, t_up, t_down, s); break;
    case CI_BF16: rc = sw ? launch_union_typed<BF16, true>(a, ni, t_up, t_down, s) : launch_union_typed<BF16, false>(a, ni, t_up, t_down, s); break;
    default: return CI_ERR_BAD_DTYPE;
  }
  if (rc != CI_OK) return rc;
  return launch_decode_reduce(a.partial, w->b_down, y, a.n_down, a.d, (int)B, dtype, s);
}

}  // namespace ci
