// Decode-stage FFN of small layers in one launch (neuron-major compact weights):
//   y = W_down_c^T act(W_up_c x [+ b]) [+ b_down]
// The two launches of ffn_decode.hip cost the host about 3.9 us each, more than the GPU needs for both where the weights
// are a few hundred kilobytes.  So every workgroup here has ALL hidden values in LDS and sums its own columns of y over all neurons: no
// partial sums and no second launch.  It computes them itself, from weights that lie in its L2, or a part of them, and takes the others' from
// memory (SHARE, below).
// What bounds it is the fill of a compute unit's L1 with the up (and gate) rows: by the slope of its time over their size 124 GB/s
// in fp32 and 85 in 16 bits, with twice the products a byte (256 x 96 to 256 x 512).  The down rows of the workgroup's columns
// are requested ahead of them and wait in registers.
// Where that fill takes longer than to hand a value on (SHARE), a workgroup computes its part of the hidden values only and stores each
// as words that say themselves that they are this call's; the others read them until they are (about 1.5 us).  Nothing depends on the
// others being there: a workgroup whose values have not come in 20 us computes them itself.  256 x 410 fp32, call by call, 6.95 ->
// 5.39 us, 256 x 512 7.6 -> 5.4, 4 tokens of 256 x 448 7.2 -> 5.8, fp16 512 x 256 6.7 -> 5.8.  The words are the library's own and shared by
// all streams, which costs little: 256 x 410 on two and three streams at once, enqueued so that calls take the same words, 5.0 to 5.2 us a
// call where one stream alone takes 4.8 and every workgroup computing all 7.3 to 14; beside dense FFNs of 2048 x 5120 x 13824, whose
// workgroups leave no room, 19 us where that takes 21 and two launches 20, and the dense FFNs the same 790 us; a wait of 4 us
// for 20 makes no difference there.
// A call gives the same bits whichever way it goes (launched or captured, apart or in place; finite weights): dot products are
// added up over the lanes as there, down rows slice by slice, and the slices in the order of decode_reduce_kernel.  That costs
// nothing measurable: 256 x 424 fp32 from a graph 6.91 us, and 6.89 with the rows spread over all threads.
#include <sys/random.h>
#include <time.h>
#include <unistd.h>

#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "decode_common.hpp"

namespace ci {

namespace {

struct SmallArgs {
  const void* x;
  const void* w_up;
  const void* w_gate;
  const void* b_up;
  const void* w_down;
  const void* b_down;
  void* y;
  int K, d;
  int n_wg;           // slices of the neurons
  uint32_t inv_n_wg;  // 2^32 / n_wg rounded up: a product below 2^20 times it, 32 bits up, is the product over n_wg
  int most_rows;      // at least the rows of any slice
};
struct SharedArgs : SmallArgs {  // arguments of the one kernel only: every launch pays for its own
  uint32_t tag[2];    // of this call and no other
  int slot;           // the first of its rows of g_hidden
  int patience;       // ticks of 10 ns that a workgroup waits for the others before it computes their values itself; 0: does not look for them
};

constexpr int kSmallThreads = 512, kSmallWaves = 8;
constexpr int kSmallQuads = 4;   // 16-byte vectors of columns of a workgroup
constexpr int kSmallRows = 8;    // rows in flight per group of lanes
constexpr int kSmallDown = 4;    // down rows a thread holds at a time
constexpr int kSmallMaxK = 4096; // hidden values in LDS
constexpr int kReduceGroups = 32;  // groups of slices in decode_reduce_kernel: 256 threads, eight column quads
constexpr int kSmallSlices = 8 * kReduceGroups;  // most slices of the neurons, two a thread

// Shared hidden values, two words each: half of the call's tag and the value's bits.  A value is there where both halves are the
// call's and both values the same, so nothing has to be cleared, and calls on other streams that come to use the same row
// (every sixteenth) can at most take each other's values away.
constexpr int kSmallCalls = 16, kSmallTokens = 4;
static __device__ unsigned long long g_hidden[kSmallCalls * kSmallTokens][kSmallMaxK][2];
static __device__ unsigned int g_gave_up;  // workgroups so far that computed all hidden values after all

// The value L lanes further on in the same sixteen (past them: zero).
template <int L>
__device__ __forceinline__ float lane_behind(float v) {
  return u2f((uint32_t)__builtin_amdgcn_mov_dpp((int)f2u(v), 0x100 + L, 0xf, 0xf, true));
}

// G lanes share a row of d elements, NI vectors each.
template <class D, int G, int NI, bool SWIGLU, bool SHARE>
__global__ __launch_bounds__(kSmallThreads) void ffn_decode_small_kernel(std::conditional_t<SHARE, SharedArgs, SmallArgs> a) {
  using T = typename D::T;
  constexpr int VEC = D::VEC;
  constexpr int GPW = 64 / G, STEP = kSmallWaves * GPW;  // rows side by side
  __shared__ float h[kSmallMaxK];
  __shared__ float sums[kSmallWaves][kSmallQuads * VEC];
  __shared__ int late;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y;
  const size_t rowbytes = (size_t)a.d * sizeof(T);
  const int vecs = a.d / VEC;
  const char* x = reinterpret_cast<const char*>(a.x) + (size_t)b * rowbytes;
  const char* up = reinterpret_cast<const char*>(a.w_up);
  const char* gate = reinterpret_cast<const char*>(a.w_gate);

  const int gl = lane % G, row0 = wave * GPW + lane / G;
  uint32_t off[NI];
  float xr[NI][VEC];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int v = i * G + gl;
    off[i] = v < vecs ? (uint32_t)v * 16u : 0u;  // a vector past the end re-reads the first; its x is zero
    uint4 xv = ld16(x + off[i]);
    // without a branch: behind one, the first rows would be requested only when x has come (4 x 154 x 48 bf16 3.93 -> 4.11 us)
    const uint32_t there = v < vecs ? 0xffffffffu : 0u;
    xv.x &= there; xv.y &= there; xv.z &= there; xv.w &= there;
    unpack<D>(xv, xr[i]);
  }
  // Columns of y: 16 bytes of them a thread, and one slice of the neurons or, of more than 128, two: rows from a0 to a1 and
  // from b0 to b1.  Lanes: two bits of the columns (neighbours, as they lie), two of the slice, two of the reduction's group.  The
  // first rows, which need no hidden value to be requested:
  const int q = lane & 3, group = wave * 4 + (lane >> 4), first = group + kReduceGroups * (lane >> 2 & 3);
  const bool two = a.n_wg > kSmallSlices / 2;  // uniform
  auto slice = [&](int w) { return w < a.n_wg ? (int)__umulhi((uint32_t)w * (uint32_t)a.K, a.inv_n_wg) : a.K; };
  const int a0 = slice(first), a1 = slice(first + 1);
  const int b0 = two ? slice(first + kSmallSlices / 2) : 0, b1 = two ? slice(first + kSmallSlices / 2 + 1) : 0;
  const int vec = blockIdx.x * kSmallQuads + q;
  const char* down = reinterpret_cast<const char*>(a.w_down) + (size_t)(vec < vecs ? vec : 0) * 16;
  // of the rows that a thread holds at a time, the second half is of its second slice, if it has one
  auto row_of = [&](int i, int r) { return two ? (i < kSmallDown / 2 ? a0 + r + i : b0 + r + i - kSmallDown / 2) : a0 + r + i; };
  auto end_of = [&](int i) { return two && i >= kSmallDown / 2 ? b1 : a1; };
  const int step = two ? kSmallDown / 2 : kSmallDown;  // rows of a slice at a time
  uint4 dn[2][kSmallDown];
  auto request_down = [&](uint4 (&to)[kSmallDown], int r) {
#pragma unroll
    for (int i = 0; i < kSmallDown; ++i) to[i] = ld16(down + (size_t)min(row_of(i, r), a.K - 1) * rowbytes);
  };
  request_down(dn[0], 0);

  constexpr int SH = G / kSmallRows;  // lanes that end with the same row's sum
  auto hidden = [&](int lo, int hi, auto sink) {  // of the rows lo .. hi - 1
    for (int r0 = lo + row0; r0 - row0 < hi; r0 += kSmallRows * STEP) {
      const int mine = r0 + gl / SH * STEP;  // the row whose sum ends in this lane
      float bias = 0.f;
      if (!SWIGLU && a.b_up) bias = to_float<D>(reinterpret_cast<const T*>(a.b_up)[min(mine, hi - 1)]);
      uint4 u[kSmallRows][NI], g[SWIGLU ? kSmallRows : 1][NI];
#pragma unroll
      for (int s = 0; s < kSmallRows; ++s) {
        const size_t row = (size_t)min(r0 + s * STEP, hi - 1) * rowbytes;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (SWIGLU) g[s][i] = ld16(gate + row + off[i]);
          u[s][i] = ld16(up + row + off[i]);
        }
      }
      float zu[kSmallRows], zg[kSmallRows];
#pragma unroll
      for (int s = 0; s < kSmallRows; ++s) {
        zu[s] = zg[s] = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          float f[VEC];
          unpack<D>(u[s][i], f);
#pragma unroll
          for (int c = 0; c < VEC; ++c) zu[s] = fmaf(f[c], xr[i][c], zu[s]);
          if (SWIGLU) {
            unpack<D>(g[s][i], f);
#pragma unroll
            for (int c = 0; c < VEC; ++c) zg[s] = fmaf(f[c], xr[i][c], zg[s]);
          }
        }
      }
      halve_rows<kSmallRows, G / 2>(zu, lane);
      if (SWIGLU) halve_rows<kSmallRows, G / 2>(zg, lane);
      if (gl % SH == 0 && mine < hi) sink(mine, SWIGLU ? silu(zg[0]) * zu[0] : fmaxf(zu[0] + bias, 0.f));
    }
  };
  auto keep = [&](int k, float v) { h[k] = v; };
  if constexpr (SHARE) {
    // an equal part of the rows each, handed to the others as they come
    const int lo = (int)((uint32_t)a.K * blockIdx.x / gridDim.x), hi = (int)((uint32_t)a.K * (blockIdx.x + 1) / gridDim.x);
    unsigned long long(*words)[2] = g_hidden[a.slot + b];
    const unsigned long long t0 = (unsigned long long)a.tag[0] << 32, t1 = (unsigned long long)a.tag[1] << 32;
    if (tid == 0) late = a.patience == 0 && hi - lo < a.K;
    hidden(lo, hi, [&](int k, float v) {
      h[k] = v;
      __hip_atomic_store(&words[k][0], t0 | f2u(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&words[k][1], t1 | f2u(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
    __syncthreads();
    const long long start = __builtin_amdgcn_s_memrealtime();
    constexpr int kAtOnce = 4;
    for (int k0 = a.patience == 0 ? a.K : tid; k0 < a.K; k0 += kAtOnce * kSmallThreads) {
      uint32_t wanted = 0;
#pragma unroll
      for (int i = 0; i < kAtOnce; ++i) {
        const int k = k0 + i * kSmallThreads;
        if (k < a.K && (k < lo || k >= hi)) wanted |= 1u << i;
      }
      while (wanted) {
        unsigned long long w0[kAtOnce], w1[kAtOnce];
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) {
          const int k = min(k0 + i * kSmallThreads, a.K - 1);
          w0[i] = __hip_atomic_load(&words[k][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          w1[i] = __hip_atomic_load(&words[k][1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int i = 0; i < kAtOnce; ++i) {
          if ((wanted >> i & 1) && w0[i] == (t0 | (uint32_t)w0[i]) && w1[i] == (t1 | (uint32_t)w0[i])) {
            h[k0 + i * kSmallThreads] = u2f((uint32_t)w0[i]);
            wanted &= ~(1u << i);
          }
        }
        if (wanted && (long long)__builtin_amdgcn_s_memrealtime() - start > a.patience) {
          late = 1;
          break;
        }
      }
      if (wanted) break;
    }
    __syncthreads();
    if (late) {
      if (tid == 0) atomicAdd(&g_gave_up, 1u);
      hidden(0, a.K, keep);
    }
  } else {
    hidden(0, a.K, keep);
  }
  if (a.most_rows > step) request_down(dn[1], step);  // uniform
  __syncthreads();

  // the slices' sums, row by row
  float acc[2][VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) acc[0][c] = acc[1][c] = 0.f;
  auto add_row = [&](const uint4& from, float hk, bool valid, float (&to)[VEC]) {
    if (valid) {
      float f[VEC];
      unpack<D>(from, f);
#pragma unroll
      for (int c = 0; c < VEC; ++c) to[c] = fmaf(hk, f[c], to[c]);
    }
  };
  auto rows = [&](const uint4 (&from)[kSmallDown], int r) {
    float hk[kSmallDown];
#pragma unroll
    for (int i = 0; i < kSmallDown; ++i) hk[i] = h[min(row_of(i, r), a.K - 1)];
#pragma unroll
    for (int i = 0; i < kSmallDown / 2; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[0]);
    if (two) {
#pragma unroll
      for (int i = kSmallDown / 2; i < kSmallDown; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[1]);
    } else {
#pragma unroll
      for (int i = kSmallDown / 2; i < kSmallDown; ++i) add_row(from[i], hk[i], row_of(i, r) < end_of(i), acc[0]);
    }
  };
  for (int r = 0; r < a.most_rows; r += 2 * step) {
    rows(dn[0], r);
    if (r + 2 * step < a.most_rows) request_down(dn[0], r + 2 * step);
    if (r + step < a.most_rows) {
      rows(dn[1], r + step);
      if (r + 3 * step < a.most_rows) request_down(dn[1], r + 3 * step);
    }
  }
  // The sums of the slices, in the order of decode_reduce_kernel: slices of a group (32 apart) one after the other, groups of
  // eight pairwise, the eights one after the other.  A slice that there is not adds zero.
#pragma unroll
  for (int c = 0; c < VEC; ++c) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (i == 0 || two) {
        t += acc[i][c];
        t += lane_behind<4>(acc[i][c]);
        t += lane_behind<8>(acc[i][c]);
        t += lane_behind<12>(acc[i][c]);
      }
    }
    const auto s16 = __builtin_amdgcn_permlane16_swap(f2u(t), f2u(t), false, false);
    t = u2f(s16[0]) + u2f(s16[1]);  // lanes 16 apart, then 32
    const auto s32 = __builtin_amdgcn_permlane32_swap(f2u(t), f2u(t), false, false);
    t = u2f(s32[0]) + u2f(s32[1]);
    if ((lane & 0x3c) == 0) sums[wave][q * VEC + c] = t;
  }
  __syncthreads();
  const int col = blockIdx.x * kSmallQuads * VEC + tid;
  if (tid < kSmallQuads * VEC && col < a.d) {
    float t = sums[0][tid] + sums[1][tid];
#pragma unroll
    for (int w = 2; w < kSmallWaves; w += 2) t += sums[w][tid] + sums[w + 1][tid];
    const float bias = a.b_down ? to_float<D>(reinterpret_cast<const T*>(a.b_down)[col]) : 0.f;
    reinterpret_cast<T*>(a.y)[(size_t)b * a.d + col] = from_float<D>(t + bias);
  }
}

template <class D, int G, int NI, bool SWIGLU>
int launch_rows(const SharedArgs& a, int B, bool share, hipStream_t s) {
  const int vecs = a.d / D::VEC;
  const dim3 grid((vecs + kSmallQuads - 1) / kSmallQuads, B), block(kSmallThreads);
  if (share) hipLaunchKernelGGL((ffn_decode_small_kernel<D, G, NI, SWIGLU, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((ffn_decode_small_kernel<D, G, NI, SWIGLU, false>), grid, block, 0, s, static_cast<const SmallArgs&>(a));
  CI_HIP_CHECK_LAUNCH();
  return CI_OK;
}

template <class D, bool SWIGLU>
int launch_typed(const SharedArgs& a, int B, bool share, hipStream_t s) {
  const int vecs = a.d / D::VEC;
  if (vecs <= 16) return launch_rows<D, 16, 1, SWIGLU>(a, B, share, s);
  if (vecs <= 32) return launch_rows<D, 32, 1, SWIGLU>(a, B, share, s);
  if (vecs <= 64) return launch_rows<D, 64, 1, SWIGLU>(a, B, share, s);
  return launch_rows<D, 64, 2, SWIGLU>(a, B, share, s);
}

template <class D>
int launch_dtype(const SharedArgs& a, int B, int act, bool share, hipStream_t s) {
  return act == CI_ACT_SWIGLU ? launch_typed<D, true>(a, B, share, s) : launch_typed<D, false>(a, B, share, s);
}

// 64 bits that no other call of this process has, from a start that no other process has (memory keeps what was in it).  Nothing in
// it throws; where the system has no random numbers ready, process and time take their place.
uint64_t first_call() noexcept {
  uint64_t v = 0;
  if (getrandom(&v, sizeof(v), GRND_NONBLOCK) == (ssize_t)sizeof(v)) return v;
  timespec t{};
  clock_gettime(CLOCK_REALTIME, &t);
  return ((uint64_t)getpid() << 32 ^ (uint64_t)t.tv_sec * 1000000000u ^ (uint64_t)t.tv_nsec) * 0x9e3779b97f4a7c15u;
}
uint64_t next_call() noexcept {
  static std::atomic<uint64_t> calls{first_call()};
  return calls.fetch_add(1, std::memory_order_relaxed);
}

}  // namespace

// Where one launch beats two, by elements of the up and gate matrices with rows rounded up to what the lanes of their loads hold.
// Launched call by call, two launches are bound by the host and one is faster up to kSmallElements, over one to four tokens,
// both activations and all types; replayed from a graph two cost no host time, and one is faster up to kSmallElementsGraph only (us,
// two launches / one; call by call, then from a graph):
//   one token     fp32  256 x 256   7.7 / 5.2, 5.7 / 5.3     256 x 288  7.8 / 5.7, 5.7 / 5.9   256 x 424 7.8 / 6.9, 5.8 / 6.9
//                       128 x 1024  7.7 / 7.6, 5.7 / 7.6     gated 512 x 72  7.8 / 6.6, 6.2 / 6.7
//                 fp16  256 x 256   7.6 / 4.8, 5.8 / 4.9     256 x 512  7.6 / 6.4, 5.9 / 6.5   gated 256 x 256 7.7 / 5.8, 6.1 / 5.8
//                 bf16  256 x 424   7.8 / 6.4, 6.0 / 6.5     gated 256 x 256 7.8 / 6.0, 6.2 / 6.0
//   four tokens   fp32  256 x 256   7.9 / 5.2, 5.9 / 5.2     256 x 512  7.8 / 7.8, 6.7 / 8.1   gated 512 x 72 7.8 / 6.9, 6.3 / 7.0
//                 fp16  256 x 512   7.9 / 6.8, 6.9 / 6.9     gated 256 x 256  7.8 / 5.6, 6.6 / 5.7
// (of 208 such layers none of up to 64 K elements was slower in either way).  Both ways give the same bits.
// Call by call the hidden values of more than 64 K elements are shared where that saves a workgroup three batches of rows or more and
// there are three workgroups or more (a call's words are its own only once, so a captured call, which runs many times, has none).  us,
// every workgroup all / shared:
//   fp32  256 x 256 (4 batches, 64 K) 5.38 / 5.33    256 x 288 (5) 5.81 / 5.33    256 x 384 (6) 6.37 / 5.31   128 x 576 (5) 5.95 / 5.69
//         512 x 192 (3) 5.84 / 6.08   512 x 224 (4) 6.86 / 6.10   gated 256 x 192 (3) 5.92 / 5.65   256 x 224 (4) 6.73 / 5.71   512 x 112 (2) 6.65 / 6.37
//         four tokens   256 x 288 6.02 / 5.80    512 x 192 5.84 / 6.11   512 x 224 6.93 / 6.20
//   fp16  256 x 384 (3) 5.59 / 5.98   256 x 448 (4) 6.26 / 5.86   512 x 224 (4) 6.62 / 5.81   1024 x 128 (2) 5.84 / 6.14   bf16 gated 256 x 256 (2) 6.11 / 6.42
//   one workgroup    fp32  16 x 1025 6.49 / 7.83, 16 x 2048 8.83 / 10.65    fp16  32 x 769 6.59 / 7.61
//   two              fp32  32 x 1025 (5 batches, 2 saved) 6.51 / 7.14   32 x 1537 (7, 3) 8.08 / 8.42   32 x 2048 (8, 4) 8.96 / 8.86
//   three            fp32  48 x 1025 (5, 3) 6.51 / 6.45   48 x 1537 (7, 4) 8.18 / 7.65   gated 48 x 1024 (4, 2) 6.84 / 7.12
// Of 164 such layers in the range of the rule none is more than 0.7 % slower shared, and with layers in turn all are 7 % faster or more.
constexpr int64_t kSmallElements = 128 * 1024, kSmallElementsGraph = 64 * 1024, kSmallBatchesSaved = 3, kSmallSharers = 3;
DecodeSmall decode_small_way(int64_t B, int64_t K, int64_t d, int dtype, int act, int n_wg, hipStream_t s) {
  const int mode = params().decode_small;
  const int64_t vec = 16 / elem_bytes(dtype), vecs = d / vec;
  if (mode == 0 || K < 1 || K > kSmallMaxK || vecs > 128 || B > kSmallTokens || n_wg > kSmallSlices) return DecodeSmall::kNo;
  const int64_t held = vecs <= 16 ? 16 : vecs <= 32 ? 32 : (vecs + 63) / 64 * 64;
  const int64_t elements = (act == CI_ACT_SWIGLU ? 2 : 1) * K * held * vec;
  if (mode == 2) return DecodeSmall::kAll;
  if (mode == 1 && elements > kSmallElements) return DecodeSmall::kNo;
  if (mode == 1 && elements <= kSmallElementsGraph) return DecodeSmall::kAll;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;  // the null stream is never captured
  if (s && !(hipStreamIsCapturing(s, &capture) == hipSuccess && capture == hipStreamCaptureStatusNone)) return DecodeSmall::kNo;
  const int64_t lanes = vecs <= 16 ? 16 : vecs <= 32 ? 32 : 64, rows = kSmallRows * kSmallWaves * (64 / lanes);
  const int64_t sharers = (vecs + kSmallQuads - 1) / kSmallQuads, batches = (K + rows - 1) / rows;
  const bool pays = sharers >= kSmallSharers && batches - (batches + sharers - 1) / sharers >= kSmallBatchesSaved;
  return mode == 3 || pays ? DecodeSmall::kShare : DecodeSmall::kAll;
}

int decode_small_gave_up(uint32_t* out) {
  return hipMemcpyFromSymbol(out, HIP_SYMBOL(g_gave_up), sizeof(*out)) == hipSuccess ? CI_OK : CI_ERR_HIP;
}

int launch_ffn_decode_small(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act, void* y, int n_wg, bool share,
                            hipStream_t s) {
  const int K = (int)w->K;
  const uint64_t call = share ? next_call() : 0;
  const SharedArgs a{{x, w->w_up, w->w_gate, w->b_up, w->w_down, w->b_down, y, K, (int)w->d, n_wg,
                      (uint32_t)(((1ull << 32) + n_wg - 1) / n_wg), (K + n_wg - 1) / n_wg},
                     {(uint32_t)(call >> 32), (uint32_t)call}, (int)(call % kSmallCalls) * kSmallTokens,
                     (int)params().decode_small_patience};
  switch (dtype) {
    case CI_F32: return launch_dtype<F32>(a, (int)B, act, share, s);
    case CI_F16: return launch_dtype<F16>(a, (int)B, act, share, s);
    case CI_BF16: return launch_dtype<BF16>(a, (int)B, act, share, s);
  }
  return CI_ERR_BAD_DTYPE;
}

}  // namespace ci
