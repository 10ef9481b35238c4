// C ABI of libcoreinfer: argument validation (host only, before any HIP
// call) and dispatch to the kernel launchers.
#include <math.h>
#include <string.h>

#include <mutex>

#include <algorithm>

#include "common.hpp"
#include "coreinfer_dev.h"
#include "gemm_common.hpp"

namespace ci {

Params& params() {
  static Params p;
  return p;
}

int device_info(DeviceInfo* out) {
  static std::mutex mu;
  static int cached_cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return CI_ERR_HIP;
  if (dev < 0 || dev >= 64) return CI_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  if (cached_cus[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
      return CI_ERR_HIP;
    cached_cus[dev] = cus;
  }
  out->cus = cached_cus[dev];
  return CI_OK;
}

namespace {

bool dtype_ok(int dt) { return dt == CI_F32 || dt == CI_F16 || dt == CI_BF16; }
bool act_ok(int a) { return a == CI_ACT_RELU || a == CI_ACT_SWIGLU; }
bool layout_ok(int l) { return l == CI_DOWN_OUT_MAJOR || l == CI_DOWN_NEURON_MAJOR; }
int vec_of(int dt) { return dt == CI_F32 ? 4 : 8; }
size_t round256(size_t n) { return (n + 255) / 256 * 256; }

// parts per million of a keep fraction; 0 if the fraction is not in (0, 1]
int64_t fraction_ppm(double frac) {
  if (!(frac > 0.0) || !(frac <= 1.0)) return 0;
  const int64_t q = (int64_t)floor(frac * 1e6 + 0.5);
  return q < 1 ? 0 : q;
}
int64_t keep(int64_t q, int64_t n) { return (q * n + 999999) / 1000000; }

constexpr int64_t kMaxSplits = 1024;

}  // namespace
}  // namespace ci

using namespace ci;

extern "C" {

const char* coreinfer_strerror(int status) {
  switch (status) {
    case CI_OK: return "ok";
    case CI_ERR_INVALID_ARG: return "invalid argument";
    case CI_ERR_BAD_DTYPE: return "unknown dtype or activation";
    case CI_ERR_BAD_LAYOUT: return "bad layout or alignment";
    case CI_ERR_WORKSPACE: return "workspace missing or too small";
    case CI_ERR_HIP: return "HIP runtime error";
    case CI_ERR_UNSUPPORTED: return "unsupported configuration";
  }
  return "unknown status";
}

int coreinfer_version(void) { return 2; }

int coreinfer_dev_fused_plan(int64_t K, int64_t d, int dtype, int act, int* out) {
  if (!out || K < 1 || d < 1 || d > (1 << 15)) return CI_ERR_INVALID_ARG;
  if (act != CI_ACT_RELU && act != CI_ACT_SWIGLU) return CI_ERR_INVALID_ARG;
  return fused_decode_plan(K, d, dtype, act, out);
}

int coreinfer_dev_decode_slices(int64_t B, int64_t K, int64_t d, int dtype, int gathered, int* slices) {
  if (!slices || B < 1 || B > 65535 || K < 1 || K > CI_MAX_NEURONS || d < 1 || d > CI_MAX_DMODEL || !dtype_ok(dtype))
    return CI_ERR_INVALID_ARG;
  *slices = decode_splits(B, K, d * elem_bytes(dtype), gathered != 0);
  return CI_OK;
}

int coreinfer_dev_decode_small(int64_t B, int64_t K, int64_t d, int dtype, int act, void* stream, int* way) {
  if (!way || B < 1 || B > 65535 || K < 1 || K > CI_MAX_NEURONS || d < 1 || d > CI_MAX_DMODEL || !dtype_ok(dtype) ||
      (act != CI_ACT_RELU && act != CI_ACT_SWIGLU))
    return CI_ERR_INVALID_ARG;
  *way = (int)decode_small_way(B, K, d, dtype, act, decode_splits(B, K, d * elem_bytes(dtype), false), (hipStream_t)stream);
  return CI_OK;
}

int coreinfer_dev_decode_small_gave_up(uint32_t* workgroups) {
  return workgroups ? decode_small_gave_up(workgroups) : CI_ERR_INVALID_ARG;
}

int coreinfer_dev_select_layout(int64_t B, int64_t M, int64_t N, int64_t* out) {
  size_t need = 0;
  if (!out || coreinfer_select_batch_workspace_size(B, M, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  const SelectScratch sc = select_scratch(nullptr, need, M, N, B);
  out[0] = (int64_t)reinterpret_cast<uintptr_t>(sc.thr);
  out[1] = (int64_t)reinterpret_cast<uintptr_t>(sc.hist);
  out[2] = (int64_t)reinterpret_cast<uintptr_t>(sc.counts);
  out[3] = sc.part ? (int64_t)reinterpret_cast<uintptr_t>(sc.part) : -1;
  return CI_OK;
}

// Development hook (coreinfer_dev.h), not part of the installed interface: launch-shape parameters for tuning sweeps
// and tests.
namespace {
struct KnobEntry {
  const char* name;
  Knob Params::*knob;
  bool (*ok)(int);
};
const KnobEntry kKnobs[] = {
    {"decode_wgs_per_cu", &Params::decode_wgs_per_cu, [](int v) { return v >= 1 && v <= 16; }},
    {"decode_wgs", &Params::decode_wgs, [](int v) { return v >= 0 && v <= 1024; }},
    {"decode_threads", &Params::decode_threads, [](int v) { return v >= 0 && v <= 1024; }},
    {"decode_depth", &Params::decode_depth, [](int v) { return v == 4 || v == 8 || v == 16; }},
    {"reduce_cq", &Params::reduce_cq, [](int v) { return v == 4 || v == 8 || v == 16; }},
    {"reduce_threads", &Params::reduce_threads, [](int v) { return v == 64 || v == 128 || v == 256 || v == 512 || v == 1024; }},
    {"decode_small", &Params::decode_small, [](int v) { return v >= 0 && v <= 3; }},
    {"decode_small_patience", &Params::decode_small_patience, [](int v) { return v >= 0 && v <= 100000; }},
    {"decode_nt_store", &Params::decode_nt_store, [](int v) { return v == 0 || v == 1; }},
    {"fused_depth", &Params::fused_depth, [](int v) { return v == 4 || v == 8; }},
    {"fused_threads", &Params::fused_threads, [](int v) { return v >= 0 && v <= 1024; }},
    {"fused_chunks", &Params::fused_chunks, [](int v) { return v >= 2 && v <= 64; }},
    {"fused_chunk_size", &Params::fused_chunk_size, [](int v) { return v >= 0 && v <= 6144; }},
    {"fused_wgs", &Params::fused_wgs, [](int v) { return v >= 0 && v <= 1024; }},
    {"fused_guard_us10", &Params::fused_guard_us10, [](int v) { return v >= 0 && v <= 1000; }},
    {"fused_chunk_cost10", &Params::fused_chunk_cost10, [](int v) { return v >= 0 && v <= 1000; }},
    {"fused_window_slots", &Params::fused_window_slots, [](int v) { return v >= 0 && v <= 1000; }},
    {"fused_ablate", &Params::fused_ablate, [](int v) { return v >= 0 && v <= 2; }},
    {"fused_aux", &Params::fused_aux, [](int v) { return v == -1 || v == -2 || v == 0 || v == 16; }},
    {"select_bytes", &Params::select_bytes, [](int v) { return v >= 0 && v <= 2; }},
    {"select_def2_single", &Params::select_def2_single, [](int v) { return v == 0 || v == 1; }},
    {"select_wgs_per_cu", &Params::select_wgs_per_cu, [](int v) { return v >= 1 && v <= 8; }},
    {"gemm_tile", &Params::gemm_tile, [](int v) { return (v >= -1 && v < kShapes) || (v >= kSlim && slim_built((v - kSlim) / 16, v % 16)); }},
    {"gemm_once", &Params::gemm_once, [](int v) { return v >= 0 && v <= 2; }},
    {"gemm_splits", &Params::gemm_splits, [](int v) { return v >= 0 && v <= 8; }},
    {"gemv_wgs_per_cu", &Params::gemv_wgs_per_cu, [](int v) { return v >= 1 && v <= 32; }},
    {"gemv_cols_wgs_per_cu", &Params::gemv_cols_wgs_per_cu, [](int v) { return v >= 1 && v <= 4; }},
    {"gathered_union", &Params::gathered_union, [](int v) { return v >= 0 && v <= 2; }},
    {"union_depth", &Params::union_depth, [](int v) { return v == 8 || v == 16; }},
    {"union_down_threads", &Params::union_down_threads, [](int v) { return v >= 64 && v <= 512; }},
    {"union_up_wgs_per_cu", &Params::union_up_wgs_per_cu, [](int v) { return v >= 1 && v <= 8; }},
    {"union_down_wgs_per_cu", &Params::union_down_wgs_per_cu, [](int v) { return v >= 1 && v <= 16; }},
    {"union_super", &Params::union_super, [](int v) { return (v == 0 || (v >= 16 && v <= 256)); }},
};

const KnobEntry* find_knob(const char* name) {
  if (name)
    for (const KnobEntry& e : kKnobs)
      if (!strcmp(name, e.name)) return &e;
  return nullptr;
}
}  // namespace

int coreinfer_dev_set_param(const char* name, int value) {
  const KnobEntry* e = find_knob(name);
  if (!e || !e->ok(value)) return CI_ERR_INVALID_ARG;
  params().*(e->knob) = value;
  return CI_OK;
}

int coreinfer_dev_get_param(const char* name, int* value) {
  const KnobEntry* e = find_knob(name);
  if (!e || !value) return CI_ERR_INVALID_ARG;
  *value = params().*(e->knob);
  return CI_OK;
}

const char* coreinfer_dev_param_name(int index) {
  return index >= 0 && index < (int)(sizeof(kKnobs) / sizeof(kKnobs[0])) ? kKnobs[index].name : nullptr;
}

int coreinfer_keep_count(double frac, int64_t n, int64_t* k) {
  if (!k || n < 0 || n > ((int64_t)1 << 40)) return CI_ERR_INVALID_ARG;
  const int64_t q = fraction_ppm(frac);
  if (q == 0) return CI_ERR_INVALID_ARG;
  *k = keep(q, n);
  return CI_OK;
}

int coreinfer_select_workspace_size(int64_t M, int64_t N, size_t* bytes) {
  if (!bytes || M < 1 || M > CI_MAX_TOKENS || N < 1 || N > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  SelectWs w;
  select_ws_layout(M, N, &w);
  *bytes = w.total;
  return CI_OK;
}

int coreinfer_select(const float* act, int64_t M, int64_t N, int64_t ld, double alpha, double beta,
                     int32_t* core_idx, int32_t* counts, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (coreinfer_select_workspace_size(M, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!act || !core_idx) return CI_ERR_INVALID_ARG;
  const int64_t qa = fraction_ppm(alpha), qb = fraction_ppm(beta);
  if (qa == 0 || qb == 0) return CI_ERR_INVALID_ARG;
  if (ld < N) return CI_ERR_BAD_LAYOUT;
  if ((reinterpret_cast<uintptr_t>(act) & 3u) || (reinterpret_cast<uintptr_t>(core_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(counts) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < select_ws_least(M, N)) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  const SelectScratch sc = select_scratch(ws, ws_bytes, M, N);
  int32_t* cnt = counts ? counts : sc.counts;
  return launch_select(act, CI_F32, 0, M, N, ld, qa, keep(qb, N), M, core_idx, cnt, &sc, kSelTokens | kSelFinal,
                       (hipStream_t)stream);
}

int coreinfer_select_batch_workspace_size(int64_t B, int64_t M, int64_t N, size_t* bytes) {
  if (!bytes || B < 1 || B > 65535 || M < 1 || M > CI_MAX_TOKENS || N < 1 || N > CI_MAX_NEURONS ||
      B * M > (int64_t)CI_MAX_TOKENS * 64)
    return CI_ERR_INVALID_ARG;
  SelectWs w;
  select_ws_layout(M, N, &w, B);
  *bytes = w.total;
  return CI_OK;
}

int coreinfer_select_batch(const float* act, int64_t B, int64_t M, int64_t N, int64_t ld, double alpha, double beta,
                           int32_t* core_idx, int32_t* counts, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (coreinfer_select_batch_workspace_size(B, M, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!act || !core_idx) return CI_ERR_INVALID_ARG;
  const int64_t qa = fraction_ppm(alpha), qb = fraction_ppm(beta);
  if (qa == 0 || qb == 0) return CI_ERR_INVALID_ARG;
  if (ld < N) return CI_ERR_BAD_LAYOUT;
  if ((reinterpret_cast<uintptr_t>(act) & 3u) || (reinterpret_cast<uintptr_t>(core_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(counts) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < select_ws_least(M, N, B)) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  const int64_t K = keep(qb, N);
  const SelectScratch sc = select_scratch(ws, ws_bytes, M, N, B);
  int32_t* cnt = counts ? counts : sc.counts;
  if (B == 1 || select_batch_ok(M, N))
    return launch_select(act, CI_F32, 0, M, N, ld, qa, K, M, core_idx, cnt, &sc, kSelTokens | kSelFinal,
                         (hipStream_t)stream, (int)B, N);
  // one sentence after the other, each in the batch's layout: its thresholds and histogram take the front of theirs,
  // and its byte counts lie behind the counters of all sentences
  for (int64_t b = 0; b < B; ++b) {
    const int rc = launch_select(act + (size_t)b * M * ld, CI_F32, 0, M, N, ld, qa, K, M, core_idx + b * K, cnt + b * N,
                                 &sc, kSelTokens | kSelFinal, (hipStream_t)stream);
    if (rc != CI_OK) return rc;
  }
  return CI_OK;
}

int coreinfer_select_hidden(const void* hidden, int dtype, int act, int64_t M, int64_t N, int64_t ld, double alpha,
                            double beta, int32_t* core_idx, int32_t* counts, void* ws, size_t ws_bytes,
                            void* stream) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  size_t need = 0;
  if (coreinfer_select_workspace_size(M, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!hidden || !core_idx) return CI_ERR_INVALID_ARG;
  const int64_t qa = fraction_ppm(alpha), qb = fraction_ppm(beta);
  if (qa == 0 || qb == 0) return CI_ERR_INVALID_ARG;
  if (ld < N) return CI_ERR_BAD_LAYOUT;
  const uintptr_t elem = dtype == CI_F32 ? 4 : 2;
  if ((reinterpret_cast<uintptr_t>(hidden) & (elem - 1)) || (reinterpret_cast<uintptr_t>(core_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(counts) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < select_ws_least(M, N)) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  const SelectScratch sc = select_scratch(ws, ws_bytes, M, N);
  int32_t* cnt = counts ? counts : sc.counts;
  return launch_select(hidden, dtype, act == CI_ACT_SWIGLU ? 1 : 0, M, N, ld, qa, keep(qb, N), M, core_idx, cnt, &sc,
                       kSelTokens | kSelFinal, (hipStream_t)stream);
}

int coreinfer_count_tokens(const float* act, int64_t M, int64_t N, int64_t ld, double alpha,
                           int32_t* counts, int accumulate, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (coreinfer_select_workspace_size(M, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!act || !counts) return CI_ERR_INVALID_ARG;
  const int64_t qa = fraction_ppm(alpha);
  if (qa == 0) return CI_ERR_INVALID_ARG;
  if (ld < N) return CI_ERR_BAD_LAYOUT;
  if ((reinterpret_cast<uintptr_t>(act) & 3u) || (reinterpret_cast<uintptr_t>(counts) & 3u)) return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < select_ws_least(M, N)) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  const SelectScratch sc = select_scratch(ws, ws_bytes, M, N);
  return launch_select(act, CI_F32, 0, M, N, ld, qa, 1, M, nullptr, counts, &sc,
                       kSelTokens | (accumulate ? kSelAccumulate : 0), (hipStream_t)stream);
}

int coreinfer_count_select(const int32_t* counts, int64_t N, int64_t max_count, double beta,
                           int32_t* core_idx, void* ws, size_t ws_bytes, void* stream) {
  if (!counts || !core_idx || N < 1 || N > CI_MAX_NEURONS || max_count < 0 || max_count > CI_MAX_TOKENS)
    return CI_ERR_INVALID_ARG;
  const int64_t qb = fraction_ppm(beta);
  if (qb == 0) return CI_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(counts) & 3u) || (reinterpret_cast<uintptr_t>(core_idx) & 3u)) return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < 256) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  // Def. 2 alone runs in one workgroup and needs no scratch
  return launch_select(nullptr, CI_F32, 0, 0, N, N, 1, keep(qb, N), max_count, core_idx, const_cast<int32_t*>(counts),
                       nullptr, kSelFinal, (hipStream_t)stream);
}

int coreinfer_group_select(const int32_t* core_sets, int64_t G, int64_t K, int64_t N, double gamma,
                           int32_t* core_idx, int32_t* counts, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (G < 1 || G > CI_MAX_TOKENS || coreinfer_select_workspace_size(G, N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!core_sets || !core_idx || K < 0 || K > N) return CI_ERR_INVALID_ARG;
  const int64_t qg = fraction_ppm(gamma);
  if (qg == 0) return CI_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(core_sets) & 3u) || (reinterpret_cast<uintptr_t>(core_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(counts) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < select_ws_least(G, N)) return CI_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) & 15u) return CI_ERR_BAD_LAYOUT;
  const SelectScratch sc = select_scratch(ws, ws_bytes, G, N);
  int32_t* cnt = counts ? counts : sc.counts;
  hipStream_t s = (hipStream_t)stream;
  // clear the counters, count the groups' members, then Def. 2 with gamma on the counters
  int rc = launch_select(nullptr, CI_F32, 0, 0, N, N, 1, 1, G, nullptr, cnt, nullptr, kSelZero, s);
  if (rc != CI_OK) return rc;
  rc = launch_scatter_count(core_sets, G * K, N, cnt, s);
  if (rc != CI_OK) return rc;
  return launch_select(nullptr, CI_F32, 0, 0, N, N, 1, keep(qg, N), G, core_idx, cnt, nullptr, kSelFinal, s);
}

int coreinfer_core_similarity(const int32_t* set_a, int64_t Ka, const int32_t* set_b, int64_t Kb,
                              int32_t* out, void* stream) {
  if (!out || Ka < 0 || Kb < 0 || Ka > CI_MAX_NEURONS || Kb > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  if ((Ka > 0 && !set_a) || (Kb > 0 && !set_b)) return CI_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(set_a) & 3u) || (reinterpret_cast<uintptr_t>(set_b) & 3u) ||
      (reinterpret_cast<uintptr_t>(out) & 3u))
    return CI_ERR_BAD_LAYOUT;
  return launch_similarity(set_a, Ka, set_b, Kb, out, (hipStream_t)stream);
}

int coreinfer_assign_group(const int32_t* set, int64_t K, const int32_t* group_sets, int64_t G, int64_t Kg,
                           int32_t* best, int32_t* inter_union, void* stream) {
  if (!best || !inter_union || G < 1 || G > CI_MAX_TOKENS || K < 0 || Kg < 0 || K > CI_MAX_NEURONS ||
      Kg > CI_MAX_NEURONS)
    return CI_ERR_INVALID_ARG;
  if ((K > 0 && !set) || (Kg > 0 && !group_sets)) return CI_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(set) & 3u) || (reinterpret_cast<uintptr_t>(group_sets) & 3u) ||
      (reinterpret_cast<uintptr_t>(best) & 3u) || (reinterpret_cast<uintptr_t>(inter_union) & 3u))
    return CI_ERR_BAD_LAYOUT;
  return launch_assign_group(set, K, group_sets, G, Kg, best, inter_union, (hipStream_t)stream);
}

int coreinfer_assign_centroid_workspace_size(int64_t N, size_t* bytes) {
  if (!bytes || N < 1 || N > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  *bytes = round256((size_t)N * sizeof(float));
  return CI_OK;
}

int coreinfer_assign_centroid(const float* act, int64_t M, int64_t N, int64_t ld, const float* centroids,
                              int64_t G, int32_t* best, float* dist, void* ws, size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (coreinfer_assign_centroid_workspace_size(N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (M < 1 || M > CI_MAX_TOKENS || G < 1 || G > CI_MAX_TOKENS) return CI_ERR_INVALID_ARG;
  if (!act || !centroids || !best || !dist) return CI_ERR_INVALID_ARG;
  if (ld < N) return CI_ERR_BAD_LAYOUT;
  if ((reinterpret_cast<uintptr_t>(act) & 3u) || (reinterpret_cast<uintptr_t>(centroids) & 3u) ||
      (reinterpret_cast<uintptr_t>(best) & 3u) || (reinterpret_cast<uintptr_t>(dist) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  return launch_assign_centroid(act, M, N, ld, centroids, G, best, dist, reinterpret_cast<float*>(ws),
                                (hipStream_t)stream);
}

int coreinfer_compact_down_ld(int64_t K, int dtype, int64_t* ld) {
  if (!dtype_ok(dtype)) return CI_ERR_BAD_DTYPE;
  if (!ld || K < 0 || K > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  *ld = compact_down_ld(K, dtype);
  return CI_OK;
}

int coreinfer_compact_preferred_layout(int64_t K, int64_t d, int dtype, int act, int* down_c_layout) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!down_c_layout || K < 0 || K > CI_MAX_NEURONS || d < 1 || d > CI_MAX_DMODEL) return CI_ERR_INVALID_ARG;
  *down_c_layout = CI_DOWN_NEURON_MAJOR;
  if (K < 1 || d % vec_of(dtype) != 0) return CI_OK;
  int plan[5];
  if (fused_decode_plan(K, d, dtype, act, plan) != CI_OK) return CI_OK;
  // Measured on MI355X (OPT-6.7B / Llama-2-7B / Llama-2-13B shapes): the two paths are within 2 % of
  // each other; the single launch wins from about 120 MB of weights per token on, where its fixed
  // cost (the exchange of the hidden values between the workgroups) is spread over more bytes.
  const double bytes = (double)(act == CI_ACT_SWIGLU ? 3 : 2) * (double)K * (double)d * (double)elem_bytes(dtype);
  if (bytes >= 120e6) *down_c_layout = CI_DOWN_OUT_MAJOR;
  return CI_OK;
}

int coreinfer_compact(const void* w_up, const void* w_gate, const void* b_up, const void* w_down,
                      int down_layout, int dtype, int act, int64_t d, int64_t N,
                      const int32_t* core_idx, int64_t K, void* w_up_c, void* w_gate_c,
                      void* b_up_c, void* w_down_c, int down_c_layout, int32_t* status, void* stream) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(down_layout) || !layout_ok(down_c_layout)) return CI_ERR_BAD_LAYOUT;
  if (d < 1 || d > CI_MAX_DMODEL || N < 1 || N > CI_MAX_NEURONS || K < 0 || K > N) return CI_ERR_INVALID_ARG;
  if (!w_up || !w_down || !w_up_c || !w_down_c || (K > 0 && !core_idx)) return CI_ERR_INVALID_ARG;
  if ((act == CI_ACT_SWIGLU) != (w_gate != nullptr) || (w_gate != nullptr) != (w_gate_c != nullptr))
    return CI_ERR_INVALID_ARG;
  if ((b_up != nullptr) != (b_up_c != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && b_up) return CI_ERR_INVALID_ARG;  // gated FFNs carry no up bias here
  if (d % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  if (!aligned16(w_up) || !aligned16(w_gate) || !aligned16(w_down) || !aligned16(w_up_c) ||
      !aligned16(w_gate_c) || !aligned16(w_down_c))
    return CI_ERR_BAD_LAYOUT;
  return launch_compact(w_up, w_gate, b_up, w_down, down_layout, dtype, d, N, core_idx, K, w_up_c,
                        w_gate_c, b_up_c, w_down_c, down_c_layout, status, (hipStream_t)stream);
}

int coreinfer_compact_update_workspace_size(int64_t N, int64_t K, size_t* bytes) {
  if (!bytes || N < 1 || N > CI_MAX_NEURONS || K < 0 || K > N) return CI_ERR_INVALID_ARG;
  *bytes = round256(((size_t)N + 3 * (size_t)K + 64) * sizeof(uint32_t));
  return CI_OK;
}

int coreinfer_compact_update(const void* w_up, const void* w_gate, const void* b_up, const void* w_down,
                             int down_layout, int dtype, int act, int64_t d, int64_t N,
                             const int32_t* new_idx, int64_t K, int32_t* slot_idx, void* w_up_c,
                             void* w_gate_c, void* b_up_c, void* w_down_c, int down_c_layout,
                             int32_t* changed, void* ws, size_t ws_bytes, void* stream) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(down_layout) || !layout_ok(down_c_layout)) return CI_ERR_BAD_LAYOUT;
  if (d < 1 || d > CI_MAX_DMODEL) return CI_ERR_INVALID_ARG;
  size_t need = 0;
  if (coreinfer_compact_update_workspace_size(N, K, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!w_up || !w_down || !w_up_c || !w_down_c || (K > 0 && (!new_idx || !slot_idx))) return CI_ERR_INVALID_ARG;
  if ((act == CI_ACT_SWIGLU) != (w_gate != nullptr) || (w_gate != nullptr) != (w_gate_c != nullptr))
    return CI_ERR_INVALID_ARG;
  if ((b_up != nullptr) != (b_up_c != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && b_up) return CI_ERR_INVALID_ARG;
  if (d % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  if (!aligned16(w_up) || !aligned16(w_gate) || !aligned16(w_down) || !aligned16(w_up_c) ||
      !aligned16(w_gate_c) || !aligned16(w_down_c) || (reinterpret_cast<uintptr_t>(new_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(slot_idx) & 3u) || (reinterpret_cast<uintptr_t>(changed) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  return launch_compact_update(w_up, w_gate, b_up, w_down, down_layout, dtype, d, N, new_idx, K, slot_idx,
                               w_up_c, w_gate_c, b_up_c, w_down_c, down_c_layout, changed,
                               reinterpret_cast<uint32_t*>(ws), (hipStream_t)stream);
}

int coreinfer_ffn_decode_workspace_size(int64_t B, int64_t K, int64_t d, size_t* bytes) {
  if (!bytes || B < 1 || B > 65535 || K < 0 || K > CI_MAX_NEURONS || d < 1 || d > CI_MAX_DMODEL)
    return CI_ERR_INVALID_ARG;
  // two-launch path: fp32 partial outputs of the neuron slices; single-launch path: a header and
  // one 8-byte word per neuron.  One size serves both, so the caller need not know the path.
  const int64_t splits = K < kMaxSplits ? K : kMaxSplits;
  const size_t two = round256((size_t)B * (size_t)splits * (size_t)d * sizeof(float)) + 256;
  const size_t one = round256(fused_decode_ws_bytes(K));
  *bytes = std::max(two, one);
  return CI_OK;
}

namespace {

// Argument checks common to the decode entry points (everything but the workspace).
int decode_check(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act, void* y) {
  if (!w) return CI_ERR_INVALID_ARG;
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(w->down_layout)) return CI_ERR_BAD_LAYOUT;
  size_t need = 0;
  if (coreinfer_ffn_decode_workspace_size(B, w->K, w->d, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!x || !y) return CI_ERR_INVALID_ARG;
  if (w->K > 0 && (!w->w_up || !w->w_down)) return CI_ERR_INVALID_ARG;
  if (w->K > 0 && (act == CI_ACT_SWIGLU) != (w->w_gate != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && w->b_up) return CI_ERR_INVALID_ARG;
  if (w->core_idx && (w->N < 1 || w->N > CI_MAX_NEURONS)) return CI_ERR_INVALID_ARG;
  if (w->d % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  const bool out_major = w->down_layout == CI_DOWN_OUT_MAJOR;
  if (out_major && w->core_idx) return CI_ERR_BAD_LAYOUT;  // gathered rows need the neuron-major matrix
  if (out_major && w->K > 0 && (w->ld_down < w->K || w->ld_down % vec_of(dtype) != 0 || w->ld_down > CI_MAX_NEURONS))
    return CI_ERR_BAD_LAYOUT;
  if (!aligned16(x) || !aligned16(y) || !aligned16(w->w_up) || !aligned16(w->w_gate) ||
      !aligned16(w->w_down) || (reinterpret_cast<uintptr_t>(w->core_idx) & 3u))
    return CI_ERR_BAD_LAYOUT;
  return CI_OK;
}

// Scratch of coreinfer_ffn_decode_static: device memory that belongs to the library, one copy per
// GPU the library runs on, held until the process ends.  Two parts that are never mixed: the tagged
// words of the single-launch path (zero when the module is loaded, which is all that path asks
// for: a call's tag is one more than the epoch the last call left) and the partial outputs of the
// two-launch path.
constexpr size_t kStaticWords = (size_t)1 << 20;     // header + 8 bytes per neuron: K <= 131024
constexpr size_t kStaticPartial = (size_t)16 << 20;  // B * slices * d fp32 partial outputs
static __device__ __align__(256) unsigned char scratch[kStaticWords + kStaticPartial];

// The array's address on the current device.  `scratch` itself is a host-side stand-in, not a device
// address: only the pointer obtained here may be handed to kernels and copies.
int static_scratch(unsigned char** out) {
  static std::mutex mu;
  static unsigned char* ptr[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return CI_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    unsigned char* p = nullptr;
    if (hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)) != hipSuccess || !p) return CI_ERR_HIP;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return CI_OK;
}

}  // namespace

int coreinfer_ffn_decode(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act,
                         void* y, void* ws, size_t ws_bytes, void* stream) {
  const int rc = decode_check(x, B, w, dtype, act, y);
  if (rc != CI_OK) return rc;
  size_t need = 0;
  if (coreinfer_ffn_decode_workspace_size(B, w->K, w->d, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  if (w->down_layout == CI_DOWN_OUT_MAJOR && w->K > 0)
    return launch_ffn_decode_fused(x, B, w, dtype, act, y, ws, (hipStream_t)stream);
  return launch_ffn_decode(x, B, w, dtype, act, y, reinterpret_cast<float*>(ws), kMaxSplits, (hipStream_t)stream);
}

int coreinfer_ffn_decode_static(const void* x, int64_t B, const ci_ffn_weights* w, int dtype, int act,
                                void* y, int32_t* status_out, void* stream) {
  const int rc = decode_check(x, B, w, dtype, act, y);
  if (rc != CI_OK) return rc;
  if (reinterpret_cast<uintptr_t>(status_out) & 3u) return CI_ERR_BAD_LAYOUT;
  const bool single = w->down_layout == CI_DOWN_OUT_MAJOR && w->K > 0;
  // what THIS call needs (not the device-independent bound of coreinfer_ffn_decode_workspace_size)
  const size_t need = single ? fused_decode_ws_bytes(w->K)
                             : (size_t)B * (size_t)decode_splits_bound(B, w->K) * (size_t)w->d * sizeof(float);
  if (need > (single ? kStaticWords : kStaticPartial)) return CI_ERR_WORKSPACE;
  unsigned char* base = nullptr;
  const int rs = static_scratch(&base);
  if (rs != CI_OK) return rs;
  hipStream_t s = (hipStream_t)stream;
  if (!single) {
    const int room = (int)std::min<size_t>(kMaxSplits, kStaticPartial / ((size_t)B * (size_t)w->d * sizeof(float)));
    const int rl = launch_ffn_decode(x, B, w, dtype, act, y, reinterpret_cast<float*>(base + kStaticWords), room, s);
    if (rl != CI_OK || !status_out) return rl;
    // the two-launch path has no bounded waits: nothing to report.  A copy, not a memset: callers may
    // be under graph capture, and base + 8 is a word of the header that no kernel writes.
    return hipMemcpyAsync(status_out, base + 8, sizeof(int32_t), hipMemcpyDeviceToDevice, s) == hipSuccess ? CI_OK
                                                                                                         : CI_ERR_HIP;
  }
  const int rl = launch_ffn_decode_fused(x, B, w, dtype, act, y, base, s);
  if (rl != CI_OK || !status_out) return rl;
  return hipMemcpyAsync(status_out, base + 4, sizeof(int32_t), hipMemcpyDeviceToDevice, s) == hipSuccess ? CI_OK
                                                                                                       : CI_ERR_HIP;
}

int coreinfer_ffn_decode_status(const void* ws, int32_t* status_out, void* stream) {
  if (!ws || !status_out) return CI_ERR_INVALID_ARG;
  if (!aligned16(ws) || (reinterpret_cast<uintptr_t>(status_out) & 3u)) return CI_ERR_BAD_LAYOUT;
  if (hipMemcpyAsync(status_out, reinterpret_cast<const char*>(ws) + 4, sizeof(int32_t), hipMemcpyDeviceToDevice,
                     (hipStream_t)stream) != hipSuccess)
    return CI_ERR_HIP;
  return CI_OK;
}

int coreinfer_union_workspace_size(int64_t N, size_t* bytes) {
  if (!bytes || N < 1 || N > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  // owner masks [N] and the number of owned neurons per block of 1024
  *bytes = round256(((size_t)(N + 63) / 64 * 64 + 1024) * sizeof(uint32_t));
  return CI_OK;
}

int coreinfer_union_build(const int32_t* core_idx, int64_t B, int64_t K, int64_t N, int64_t max_rows,
                          int32_t* union_idx, uint32_t* union_mask, int32_t* union_count, void* ws,
                          size_t ws_bytes, void* stream) {
  size_t need = 0;
  if (coreinfer_union_workspace_size(N, &need) != CI_OK) return CI_ERR_INVALID_ARG;
  if (B < 1 || B > CI_MAX_UNION_SENTENCES || K < 0 || K > N) return CI_ERR_INVALID_ARG;
  if ((K > 0 && !core_idx) || !union_idx || !union_mask || !union_count) return CI_ERR_INVALID_ARG;
  const int64_t worst = B * K < N ? B * K : N;  // the union cannot have more rows than this
  if (max_rows < 1 || max_rows < worst || max_rows > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(core_idx) & 3u) || (reinterpret_cast<uintptr_t>(union_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(union_mask) & 3u) || (reinterpret_cast<uintptr_t>(union_count) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  return launch_union_build(core_idx, B, K, N, max_rows, union_idx, union_mask, union_count,
                            reinterpret_cast<uint32_t*>(ws), nullptr, (hipStream_t)stream);
}

int coreinfer_ffn_decode_union_workspace_size(int64_t B, int64_t max_rows, int64_t d, int dtype, int act,
                                              size_t* bytes) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!bytes || B < 1 || B > CI_MAX_UNION_SENTENCES || max_rows < 1 || max_rows > CI_MAX_NEURONS ||
      d < 1 || d > CI_MAX_DMODEL)
    return CI_ERR_INVALID_ARG;
  if (d % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  const int64_t chunks = union_up_chunks(d / vec_of(dtype));
  const int64_t ndot = act == CI_ACT_SWIGLU ? 2 : 1;
  // partial dots [chunks][ndot][max_rows][8] and partial sums [B][<= 256 slices][d], fp32
  const size_t hp = ((size_t)chunks * ndot * (size_t)max_rows * 8 + 63) / 64 * 64;
  *bytes = round256((hp + (size_t)B * 256 * (size_t)d) * sizeof(float)) + 256;
  return CI_OK;
}

int coreinfer_ffn_decode_union(const void* x, int64_t B, const ci_ffn_weights* w,
                               const int32_t* union_idx, const uint32_t* union_mask,
                               const int32_t* union_count, int64_t max_rows, int dtype, int act,
                               void* y, void* ws, size_t ws_bytes, void* stream) {
  if (!w) return CI_ERR_INVALID_ARG;
  size_t need = 0;
  const int rc = coreinfer_ffn_decode_union_workspace_size(B, max_rows, w->d, dtype, act, &need);
  if (rc != CI_OK) return rc;
  if (!x || !y || !union_idx || !union_mask || !union_count) return CI_ERR_INVALID_ARG;
  if (!w->w_up || !w->w_down || w->N < 1 || w->N > CI_MAX_NEURONS) return CI_ERR_INVALID_ARG;
  if ((act == CI_ACT_SWIGLU) != (w->w_gate != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && w->b_up) return CI_ERR_INVALID_ARG;
  if (!aligned16(x) || !aligned16(y) || !aligned16(w->w_up) || !aligned16(w->w_gate) ||
      !aligned16(w->w_down) || (reinterpret_cast<uintptr_t>(union_idx) & 3u) ||
      (reinterpret_cast<uintptr_t>(union_mask) & 3u) || (reinterpret_cast<uintptr_t>(union_count) & 3u))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  return launch_ffn_decode_union(x, B, w, union_idx, union_mask, union_count, max_rows, dtype, act, y,
                                 reinterpret_cast<float*>(ws), (hipStream_t)stream);
}

// Sums of tiles split along k, whichever layout the down matrix has.
static size_t dense_sums_bytes(int64_t M, int64_t d, int64_t N, int dtype) {
  return std::max(gemm_plan_bytes(gemm_down_plan(M, d, N, CI_DOWN_OUT_MAJOR, dtype, false, SIZE_MAX)),
                  gemm_plan_bytes(gemm_down_plan(M, d, N, CI_DOWN_NEURON_MAJOR, dtype, false, SIZE_MAX)));
}

static bool dense_sizes_ok(int64_t M, int64_t d, int64_t N) {
  return M >= 1 && M <= CI_MAX_TOKENS && d >= 1 && d <= CI_MAX_DMODEL && N >= 1 && N <= CI_MAX_NEURONS;
}
// Decode partials of up to four tokens over a neuron-major down matrix.
static size_t dense_partial_bytes(int64_t M, int64_t d, int64_t N) {
  return round256((size_t)M * (size_t)(N < kMaxSplits ? N : kMaxSplits) * (size_t)d * sizeof(float));
}

int coreinfer_dev_dense_plan(int64_t M, int64_t d, int64_t N, int dtype, int act, int down_layout, int64_t room,
                             int64_t* out) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(down_layout)) return CI_ERR_BAD_LAYOUT;
  if (!out || room < 0 || !dense_sizes_ok(M, d, N)) return CI_ERR_INVALID_ARG;
  if (M <= 4 || dtype == CI_F32) return CI_ERR_UNSUPPORTED;
  const GemmPlan up = gemm_up_plan(M, d, N, dtype, act);
  const GemmPlan down = gemm_down_plan(M, d, N, down_layout, dtype, act == CI_ACT_SWIGLU, (size_t)room);
  const int64_t values[] = {up.shape, up.full, down.shape, down.full, down.tail, down.splits,
                            (int64_t)gemm_plan_bytes(down), up.once, down.once};
  std::copy(std::begin(values), std::end(values), out);
  return CI_OK;
}

int coreinfer_ffn_dense_workspace_size(int64_t M, int64_t d, int64_t N, int dtype, size_t* bytes) {
  if (!dtype_ok(dtype)) return CI_ERR_BAD_DTYPE;
  if (!bytes || !dense_sizes_ok(M, d, N)) return CI_ERR_INVALID_ARG;
  // hidden matrix H [M, N]: fp32 on the row-dot path (M <= 4), element type
  // on the matrix-core path; plus the decode partials, or the sums of tiles split along k.
  *bytes = round256((size_t)M * (size_t)N * sizeof(float)) +
           (M <= 4 ? dense_partial_bytes(M, d, N) : round256(dense_sums_bytes(M, d, N, dtype))) + 256;
  return CI_OK;
}

// Up to four tokens over neuron-major weights: hidden values first, then the down rows, each weight read once;
// or the decode kernel with all neurons as the core set, which reads the weights once per token and, for the
// scores, the up matrices once more.  The latter has shorter launches, and one fewer where no scores are asked for.
// Where the line lies, by bytes of the weights (decode kernel / columns, us).  With scores, one token: 13 MB (512 x 2048
// gated fp32, 12.6 MB: 12.5 / 14.1; 768 x 3072 gated fp32, 28 MB: 15.6 / 13.8), 60 MB for rows of whole 4 KB (1024 x 4096 fp32,
// 34 MB: 14.8 / 20.3); two: 9 MB, gated 3 MB (384 x 1536 fp32, 4.7 MB: 12.6 / 13.5; gated 512 x 2048 fp16, 6.3 MB: 16.5 /
// 13.6); three and four: 3 MB, gated 1.5 MB (256 x 1024 fp32, 2.1 MB: 12.1 / 13.0; gated fp16, 1.6 MB: 15.5 / 14.8).  Without
// scores, two tokens: 200 MB (2048 x 8192 fp32 30 / 36; 4096 x 16384 fp16 55 / 48); three and four: 9 MB (512 x 2048 fp32,
// 8.4 MB: 13.2 / 14.5; 768 x 3072 fp16, 9.4 MB: 20.4 / 15.9); one: never.  (Rows that the decode kernel does not take are
// refused in either case.)
static bool dense_cols_pays(int64_t M, int64_t d, int64_t N, int dtype, int act, bool scores) {
  if (d / vec_of(dtype) > 4096) return false;
  const bool gated = act == CI_ACT_SWIGLU;
  const int64_t row = d * elem_bytes(dtype);
  const double bytes = (double)(gated ? 3 : 2) * (double)row * (double)N;
  if (!scores) return M > 1 && bytes >= (M == 2 ? 200e6 : 9e6);
  if (M == 1) return bytes >= (row % 4096 == 0 ? 60e6 : 13e6);
  return bytes >= (M == 2 ? (gated ? 3e6 : 9e6) : (gated ? 1.5e6 : 3e6));
}

int coreinfer_ffn_dense(const void* X, int64_t M, const void* w_up, const void* w_gate,
                        const void* b_up, const void* w_down, const void* b_down, int down_layout,
                        int dtype, int act, int64_t d, int64_t N, void* Y, float* A, void* ws,
                        size_t ws_bytes, void* stream) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(down_layout)) return CI_ERR_BAD_LAYOUT;
  if (!dense_sizes_ok(M, d, N)) return CI_ERR_INVALID_ARG;
  const size_t hidden = round256((size_t)M * (size_t)N * sizeof(float));
  // without room for the sums of split tiles none is split
  const size_t need = hidden + (M <= 4 ? dense_partial_bytes(M, d, N) : 0) + 256;
  if (!X || !w_up || (!Y && !A) || (Y && !w_down)) return CI_ERR_INVALID_ARG;
  if ((act == CI_ACT_SWIGLU) != (w_gate != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && b_up) return CI_ERR_INVALID_ARG;
  if (d % vec_of(dtype) != 0 || N % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  if (!aligned16(X) || !aligned16(w_up) || !aligned16(w_gate) || !aligned16(w_down) ||
      !aligned16(Y) || !aligned16(A))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < need) return CI_ERR_WORKSPACE;
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  hipStream_t s = (hipStream_t)stream;

  if (M <= 4) {
    float* H = reinterpret_cast<float*>(ws);
    float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + hidden);
    if (down_layout == CI_DOWN_NEURON_MAJOR && Y && dense_cols_pays(M, d, N, dtype, act, A != nullptr)) {
      const int rc = launch_up_rows(X, M, w_up, w_gate, b_up, dtype, act, d, N, H, A, s);
      return rc != CI_OK ? rc : launch_down_cols(H, M, w_down, b_down, dtype, d, N, Y, partial, s);
    }
    if (down_layout == CI_DOWN_NEURON_MAJOR && Y) {
      // all three matrices are neuron-major: this is the decode kernel with S = all neurons
      if (A) {
        int rc = launch_up_rows(X, M, w_up, w_gate, b_up, dtype, act, d, N, nullptr, A, s);
        if (rc != CI_OK) return rc;
      }
      ci_ffn_weights w;
      w.w_up = w_up; w.w_gate = w_gate; w.b_up = b_up; w.w_down = w_down; w.b_down = b_down;
      w.core_idx = nullptr; w.K = N; w.d = d; w.N = N;
      w.ld_down = 0; w.down_layout = CI_DOWN_NEURON_MAJOR;
      return launch_ffn_decode(X, M, &w, dtype, act, Y, partial, kMaxSplits, s);
    }
    int rc = launch_up_rows(X, M, w_up, w_gate, b_up, dtype, act, d, N, Y ? H : nullptr, A, s);
    if (rc != CI_OK || !Y) return rc;
    return launch_down_rows(H, M, w_down, b_down, dtype, d, N, Y, s);
  }
  const GemmPlan plan = gemm_down_plan(M, d, N, down_layout, dtype, w_gate != nullptr, ws_bytes - hidden);
  void* H = Y ? ws : nullptr;
  int rc = launch_gemm_up(X, M, w_up, w_gate, b_up, dtype, act, d, N, H, A, s);
  if (rc != CI_OK || !Y) return rc;
  float* partial = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + hidden);
  return launch_gemm_down(H, M, w_down, b_down, down_layout, dtype, d, N, Y, partial, plan, s);
}

int coreinfer_ffn_dense_hidden_workspace_size(int64_t M, int64_t d, int64_t N, int dtype, size_t* bytes) {
  if (!dtype_ok(dtype)) return CI_ERR_BAD_DTYPE;
  if (!bytes || !dense_sizes_ok(M, d, N)) return CI_ERR_INVALID_ARG;
  *bytes = round256(dense_sums_bytes(M, d, N, dtype)) + 256;  // sums of tiles split along k
  return CI_OK;
}

int coreinfer_ffn_dense_hidden(const void* X, int64_t M, const void* w_up, const void* w_gate, const void* b_up,
                               const void* w_down, const void* b_down, int down_layout, int dtype, int act,
                               int64_t d, int64_t N, void* Y, void* H, void* ws, size_t ws_bytes, void* stream) {
  if (!dtype_ok(dtype) || !act_ok(act)) return CI_ERR_BAD_DTYPE;
  if (!layout_ok(down_layout)) return CI_ERR_BAD_LAYOUT;
  if (!dense_sizes_ok(M, d, N)) return CI_ERR_INVALID_ARG;
  if (!X || !w_up || !H || (Y && !w_down)) return CI_ERR_INVALID_ARG;
  if ((act == CI_ACT_SWIGLU) != (w_gate != nullptr)) return CI_ERR_INVALID_ARG;
  if (act == CI_ACT_SWIGLU && b_up) return CI_ERR_INVALID_ARG;
  if (d % vec_of(dtype) != 0 || N % vec_of(dtype) != 0) return CI_ERR_BAD_LAYOUT;
  if (!aligned16(X) || !aligned16(w_up) || !aligned16(w_gate) || !aligned16(w_down) || !aligned16(Y) ||
      !aligned16(H))
    return CI_ERR_BAD_LAYOUT;
  if (!ws || ws_bytes < 256) return CI_ERR_WORKSPACE;  // without room for the sums of split tiles none is split
  if (!aligned16(ws)) return CI_ERR_BAD_LAYOUT;
  const GemmPlan plan = gemm_down_plan(M, d, N, down_layout, dtype, w_gate != nullptr, ws_bytes);
  hipStream_t s = (hipStream_t)stream;
  int rc = launch_gemm_up(X, M, w_up, w_gate, b_up, dtype, act, d, N, H, nullptr, s);
  if (rc != CI_OK || !Y) return rc;
  return launch_gemm_down(H, M, w_down, b_down, down_layout, dtype, d, N, Y, reinterpret_cast<float*>(ws), plan, s);
}

}  // extern "C"
