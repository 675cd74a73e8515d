// Clip-weighted sum and materialised norms: which kernel takes a layer, how a
// sum's K range is split, the split-K reduction, and the VALU kernel for layers
// with a tiny gradient.
//
// Paper: Section 2.2 aggregation sum_i g_bar_i with g_bar_i = c_i g_i and
// g_i = G_i^T A_i; GPU-side algorithm, clip and average steps.
//
// Split K. Small outputs are split along K to fill the GPU; each split writes
// its own fp32 partial and a second kernel adds them in split order, so the
// result is deterministic.
#include <algorithm>

#include "mma.h"

namespace dpsgd {
namespace {

enum EpiMode : int { EPI_STORE = 0, EPI_SUMSQ = 1 };

// --------------------------------------------------------- split-K reduce

struct SplitEntry {
  float* grad;
  const float* part;     // [splits][numel]
  int64_t numel;
  int32_t splits;
  int32_t accumulate;
  uint32_t wg_begin;
  int32_t vec;           // grad, part 16-byte aligned and numel % 4 == 0
};
struct SplitArgs {
  SplitEntry L[kMaxLayersPerLaunch];
  int32_t n;
};

constexpr int kSplitElemsPerWG = kThreads * 4;  // one float4 per thread

// Adds the partials in split order. A layer can have tens of splits, so the
// loads of eight consecutive splits are issued before their adds (the order
// of the additions does not change) and each thread owns one float4, which
// gives enough workgroups to cover the GPU.
__global__ __launch_bounds__(kThreads) void split_reduce_kernel(SplitArgs args) {
  int lo = 0, hi = args.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (args.L[mid].wg_begin <= blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const SplitEntry& E = args.L[lo];
  const int64_t e = (int64_t)(blockIdx.x - E.wg_begin) * kSplitElemsPerWG + (int64_t)threadIdx.x * 4;
  if (e >= E.numel) return;
  const int S = E.splits;
  if (E.vec) {
    float4 v = E.accumulate ? *reinterpret_cast<const float4*>(E.grad + e)
                            : make_float4(0.f, 0.f, 0.f, 0.f);
    const float* part = E.part + e;
    int s = 0;
    for (; s + 8 <= S; s += 8) {
      float4 p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = *reinterpret_cast<const float4*>(part + (int64_t)(s + u) * E.numel);
#pragma unroll
      for (int u = 0; u < 8; ++u) { v.x += p[u].x; v.y += p[u].y; v.z += p[u].z; v.w += p[u].w; }
    }
    for (; s < S; ++s) {
      const float4 p = *reinterpret_cast<const float4*>(part + (int64_t)s * E.numel);
      v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
    }
    *reinterpret_cast<float4*>(E.grad + e) = v;
  } else {
    // Element loads, 32 in flight (7 -> 70, T = 256, B = 256, 512 splits: 302 us a call
    // with one load at a time, 72 so).
    int64_t at[4];
    float v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      at[k] = e + k < E.numel ? e + k : E.numel - 1;
      v[k] = E.accumulate ? E.grad[at[k]] : 0.f;
    }
    int s = 0;
    for (; s + 8 <= S; s += 8) {
      float p[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) p[u][k] = E.part[(int64_t)(s + u) * E.numel + at[k]];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += p[u][k];
    }
    for (; s < S; ++s)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += E.part[(int64_t)s * E.numel + at[k]];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (e + k < E.numel) E.grad[e + k] = v[k];
  }
}

// ------------------------------------------------------ tiny layers (VALU)
//
// Some layers with at most kTinyMaxOut entries in g_i = G_i^T A_i form each
// example's gradient directly: its rows are staged in LDS a chunk at a time
// and thread t accumulates entries t and t + 256 of g_i in float32. The norm
// variant sums g_i's squares per example; the clip variant adds c_i g_i to the
// job's partial sum (an example with c_i = 0 is skipped, its rows are never
// read). Which layers: tiny_norm_ok and tiny_clip_ok below.

constexpr int kTinyMaxOut = 2 * kThreads;     // d_in * d_out
constexpr int kTinyLdsFloats = 16384;         // 64 KB of staged rows
constexpr int kTinyBatch = 16;                // loads in flight per thread while staging

struct TinyEntry {
  const void* A;          // [B*T][N]
  const void* G;          // [B*T][M]
  float* out;             // EPI_STORE: grad (one job) or this layer's per-job partials
  int32_t M, N, T;
  int32_t ex_per_job;
  int32_t jobs;
  uint32_t wg_begin;
  int32_t partial_col;    // EPI_SUMSQ
  int32_t accumulate;     // EPI_STORE, jobs == 1
};

struct TinyArgs {
  TinyEntry L[kMaxLayersPerLaunch];
  int32_t n;
  int32_t B;
  const float* factors;
  float* partials;
  int64_t P;
};

template <typename TIn, int EPI>
__global__ __launch_bounds__(kThreads) void tiny_kernel(TinyArgs args) {
  __shared__ float rows[kTinyLdsFloats];
  __shared__ float red[4];
  int lo = 0, hi = args.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (args.L[mid].wg_begin <= blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const TinyEntry& E = args.L[lo];
  const int job = (int)(blockIdx.x - E.wg_begin);
  const int M = E.M, N = E.N, T = E.T, W = M + N;
  const int rc = kTinyLdsFloats / W;   // rows per chunk
  const TIn* A = static_cast<const TIn*>(E.A);
  const TIn* G = static_cast<const TIn*>(E.G);
  const int tid = threadIdx.x;
  const int n_out = M * N;
  const int o0 = tid, o1 = tid + kThreads;
  const int m0 = o0 / N, n0 = o0 - m0 * N, m1 = o1 / N, n1 = o1 - m1 * N;
  float sum0 = 0.f, sum1 = 0.f;   // EPI_STORE: sum over this job's examples of c_i g_i
  const int ex_begin = job * E.ex_per_job;
  const int ex_end = min(ex_begin + E.ex_per_job, args.B);
  for (int ex = ex_begin; ex < ex_end; ++ex) {
    const float c = EPI == EPI_STORE ? args.factors[ex] : 1.0f;
    if (EPI == EPI_STORE && c == 0.0f) continue;   // uniform over the workgroup
    float g0 = 0.f, g1 = 0.f;
    for (int r0 = 0; r0 < T; r0 += rc) {
      const int nr = min(rc, T - r0);
      const int64_t row = (int64_t)ex * T + r0;
      // Staged chunk: rows [r][0, M) hold G, [r][M, M + N) hold A.
      __syncthreads();   // the previous chunk is no longer read
      // kTinyBatch independent loads per thread, then their LDS stores, so the
      // staging waits for one memory latency per batch rather than per element.
      const int n_el = nr * W;
      for (int i0 = 0; i0 < n_el; i0 += kThreads * kTinyBatch) {
        float v[kTinyBatch];
#pragma unroll
        for (int u = 0; u < kTinyBatch; ++u) {
          const int i = i0 + u * kThreads + tid;
          v[u] = 0.f;
          if (i < n_el) {
            const int r = i / W, k = i - r * W;
            v[u] = k < M ? load_elem(G + (row + r) * M + k) : load_elem(A + (row + r) * N + (k - M));
          }
        }
#pragma unroll
        for (int u = 0; u < kTinyBatch; ++u) {
          const int i = i0 + u * kThreads + tid;
          if (i < n_el) rows[i] = v[u];
        }
      }
      __syncthreads();
      if (o0 < n_out)
        for (int r = 0; r < nr; ++r) g0 = fmaf(rows[r * W + m0], rows[r * W + M + n0], g0);
      if (o1 < n_out)
        for (int r = 0; r < nr; ++r) g1 = fmaf(rows[r * W + m1], rows[r * W + M + n1], g1);
    }
    if (EPI == EPI_SUMSQ) {
      const float s = block_sum(g0 * g0 + g1 * g1, red);
      if (tid == 0) args.partials[(int64_t)ex * args.P + E.partial_col] = s;
    } else {
      sum0 = fmaf(c, g0, sum0);
      sum1 = fmaf(c, g1, sum1);
    }
  }
  if (EPI == EPI_STORE) {
    float* out = E.out + (E.jobs > 1 ? (int64_t)job * n_out : 0);
    const bool add = E.jobs == 1 && E.accumulate;
    if (o0 < n_out) out[o0] = add ? out[o0] + sum0 : sum0;
    if (o1 < n_out) out[o1] = add ? out[o1] + sum1 : sum1;
  }
}

template <typename TIn, int EPI>
int launch_tiny_group(const dpsgd_layer* layers, const int* idx, int n, const float* factors,
                      float* const* outs, const int* jobs, const int* accumulate,
                      const int64_t* cols, float* partials, int64_t P, hipStream_t stream) {
  for (int base = 0; base < n; base += kMaxLayersPerLaunch) {
    const int m = n - base < kMaxLayersPerLaunch ? n - base : kMaxLayersPerLaunch;
    TinyArgs args{};
    args.n = m;
    args.B = (int32_t)layers[idx[base]].B;
    args.factors = factors;
    args.partials = partials;
    args.P = P;
    int64_t wgs = 0;
    for (int k = 0; k < m; ++k) {
      const int li = idx[base + k];
      const dpsgd_layer& L = layers[li];
      TinyEntry& E = args.L[k];
      E.A = L.A;
      E.G = L.G;
      E.M = (int32_t)L.d_out;
      E.N = (int32_t)L.d_in;
      E.T = (int32_t)L.T;
      E.wg_begin = (uint32_t)wgs;
      if (EPI == EPI_STORE) {
        E.out = outs[base + k];
        E.jobs = jobs[base + k];
        E.accumulate = accumulate ? accumulate[base + k] : 0;
      } else {
        E.jobs = (int32_t)L.B;
        E.partial_col = (int32_t)cols[li];
      }
      // A job past the last example writes zeros, so the count may overshoot.
      E.ex_per_job = (int32_t)ceil_div(L.B, E.jobs);
      wgs += E.jobs;
    }
    if (wgs > 0x7FFFFFFF) return DPSGD_ERR_INVALID_ARG;
    hipLaunchKernelGGL((tiny_kernel<TIn, EPI>), dim3((uint32_t)wgs), dim3(kThreads), 0, stream, args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

}  // namespace

int tiny_jobs(const dpsgd_layer& L) {
  // About two workgroups per CU, each over ceil(B / jobs) consecutive examples.
  const int64_t want = L.B < 2 * (int64_t)tr_cu_count() ? L.B : 2 * (int64_t)tr_cu_count();
  return (int)ceil_div(L.B, ceil_div(L.B, want));
}

// A tiny layer goes to the VALU kernel or to an MFMA tile that stays mostly
// empty. The VALU kernel's time grows with the entries a thread accumulates (one
// or two) and the elements it stages, and it runs a workgroup per example; the
// MFMA kernel takes 16 rows at a time whatever the width, is slower where rows
// are below 16 bytes (any_slow) and splits long examples.
bool tiny_norm_ok(const dpsgd_layer& L) {
  if (L.d_in * L.d_out > kTinyMaxOut) return false;
  if (any_tiles(L) > 1) return true;
  // Norm calls in us, VALU and MFMA: float32 16 -> 16, T = 1024, B = 256 67 and 70, 3 -> 16
  // 59 and 105, 27 -> 16 116 and 70; T = 100, B = 32 16 and 13; T = 4, B = 4096 22 and
  // 27. bf16 16 -> 16, T = 16, B = 512 9 and 10, T = 64, B = 1024 16 and 12; 3 -> 64
  // (any_slow), T = 64, B = 1024 21 and 21, T = 256, B = 256 32 and 19; 2 -> 2, T = 1024 52
  // and 54.
  if (L.dtype == DPSGD_F32) return L.d_in * L.d_out <= kThreads || L.T < 32;
  return any_slow(L) ? L.T * (L.d_in + L.d_out) < 4500 : L.T < 16;
}

bool tiny_clip_ok(const dpsgd_layer& L) {
  if (L.d_in * L.d_out > kTinyMaxOut) return false;
  // Clip calls in us, VALU and MFMA: float32 2 -> 2, T = 256, B = 256 28 and 38, 3 -> 16
  // 30 and 38, 27 -> 16 48 and 40; 2 -> 32 and 32 -> 5, T = 1024 88 and 124; 16 -> 16, T = 64,
  // B = 1024 39 and 38, T = 1024, B = 16 69 and 21, T = 16, B = 512 31 and 16.
  if (L.dtype == DPSGD_F32)
    return L.d_in * L.d_out <= kThreads && L.d_in + L.d_out <= 72 && L.B >= tr_cu_count() &&
           L.B * L.T >= 32768;
  // bf16 with the weight on the MFMA operand would round it to bf16. Otherwise:
  // 3 -> 64, T = 100, B = 32 18 and 23, T = 256, B = 256 45 and 32; 2 -> 2, T = 100, B = 32
  // 14 and 24, T = 64, B = 1024 34 and 32; 16 -> 16, T = 100, B = 32 15 and 15.
  return any_flat(L) || (any_slow(L) && L.T <= 300 && L.T * (L.d_in + L.d_out) < 7000 && L.B <= 256);
}
int64_t mat_tile_count(const dpsgd_layer& L) {
  return tr_tile_ok(L) ? (L.d_out / 256) * (L.d_in / 256) : any_tiles(L);
}

namespace {

// Launch of the any-shape kernel that takes a layer (one dtype in a call).
// Both tile shapes, and layers with rows below 16 bytes (any_slow) and others,
// share a launch when the launch is short (a launch costs about 4 us) and have
// one each when it is long: their slices differ in cost, and a plan of its own
// fills the rounds better (the convolutions of WRN-16-4, B = 256: 1.46 against
// 1.42 ms, and half the partial sums).
constexpr int kAnyGroups = 8;
constexpr double kMergeFlops = 1.0e10;
int any_group(const dpsgd_layer& L, bool merge) {
  return (any_flat(L) ? 0 : 1) + (merge ? 0 : 2 * (any_slow(L) ? 1 : 0) + 4 * any_shape(L));
}
double clip_flops(const dpsgd_layer& L) {
  return 2.0 * (double)(L.B * L.T) * (double)L.d_in * (double)L.d_out;
}

// Launches of a clipped sum: the any-shape ones, then the other kernels'.
enum ClipGroup : int {
  kTr = kAnyGroups,
  kWide = kAnyGroups + 1,
  kTiny = kAnyGroups + 2,
  kRagged = kAnyGroups + 3,   // 384x256 tiles with padding, if the launch uses them
  kClipGroups = kAnyGroups + 4
};
// The group of a layer's clipped sum; any-shape layers get kAnyGroups' first.
int clip_class(const dpsgd_layer& L) {
  return wide_tile_ok(L)     ? kWide
         : tr_tile_ok(L)     ? kTr
         : wide_ragged_ok(L) ? kRagged
         : tiny_clip_ok(L)   ? kTiny
                             : 0;
}

// The same for the layers of a launch.
void clip_classes(const dpsgd_layer* layers, int n, int8_t* group) {
  bool any_launch = false;
  for (int l = 0; l < n; ++l) {
    group[l] = (int8_t)clip_class(layers[l]);
    any_launch = any_launch || group[l] == 0;
  }
  // Where an any-shape launch runs in any case, a tiny layer joins it (unless its
  // weights would be rounded there): that costs less than a launch.
  for (int l = 0; l < n && any_launch; ++l)
    if (group[l] == kTiny && !(layers[l].dtype == DPSGD_BF16 && any_flat(layers[l]))) group[l] = 0;
}

}  // namespace

void plan_clip(const dpsgd_layer* layers, int n_layers, ClipPlan* plan) {
  // Layers on the 256- and 384x256-tile kernels are balanced by their own
  // plans (whole tiles, then a split tail). The layers of an any-shape launch
  // split their K range so that every workgroup of the launch gets about the
  // same number of slices: the layers of one call can differ by orders of
  // magnitude in B * T (a convolution's positions) and in output tiles, and a
  // layer with few output tiles but a long K range would otherwise run on a
  // handful of CUs.
  // The balance is per launch (launches run one after the other, so each fills
  // the GPU on its own).
  const int cus = tr_cu_count();
  // The 384x256 tiles of the layers that they suit only with padding pay off
  // once the launch holds enough work for its prologues and partial tiles:
  // single layers of 8, 10, 12 and 13 GFLOP took 37.9, 38.9, 42.9 and 45.3 us
  // against 35.3, 36.6, 42.9 and 41.1 on the any-shape kernel, layers of 29,
  // 33, 48 and 164 GFLOP 72.9, 64.1, 79.5 and 180 against 79.2, 72.7, 98.9 and
  // 300 us. With fewer than nine tiles the launch has too few ranges for the CUs,
  // or ranges too short for their partial tiles: 192 -> 1000 (3 tiles, 25 GFLOP) 164
  // us and 91, 392 -> 768 (4, 48) 192 and 118, 192 -> 200 (1, 56) 1687 and 178; 1000
  // -> 520 (8, 96) 215 and 227, 760 -> 776 (9, 66) 144 and 149, 776 -> 776 (12, 36) 88
  // and 98, 1544 -> 1000 (21, 53) 89 and 131.
  constexpr double kMinRaggedFlops = 2.0e10;
  constexpr int64_t kMinRaggedTiles = 9;
  double ragged_flops = 0.0, any_flops = 0.0;
  int64_t ragged_tiles = 0;
  clip_classes(layers, n_layers, plan->group);
  for (int l = 0; l < n_layers; ++l) {
    if (plan->group[l] == kRagged) {
      ragged_flops += clip_flops(layers[l]);
      ragged_tiles += wide_tiles(layers[l]);
    }
    if (plan->group[l] == 0) any_flops += clip_flops(layers[l]);
  }
  const bool ragged = ragged_flops >= kMinRaggedFlops && ragged_tiles >= kMinRaggedTiles;
  if (!ragged) any_flops += ragged_flops;
  const bool merge = any_flops <= kMergeFlops;
  int idx[kClipGroups][kMaxLayersPerLaunch], cnt[kClipGroups] = {};
  for (int l = 0; l < n_layers; ++l) {
    int g = plan->group[l];
    if (g == 0 || (g == kRagged && !ragged)) g = any_group(layers[l], merge);
    plan->group[l] = (int8_t)g;
    idx[g][cnt[g]++] = l;
  }
  constexpr int64_t kMinSlicesPerSplit = 4;
  constexpr int64_t kMaxSplits = 1024;
  auto split_count = [](int64_t q_total, int64_t chunk) {
    int64_t s = ceil_div(q_total, chunk);
    if (s > q_total / kMinSlicesPerSplit) s = q_total / kMinSlicesPerSplit;
    if (s > kMaxSplits) s = kMaxSplits;
    return s < 1 ? (int64_t)1 : s;
  };
  int64_t chunk_of[kAnyGroups];
  for (int64_t& c : chunk_of) c = 1;
  for (int g = 0; g < kAnyGroups; ++g) {
    if (cnt[g] == 0) continue;
    // A launch runs in rounds of as many workgroups as the GPU holds, and a
    // round that is only partly filled costs as much as a full one, so the
    // chunk (slices per workgroup) is chosen per launch: for r = 1 .. 8
    // rounds, the smallest chunk whose workgroups fit r rounds, keeping the r
    // with the least estimated time: r x (longest workgroup) plus the partial
    // sums written and read back. The rates are what the kernel and the
    // reduction sustain (a slice at the kernel's rate on a full GPU).
    const dpsgd_layer& L0 = layers[idx[g][0]];
    const int64_t slots = (int64_t)any_workgroups_per_cu() * cus;
    const double rate = L0.dtype == DPSGD_F32 ? 1.4e14 : 6.0e14;
    const double t_slice = 2.0 * 128 * 128 * any_slice_rows(L0) * (double)slots / rate;
    constexpr double kHbm = 4.0e12;
    int64_t q_max = 1;
    for (int k = 0; k < cnt[g]; ++k) q_max = std::max(q_max, any_slices(layers[idx[g][k]]));
    // Workgroups of the launch for a given chunk, its longest K range and the
    // bytes of its partial sums.
    auto eval = [&](int64_t chunk, int64_t* longest, double* bytes) {
      int64_t wgs = 0, lg = 0;
      double by = 0.0;
      for (int k = 0; k < cnt[g]; ++k) {
        const dpsgd_layer& L = layers[idx[g][k]];
        const int64_t q = any_slices(L);
        const int64_t sp = split_count(q, chunk);
        wgs += any_tiles(L) * sp;
        lg = std::max(lg, ceil_div(q, sp));
        if (sp > 1) by += 4.0 * (double)sp * (double)L.d_in * (double)L.d_out;
      }
      if (longest) *longest = lg;
      if (bytes) *bytes = by;
      return wgs;
    };
    int64_t best_chunk = q_max;
    double best_cost = -1.0;
    for (int64_t r = 1; r <= 8; ++r) {
      if (eval(q_max, nullptr, nullptr) > r * slots) continue;   // not even one split per layer fits
      int64_t lo = std::min(kMinSlicesPerSplit, q_max), hi = q_max;
      while (lo < hi) {   // smallest chunk with at most r rounds of workgroups
        const int64_t mid = (lo + hi) / 2;
        if (eval(mid, nullptr, nullptr) <= r * slots) hi = mid; else lo = mid + 1;
      }
      int64_t longest = 0;
      double bytes = 0.0;
      eval(lo, &longest, &bytes);
      const double cost = (double)(r * longest) * t_slice + 2.0 * bytes / kHbm;
      if (best_cost < 0.0 || cost < best_cost) { best_cost = cost; best_chunk = lo; }
    }
    chunk_of[g] = best_chunk;
  }
  size_t off = 0;
  for (int l = 0; l < n_layers; ++l) {
    const dpsgd_layer& L = layers[l];
    int64_t s = 1;
    const int g = plan->group[l];
    if (g < kAnyGroups) s = split_count(any_slices(L), chunk_of[g]);
    else if (g == kTiny) s = tiny_jobs(L);   // one partial per job of consecutive examples
    plan->splits[l] = (int)s;
    plan->partial_offset[l] = off;
    if (s > 1) off += round_up((size_t)s * (size_t)L.d_out * (size_t)L.d_in * sizeof(float), 256);
  }
  plan_tr_clip(layers, idx[kTr], cnt[kTr], cus, &plan->tr);
  plan_wide_clip(layers, idx[kWide], cnt[kWide], cus, &plan->wide);
  plan->tr_offset = off;
  plan->wide_offset = off + round_up(plan->tr.tail_bytes, 256);
  plan_wide_clip(layers, idx[kRagged], cnt[kRagged], cus, &plan->ragged);
  plan->ragged_offset = plan->wide_offset + round_up(plan->wide.tail_bytes, 256);
  plan->partial_bytes = plan->ragged_offset + round_up(plan->ragged.tail_bytes, 256);
}

bool clip_from_norms(const dpsgd_layer* layers, int n_layers) {
  // Forming a factor takes about 30 instructions a slice and lane, next to the
  // 150 of a float32 slice; a launch for the factors takes about 4 us with its
  // gap. The whole call has to be one launch of any_flat layers.
  constexpr double kMostFlops = 2.0e9;   // about 20 us of the kernel
  if (n_layers > kMaxLayersPerLaunch) return false;
  int8_t group[kMaxLayersPerLaunch];
  clip_classes(layers, n_layers, group);
  double flops = 0.0;
  for (int l = 0; l < n_layers; ++l) {
    const dpsgd_layer& L = layers[l];
    if (group[l] != 0 || any_group(L, true) != any_group(layers[0], true) || !any_flat(L)) return false;
    flops += clip_flops(L);
  }
  return flops <= kMostFlops;
}

int launch_clip_sum(const dpsgd_layer* layers, int n_layers, const ClipWeights& weights,
                    float* const* grads, int accumulate, float* partial_base, const ClipPlan& plan,
                    hipStream_t stream) {
  // Group layers by kernel variant; each group is one grouped launch.
  int idx[kClipGroups][kMaxLayersPerLaunch];
  float* outs[kClipGroups][kMaxLayersPerLaunch];
  int spl[kClipGroups][kMaxLayersPerLaunch];
  int acc[kClipGroups][kMaxLayersPerLaunch];
  int cnt[kClipGroups] = {};
  for (int l = 0; l < n_layers; ++l) {
    const int g = plan.group[l];
    const int k = cnt[g]++;
    idx[g][k] = l;
    spl[g][k] = plan.splits[l];
    outs[g][k] = plan.splits[l] > 1
                     ? reinterpret_cast<float*>(reinterpret_cast<char*>(partial_base) +
                                                plan.partial_offset[l])
                     : grads[l];
    acc[g][k] = accumulate;
  }
  const float* factors = weights.factors;
  int st = DPSGD_OK;
  if (cnt[kTr])
    st = launch_tr_clip(layers, idx[kTr], cnt[kTr], factors, outs[kTr], accumulate, plan.tr,
                        reinterpret_cast<float*>(reinterpret_cast<char*>(partial_base) +
                                                 plan.tr_offset),
                        stream);
  if (st == DPSGD_OK && cnt[kWide])
    st = launch_wide_clip(layers, idx[kWide], cnt[kWide], factors, outs[kWide], accumulate, plan.wide,
                          reinterpret_cast<float*>(reinterpret_cast<char*>(partial_base) +
                                                   plan.wide_offset),
                          false, stream);
  if (st == DPSGD_OK && cnt[kRagged])
    st = launch_wide_clip(layers, idx[kRagged], cnt[kRagged], factors, outs[kRagged], accumulate,
                          plan.ragged,
                          reinterpret_cast<float*>(reinterpret_cast<char*>(partial_base) +
                                                   plan.ragged_offset),
                          true, stream);
  for (int g = 0; g < kAnyGroups; ++g)
    if (st == DPSGD_OK && cnt[g])
      st = launch_any_clip(layers, idx[g], cnt[g], weights, outs[g], spl[g], acc[g], stream);
  if (st == DPSGD_OK && cnt[kTiny])
    st = layers[0].dtype == DPSGD_BF16
             ? launch_tiny_group<uint16_t, EPI_STORE>(layers, idx[kTiny], cnt[kTiny], factors, outs[kTiny],
                                                      spl[kTiny], acc[kTiny], nullptr, nullptr, 0, stream)
             : launch_tiny_group<float, EPI_STORE>(layers, idx[kTiny], cnt[kTiny], factors, outs[kTiny],
                                                   spl[kTiny], acc[kTiny], nullptr, nullptr, 0, stream);
  if (st != DPSGD_OK) return st;

  // Split-K fix-up for the layers that were split.
  SplitArgs sargs{};
  int64_t wgs = 0;
  for (int l = 0; l < n_layers; ++l) {
    if (plan.splits[l] <= 1) continue;
    SplitEntry& E = sargs.L[sargs.n++];
    E.grad = grads[l];
    E.part = reinterpret_cast<const float*>(reinterpret_cast<const char*>(partial_base) +
                                            plan.partial_offset[l]);
    E.numel = layers[l].d_out * layers[l].d_in;
    E.splits = plan.splits[l];
    E.accumulate = accumulate;
    E.wg_begin = (uint32_t)wgs;
    E.vec = (aligned16(E.grad) && aligned16(E.part) && E.numel % 4 == 0) ? 1 : 0;
    wgs += ceil_div(E.numel, kSplitElemsPerWG);
  }
  if (sargs.n > 0) {
    if (wgs > 0x7FFFFFFF) return DPSGD_ERR_INVALID_ARG;
    hipLaunchKernelGGL(split_reduce_kernel, dim3((uint32_t)wgs), dim3(kThreads), 0, stream, sargs);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

int launch_mat_norms(const dpsgd_layer* layers, const int* idx, int n, const int64_t* cols,
                     float* partials, int64_t P, hipStream_t stream) {
  const bool bf16 = layers[idx[0]].dtype == DPSGD_BF16;
  int ib[256], it[256], ia[2][256], nb = 0, nt = 0, na[2] = {0, 0};
  double flops = 0.0;
  for (int k = 0; k < n; ++k) flops += clip_flops(layers[idx[k]]);
  const bool merge = flops <= kMergeFlops;
  // A tiny layer that an MFMA tile covers joins the any-shape launch of a layer
  // whose examples are at least as long: it ends no later there, and a launch of
  // the VALU kernel comes on top. (Either way it has one norm partial.)
  int64_t longest = 0;
  for (int k = 0; k < n; ++k) {
    const dpsgd_layer& L = layers[idx[k]];
    if (!tr_tile_ok(L) && !tiny_norm_ok(L)) longest = std::max(longest, L.T);
  }
  for (int k = 0; k < n; ++k) {
    const dpsgd_layer& L = layers[idx[k]];
    const int g = any_slow(L) && !merge ? 1 : 0;
    if (tr_tile_ok(L)) ib[nb++] = idx[k];
    else if (tiny_norm_ok(L) && !(merge && any_tiles(L) == 1 && L.T <= longest)) it[nt++] = idx[k];
    else ia[g][na[g]++] = idx[k];
  }
  int st = DPSGD_OK;
  if (nb) st = launch_tr_mat_norms(layers, ib, nb, cols, partials, P, stream);
  for (int g = 0; g < 2; ++g)
    if (st == DPSGD_OK && na[g]) st = launch_any_norms(layers, ia[g], na[g], cols, partials, P, stream);
  if (st == DPSGD_OK && nt)
    st = bf16 ? launch_tiny_group<uint16_t, EPI_SUMSQ>(layers, it, nt, nullptr, nullptr, nullptr,
                                                       nullptr, cols, partials, P, stream)
              : launch_tiny_group<float, EPI_SUMSQ>(layers, it, nt, nullptr, nullptr, nullptr, nullptr,
                                                    cols, partials, P, stream);
  return st;
}

}  // namespace dpsgd
