// Per-example gradient norms and clip factors of the DP-SGD step.
//
// Paper: Section 2.2, per-example clipping by ||g_t(x_i)||_2 over all trainable
// parameters; GPU-side algorithm, clip step. For a linear layer the squared
// norm of g_i = G_i^T A_i can be formed without the [d_out, d_in] gradient:
//
//   T = 1:   ||g_i||^2 = ||a_i||^2 ||g_i||^2                       (rank one)
//   ghost:   ||g_i||^2 = sum_{t,s} (a_t . a_s)(g_t . g_s)
//                      = <A_i A_i^T, G_i G_i^T>_F                  (Gram form)
//   materialise: square-sum of G_i^T A_i tiles kept in registers   (gemm.hip)
//
// The ghost kernel evaluates the Gram form on 128x128 (t, s) tiles of the
// upper triangle (off-diagonal tiles count twice): one MFMA K-loop over d_in
// builds the activation Gram tile, a second over d_out builds the
// output-gradient Gram tile in the same register layout, and the two are
// multiplied element-wise and summed. Each tile writes one float partial;
// a final fixed-order reduction adds the partials of every layer of the call
// into norms_sq, so the result does not depend on scheduling.
#include <algorithm>
#include <vector>

#include "mma.h"

namespace dpsgd {
namespace {

// ------------------------------------------------------------------ T = 1

struct T1Entry {
  const void* A;
  const void* G;
  int32_t d_in, d_out;
  int32_t partial_col;
  int32_t pad;
};
struct T1Args {
  T1Entry L[kMaxLayersPerLaunch];
  int32_t n;
  int64_t P;
  float* partials;
};

template <typename TIn>
__global__ __launch_bounds__(kThreads) void t1_norm_kernel(T1Args args) {
  __shared__ float red[4];
  const int64_t i = blockIdx.x;
  const T1Entry& E = args.L[blockIdx.y];
  const TIn* a = static_cast<const TIn*>(E.A) + i * E.d_in;
  const TIn* g = static_cast<const TIn*>(E.G) + i * E.d_out;
  float sa = 0.f, sg = 0.f;
  for (int e = threadIdx.x; e < E.d_in; e += kThreads) { const float v = load_elem(a + e); sa = fmaf(v, v, sa); }
  for (int e = threadIdx.x; e < E.d_out; e += kThreads) { const float v = load_elem(g + e); sg = fmaf(v, v, sg); }
  sa = block_sum(sa, red);
  sg = block_sum(sg, red);
  if (threadIdx.x == 0) args.partials[i * args.P + E.partial_col] = sa * sg;
}

// ------------------------------------------------------------------ ghost

struct GhostEntry {
  const void* A;
  const void* G;
  int32_t d_in, d_out, T;
  int32_t nt;          // 128-row tiles along T
  int32_t pairs;       // nt (nt + 1) / 2 upper-triangle tile pairs
  uint32_t wg_begin;   // first workgroup of this layer in the launch
  int32_t partial_col;
  int32_t load;        // LoadMode
};
struct GhostArgs {
  GhostEntry L[kMaxLayersPerLaunch];
  int32_t n;
  int64_t P;
  float* partials;
};

// How a tile's 16-byte chunks are loaded: LD_VEC (widths that are multiples of
// 16 bytes) and LD_ANY (other widths of at least 16 bytes; global loads need no
// alignment) unconditionally and two slices ahead; LD_FEW (widths as LD_VEC's
// that make few slices) and LD_SHORT (widths below 16 bytes, element by element)
// only where the tile has data, and one slice ahead.
enum LoadMode : int { LD_VEC = 0, LD_ANY = 1, LD_FEW = 2, LD_SHORT = 3 };

// Chunks of a 128-row x BK tile of a row-major matrix with rows of length ld, of
// whose columns the first d (from X) belong to the tile. LD_VEC and LD_ANY: a
// chunk outside the tile loads one inside (its row's last) and is cleared by
// mend_tile_rows; with branches around the loads the compiler waits for each in
// turn.
template <typename TIn, int LD>
__device__ __forceinline__ void load_tile_rows(const TIn* X, int64_t ld, int rows_valid, int k0,
                                               int d, uint4 (&r)[4]) {
  constexpr int E = TileCfg<TIn>::E;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = threadIdx.x + kThreads * u, row = c >> 3, k = k0 + (c & 7) * E;
    if (LD == LD_VEC || LD == LD_ANY) {
      __builtin_memcpy(&r[u], X + (int64_t)min(row, rows_valid - 1) * ld + min(k, d - E), 16);
      continue;
    }
    r[u] = make_uint4(0u, 0u, 0u, 0u);
    if (row >= rows_valid) continue;
    const TIn* p = X + (int64_t)row * ld + k;
    if (LD == LD_FEW) {
      if (k < d) r[u] = *reinterpret_cast<const uint4*>(p);
    } else {
      uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (k + e < d) {
          if (E == 8) w[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(p)[e] << (16 * (e & 1));
          else w[e] = reinterpret_cast<const uint32_t*>(p)[e];
        }
      r[u] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// Clears what lies outside the tile (uniform branches: whole tiles skip them).
template <typename TIn, int LD>
__device__ __forceinline__ void mend_tile_rows(int rows_valid, int k0, int d, uint4 (&r)[4]) {
  constexpr int E = TileCfg<TIn>::E;
  if (LD == LD_FEW || LD == LD_SHORT) return;
  if (k0 + TileCfg<TIn>::BK > d) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // The chunk was loaded `over` elements early.
      const int over = max(0, k0 + (((int)threadIdx.x + kThreads * u) & 7) * E + E - d);
      r[u] = LD == LD_VEC ? (over > 0 ? make_uint4(0u, 0u, 0u, 0u) : r[u])
                          : shift_chunk<(int)sizeof(TIn)>(r[u], over);
    }
  }
  if (rows_valid < kTile) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if ((((int)threadIdx.x + kThreads * u) >> 3) >= rows_valid) r[u] = make_uint4(0u, 0u, 0u, 0u);
  }
}

template <typename TIn>
__device__ __forceinline__ void store_tile_rows(TIn* Xs, const uint4 (&r)[4]) {
  constexpr int E = TileCfg<TIn>::E;
  constexpr int SK = TileCfg<TIn>::SK;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = threadIdx.x + kThreads * u;
    *reinterpret_cast<uint4*>(Xs + (c >> 3) * SK + (c & 7) * E) = r[u];
  }
}

// acc = Xp[rows_p] Xq[rows_q]^T over k in [0, d) of rows of length ld. Slice s is
// multiplied while slice s + 1 waits in registers and slice s + 2 is on its way.
// Load latency bounds the short row blocks: 640 -> 1295 at B = 16, T = 437 in bf16
// 51 us with branches around the loads and one slice ahead, 38 us so; 768 ->
// 50257 at B = 4, T = 128 36.6 and 30.3 us.
template <typename TIn, int LD>
__device__ __forceinline__ void gram_phase(const TIn* Xp, const TIn* Xq, int64_t ld, int d,
                                           int rows_p, int rows_q, bool diag,
                                           f32x4_t (&acc)[4][4],
                                           TIn* lds /* [2 stages][2 operands][OPE] */) {
  constexpr int BK = TileCfg<TIn>::BK;
  constexpr int SK = TileCfg<TIn>::SK;
  constexpr int OPE = lds_operand_elems<TIn>();
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int nsteps = (d + BK - 1) / BK;
  struct Slice {
    uint4 p[4], q[4];
  };
  Slice S0, S1;
  zero_acc(acc);
  auto fetch = [&](int k0, Slice& S) {
    load_tile_rows<TIn, LD>(Xp, ld, rows_p, k0, d, S.p);
    if (!diag) load_tile_rows<TIn, LD>(Xq, ld, rows_q, k0, d, S.q);
  };
  auto commit = [&](int s, Slice& S, int buf) {
    TIn* N = lds + buf * 2 * OPE;
    mend_tile_rows<TIn, LD>(rows_p, s * BK, d, S.p);
    store_tile_rows<TIn>(N, S.p);
    if (!diag) {
      mend_tile_rows<TIn, LD>(rows_q, s * BK, d, S.q);
      store_tile_rows<TIn>(N + OPE, S.q);
    }
  };
  auto multiply = [&](int cur) {
    const TIn* P = lds + cur * 2 * OPE;
    const TIn* Q = diag ? P : P + OPE;
    mma_step(P + wm * 64 * SK, Q + wn * 64 * SK, acc, lane);
  };
  fetch(0, S0);
  if (LD == LD_FEW || LD == LD_SHORT) {   // one slice ahead
    commit(0, S0, 0);
    __syncthreads();
    for (int s = 0; s < nsteps; ++s) {
      const bool more = s + 1 < nsteps;
      if (more) fetch((s + 1) * BK, S0);
      multiply(s & 1);
      if (more) commit(s + 1, S0, (s & 1) ^ 1);
      __syncthreads();
    }
    return;
  }
  // (Slices past the end load columns of the last one and are not used: a branch
  // around the loads would make the compiler wait for all of them.)
  auto body = [&](int s, int cur, Slice& next, Slice& after) {
    fetch(min(s + 2, nsteps - 1) * BK, after);
    multiply(cur);
    if (s + 1 < nsteps) commit(s + 1, next, cur ^ 1);
    __syncthreads();
  };
  fetch(BK, S1);
  commit(0, S0, 0);
  __syncthreads();
  for (int s = 0; s < nsteps; s += 2) {
    body(s, 0, S1, S0);
    if (s + 1 < nsteps) body(s + 1, 1, S0, S1);
  }
}

// One tile of a Gram launch.
template <typename TIn, int LD>
__device__ __forceinline__ void ghost_tile(const GhostArgs& args, const GhostEntry& E, TIn* lds,
                                           float* red) {
  const uint32_t w = blockIdx.x - E.wg_begin;
  const int64_t i = w / (uint32_t)E.pairs;
  const int pr = (int)(w % (uint32_t)E.pairs);
  int p = 0, rem = pr;
  while (rem >= E.nt - p) { rem -= E.nt - p; ++p; }
  const int q = p + rem;
  const int rows_p = min(kTile, E.T - p * kTile);
  const int rows_q = min(kTile, E.T - q * kTile);
  const bool diag = p == q;

  const TIn* A = static_cast<const TIn*>(E.A) + i * (int64_t)E.T * E.d_in;
  const TIn* G = static_cast<const TIn*>(E.G) + i * (int64_t)E.T * E.d_out;

  f32x4_t accA[4][4], accG[4][4];
  gram_phase<TIn, LD>(A + (int64_t)p * kTile * E.d_in, A + (int64_t)q * kTile * E.d_in, E.d_in,
                       E.d_in, rows_p, rows_q, diag, accA, lds);
  gram_phase<TIn, LD>(G + (int64_t)p * kTile * E.d_out, G + (int64_t)q * kTile * E.d_out, E.d_out,
                       E.d_out, rows_p, rows_q, diag, accG, lds);
  float s = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) s = fmaf(accA[a][b][v], accG[a][b][v], s);
  s = block_sum(s, red);
  if (threadIdx.x == 0) args.partials[i * args.P + E.partial_col + pr] = diag ? s : 2.0f * s;
}

// Layers of all load modes run in one launch: small layers of one call often
// differ in it, and launches one after the other cost more than the tiles (24 ->
// 1 -> 17 -> 10 in float32 at B = 8, T = 256: 22 us with a launch for each mode).
template <typename TIn>
__global__ __launch_bounds__(kThreads, 2) void ghost_kernel(GhostArgs args) {
  __shared__ __attribute__((aligned(16))) TIn lds[2 * 2 * lds_operand_elems<TIn>()];
  __shared__ float red[4];
  int lo = 0, hi = args.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (args.L[mid].wg_begin <= blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const GhostEntry& E = args.L[lo];
  if (E.load == LD_VEC) ghost_tile<TIn, LD_VEC>(args, E, lds, red);
  else if (E.load == LD_ANY) ghost_tile<TIn, LD_ANY>(args, E, lds, red);
  else if (E.load == LD_FEW) ghost_tile<TIn, LD_FEW>(args, E, lds, red);
  else ghost_tile<TIn, LD_SHORT>(args, E, lds, red);
}

// ------------------------------------------- ghost, tiles split by columns
//
// A call with few examples and short sequences has fewer tiles than the GPU
// has CUs, and each tile would walk all d_in + d_out columns alone. Here the
// column slices of every tile are dealt to `parts` workgroups (parts_a of them
// take A's slices, the rest G's). Each writes its float32 partial Gram tile to
// the workspace, in register order (64 KB, 16 bytes a lane), and a second
// kernel adds a tile's parts in order, multiplies GA by GG and sums. 768 ->
// 50257 in bf16 with B = 4, T = 128: 4.6 ms with one workgroup a tile (four in
// all), 30 us split (norms and clipped sum together 6.91 -> 0.12 ms, most of the
// rest in the sum's kernel). At most kGsMaxJobs parts run, so that the partial tiles fit the
// allocation-free call's scratch and both calls run the same kernels.

constexpr int kGsTileFloats = kTile * kTile;   // one partial Gram tile
constexpr int64_t kGsMaxJobs = 112;            // partial tiles of a call (7 MB)
constexpr int kGsChunks = 16;                  // combine workgroups (and norm partials) per tile


struct GsEntry {
  const void* A;
  const void* G;
  int32_t d_in, d_out, T;
  int32_t nt, pairs;
  int32_t parts_a, parts;
  uint32_t wg_begin;      // first part job of this layer in the launch
  uint32_t tile_begin;    // first tile of this layer in the launch
  int32_t partial_col;
  int32_t load;           // LoadMode
};
struct GsArgs {
  GsEntry L[kMaxLayersPerLaunch];
  int32_t n;
  int64_t P;
  float* partials;
  float* park;            // [jobs][kGsTileFloats]
};

// Row blocks (p, q), p <= q, of tile pr of the row-major upper triangle.
__device__ __forceinline__ void tile_pair(int nt, int pr, int* p, int* q) {
  int pp = 0, rem = pr;
  while (rem >= nt - pp) { rem -= nt - pp; ++pp; }
  *p = pp;
  *q = pp + rem;
}

template <typename TIn, int LD>
__device__ __forceinline__ void ghost_part(const GsArgs& args, const GsEntry& E, TIn* lds) {
  constexpr int BK = TileCfg<TIn>::BK;
  const uint32_t w = blockIdx.x - E.wg_begin;
  const int part = (int)(w % (uint32_t)E.parts);
  const uint32_t tile = w / (uint32_t)E.parts;
  const int64_t i = tile / (uint32_t)E.pairs;
  int p, q;
  tile_pair(E.nt, (int)(tile % (uint32_t)E.pairs), &p, &q);
  const bool is_a = part < E.parts_a;
  const int d = is_a ? E.d_in : E.d_out;
  const int np = is_a ? E.parts_a : E.parts - E.parts_a, pi = is_a ? part : part - E.parts_a;
  const int slices = (d + BK - 1) / BK;
  const int k0 = (int)((int64_t)slices * pi / np) * BK;
  const int k1 = min((int)((int64_t)slices * (pi + 1) / np) * BK, d);
  const TIn* X = static_cast<const TIn*>(is_a ? E.A : E.G) + i * (int64_t)E.T * d + k0;
  f32x4_t acc[4][4];
  gram_phase<TIn, LD>(X + (int64_t)p * kTile * d, X + (int64_t)q * kTile * d, d, k1 - k0,
                       min(kTile, E.T - p * kTile), min(kTile, E.T - q * kTile), p == q, acc, lds);
  float* dst = args.park + (int64_t)blockIdx.x * kGsTileFloats + 4 * threadIdx.x;
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
      *reinterpret_cast<f32x4_t*>(dst + (4 * a + b) * 4 * kThreads) = acc[a][b];
}

template <typename TIn>
__global__ __launch_bounds__(kThreads, 2) void ghost_part_kernel(GsArgs args) {
  __shared__ __attribute__((aligned(16))) TIn lds[2 * 2 * lds_operand_elems<TIn>()];
  int l = 0;
  while (l + 1 < args.n && args.L[l + 1].wg_begin <= blockIdx.x) ++l;
  const GsEntry& E = args.L[l];
  if (E.load == LD_VEC) ghost_part<TIn, LD_VEC>(args, E, lds);
  else if (E.load == LD_ANY) ghost_part<TIn, LD_ANY>(args, E, lds);
  else if (E.load == LD_FEW) ghost_part<TIn, LD_FEW>(args, E, lds);
  else ghost_part<TIn, LD_SHORT>(args, E, lds);
}

// One workgroup per tile and 1/16 of its elements (one float4 a thread).
__global__ __launch_bounds__(kThreads) void ghost_part_combine_kernel(GsArgs args) {
  __shared__ float red[4];
  const uint32_t tile_g = blockIdx.x / kGsChunks;
  const int chunk = (int)(blockIdx.x % kGsChunks);
  int l = 0;
  while (l + 1 < args.n && args.L[l + 1].tile_begin <= tile_g) ++l;
  const GsEntry& E = args.L[l];
  const uint32_t tile = tile_g - E.tile_begin;
  const int64_t i = tile / (uint32_t)E.pairs;
  const int pr = (int)(tile % (uint32_t)E.pairs);
  const float* src = args.park + ((int64_t)E.wg_begin + (int64_t)tile * E.parts) * kGsTileFloats +
                     chunk * 4 * kThreads + 4 * threadIdx.x;
  f32x4_t ga = {0.f, 0.f, 0.f, 0.f}, gg = {0.f, 0.f, 0.f, 0.f};
  const int na = E.parts_a, n = E.parts;
#pragma unroll 8
  for (int s = 0; s < na; ++s) ga += *reinterpret_cast<const f32x4_t*>(src + (int64_t)s * kGsTileFloats);
#pragma unroll 8
  for (int s = na; s < n; ++s) gg += *reinterpret_cast<const f32x4_t*>(src + (int64_t)s * kGsTileFloats);
  float v = fmaf(ga[0], gg[0], fmaf(ga[1], gg[1], fmaf(ga[2], gg[2], ga[3] * gg[3])));
  v = block_sum(v, red);
  int p, q;
  tile_pair(E.nt, pr, &p, &q);
  if (threadIdx.x == 0)
    args.partials[i * args.P + E.partial_col + pr * kGsChunks + chunk] = p == q ? v : 2.0f * v;
}

// ---------------------------------------------------------- reduce, factors

// FACTORS: also the example's clip factor (one launch for a call that goes on
// to the clipped sum).
template <bool FACTORS>
__global__ __launch_bounds__(kThreads) void norms_reduce_kernel(const float* __restrict__ partials,
                                                                int64_t P, int64_t B,
                                                                float* __restrict__ norms_sq,
                                                                int accumulate, float C,
                                                                float* factors, float* factors_out,
                                                                uint8_t* mask_out) {
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= B) return;  // uniform per wave
  const int lane = threadIdx.x & 63;
  float s = 0.f;
  for (int64_t j = lane; j < P; j += 64) s += partials[i * P + j];
  s = wave_sum(s);
  if (lane == 0) {
    if (accumulate) s += norms_sq[i];
    norms_sq[i] = s;
    if (FACTORS) write_factor(s, C, i, factors, factors_out, mask_out);
  }
}

__global__ __launch_bounds__(kThreads) void clip_factors_kernel(const float* __restrict__ norms_sq,
                                                                int64_t B, float C,
                                                                float* __restrict__ factors,
                                                                float* __restrict__ factors_out,
                                                                uint8_t* __restrict__ mask_out) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < B) write_factor(norms_sq[i], C, i, factors, factors_out, mask_out);
}

// Calls of a few layers that all have T = 1: W waves per example take every
// layer and write the squared norm themselves, so the call is one launch instead
// of two (784 -> 512 -> 10, float32, B = 256: one kernel of 4.6 us for two of
// 3.1 and 2.3 us and the gap between them). With more layers than kT1Layers one
// workgroup per example and layer and a reduction finish sooner.
constexpr int kT1Layers = 4;
constexpr int kT1Waves = kThreads / 64;
struct T1SumArgs {
  T1Entry L[kT1Layers];
  int32_t n;
  int32_t accumulate;
  int64_t B;
  float* norms_sq;
};

// Wave w's share (of W) of the sum of squares of n elements at p (any alignment),
// over its lanes. A wave walks its share alone, a kilobyte a load, so four loads
// are in flight, and examples of 48 KB or more take four waves: three 4096 ->
// 4096 layers in float32 at B = 128 25.4 us with one load and one wave, 10.0 with
// four loads, 5.8 with both (7.8 to 9.5 for the two kernels above); with shorter
// examples one wave is as fast, and faster with many (four 1024 -> 1024 layers in
// bf16 at B = 8192: 21 us and 35).
template <typename TIn, int W>
__device__ __forceinline__ float t1_sum_sq(const TIn* p, int n, int w, int lane) {
  constexpr int E = 16 / (int)sizeof(TIn), kStep = 64 * E * W, kU = 4;
  float s = 0.f;
  auto add = [&](const uint4& v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (E == 8) {
        s = fmaf(bf16_lo(w[k]), bf16_lo(w[k]), s);
        s = fmaf(bf16_hi(w[k]), bf16_hi(w[k]), s);
      } else {
        s = fmaf(__uint_as_float(w[k]), __uint_as_float(w[k]), s);
      }
    }
  };
  int64_t e = (64 * w + lane) * E;
  for (; e + (kU - 1) * kStep + E <= n; e += kU * kStep) {
    uint4 v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) __builtin_memcpy(&v[u], p + e + u * kStep, 16);
#pragma unroll
    for (int u = 0; u < kU; ++u) add(v[u]);
  }
  for (; e + E <= n; e += kStep) {
    uint4 v;
    __builtin_memcpy(&v, p + e, 16);
    add(v);
  }
  for (int k = 0; k < E - 1; ++k)
    if (e + k < n) {
      const float v = load_elem(p + e + k);
      s = fmaf(v, v, s);
    }
  return s;
}

template <typename TIn, int W>
__global__ __launch_bounds__(kThreads) void t1_sum_kernel(T1SumArgs args) {
  __shared__ float red[2][W];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t i = W == 1 ? (int64_t)blockIdx.x * kT1Waves + wave : (int64_t)blockIdx.x;
  if (i >= args.B) return;   // uniform per wave; never with W > 1
  const int w = W == 1 ? 0 : wave;
  float total = args.accumulate ? args.norms_sq[i] : 0.0f;
  for (int l = 0; l < args.n; ++l) {
    const T1Entry& E = args.L[l];
    float sa = t1_sum_sq<TIn, W>(static_cast<const TIn*>(E.A) + i * E.d_in, E.d_in, w, lane);
    float sg = t1_sum_sq<TIn, W>(static_cast<const TIn*>(E.G) + i * E.d_out, E.d_out, w, lane);
    sa = wave_sum(sa);
    sg = wave_sum(sg);
    if constexpr (W > 1) {
      static_assert(W == 4, "four waves' sums");
      __syncthreads();   // the previous layer's sums are read
      if (lane == 0) {
        red[0][w] = sa;
        red[1][w] = sg;
      }
      __syncthreads();
      sa = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
      sg = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    }
    total = fmaf(sa, sg, total);
  }
  if (lane == 0 && w == 0) args.norms_sq[i] = total;
}

template <typename TIn>
int launch_t1_sum(const dpsgd_layer* layers, int n, float* norms_sq, int accumulate,
                  hipStream_t stream) {
  T1SumArgs args{};
  args.n = n;
  args.accumulate = accumulate;
  args.B = layers[0].B;
  args.norms_sq = norms_sq;
  for (int l = 0; l < n; ++l) {
    args.L[l].A = layers[l].A;
    args.L[l].G = layers[l].G;
    args.L[l].d_in = (int32_t)layers[l].d_in;
    args.L[l].d_out = (int32_t)layers[l].d_out;
  }
  int64_t bytes = 0;   // of an example
  for (int l = 0; l < n; ++l) bytes += (layers[l].d_in + layers[l].d_out) * (int64_t)sizeof(TIn);
  if (bytes < (48 << 10))
    hipLaunchKernelGGL((t1_sum_kernel<TIn, 1>), dim3((uint32_t)ceil_div(args.B, kT1Waves)),
                       dim3(kThreads), 0, stream, args);
  else
    hipLaunchKernelGGL((t1_sum_kernel<TIn, kT1Waves>), dim3((uint32_t)args.B), dim3(kThreads), 0, stream,
                       args);
  return check_launch();
}

template <typename TIn>
int launch_t1_group(const dpsgd_layer* layers, const int* idx, int n, const int64_t* cols,
                    float* partials, int64_t P, int64_t B, hipStream_t stream) {
  for (int base = 0; base < n; base += kMaxLayersPerLaunch) {
    const int m = n - base < kMaxLayersPerLaunch ? n - base : kMaxLayersPerLaunch;
    T1Args args{};
    args.n = m;
    args.P = P;
    args.partials = partials;
    for (int k = 0; k < m; ++k) {
      const dpsgd_layer& L = layers[idx[base + k]];
      args.L[k].A = L.A;
      args.L[k].G = L.G;
      args.L[k].d_in = (int32_t)L.d_in;
      args.L[k].d_out = (int32_t)L.d_out;
      args.L[k].partial_col = (int32_t)cols[idx[base + k]];
    }
    hipLaunchKernelGGL(t1_norm_kernel<TIn>, dim3((uint32_t)B, (uint32_t)m), dim3(kThreads), 0,
                       stream, args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

// (The ABI requires 16-byte aligned A and G.)
// LD_FEW: up to 384 columns of A and G together (padded to slices). Loads past
// the last slice are then a good part of all: 32 -> 48 in bf16 at B = 2048, T = 65
// 21.0 us two slices ahead, 19.3 one; 64 -> 12 in float32 at B = 512 19.7 and 17.7;
// from about 500 columns on two ahead is as fast or faster.
template <typename TIn>
LoadMode ghost_load_mode(const dpsgd_layer& L) {
  constexpr int E = TileCfg<TIn>::E, BK = TileCfg<TIn>::BK;
  if (L.d_in < E || L.d_out < E) return LD_SHORT;
  if (L.d_in % E != 0 || L.d_out % E != 0) return LD_ANY;
  return (ceil_div(L.d_in, BK) + ceil_div(L.d_out, BK)) * BK <= 384 ? LD_FEW : LD_VEC;
}

template <typename TIn>
int launch_ghost_group(const dpsgd_layer* layers, int* idx, int n, const int64_t* cols,
                       float* partials, int64_t P, hipStream_t stream) {
  // The widest tiles first, so that no CU gets two of them while others have a
  // narrow one.
  std::stable_sort(idx, idx + n, [&](int a, int b) {
    return layers[a].d_in + layers[a].d_out > layers[b].d_in + layers[b].d_out;
  });
  for (int base = 0; base < n; base += kMaxLayersPerLaunch) {
    const int m = n - base < kMaxLayersPerLaunch ? n - base : kMaxLayersPerLaunch;
    GhostArgs args{};
    args.n = m;
    args.P = P;
    args.partials = partials;
    int64_t wgs = 0;
    for (int k = 0; k < m; ++k) {
      const dpsgd_layer& L = layers[idx[base + k]];
      GhostEntry& E = args.L[k];
      E.A = L.A;
      E.G = L.G;
      E.d_in = (int32_t)L.d_in;
      E.d_out = (int32_t)L.d_out;
      E.T = (int32_t)L.T;
      E.nt = (int32_t)ceil_div(L.T, kTile);
      E.pairs = E.nt * (E.nt + 1) / 2;
      E.wg_begin = (uint32_t)wgs;
      E.partial_col = (int32_t)cols[idx[base + k]];
      E.load = ghost_load_mode<TIn>(L);
      wgs += L.B * (int64_t)E.pairs;
    }
    if (wgs > 0x7FFFFFFF) return DPSGD_ERR_INVALID_ARG;
    hipLaunchKernelGGL(ghost_kernel<TIn>, dim3((uint32_t)wgs), dim3(kThreads), 0, stream,
                       args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

// Parts of a split layer's A and G columns when a part takes `chunk` slices.
struct GsParts {
  int64_t a, g;
};
GsParts gs_parts(const dpsgd_layer& L, int64_t chunk) {
  const int64_t bk = L.dtype == DPSGD_BF16 ? TileCfg<uint16_t>::BK : TileCfg<float>::BK;
  return {ceil_div(ceil_div(L.d_in, bk), chunk), ceil_div(ceil_div(L.d_out, bk), chunk)};
}
int64_t gs_tiles(const dpsgd_layer& L) {
  const int64_t nt = ceil_div(L.T, kTile);
  return L.B * (nt * (nt + 1) / 2);
}
int64_t gs_jobs(const dpsgd_layer* layers, const int* idx, int n, int64_t chunk) {
  int64_t jobs = 0;
  for (int k = 0; k < n; ++k) {
    const GsParts s = gs_parts(layers[idx[k]], chunk);
    jobs += gs_tiles(layers[idx[k]]) * (s.a + s.g);
  }
  return jobs;
}
// Slices per part: the fewest (at least four) whose parts fit kGsMaxJobs.
int64_t gs_chunk(const dpsgd_layer* layers, const int* idx, int n) {
  int64_t lo = 4, hi = 4;
  while (gs_jobs(layers, idx, n, hi) > kGsMaxJobs && hi < (INT64_C(1) << 32)) hi *= 2;
  while (lo < hi) {
    const int64_t mid = (lo + hi) / 2;
    if (gs_jobs(layers, idx, n, mid) <= kGsMaxJobs) hi = mid; else lo = mid + 1;
  }
  return lo;
}

template <typename TIn>
int launch_ghost_split(const dpsgd_layer* layers, const int* idx, int n, int64_t chunk,
                       const int64_t* cols, float* partials, int64_t P, float* park,
                       hipStream_t stream) {
  for (int base = 0; base < n; base += kMaxLayersPerLaunch) {
    const int m = n - base < kMaxLayersPerLaunch ? n - base : kMaxLayersPerLaunch;
    GsArgs args{};
    args.n = m;
    args.P = P;
    args.partials = partials;
    args.park = park;
    int64_t jobs = 0, tiles = 0;
    for (int k = 0; k < m; ++k) {
      const dpsgd_layer& L = layers[idx[base + k]];
      const GsParts s = gs_parts(L, chunk);
      GsEntry& E = args.L[k];
      E.A = L.A;
      E.G = L.G;
      E.d_in = (int32_t)L.d_in;
      E.d_out = (int32_t)L.d_out;
      E.T = (int32_t)L.T;
      E.nt = (int32_t)ceil_div(L.T, kTile);
      E.pairs = E.nt * (E.nt + 1) / 2;
      E.parts_a = (int32_t)s.a;
      E.parts = (int32_t)(s.a + s.g);
      E.wg_begin = (uint32_t)jobs;
      E.tile_begin = (uint32_t)tiles;
      E.partial_col = (int32_t)cols[idx[base + k]];
      E.load = ghost_load_mode<TIn>(L);
      jobs += gs_tiles(L) * E.parts;
      tiles += gs_tiles(L);
    }
    hipLaunchKernelGGL(ghost_part_kernel<TIn>, dim3((uint32_t)jobs), dim3(kThreads), 0,
                       stream, args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
    hipLaunchKernelGGL(ghost_part_combine_kernel, dim3((uint32_t)(tiles * kGsChunks)),
                       dim3(kThreads), 0, stream, args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

template <typename TIn>
int launch_norms_typed(const dpsgd_layer* layers, const NormForm* forms, int n_layers,
                       float* partials, int64_t P, const int64_t* cols, float* park,
                       hipStream_t stream) {
  const int64_t B = layers[0].B;
  int idx_t1[256], n_t1 = 0;
  int idx_gm[256], n_gm = 0;   // general tiles
  int idx_gd[256], n_gd = 0;
  int idx_g4[256], n_g4 = 0;
  int idx_g64[256], n_g64 = 0;
  int idx_mat[256], n_mat = 0;
  int idx_sm[256], n_sm = 0;   // split tiles
  // The part size is planned over all split layers of the call.
  std::vector<int> split;
  for (int l = 0; l < n_layers; ++l)
    if (forms[l] == FORM_GHOST_SPLIT) split.push_back(l);
  const int64_t chunk = split.empty() ? 0 : gs_chunk(layers, split.data(), (int)split.size());
  for (int base = 0; base < n_layers; base += 256) {
    n_t1 = n_gm = n_sm = n_gd = n_g4 = n_g64 = n_mat = 0;
    const int m = n_layers - base < 256 ? n_layers - base : 256;
    for (int k = 0; k < m; ++k) {
      const int l = base + k;
      switch (forms[l]) {
        case FORM_T1: idx_t1[n_t1++] = l; break;
        case FORM_STORED: break;   // skinny.hip
        case FORM_GHOST256: idx_g4[n_g4++] = l; break;
        case FORM_GHOST_SPLIT: idx_sm[n_sm++] = l; break;
        case FORM_GHOST:
          if (ghost_dma_ok(layers[l])) idx_gd[n_gd++] = l;
          else if (gram64_ok(layers[l])) idx_g64[n_g64++] = l;
          else idx_gm[n_gm++] = l;
          break;
        default: idx_mat[n_mat++] = l; break;
      }
    }
    int st = DPSGD_OK;
    if (n_t1) st = launch_t1_group<TIn>(layers, idx_t1, n_t1, cols, partials, P, B, stream);
    if (st == DPSGD_OK && n_gm)
      st = launch_ghost_group<TIn>(layers, idx_gm, n_gm, cols, partials, P, stream);
    if (st == DPSGD_OK && n_sm)
      st = launch_ghost_split<TIn>(layers, idx_sm, n_sm, chunk, cols, partials, P, park, stream);
    if (st == DPSGD_OK && n_gd) st = launch_ghost_dma(layers, idx_gd, n_gd, cols, partials, P, stream);
    if (st == DPSGD_OK && n_g4)
      st = launch_ghost256(layers, idx_g4, n_g4, cols, partials, P, park, stream);
    if (st == DPSGD_OK && n_g64) st = launch_gram64(layers, idx_g64, n_g64, cols, partials, P, stream);
    if (st == DPSGD_OK && n_mat)
      st = launch_mat_norms(layers, idx_mat, n_mat, cols, partials, P, stream);
    if (st != DPSGD_OK) return st;
  }
  return DPSGD_OK;
}

}  // namespace

bool ghost_split_wanted(const dpsgd_layer* layers, const int* idx, int n) {
  // At most a third as many tiles as parts, and a part at most a third of the
  // longest walk over a tile's columns: then the extra pass over the partial
  // tiles is paid back. (Every tile takes a part for A and one for G.)
  int64_t tiles = 0, longest = 0;
  for (int k = 0; k < n; ++k) {
    const GsParts s = gs_parts(layers[idx[k]], 1);
    tiles += gs_tiles(layers[idx[k]]);
    if (s.a + s.g > longest) longest = s.a + s.g;
  }
  if (n <= 0 || 3 * tiles > kGsMaxJobs) return false;
  return longest >= 3 * gs_chunk(layers, idx, n);
}

size_t ghost_split_park_bytes(const dpsgd_layer* layers, const int* idx, int n) {
  if (n <= 0) return 0;
  return (size_t)gs_jobs(layers, idx, n, gs_chunk(layers, idx, n)) * kGsTileFloats * sizeof(float);
}

// Gram form where it issues less MFMA work than `tiles` materialised tiles of
// 128 x 128; work of the Gram kernels counts `weight` times.
static bool gram_is_less(const dpsgd_layer& L, double weight, double tiles) {
  const int64_t bk = L.dtype == DPSGD_BF16 ? TileCfg<uint16_t>::BK : TileCfg<float>::BK;
  const int64_t nt = ceil_div(L.T, kTile);
  // (The float32 kernel for T <= 64 takes one 64 x 64 tile: a quarter of the
  // 128 x 128 one.)
  const double ghost = gram64_ok(L) ? (double)(L.d_in + L.d_out) / 4.0
                                    : (double)(nt * (nt + 1) / 2) *
                                          (double)(ceil_div(L.d_in, bk) * bk + ceil_div(L.d_out, bk) * bk);
  return ghost * weight <= tiles * (double)(ceil_div(L.T, bk) * bk);
}
static double any_tiles_128(const dpsgd_layer& L) {
  return (double)any_tiles(L) * any_tile_area(L) / (kTile * kTile);
}

NormForm resolve_norm_form(const dpsgd_layer& L, int32_t mode) {
  if (L.T == 1) return FORM_T1;
  if (mode == DPSGD_NORM_GHOST) return FORM_GHOST;
  if (mode == DPSGD_NORM_MATERIALIZE) return FORM_MAT;
  const double tiles = gram64_ok(L) ? any_tiles_128(L)
                                    : (double)(ceil_div(L.d_out, kTile) * ceil_div(L.d_in, kTile));
  return gram_is_less(L, 1.0, tiles) ? FORM_GHOST : FORM_MAT;
}

// Estimated times of the two forms in microseconds, without launches, fitted to
// 240 layers (B = 8 to 2048, T = 50 to 512, widths 2 to 1152) within about 10 %.
// Gram: columns of a tile, at one workgroup a CU, then two, then in rounds (a last
// round of one workgroup a CU takes half the time of a whole one).
static double gram_us(const dpsgd_layer& L) {
  const bool bf16 = L.dtype == DPSGD_BF16;
  const int64_t bk = bf16 ? TileCfg<uint16_t>::BK : TileCfg<float>::BK, nt = ceil_div(L.T, kTile);
  const int64_t jobs = L.B * (nt * (nt + 1) / 2), cus = tr_cu_count(), rest = jobs % (2 * cus);
  const double rounds = (double)(jobs / (2 * cus)) + (rest == 0 ? 0.0 : rest <= cus ? 0.5 : 1.0);
  const double cols = (double)((ceil_div(L.d_in, bk) + ceil_div(L.d_out, bk)) * bk);
  const double col_us = jobs <= cus ? (bf16 ? 0.018 : 0.066)
                                    : (bf16 ? 0.022 : 0.13) * rounds;
  return cols * col_us * (any_slow(L) ? (bf16 ? 2.0 : 1.2) : 1.0);
}
// Materialised: 16-row groups of a tile alone, or of all tiles with two
// workgroups a CU; or the VALU kernel's rows (one or two entries a thread,
// d_in + d_out staged elements).
double mat_us(const dpsgd_layer& L) {
  const bool bf16 = L.dtype == DPSGD_BF16;
  const double slots = 2.0 * tr_cu_count(), groups = (double)ceil_div(L.T, 16);
  if (tiny_norm_ok(L)) {
    const double n = L.d_in * L.d_out > kThreads ? 2.0 : 1.0, w = (double)(L.d_in + L.d_out);
    const double row = (bf16 ? 8.0 + 41.0 * n + w : 6.0 + 41.0 * n + 0.65 * w) / 1024.0;
    return std::max(1.0, (double)L.B / slots) * (double)L.T * row;
  }
  const double alone = (bf16 ? 0.5 : 0.9) * groups;
  const double full = (bf16 ? 0.8 : 1.4) * (double)L.B * (double)any_tiles(L) * groups / slots;
  return std::max(alone, full) * (any_slow(L) ? (bf16 ? 2.0 : 1.4) : 1.0);
}

// Layers near the line, where the tiles' work alone misjudges: float32 up to 2.5
// times on the Gram side (whose kernels multiply on the float32 matrix cores,
// the materialised form as products of bf16 parts, but a call with few
// examples leaves most CUs without a Gram tile), and bf16 with d_out <= 64 (tiles
// of 3/4 the area). Gram and materialised, us: float32 768 -> 3072 at B = 8, T = 512
// 283 and 119; 768 -> 256 at B = 64, T = 100 74 and 23; 768 -> 1152 at B = 512, T = 256
// 757 and 1270; 576 -> 512 at T = 128 141 and 253; bf16 144 -> 12 at B = 2048, T = 65 29
// and 24; 16 -> 48 19 and 25. The kernels for T <= 64 in float32 and for 256-row tiles keep
// the plain comparison.
bool may_materialise(const dpsgd_layer& L, int32_t mode) {
  if (mode != DPSGD_NORM_AUTO || L.T == 1 || gram64_ok(L) || ghost256_ok(L)) return false;
  return !gram_is_less(L, L.dtype == DPSGD_F32 ? 2.5 : 1.0, any_tiles_128(L));
}
bool prefer_materialised(const dpsgd_layer& L) { return mat_us(L) < gram_us(L); }

int64_t norm_partials_per_example(const dpsgd_layer& L, NormForm form) {
  switch (form) {
    case FORM_T1: return 1;
    case FORM_STORED: return skinny_chunks(L);
    case FORM_GHOST256: return ghost256_cols(L);
    case FORM_GHOST_SPLIT: {
      const int64_t nt = ceil_div(L.T, kTile);
      return kGsChunks * (nt * (nt + 1) / 2);
    }
    case FORM_GHOST: {
      const int64_t nt = ceil_div(L.T, kTile);
      return nt * (nt + 1) / 2;
    }
    default: return tiny_norm_ok(L) && !tr_tile_ok(L) ? 1 : mat_tile_count(L);
  }
}

int launch_norm_partials(const dpsgd_layer* layers, const NormForm* forms, int n_layers,
                         float* partials, int64_t P, const int64_t* cols, float* park,
                         hipStream_t stream) {
  return layers[0].dtype == DPSGD_BF16
             ? launch_norms_typed<uint16_t>(layers, forms, n_layers, partials, P, cols, park, stream)
             : launch_norms_typed<float>(layers, forms, n_layers, partials, P, cols, park, stream);
}

int launch_norms_reduce(const float* partials, int64_t P, int64_t B, float* norms_sq,
                        int accumulate, hipStream_t stream) {
  const int64_t wgs = ceil_div(B, 4);
  hipLaunchKernelGGL(norms_reduce_kernel<false>, dim3((uint32_t)wgs), dim3(kThreads), 0, stream,
                     partials, P, B, norms_sq, accumulate, 0.0f, nullptr, nullptr, nullptr);
  return check_launch();
}

int launch_norms_reduce_factors(const float* partials, int64_t P, int64_t B, float* norms_sq,
                                float C, float* factors, float* factors_out, uint8_t* mask_out,
                                hipStream_t stream) {
  const int64_t wgs = ceil_div(B, 4);
  hipLaunchKernelGGL(norms_reduce_kernel<true>, dim3((uint32_t)wgs), dim3(kThreads), 0, stream,
                     partials, P, B, norms_sq, 0, C, factors, factors_out, mask_out);
  return check_launch();
}

int launch_norms(const dpsgd_layer* layers, const NormForm* forms, int n_layers, float* norms_sq,
                 int accumulate, float* partials, int64_t P, const int64_t* cols, float* park,
                 hipStream_t stream) {
  bool all_t1 = n_layers <= kT1Layers;
  for (int l = 0; l < n_layers; ++l) all_t1 = all_t1 && forms[l] == FORM_T1;
  if (all_t1)
    return layers[0].dtype == DPSGD_BF16
               ? launch_t1_sum<uint16_t>(layers, n_layers, norms_sq, accumulate, stream)
               : launch_t1_sum<float>(layers, n_layers, norms_sq, accumulate, stream);
  const int st = launch_norm_partials(layers, forms, n_layers, partials, P, cols, park, stream);
  if (st != DPSGD_OK) return st;
  return launch_norms_reduce(partials, P, layers[0].B, norms_sq, accumulate, stream);
}

int launch_clip_factors(const float* norms_sq, int64_t B, float C, float* factors,
                        float* factors_out, uint8_t* mask_out, hipStream_t stream) {
  const int64_t wgs = ceil_div(B, kThreads);
  hipLaunchKernelGGL(clip_factors_kernel, dim3((uint32_t)wgs), dim3(kThreads), 0, stream,
                     norms_sq, B, C, factors, factors_out, mask_out);
  return check_launch();
}

}  // namespace dpsgd
