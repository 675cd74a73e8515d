// Transposed-operand MFMA GEMM for layers of any width and any number of
// positions (clip-weighted sum and materialised norms):
//
//   clip-weighted sum:  S[m][n] = sum_k w_k G[k][m] A[k][n]     k = (i, t), w_k = c_i
//   materialised norm:  sum_{m,n} (sum_t G_i[t][m] A_i[t][n])^2   per example i
//
// (paper: Section 2.2, the clipped per-example gradients c_i g_i with
// g_i = G_i^T A_i, their sum over the batch, and the 2-norm of g_i.) bf16
// layers whose widths and T suit the larger tiles of gemm_wide.hip and
// gemm_tr.hip go there; this kernel takes every other bf16 layer and every
// float32 layer.
//
// Both operands are stored k-major. A slice of BK rows is loaded into
// registers (16 bytes a lane, eight lanes a row: whole 128-byte lines; global
// loads need no alignment, so widths that are no multiple of 16 bytes load the
// same way), written to LDS k-major and read back transposed with
// ds_read_b64_tr_b16. One LDS slice is filled while the other is multiplied.
// In LDS a 256-byte unit holds 32 columns (64 bytes) of four consecutive
// k-rows: a transposed read of a half-wave covers exactly one unit, hence
// every bank once, and so does each 16- or 32-lane group of the writes (the
// bf16 writes span two column blocks; odd blocks store their rows rotated by
// two places).
//
// float32 on the bf16 matrix cores. A float32 number is the sum of three bf16
// numbers h + m + l (x rounded to bf16, the rest rounded, the rest of that; 24
// significand bits). Both operands are multiplied by 2^24 first (G with its
// clip weight, in one multiplication) and the sums by 2^-48, so that also the
// smallest number's l is a bf16 number (unscaled, operands below 2^-110 lost
// their low bits). The six products of
// weight 2^-18 or more (l h, h l, m m, m h, h m, h h) are accumulated in
// float32; bf16 products are exact there, and the products left out are below
// 2^-26 of a term. Six v_mfma_f32_32x32x16_bf16 take the place of eight
// v_mfma_f32_32x32x2_f32 in 3/8 of the cycles. An infinity has no such parts
// (inf - inf is NaN, and so is inf times a zero part), and operands from 2^103
// or sums from 2^80 leave the range when scaled, so a wave whose result is not
// finite recomputes its block with float32 MFMAs (recompute_f32: about five times
// the time of a sum whose every wave does; a NaN clip factor, after which all
// entries are NaN, is told apart first).
// What bounds it: the matrix cores and, next to them, the conversion on the
// VALU (5.5 instructions an element), so the loads' addresses cost one
// instruction each (a scalar base and a fixed 32-bit lane offset).
// The sixteen convolutions of WRN-16-4 (B = 256, T = 1024, 256 and 64; 343
// GFLOP in all): norms of the materialised ones 1.53 -> 1.05 ms and clipped
// sums 2.18 -> 1.41 ms against float32 MFMAs, the whole call 3.91 -> 2.49 ms
// (two accumulator sets included, which cost 10 % but bring the error against
// float64 from 2.1e-6 to 4.4e-7; 6.8e-7 before; the scaling costs 1 %). A launch
// of 137 GFLOP takes 0.85 ms: with six products each 0.97 PFLOP/s, 70 % of what a
// large bf16 product reaches here (1.5 GHz in a loop of them: the power limit).
// bf16, T = 1 (768 -> 768 and 768 -> 10, B = 2048): 72 -> 17 us.
//
// Clip weights. FLAT (float32, and bf16 with short or badly padded T): rows
// run on through the batch and the weight is multiplied into G on the way to
// LDS (float32 exactly as the definition; for bf16 one rounding of c_i G to
// bf16). EX (bf16): K advances in groups of 16 rows that lie inside one
// example, the accumulator is kept in units of the current example's factor
// and multiplied by c_prev / c_next at each example boundary, so the weights
// are applied in float32. Rows of an example whose factor is 0 are read as
// zeros on both sides: it adds exactly nothing, also when its inputs are not
// finite.
#include <algorithm>

#include "mma.h"

namespace dpsgd {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

enum AnyMode : int { ANY_FLAT = 0, ANY_EX = 1, ANY_SUMSQ = 2 };

// SHAPE 0: 128 x 128 tile, each wave 64 x 64 as 2 x 2 blocks of 32 x 32.
// SHAPE 1 (d_out <= 64): 64 x 192 tile, each wave 32 x 96 as 1 x 3 blocks (a
// convolution's 9 c_in columns are a multiple of 192 for c_in % 64 == 0; on
// 64 x 256 tiles the last of 2.25 tiles of 576 columns kept one wave of four
// busy). Both: waves 2 x 2, eight column blocks of 32, two workgroups per CU.
constexpr int kAnyPerCu = 2;
constexpr float kAnyScale = 0x1p24f, kAnyUnscale = 0x1p-48f;   // float32 operands, sums
constexpr int kAnyBlocks = 8;

template <typename TIn, int SHAPE>
struct AnyCfg {
  static constexpr bool kF32 = sizeof(TIn) == 4;
  static constexpr int kParts = kF32 ? 3 : 1;              // bf16 parts of an element
  static constexpr int kMB = SHAPE ? 1 : 2, kNB = SHAPE ? 3 : 2;   // 32 x 32 blocks per wave
  static constexpr int kTM = 64 * kMB, kTN = 64 * kNB;
  static constexpr int kBlocksM = 2 * kMB;
  static constexpr int kBK = kF32 ? 16 : 64;               // k rows per slice
  static constexpr int kGroups = kBK / 16;                 // 16-row groups per slice
  static constexpr int kE = 16 / (int)sizeof(TIn);         // elements per 16-byte load
  static constexpr int kBlockBytes = kBK / 4 * 256;        // one column block of a slice
  static constexpr int kPartBytes = kAnyBlocks * kBlockBytes;
  static constexpr int kStageBytes = kParts * kPartBytes;  // 24 KB float32, 32 KB bf16
  static constexpr int kLoads = kAnyBlocks * 32 * kBK * (int)sizeof(TIn) / 16 / kThreads;
  static constexpr int kLoadsM = kBlocksM * 32 * kBK * (int)sizeof(TIn) / 16 / kThreads;
  static constexpr int kWaveGroups = kBK == 64 ? 2 : 1;    // groups of a slice one wave loads
};

struct AnyEntry {
  const void* G;         // [B*T][M]
  const void* A;         // [B*T][N]
  float* out;            // sums: grad (splits == 1) or this layer's split partials
  int64_t k_total;       // FLAT: rows B*T; otherwise 16-row groups B * ceil(T / 16)
  int32_t M, N, T;
  int32_t tiles_n;
  int32_t splits;        // sums: K ranges
  int32_t q_per_split;   // sums: slices per range
  uint32_t wg_begin;     // first workgroup of this layer in the launch
  int32_t partial_col;   // norms: first partial slot (one per tile)
  int32_t accumulate;    // sums, splits == 1: add to grad
  int32_t ex_per_job;    // norms: consecutive examples of one job
  int32_t shape;
  int32_t slow;          // any_slow
  uint32_t magic;        // FLAT: divides a row by T; otherwise a group by ceil(T / 16)
  int32_t shift;         // -1: the divisor is 1
};

struct AnyArgs {
  AnyEntry L[kMaxLayersPerLaunch];
  int32_t n;
  int32_t B;
  const float* factors;
  float* partials;       // norms
  int64_t P;
  // FLAT without `factors`: the weights come from the squared norms, and the
  // workgroups after the jobs write them out (either output may be null).
  const float* norms_sq;
  float C;
  float* factors_out;
  uint8_t* mask_out;
  uint32_t jobs;
};

// n / d for n < 2^31 (divide_magic).
__device__ __forceinline__ uint32_t any_div(uint32_t n, uint32_t magic, int shift) {
  return shift < 0 ? n : __umulhi(n, magic) >> shift;
}

// Two transposed reads: k 0..3 and k 4..7 of the lane's eight (of one row).
__device__ __forceinline__ bf16x8_t any_frag(const char* p) {
  typedef short v4i16_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4i16_t lds_v4i16;
  const v4i16_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)p);
  const v4i16_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(p + 256));
  typedef short v8i16_t __attribute__((ext_vector_type(8)));
  const v8i16_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8_t, v);
}

// The wave's block over global rows [r0, r1), by float32 MFMAs with both
// operands straight from memory (lane l: column l % 32 of a block, row l / 32
// of two): for results that are not finite.
template <int MB, int NB>
__device__ __forceinline__ void recompute_f32(const float* G, const float* A, int M, int N,
                                              int m_base, int n_base, int64_t r0, int64_t r1, int T,
                                              const float* factors, const float* norms_sq,
                                              float clip, f32x16_t (&acc)[MB][NB]) {
  const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31;
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f32x16_t{};
  for (int64_t r = r0; r < r1; r += 2) {
    const int64_t row = r + h;
    float c = 1.0f;
    if (factors && row < r1) c = factors[row / T];
    if (norms_sq && row < r1) c = clip_factor(norms_sq[row / T], clip);
    const bool use = row < r1 && c != 0.0f;
    float g[MB], x[NB];
#pragma unroll
    for (int a = 0; a < MB; ++a) {
      const int m = m_base + 32 * a + c32;
      g[a] = use && m < M ? c * G[row * M + m] : 0.0f;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = n_base + 32 * b + c32;
      x[b] = use && n < N ? A[row * N + n] : 0.0f;
    }
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(g[a], x[b], acc[a][b], 0, 0, 0);
  }
}

// One job of a launch. SLOW: layers whose rows the 32-bit lane offsets or the
// 16-byte loads do not suit (any_slow). NSQ (FLAT): see AnyArgs::norms_sq.
// lds: two stages; ended (norms): [2][groups of a slice][4], the four waves'
// sums of the examples that ended in a slice (at most one per group), added
// and stored after the slice's barrier.
template <typename TIn, int SHAPE, int MODE, bool SLOW, bool NSQ>
__device__ __forceinline__ void any_job(const AnyArgs& args, const AnyEntry& E, char* lds,
                                        float (*ended)[4][4]) {
  using C = AnyCfg<TIn, SHAPE>;
  constexpr int ES = (int)sizeof(TIn);
  const int M = E.M, N = E.N, T = E.T;
  const uint32_t magic = E.magic;
  const int shift = E.shift;
  const char* Gb = static_cast<const char*>(E.G);
  const char* Ab = static_cast<const char*>(E.A);
  const int tiles_mn = ((M + C::kTM - 1) / C::kTM) * E.tiles_n;
  // Within a layer, consecutive jobs (the tiles of one K range) run on one XCD
  // and share its L2; every XCD takes an equal share of each layer.
  const int n_outer = MODE == ANY_SUMSQ ? (args.B + E.ex_per_job - 1) / E.ex_per_job : E.splits;
  const uint32_t n_l = (uint32_t)tiles_mn * (uint32_t)n_outer;
  const uint32_t w = xcd_two_class_index(blockIdx.x - E.wg_begin, n_l, n_l);
  const int outer = (int)(w / (uint32_t)tiles_mn);   // K range, or group of examples
  const int tile = (int)(w % (uint32_t)tiles_mn);
  const int tm = tile / E.tiles_n, tn = tile % E.tiles_n;

  // The job's nq slices start at row (FLAT) or 16-row group k0 and end at k1.
  constexpr int kPerSlice = MODE == ANY_FLAT ? C::kBK : C::kGroups;
  const int gpe = (T + 15) >> 4;   // groups per example
  int64_t k0, k1;
  if (MODE == ANY_SUMSQ) {
    k0 = (int64_t)outer * E.ex_per_job * gpe;
    k1 = min((int64_t)(outer + 1) * E.ex_per_job, (int64_t)args.B) * gpe;
  } else {
    k0 = (int64_t)outer * E.q_per_split * kPerSlice;
    k1 = min(k0 + (int64_t)E.q_per_split * kPerSlice, E.k_total);
  }
  const int nq = k1 <= k0 ? 0 : (int)((k1 - k0 + kPerSlice - 1) / kPerSlice);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int m_base = tm * C::kTM + wm * 32 * C::kMB, n_base = tn * C::kTN + wn * 32 * C::kNB;
  const bool inside = m_base < M && n_base < N;   // some of the wave's block is in the matrix
  typedef __attribute__((address_space(4))) const float const_float;
  const const_float* fac = (const const_float*)args.factors;

  // Loads. A wave instruction takes eight rows (lane / 8) of 128 bytes (32
  // float32 or 64 bf16 columns). float32: load u of wave w is rows 8 (w % 2)
  // of the slice's one group, column block w / 2 + 2 u. bf16: load u = W v + gi
  // (W = kWaveGroups) is rows 8 (w % 2) of group w / 2 + 2 gi, column block
  // pair v. The blocks of G come first, then those of A.
  const int rl = 8 * (wave & 1) + (lane >> 3);   // row within its 16-row group
  const int lcol = C::kF32 ? 32 * (wave >> 1) + 4 * (lane & 7) : 8 * (lane & 7);
  constexpr int kColStep = 64;                   // columns from one load to the next (of a group)
  const int gcol = tm * C::kTM + lcol, acol = tn * C::kTN + lcol;
  // A 16-byte load that would overrun its row takes the row's last 16 bytes
  // instead and is shifted down in commit().
  const bool g_edge = (tm + 1) * C::kTM > M, a_edge = (tn + 1) * C::kTN > N;
  constexpr int kPerGroup = C::kLoads / C::kWaveGroups, kPerGroupM = C::kLoadsM / C::kWaveGroups;
  const uint32_t g_stride = (uint32_t)M * ES, a_stride = (uint32_t)N * ES;   // !SLOW: < 2^28
  uint32_t voff[kPerGroup];   // from the group's first row
#pragma unroll
  for (int v = 0; v < kPerGroup; ++v)
    voff[v] = v < kPerGroupM
                  ? (uint32_t)rl * g_stride + (uint32_t)min(gcol + kColStep * v, M - C::kE) * ES
                  : (uint32_t)rl * a_stride +
                        (uint32_t)min(acol + kColStep * (v - kPerGroupM), N - C::kE) * ES;
  const int rows_total = args.B * T;

  // One slice on its way from memory to LDS. Loads are unconditional: lanes
  // whose row does not exist load something else of the tensor and are cleared
  // in commit(). With branches around the loads the compiler waits for each
  // load in turn.
  struct Slice {
    uint4 r[C::kLoads];
    float w[C::kWaveGroups];    // FLAT: clip weight of this lane's row
    int nv[C::kWaveGroups];     // valid rows of the group
  };
  // fetch() takes the slices in order: example and 16-row group within it of
  // the next group this wave loads (EX, SUMSQ), and its number in the job.
  int f_ex[C::kWaveGroups], f_lt[C::kWaveGroups], f_k = 0;
  if (MODE != ANY_FLAT) {
#pragma unroll
    for (int gi = 0; gi < C::kWaveGroups; ++gi) {
      const uint32_t gg = (uint32_t)k0 + (C::kF32 ? 0 : (wave >> 1) + 2 * gi);
      f_ex[gi] = (int)any_div(gg, magic, shift);
      f_lt[gi] = (int)(gg - (uint32_t)f_ex[gi] * (uint32_t)gpe);
    }
  }
  const int nk = (int)max((int64_t)0, k1 - k0);   // rows or groups of the job

  auto fetch = [&](Slice& S) {
#pragma unroll
    for (int gi = 0; gi < C::kWaveGroups; ++gi) {
      const int g = C::kF32 ? 0 : (wave >> 1) + 2 * gi;
      int row0, nv;
      if (MODE == ANY_FLAT) {
        row0 = (int)k0 + f_k + 16 * g;
        nv = min(16, nk - f_k - 16 * g);
      } else {
        row0 = f_ex[gi] * T + 16 * f_lt[gi];
        nv = f_k + g < nk ? min(16, T - 16 * f_lt[gi]) : 0;
        if (MODE == ANY_EX && nv > 0 && fac[f_ex[gi]] == 0.0f) nv = 0;   // its rows count as zeros
        f_lt[gi] += C::kGroups;
        while (f_lt[gi] >= gpe) {
          f_lt[gi] -= gpe;
          ++f_ex[gi];
        }
      }
      if (nv <= 0) {   // nothing of the group is used: any rows serve
        nv = 0;
        row0 = 0;
      }
      S.nv[gi] = nv;
      if (MODE == ANY_FLAT)
        S.w[gi] = (NSQ ? args.norms_sq : args.factors)[any_div(
            (uint32_t)min(row0 + rl, rows_total - 1), magic, shift)];
      if constexpr (SLOW) {
        const int64_t row = min(row0 + rl, rows_total - 1);
#pragma unroll
        for (int v = 0; v < kPerGroup; ++v) {
          const bool gs = v < kPerGroupM;
          const char* p = gs ? Gb + row * M * ES : Ab + row * N * ES;
          const int width = gs ? M : N;
          const int col = gs ? gcol + kColStep * v : acol + kColStep * (v - kPerGroupM);
          uint4 x;
          if (width < C::kE) {   // uniform
            uint32_t y[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < C::kE - 1; ++e)
              if (col + e < width) {
                if (C::kF32) y[e] = reinterpret_cast<const uint32_t*>(p)[col + e];
                else y[e >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(p)[col + e] << (16 * (e & 1));
              }
            x = make_uint4(y[0], y[1], y[2], y[3]);
          } else {
            __builtin_memcpy(&x, p + (int64_t)min(col, width - C::kE) * ES, 16);
          }
          S.r[C::kWaveGroups * v + gi] = x;
        }
      } else {
        // Offsets that stay inside the tensor (its last rows may be fewer than 16).
        const int left = rows_total - row0;
        const uint32_t g_end = left < 16 ? (uint32_t)left * g_stride - 16u : 0xFFFFFFFFu;
        const uint32_t a_end = left < 16 ? (uint32_t)left * a_stride - 16u : 0xFFFFFFFFu;
        const char* pg = Gb + (uint64_t)(uint32_t)row0 * g_stride;
        const char* pa = Ab + (uint64_t)(uint32_t)row0 * a_stride;
#pragma unroll
        for (int v = 0; v < kPerGroup; ++v)
          __builtin_memcpy(&S.r[C::kWaveGroups * v + gi],
                           v < kPerGroupM ? pg + min(voff[v], g_end) : pa + min(voff[v], a_end), 16);
      }
    }
    f_k += MODE == ANY_FLAT ? C::kBK : C::kGroups;
  };

  // LDS byte of this lane's 16 bytes (bf16) or 8 bytes a part (float32) of
  // load u = 0, relative to the stage.
  uint32_t woff;
  if (C::kF32) {
    woff = (uint32_t)((wave >> 1) * C::kBlockBytes + 512 * (wave & 1) + 8 * lane);
  } else {
    const int odd = (lane >> 2) & 1, rr = (lane >> 3) & 3;
    woff = (uint32_t)(odd * C::kBlockBytes + 256 * (4 * (wave >> 1) + 2 * (wave & 1) + (lane >> 5)) +
                      64 * ((rr + 2 * odd) & 3) + 16 * (lane & 3));
  }

  auto commit = [&](Slice& S, int buf) {
    char* dst = lds + buf * C::kStageBytes + woff;
    if (NSQ) {
#pragma unroll
      for (int gi = 0; gi < C::kWaveGroups; ++gi) S.w[gi] = clip_factor(S.w[gi], args.C);
    }
    // Overrunning loads of edge tiles (uniform branches).
    if (g_edge && (!SLOW || M >= C::kE)) {
#pragma unroll
      for (int u = 0; u < C::kLoadsM; ++u)
        S.r[u] = shift_chunk<ES>(S.r[u], max(0, gcol + kColStep * (u / C::kWaveGroups) + C::kE - M));
    }
    if (a_edge && (!SLOW || N >= C::kE)) {
#pragma unroll
      for (int u = C::kLoadsM; u < C::kLoads; ++u)
        S.r[u] = shift_chunk<ES>(
            S.r[u], max(0, acol + kColStep * ((u - C::kLoadsM) / C::kWaveGroups) + C::kE - N));
    }
    // Rows that do not exist or whose clip factor is 0.
#pragma unroll
    for (int gi = 0; gi < C::kWaveGroups; ++gi) {
      const bool no_weight = MODE == ANY_FLAT && S.w[gi] == 0.0f;
      if (S.nv[gi] < 16 || (MODE == ANY_FLAT && __builtin_amdgcn_ballot_w64(no_weight) != 0)) {
        const bool zero = rl >= S.nv[gi] || no_weight;
#pragma unroll
        for (int u = 0; u < C::kLoads; ++u)
          if (u % C::kWaveGroups == gi && zero) S.r[u] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
#pragma unroll
    for (int u = 0; u < C::kLoads; ++u) {
      const bool weigh = MODE == ANY_FLAT && u < C::kLoadsM;
      const int gi = u % C::kWaveGroups, v = u / C::kWaveGroups;
      const uint4 in = S.r[u];
      const float f = C::kF32 ? (weigh ? S.w[gi] * kAnyScale : kAnyScale) : S.w[gi];
      if (C::kF32) {
        float x[4] = {__uint_as_float(in.x), __uint_as_float(in.y), __uint_as_float(in.z),
                      __uint_as_float(in.w)};
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] *= f;
#pragma unroll
        for (int part = 0; part < 3; ++part) {
          const uint2 o = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
          *reinterpret_cast<uint2*>(dst + part * C::kPartBytes + 2 * v * C::kBlockBytes) = o;
          if (part < 2) {
            x[0] -= bf16_lo(o.x);
            x[1] -= bf16_hi(o.x);
            x[2] -= bf16_lo(o.y);
            x[3] -= bf16_hi(o.y);
          }
        }
      } else {
        uint4 o = in;
        if (weigh) {
          o.x = pack_bf16x2(bf16_lo(in.x) * f, bf16_hi(in.x) * f);
          o.y = pack_bf16x2(bf16_lo(in.y) * f, bf16_hi(in.y) * f);
          o.z = pack_bf16x2(bf16_lo(in.z) * f, bf16_hi(in.z) * f);
          o.w = pack_bf16x2(bf16_lo(in.w) * f, bf16_hi(in.w) * f);
        }
        *reinterpret_cast<uint4*>(dst + 2 * v * C::kBlockBytes + gi * 8 * 256) = o;
      }
    }
  };

  // Transposed reads: lane group g = lane / 16, s = lane % 16 takes k-row
  // 8 (g / 2) + 4 h + s / 4 (h = 0, 1: the two units of any_frag), columns
  // 16 (g % 2) + 4 (s % 4) of a block (bf16: rows of odd blocks are rotated by
  // two places).
  uint32_t rg[C::kMB], ra[C::kNB];
  {
    const int g = lane >> 4, s = lane & 15;
    const int in = 512 * (g >> 1) + 32 * (g & 1) + 8 * (s & 3);
    auto at = [&](int block) {
      const int pos = C::kF32 ? (s >> 2) : (((s >> 2) + 2 * (block & 1)) & 3);
      return (uint32_t)(block * C::kBlockBytes + in + 64 * pos);
    };
#pragma unroll
    for (int i = 0; i < C::kMB; ++i) rg[i] = at(C::kMB * wm + i);
#pragma unroll
    for (int i = 0; i < C::kNB; ++i) ra[i] = at(C::kBlocksM + C::kNB * wn + i);
  }

  // float32: the products below the leading one go to accumulators of their
  // own. They are 2^-8 of it or less, and so are their rounding errors; the
  // main accumulators then take one rounding per 16 products.
  f32x16_t acc[C::kMB][C::kNB], low[C::kF32 ? C::kMB : 1][C::kF32 ? C::kNB : 1];
  auto clear = [&]() {
#pragma unroll
    for (int a = 0; a < C::kMB; ++a)
#pragma unroll
      for (int b = 0; b < C::kNB; ++b) {
        acc[a][b] = f32x16_t{};
        if constexpr (C::kF32) low[a][b] = f32x16_t{};
      }
  };
  auto scale = [&](float c) {
#pragma unroll
    for (int a = 0; a < C::kMB; ++a)
#pragma unroll
      for (int b = 0; b < C::kNB; ++b) acc[a][b] *= c;
  };
  auto join_parts = [&]() {
    if constexpr (C::kF32) {
#pragma unroll
      for (int a = 0; a < C::kMB; ++a)
#pragma unroll
        for (int b = 0; b < C::kNB; ++b) acc[a][b] = (acc[a][b] + low[a][b]) * kAnyUnscale;
    }
  };
  clear();
  float c_cur = 1.0f;    // EX: accumulator unit, acc * c_cur is the weighted sum
  bool started = false;
  // Example and 16-row group within it of the next group to multiply.
  int ex = 0, lt = 0;
  if (MODE != ANY_FLAT) {
    ex = (int)any_div((uint32_t)k0, magic, shift);
    lt = (int)(k0 - (int64_t)ex * gpe);
  }

  int n_ended = 0, ended_ex = 0;   // norms: examples that ended in the last slice
  auto flush_ended = [&](int buf) {
    if (MODE == ANY_SUMSQ && tid < n_ended) {
      const float* e = ended[buf][tid];
      args.partials[(int64_t)(ended_ex + tid) * args.P + E.partial_col + tile] =
          (e[0] + e[1]) + (e[2] + e[3]);
    }
  };

  auto multiply = [&](const char* base) {
    bf16x8_t g[C::kParts][C::kMB], x[C::kParts][C::kNB];
#pragma unroll
    for (int p = 0; p < C::kParts; ++p) {
#pragma unroll
      for (int i = 0; i < C::kMB; ++i) g[p][i] = any_frag(base + rg[i] + p * C::kPartBytes);
#pragma unroll
      for (int i = 0; i < C::kNB; ++i) x[p][i] = any_frag(base + ra[i] + p * C::kPartBytes);
    }
    if constexpr (C::kF32) {
      constexpr int pg[6] = {2, 0, 1, 1, 0, 0}, px[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int a = 0; a < C::kMB; ++a)
#pragma unroll
          for (int b = 0; b < C::kNB; ++b) {
            f32x16_t& to = t < 5 ? low[a][b] : acc[a][b];
            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[pg[t]][a], x[px[t]][b], to, 0, 0, 0);
          }
    } else {
#pragma unroll
      for (int a = 0; a < C::kMB; ++a)
#pragma unroll
        for (int b = 0; b < C::kNB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(g[0][a], x[0][b], acc[a][b], 0, 0, 0);
    }
  };

  // Norms, at the end of an example: this wave's share of ||G_i^T A_i||_F^2
  // over the tile. Entries past the edges are 0 for finite inputs, but 0 times
  // an infinity is not, so they are cleared when the sum is not finite.
  auto sum_squares = [&]() {
    float s = 0.f;
    auto square = [&]() {
      s = 0.f;
#pragma unroll
      for (int a = 0; a < C::kMB; ++a)
#pragma unroll
        for (int b = 0; b < C::kNB; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) s = fmaf(acc[a][b][v], acc[a][b][v], s);
      s = wave_sum(s);
    };
    join_parts();
    square();
    if (inside && !(s < __builtin_inff())) {
      if constexpr (C::kF32)
        recompute_f32<C::kMB, C::kNB>(reinterpret_cast<const float*>(Gb),
                                      reinterpret_cast<const float*>(Ab), M, N, m_base, n_base,
                                      (int64_t)ex * T, (int64_t)(ex + 1) * T, T, nullptr, nullptr,
                                      0.f, acc);
      // (The lane index is made here and the conditions are sign bits: otherwise
      // the compiler keeps them in hundreds of scalar registers across the loop.)
      int li;
      asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(li));
      const int rows = M - 1 - m_base - 4 * (li >> 5), cols = N - 1 - n_base - (li & 31);
#pragma unroll
      for (int a = 0; a < C::kMB; ++a)
#pragma unroll
        for (int b = 0; b < C::kNB; ++b)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int past = ((rows - 32 * a - 8 * (v >> 2) - (v & 3)) | (cols - 32 * b)) >> 31;
            acc[a][b][v] = __int_as_float(__float_as_int(acc[a][b][v]) & ~past);
          }
      square();
    }
    clear();
    return s;
  };

  // Slice q is multiplied while slice q + 1 waits in registers and slice q + 2
  // is on its way.
  Slice S0, S1;
  auto body = [&](int q, int cur, Slice& next, Slice& after) {
    fetch(after);
    if (MODE == ANY_SUMSQ) {
      flush_ended(cur ^ 1);
      n_ended = 0;
      ended_ex = ex;
    }
    const char* base = lds + cur * C::kStageBytes;
#pragma unroll
    for (int ks = 0; ks < C::kGroups; ++ks) {
      if (MODE != ANY_FLAT && q * C::kGroups + ks >= nk) break;   // uniform
      if (MODE == ANY_EX && (lt == 0 || !started)) {
        const float c_new = fac[ex];
        if (c_new != 0.0f) {
          if (started && c_cur != c_new) scale(c_cur / c_new);
          c_cur = c_new;
          started = true;
        }
      }
      if (inside) multiply(base + ks * 1024);
      if (MODE != ANY_FLAT && ++lt == gpe) {
        if (MODE == ANY_SUMSQ) {
          const float s = sum_squares();
          if (lane == 0) ended[cur][n_ended][wave] = s;
          ++n_ended;
        }
        lt = 0;
        ++ex;
      }
    }
    if (q + 1 < nq) commit(next, cur ^ 1);
    __syncthreads();
  };
  if (nq > 0) {
    fetch(S0);
    fetch(S1);
    commit(S0, 0);
  }
  __syncthreads();
  for (int q = 0; q < nq; q += 2) {
    body(q, 0, S1, S0);
    if (q + 1 < nq) body(q + 1, 1, S0, S1);
  }
  if (MODE == ANY_SUMSQ) {
    flush_ended((nq - 1) & 1);
    return;
  }

  if (!inside) return;
  join_parts();
  if (MODE == ANY_EX) scale(c_cur);
  if constexpr (C::kF32) {
    float bad = 0.f;   // NaN once an entry is not finite
#pragma unroll
    for (int a = 0; a < C::kMB; ++a)
#pragma unroll
      for (int b = 0; b < C::kNB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) bad = fmaf(acc[a][b][v], 0.0f, bad);
    bool again = __builtin_amdgcn_ballot_w64(bad != bad) != 0;
    if (again) {
      // A NaN factor makes every entry NaN, which it is already.
      bool nan = false;
      for (int64_t i = k0 / T + lane; i <= (k1 - 1) / T; i += 64) {
        const float c = NSQ ? clip_factor(args.norms_sq[i], args.C) : args.factors[i];
        nan = nan || c != c;
      }
      again = __builtin_amdgcn_ballot_w64(nan) == 0;
    }
    if (again)
      recompute_f32<C::kMB, C::kNB>(reinterpret_cast<const float*>(Gb),
                                    reinterpret_cast<const float*>(Ab), M, N, m_base, n_base, k0, k1,
                                    T, NSQ ? nullptr : args.factors, NSQ ? args.norms_sq : nullptr,
                                    args.C, acc);
  }
  // Element v of block (a, b) in lane l: row 32 a + 8 (v / 4) + 4 (l / 32) +
  // v % 4, column 32 b + l % 32.
  float* out = E.out + (E.splits > 1 ? (int64_t)outer * M * N : 0);
  const bool add = E.splits == 1 && E.accumulate;
  // Blocks that lie inside the matrix store without a branch per element, and
  // the loads of an accumulated sum are issued 16 at a time: with short K ranges
  // the stores are a good part of a job (768 -> 50257, B = 4, T = 128: 94 -> 85 us;
  // 768 -> 768, T = 1, B = 2048: 25.9 -> 23.6 us).
#pragma unroll
  for (int a = 0; a < C::kMB; ++a)
#pragma unroll
    for (int b = 0; b < C::kNB; ++b) {
      const int m0 = m_base + 32 * a, n0 = n_base + 32 * b, n = n0 + (lane & 31);
      if (m0 >= M || n0 >= N) continue;
      float* p = out + (int64_t)min(m0 + 4 * (lane >> 5), M - 1) * N + min(n, N - 1);
      if (add) {
        float old[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = m0 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
          old[v] = out[(int64_t)min(m, M - 1) * N + min(n, N - 1)];
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = old[v] + acc[a][b][v];
      }
      if (m0 + 32 <= M && n0 + 32 <= N) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          p[(int64_t)(8 * (v >> 2) + (v & 3)) * N] = acc[a][b][v];
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = 8 * (v >> 2) + (v & 3);
          if (m0 + 4 * (lane >> 5) + m < M && n < N) p[(int64_t)m * N] = acc[a][b][v];
        }
      }
    }
}

// Layers of both shapes run in one launch (their LDS is the same size); SLOW: so
// do layers with and without any_slow.
template <typename TIn, int MODE, bool SLOW, bool NSQ>
__global__ __launch_bounds__(kThreads, kAnyPerCu) void tgemm_any_kernel(AnyArgs args) {
  using C = AnyCfg<TIn, 0>;
  static_assert(C::kStageBytes == AnyCfg<TIn, 1>::kStageBytes && C::kGroups <= 4, "one LDS layout");
  __shared__ __attribute__((aligned(1024))) char lds[2 * C::kStageBytes];
  __shared__ float ended[2][4][4];
  if (NSQ && blockIdx.x >= args.jobs) {
    const int i = (int)(blockIdx.x - args.jobs) * kThreads + (int)threadIdx.x;
    if (i < args.B) write_factor(args.norms_sq[i], args.C, i, nullptr, args.factors_out, args.mask_out);
    return;
  }
  int lo = 0, hi = args.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (args.L[mid].wg_begin <= blockIdx.x) lo = mid; else hi = mid - 1;
  }
  const AnyEntry& E = args.L[lo];
  if (SLOW && E.slow) {
    if (E.shape) any_job<TIn, 1, MODE, SLOW, NSQ>(args, E, lds, ended);
    else any_job<TIn, 0, MODE, SLOW, NSQ>(args, E, lds, ended);
  } else {
    if (E.shape) any_job<TIn, 1, MODE, false, NSQ>(args, E, lds, ended);
    else any_job<TIn, 0, MODE, false, NSQ>(args, E, lds, ended);
  }
}

template <typename TIn, int MODE, bool SLOW, bool NSQ>
int launch_any(const dpsgd_layer* layers, const int* idx, int n, const ClipWeights& weights,
               float* const* outs, const int* splits, const int* accumulate, const int64_t* cols,
               float* partials, int64_t P, hipStream_t stream) {
  for (int base = 0; base < n; base += kMaxLayersPerLaunch) {
    const int m = n - base < kMaxLayersPerLaunch ? n - base : kMaxLayersPerLaunch;
    AnyArgs args{};
    args.n = m;
    args.B = (int32_t)layers[idx[base]].B;
    args.factors = weights.factors;
    args.norms_sq = weights.norms_sq;
    args.C = weights.C;
    // One of the call's launches writes the factors out.
    args.factors_out = base == 0 ? weights.factors_out : nullptr;
    args.mask_out = base == 0 ? weights.mask_out : nullptr;
    args.partials = partials;
    args.P = P;
    int64_t wgs = 0;
    for (int k = 0; k < m; ++k) {
      const int li = idx[base + k];
      const dpsgd_layer& L = layers[li];
      AnyEntry& E = args.L[k];
      const int64_t gpe = ceil_div(L.T, 16);
      E.G = L.G;
      E.A = L.A;
      E.shape = any_shape(L);
      E.slow = any_slow(L) ? 1 : 0;
      E.M = (int32_t)L.d_out;
      E.N = (int32_t)L.d_in;
      E.T = (int32_t)L.T;
      E.k_total = MODE == ANY_FLAT ? L.B * L.T : L.B * gpe;
      divide_magic(MODE == ANY_FLAT ? L.T : gpe, &E.magic, &E.shift);
      E.tiles_n = (int32_t)any_tiles_n(L);
      E.wg_begin = (uint32_t)wgs;
      if (MODE == ANY_SUMSQ) {
        E.partial_col = (int32_t)cols[li];
        E.ex_per_job = any_ex_per_job(L);
        wgs += any_tiles(L) * ceil_div(L.B, E.ex_per_job);
      } else {
        E.out = outs[base + k];
        E.splits = splits[base + k];
        E.q_per_split = (int32_t)ceil_div(any_slices(L), E.splits);
        E.accumulate = accumulate ? accumulate[base + k] : 0;
        wgs += any_tiles(L) * E.splits;
      }
    }
    args.jobs = (uint32_t)wgs;
    if (NSQ && (args.factors_out || args.mask_out)) wgs += ceil_div(args.B, kThreads);
    if (wgs > 0x7FFFFFFF) return DPSGD_ERR_INVALID_ARG;
    hipLaunchKernelGGL((tgemm_any_kernel<TIn, MODE, SLOW, NSQ>), dim3((uint32_t)wgs), dim3(kThreads), 0,
                       stream, args);
    if (check_launch() != DPSGD_OK) return DPSGD_ERR_HIP;
  }
  return DPSGD_OK;
}

}  // namespace

bool any_flat(const dpsgd_layer& L) {
  if (L.dtype == DPSGD_F32) return true;
  // bf16: the weight goes to the accumulator when the zero rows that fill up
  // an example's last 16-row group (or 64-row slice) are at most 1/8 of T; a
  // rescale of the accumulators costs half of a 64-row slice's products, so T
  // is at least 57.
  const int64_t pad16 = ceil_div(L.T, 16) * 16 - L.T, pad64 = ceil_div(L.T, 64) * 64 - L.T;
  return !(pad64 * 8 <= L.T || (L.T >= 64 && pad16 * 8 <= L.T));
}
int any_shape(const dpsgd_layer& L) { return L.d_out <= 64 ? 1 : 0; }
int64_t any_tiles_n(const dpsgd_layer& L) { return ceil_div(L.d_in, any_shape(L) ? 192 : 128); }
int64_t any_tiles(const dpsgd_layer& L) {
  return ceil_div(L.d_out, any_shape(L) ? 64 : 128) * any_tiles_n(L);
}
double any_tile_area(const dpsgd_layer& L) { return any_shape(L) ? 64.0 * 192 : 128.0 * 128; }
int any_slice_rows(const dpsgd_layer& L) { return L.dtype == DPSGD_F32 ? 16 : 64; }
int64_t any_slices(const dpsgd_layer& L) {
  const int64_t bk = any_slice_rows(L);
  return any_flat(L) ? ceil_div(L.B * L.T, bk) : ceil_div(L.B * ceil_div(L.T, 16), bk / 16);
}
int any_workgroups_per_cu() { return kAnyPerCu; }
int any_ex_per_job(const dpsgd_layer& L) {
  // A norm job covers consecutive examples of one tile so that a short T does
  // not leave it mostly in its prologue and epilogue: about 1024 rows, at
  // most 8 examples, and no more than leaves about three rounds of jobs.
  int64_t e = 1024 / (ceil_div(L.T, 16) * 16);
  const int64_t most = L.B * any_tiles(L) / (6 * (int64_t)tr_cu_count());
  if (e > 8) e = 8;
  if (e > most) e = most;
  return (int)(e < 1 ? 1 : e);
}

bool any_slow(const dpsgd_layer& L) {
  // A width below 16 bytes, or rows so long that 16 of them exceed the 32-bit
  // lane offsets.
  const int64_t es = L.dtype == DPSGD_F32 ? 4 : 2;
  return std::min(L.d_in, L.d_out) * es < 16 || std::max(L.d_in, L.d_out) * es >= (INT64_C(1) << 28);
}

// Whether a launch needs the kernel that also takes any_slow layers.
static bool some_slow(const dpsgd_layer* layers, const int* idx, int n) {
  bool slow = false;
  for (int k = 0; k < n; ++k) slow = slow || any_slow(layers[idx[k]]);
  return slow;
}

int launch_any_clip(const dpsgd_layer* layers, const int* idx, int n, const ClipWeights& weights,
                    float* const* outs, const int* splits, const int* accumulate,
                    hipStream_t stream) {
  const dpsgd_layer& L = layers[idx[0]];
  const bool slow = some_slow(layers, idx, n), nsq = weights.norms_sq != nullptr;
#define DPSGD_ANY(T_, M_, S_, Q_) \
  launch_any<T_, M_, S_, Q_>(layers, idx, n, weights, outs, splits, accumulate, nullptr, nullptr, 0, stream)
#define DPSGD_ANY_FLAT(T_)                                                                  \
  (slow ? (nsq ? DPSGD_ANY(T_, ANY_FLAT, true, true) : DPSGD_ANY(T_, ANY_FLAT, true, false)) \
        : (nsq ? DPSGD_ANY(T_, ANY_FLAT, false, true) : DPSGD_ANY(T_, ANY_FLAT, false, false)))
  if (L.dtype == DPSGD_F32) return DPSGD_ANY_FLAT(float);
  if (any_flat(L)) return DPSGD_ANY_FLAT(uint16_t);
  return slow ? DPSGD_ANY(uint16_t, ANY_EX, true, false) : DPSGD_ANY(uint16_t, ANY_EX, false, false);
#undef DPSGD_ANY_FLAT
#undef DPSGD_ANY
}

int launch_any_norms(const dpsgd_layer* layers, const int* idx, int n, const int64_t* cols,
                     float* partials, int64_t P, hipStream_t stream) {
  const dpsgd_layer& L = layers[idx[0]];
#define DPSGD_ANY(T_, S_)                                                                         \
  launch_any<T_, ANY_SUMSQ, S_, false>(layers, idx, n, ClipWeights{}, nullptr, nullptr, nullptr, cols, \
                                       partials, P, stream)
  const bool slow = some_slow(layers, idx, n);
  if (L.dtype == DPSGD_F32) return slow ? DPSGD_ANY(float, true) : DPSGD_ANY(float, false);
  return slow ? DPSGD_ANY(uint16_t, true) : DPSGD_ANY(uint16_t, false);
#undef DPSGD_ANY
}

}  // namespace dpsgd
