// Quantiser side: the E- and M-step of the Hessian-weighted EM that initialises a group's
// codebook (paragraph "Codebook Initialization": eq. "hessian_e_step" and the closed form
// below eq. "hessian_m_step"); the E-step is also the VQ_quant operation of Algorithm 2.
//
//   E-step:  a_i = argmin_m  sum_t h[c+t] * (x_i[t] - c_m[t])^2
//   M-step:  c_m[t] = sum_{i in I_m} h[c_i+t] * x_i[t] / sum_{i in I_m} h[c_i+t]   (0 if the sum of weights is 0)
//
// with x_i = W[r, c .. c+d-1] and h[c] = 1 / [H^-1]_cc, the diagonal weight of column c.
// em_assign_kernel: d = 2, groups of 8 x 256 weights.  One wave per group, lane L owns columns
// 4L .. 4L+3 (two vectors) of the group's 8 rows, exactly as in the matrix-vector kernels.
// em_assign_any_kernel: d = 1, 2 or 4 and groups of 1, 4, 8, 16, ... 256 rows x 256 columns (every group
// shape the decode formats use), the same lane ownership.  Both take large codebooks through
// em_assign_filtered, where the matrix cores leave 8 candidates of the k.  em_update_small_kernel / em_update_kernel: the M-step with
// a table per lane or per wave.
//
// The E-step is a decision taken in floating point, so its arithmetic is fixed: binary32,
// every operation rounded on its own (no fused multiply-add), in the order subtract, square,
// times weight, add; the smallest distance wins, the lowest m wins a tie.  The M-step's sums are
// deterministic (see there).
#include "vq_device.h"
#include "vq_internal.h"

namespace vq {
namespace {

// E-step on the matrix cores.  The objective without the part that all centroids share,
//   s_m = sum_t h_t * c_m[t]^2 - 2 * (h_t * x_t) * c_m[t],
// is a product of 2 * D features of the vector (h_t, h_t x_t) with 2 * D features of the centroid.  Each
// feature is split into two fp16 halves and all four half products are taken (K = 16 for d = 2, twice 16
// for d = 4, half of 16 for d = 1): v_mfma_f32_32x32x16_f16 gives the scores of 32 centroids x 32 vectors.
// Powers of two bring the largest coordinate of the codebook and the largest weight of each vector to
// [2^5, 2^6).  The scores are only a filter.  Per vector the smallest block of 8 centroids and the second
// smallest are kept (7 instructions per 8 scores, the block number in the low bits of the score); if the
// second lies above the first by more than the scores can be off by, the assignment is found in the first
// block with the arithmetic that defines the E-step, otherwise in the whole codebook, so the result is the
// defined one bit for bit.
//   How far scores can be off: with X = sum h x^2, a centroid at weighted distance dist from the vector has
// S = sum h c^2 + 2 h |x c| <= 5 X + 3 dist, and only centroids as near as the first block's matter.  Relative to S
// the vector's halves (rounded towards zero) are off by 2^-20, the centroid's by 2^-22, rounded features by 2^-22, and
// the accumulation of 8 D products by 2^-20 D if every addition truncates (2^-23 of the sum so far): kScoreError
// * 2^-20 in all, for each of the two scores compared.  The block number moves a score by 2^-18 of X + dist, and the
// defined arithmetic itself rounds to 2^-21 of dist.  With dist = first + X that is, in 2^-20,
// (16 kScoreError + 17) X + (6 kScoreError + 9) first; a tenth is added for the terms of second order.
// kScoreTiny covers halves that are subnormal: 2^-24 each (the matrix cores keep subnormals) times the largest
// value of the feature they meet, at most 60,000.  Codebooks, weights or vectors outside the ranges checked
// below (NaN, infinities, negative or very uneven weights) take the whole codebook.
//   Bound: vector instructions, the minima first.  The loop over centroids that this replaces takes 18
// (d = 4) or 11 (d = 2) instructions per centroid and vector.
template <int D>
struct EmMargin {
  static constexpr float kScoreError = 1.5f + 1.0f * D;
  static constexpr float kX = 1.1f * (16.f * kScoreError + 17.f) / 1048576.f;
  static constexpr float kFirst = 1.f + 1.1f * (6.f * kScoreError + 9.f) / 1048576.f;
};
constexpr float kScoreTiny = 0.0112f;      // per coordinate
// h x^2 of a vector up to which |h x| <= sqrt(2^6 * 2^25) < 60,000 (scaled)
constexpr float kMaxNorm = 0x1p25f;

typedef _Float16 h8v_t __attribute__((ext_vector_type(8)));

// v as two fp16 halves, each in both halves of a dword; rounded towards zero
__device__ __forceinline__ void split_twice(float v, uint32_t& hi, uint32_t& lo) {
  const auto h = __builtin_amdgcn_cvt_pkrtz(v, v);
  const float rest = v - (float)h[0];
  hi = __builtin_bit_cast(uint32_t, h);
  lo = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(rest, rest));
}
// v as (high half, low half) of one dword; rounded to nearest
__device__ __forceinline__ uint32_t split_once(float v) {
  const _Float16 hi = (_Float16)v;
  const _Float16 lo = (_Float16)(v - (float)hi);
  return __builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
// The power of two that brings v (a positive normal number) to [2^5, 2^6).
__device__ __forceinline__ float scale_to_32(float v) {
  return __builtin_bit_cast(float, (uint32_t)(259 - (int)((__builtin_bit_cast(uint32_t, v) >> 23) & 0xffu)) << 23);
}
__device__ __forceinline__ float power_inverse(float p) { return __builtin_bit_cast(float, 0x7f000000u - __builtin_bit_cast(uint32_t, p)); }
__device__ __forceinline__ float min_nn(float a, float b) { return __builtin_elementwise_minimum(a, b); }
__device__ __forceinline__ float max_nn(float a, float b) { return __builtin_elementwise_maximum(a, b); }

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_inf(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0x7f800000, __builtin_bit_cast(int, v), CTRL, ROWS, 0xf, false));
}
// Minimum over the 64 lanes (no NaN), in every lane.
__device__ __forceinline__ float wave_min(float v) {
  v = min_nn(v, dpp_or_inf<0x111, 0xf>(v));   // row_shr 1, 2, 4, 8: lane 15 of a row of 16 holds the row's
  v = min_nn(v, dpp_or_inf<0x112, 0xf>(v));
  v = min_nn(v, dpp_or_inf<0x114, 0xf>(v));
  v = min_nn(v, dpp_or_inf<0x118, 0xf>(v));
  v = min_nn(v, dpp_or_inf<0x142, 0xa>(v));   // row_bcast 15 and 31: lane 63 holds the wave's
  v = min_nn(v, dpp_or_inf<0x143, 0xc>(v));
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// The values that lanes L and L + 32 hold, in both of them.
__device__ __forceinline__ void both_halves(uint32_t v, uint32_t& lower, uint32_t& upper) {
  const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  lower = r[0];
  upper = r[1];
}
__device__ __forceinline__ void both_halves(float v, float& lower, float& upper) {
  uint32_t a, b;
  both_halves(__builtin_bit_cast(uint32_t, v), a, b);
  lower = __builtin_bit_cast(float, a);
  upper = __builtin_bit_cast(float, b);
}

// The defined arithmetic: binary32, every operation rounded on its own.
template <int D>
__device__ __forceinline__ float em_distance(const float (&x)[D], const float (&h)[D], const float* cm) {
#pragma clang fp contract(off)
  const float e0 = x[0] - cm[0];
  float dist = h[0] * (e0 * e0);
#pragma unroll
  for (int t = 1; t < D; ++t) {
    const float e = x[t] - cm[t];
    dist = dist + h[t] * (e * e);
  }
  return dist;
}

template <int D>
__device__ __forceinline__ void load_coords(const float* p, float (&v)[D]) {
  if constexpr (D == 4) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else if constexpr (D == 2) {
    const float2 t = *reinterpret_cast<const float2*>(p);
    v[0] = t.x; v[1] = t.y;
  } else {
    v[0] = *p;
  }
}

// The q-th coordinate whose features a half-wave holds: d = 4: 2 * half + q; d = 2: half; d = 1: the lower half only.
template <int D>
__device__ __forceinline__ float own_coord(const float (&v)[D], int q, int half) {
  const float lower = v[D == 4 ? q : 0];
  const float upper = D == 1 ? 0.f : v[D == 4 ? D / 2 + q : D - 1];
  return half ? upper : lower;
}

// Where centroid m lies in LDS (floats): a gap after every eighth spreads the blocks that lanes read over the banks.
template <int D>
__device__ __forceinline__ int em_place(int m) { return D * (m + (m >> 3)); }

// The whole codebook for 8 rows of 32 vectors: lanes L and L + 32 take four rows each of the vectors in column
// place L, so that a read of a centroid serves four vectors.  Per 8 centroids only the smallest distance is kept
// (the first block that has it), and its place is found in that block afterwards: 8 (d = 2) or 15 (d = 4)
// instructions per centroid and vector where keeping the place takes 10 or 18.  A NaN distance is never the smallest.
template <int K, int D>
__device__ __forceinline__ void em_assign_whole(const float* cbs, const float* __restrict__ Wl, int in_features,
                                                const float (&h)[D], uint8_t* __restrict__ out) {
#pragma clang fp contract(off)
  float x[4][D], best[4];
  uint32_t blk[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    load_coords<D>(Wl + (size_t)r * in_features, x[r]);
    best[r] = __builtin_inff();
    blk[r] = 0;
  }
  float ahead[8][D];                          // the next 8 centroids; the same address in every lane
#pragma unroll
  for (int j = 0; j < 8; ++j) load_coords<D>(cbs + j * D, ahead[j]);
#pragma unroll 1
  for (uint32_t b = 0; b < K / 8; ++b) {
    float cm[8][D], low[4];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int t = 0; t < D; ++t) cm[j][t] = ahead[j][t];
    const float* next = cbs + em_place<D>(8) * (int)(b + 1 < K / 8 ? b + 1 : b);
#pragma unroll
    for (int j = 0; j < 8; ++j) load_coords<D>(next + j * D, ahead[j]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float dist = em_distance<D>(x[r], h, cm[j]);
        low[r] = j == 0 ? dist : __builtin_fminf(low[r], dist);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (low[r] < best[r]) { best[r] = low[r]; blk[r] = b; }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float* cand = cbs + em_place<D>(8) * (int)blk[r];
    float low = __builtin_inff();
    uint32_t arg = 8 * blk[r];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float dist = em_distance<D>(x[r], h, cand + j * D);
      if (dist < low) { low = dist; arg = 8 * blk[r] + j; }
    }
    out[(size_t)r * (in_features / D)] = (uint8_t)arg;
  }
}

// Workgroups of one wave, one per (8-row block, col-block).  A step is 32 vectors of one row: lanes L and
// L + 32 share vector L, and each scores half of every tile of 32 centroids.
template <int K, int D>
__device__ __forceinline__ void em_assign_filtered(const float* __restrict__ W, const float* __restrict__ hdiag,
                                                   const float* __restrict__ cb, uint8_t* __restrict__ assign,
                                                   int n_cb, int in_features, int group_rows) {
#pragma clang fp contract(off)
  constexpr int TILES = K / 32;
  constexpr int SETS = 8 / D;                 // steps per row
  constexpr int NM = D == 4 ? 2 : 1;          // coordinates per half-wave = matrix instructions per tile
  constexpr uint32_t kBlockMask = 4 * TILES - 1;   // block number: tile, half-wave, upper or lower 8
  constexpr int R = D == 4 ? 2 : 4;           // steps filtered together
  // Undecided vectors of a step from which the whole codebook is faster: a vector taken by itself costs 25, 17, 13 us
  // per 4096 x 4096 and vector of a step, the filter 106, 85, 40, the whole codebook 300, 300, 85 (d = 2 and d = 4 with
  // k = 256, d = 4 with k = 64).  Judged by the first rows of a set; later ones, whose set would be done twice, need
  // twice as many.
  constexpr int kMostUndecided = D == 2 ? 7 : K == 256 ? 13 : 3;
  __shared__ __attribute__((aligned(16))) float cbs[(K + K / 8) * D];
  const int lane = threadIdx.x;
  const int half = lane >> 5, n = lane & 31;
  const uint32_t strip = blockIdx.x / (uint32_t)n_cb;
  const int c = (int)(blockIdx.x - strip * (uint32_t)n_cb);
  const long long row0 = (long long)strip * 8;

  {
    const float* cg = cb + ((long long)((uint32_t)row0 / (uint32_t)group_rows) * n_cb + c) * (K * D);
#pragma unroll
    for (int i = 0; i < (K + 63) / 64; ++i) {
      const int m = i * 64 + lane;
      if (m < K) {
        float v[D];
        load_coords<D>(cg + m * D, v);
#pragma unroll
        for (int t = 0; t < D; ++t) cbs[em_place<D>(m) + t] = v[t];
      }
    }
  }
  const float* Wb = W + (size_t)row0 * in_features + (size_t)c * 256;
  const float* hb = hdiag + (size_t)c * 256;
  uint8_t* ab = assign + (size_t)row0 * (in_features / D) + (size_t)c * (256 / D);
  float xn[R][D];                             // the next R steps' vectors
#pragma unroll
  for (int r = 0; r < R; ++r) load_coords<D>(Wb + (size_t)r * in_features + n * D, xn[r]);
  wave_lds_sync();

  // Centroid features: row j of a tile is given centroid 16 * ((j >> 2) & 1) + 4 * (j >> 3) + (j & 3), so that a
  // lane's 16 scores of a tile are those of centroids 16 * half .. + 15, in order.  K slots of a half-wave, per
  // coordinate: (h hi, h hi, h lo, h lo, hx hi, hx hi, hx lo, hx lo) against (c^2 hi, c^2 lo, twice; -2c hi, -2c lo, twice).
  float top = 0.f;                            // largest coordinate of the codebook (NaN if there is one)
#pragma unroll
  for (int i = 0; i < (K + 63) / 64; ++i)
#pragma unroll
    for (int t = 0; t < D; ++t) top = max_nn(top, __builtin_fabsf(cbs[em_place<D>((i * 64 + lane) % K) + t]));
  const bool nan_c = __any(!(top >= 0.f));
  top = -wave_min(nan_c ? 0.f : -top);
  const bool ok_c = !nan_c && top >= 0x1p-40f && top <= 0x1p20f;
  const float c_scale = ok_c ? scale_to_32(top) : 1.f;
  const float margin_x = EmMargin<D>::kX * c_scale, max_norm = kMaxNorm * power_inverse(c_scale);   // X below lacks one factor c_scale
  const int row_centroid = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  uint4 A[TILES][NM];
#pragma unroll
  for (int t = 0; t < TILES; ++t)
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const bool has = D > 1 || half == 0;    // d = 1: the upper half-wave has no coordinate
      const float cv = has ? c_scale * cbs[em_place<D>(32 * t + row_centroid) + (D > 1 ? NM * half + q : 0)] : 0.f;
      const uint32_t sq = split_once(cv * cv), mul = split_once(-2.f * cv);
      A[t][q] = make_uint4(sq, sq, mul, mul);
    }

  float h[D], hs[D];                          // weights, and weights times both scales
  uint4 B[NM];
  bool filter = ok_c;
#pragma unroll 1
  for (int set = 0, row = 0; set < SETS;) {   // R steps each: 32 vectors of R rows
    bool whole = !filter;                     // this set's vectors against the whole codebook
    const int col = set * 32 + n;             // the vector's place in the row
    if (row == 0) {
      load_coords<D>(hb + col * D, h);
      float h_top = h[0], h_low = h[0];
#pragma unroll
      for (int t = 1; t < D; ++t) {
        h_top = max_nn(h_top, h[t]);
        h_low = min_nn(h_low, h[t]);
      }
      // with h_low >= 2^-20 h_top the bound on h x below is one on x
      const bool good = h_low >= 0x1p-30f && h_top <= 0x1p30f && h_low >= 0x1p-20f * h_top;
      whole = whole || !__all(good);
      const float h_scale = good ? scale_to_32(h_top) : 1.f;
      float hq[D];
#pragma unroll
      for (int t = 0; t < D; ++t) {
        hq[t] = h[t] * h_scale;
        hs[t] = hq[t] * c_scale;
      }
#pragma unroll
      for (int p = 0; p < NM; ++p) split_twice(own_coord<D>(hq, p, half), B[p].x, B[p].y);
    }
    float xs[R][D];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < D; ++t) xs[r][t] = xn[r][t];
    const int row_now = row;
    row = row + R < 8 ? row + R : 0;
    set += row == 0 ? 1 : 0;
    {   // past the end: a harmless re-read
      const int ahead = set < SETS ? set : 0;
#pragma unroll
      for (int r = 0; r < R; ++r)
        load_coords<D>(Wb + (size_t)(row + r) * in_features + (uint32_t)((ahead * 32 + n) * D), xn[r]);
    }
    uint32_t args[R], unsures[R];
    bool in_upper[R];                         // which of lanes L and L + 32 holds the result
    if (!whole) {     // R steps' filters, without a branch between them
      uint4 Bx[R][NM];
      float X[R], m1[R], m2[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float hx[D];
        X[r] = 0.f;
#pragma unroll
        for (int t = 0; t < D; ++t) {
          hx[t] = hs[t] * xs[r][t];
          X[r] = X[r] + hx[t] * xs[r][t];
        }
#pragma unroll
        for (int p = 0; p < NM; ++p) {
          Bx[r][p] = B[p];
          split_twice(own_coord<D>(hx, p, half), Bx[r][p].z, Bx[r][p].w);
        }
        m1[r] = m2[r] = __builtin_inff();
      }
      // The scores of the next tile are on the matrix cores while this one's minima are taken; the compiler
      // would put them one behind the other to save registers.
      auto score = [&](int i, f16v_t& sc) {
#pragma unroll
        for (int j = 0; j < 16; ++j) sc[j] = 0.f;
#pragma unroll
        for (int p = 0; p < NM; ++p)
          sc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8v_t, A[i % TILES][p]),
                                                      __builtin_bit_cast(h8v_t, Bx[i / TILES][p]), sc, 0, 0, 0);
      };
      f16v_t sc[2];
      score(0, sc[0]);
#pragma unroll
      for (int i = 0; i < R * TILES; ++i) {
        if (i + 1 < R * TILES) score(i + 1, sc[(i + 1) & 1]);
        const f16v_t& v = sc[i & 1];
        const int r = i / TILES;
#pragma unroll
        for (int k8 = 0; k8 < 2; ++k8) {
          float e = min_nn(min_nn(v[8 * k8], v[8 * k8 + 1]), v[8 * k8 + 2]);
          e = min_nn(min_nn(e, v[8 * k8 + 3]), v[8 * k8 + 4]);
          e = min_nn(min_nn(e, v[8 * k8 + 5]), v[8 * k8 + 6]);
          e = min_nn(e, v[8 * k8 + 7]);
          e = __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, e) & ~kBlockMask) | (uint32_t)(4 * (i % TILES) + k8));
          m2[r] = __builtin_amdgcn_fmed3f(e, m1[r], m2[r]);   // m1 <= m2: the middle one is the new second smallest
          m1[r] = min_nn(m1[r], e);
        }
        if (i + 1 < R * TILES) __builtin_amdgcn_sched_group_barrier(0x8, NM, 0);   // matrix instructions,
        __builtin_amdgcn_sched_group_barrier(0x2, 14, 0);                          // then vector instructions
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float lo1, hi1, lo2, hi2;      // both halves of the codebook
        both_halves(__builtin_bit_cast(float, __builtin_bit_cast(uint32_t, m1[r]) | (uint32_t)(2 * half)), lo1, hi1);
        both_halves(m2[r], lo2, hi2);
        const float first = min_nn(lo1, hi1);
        const float second = min_nn(max_nn(lo1, hi1), min_nn(lo2, hi2));
        const float limit = first * EmMargin<D>::kFirst + (X[r] * margin_x + D * kScoreTiny);
        // NaN anywhere makes a comparison false; lanes L and L + 32 agree
        unsures[r] = ~((uint32_t)__ballot(second > limit) & (uint32_t)__ballot(X[r] <= max_norm));
        // the 8 centroids of the first block, four per half-wave
        const uint32_t blk = __builtin_bit_cast(uint32_t, first) & kBlockMask;
        const float* cand = cbs + em_place<D>(8) * (int)blk + 4 * D * half;
        float best = em_distance<D>(xs[r], h, cand);
        uint32_t arg = 8 * blk + 4 * half;
        const uint32_t m0 = arg;
#pragma unroll
        for (int j = 1; j < 4; ++j) {
          const float dist = em_distance<D>(xs[r], h, cand + j * D);
          if (dist < best) { best = dist; arg = m0 + j; }
        }
        float bl, bu;
        both_halves(best, bl, bu);
        args[r] = arg;
        in_upper[r] = bu < bl;         // the lower half-wave holds the lower indices
      }
      uint32_t any = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) any |= unsures[r];
      if (any != 0) {
        int undecided = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) undecided += __builtin_popcount(unsures[r]);
        if (undecided > kMostUndecided * R * (row_now == 0 ? 1 : 2)) {
          filter = false;                     // the sets to come will be no better
          goto whole_codebook;
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float (&x)[D] = xs[r];
        uint32_t arg = args[r], left = unsures[r];
        while (left != 0) {      // one vector at a time, K / 64 centroids per lane
          const int src = __builtin_ctz(left);
          left &= left - 1;
          float xv[D], hv[D];
#pragma unroll
          for (int t = 0; t < D; ++t) {
            xv[t] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x[t]), src));
            hv[t] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, h[t]), src));
          }
          float db = __builtin_inff();
          int dj = 0;
#pragma unroll
          for (int j = 0; j < K / 64; ++j) {
            const float dist = em_distance<D>(xv, hv, cbs + em_place<D>(j * 64 + lane));
            if (dist < db) { db = dist; dj = j; }
          }
          // the lowest index that has the smallest distance; no distance below infinity: index 0
          const float mn = wave_min(db);
          int found = 0;
          if (mn < __builtin_inff()) {
            found = -1;
#pragma unroll
            for (int j = 0; j < K / 64; ++j) {
              const unsigned long long at = __ballot(db == mn && dj == j);
              if (found < 0 && at != 0) found = j * 64 + __builtin_ctzll(at);
            }
          }
          if (n == src) arg = (uint32_t)found;
        }
        uint8_t* const out = ab + (size_t)(row_now + r) * (in_features / D);
        if (in_upper[r] == (half != 0)) out[(uint32_t)col] = (uint8_t)arg;
      }
      continue;
    }
  whole_codebook:
    const int now = row == 0 ? set - 1 : set;
    set = now + 1;
    row = 0;
    const int ahead = set < SETS ? set : 0;
#pragma unroll
    for (int r = 0; r < R; ++r)   // before the stores, as on the way past this: a wait for them is one for these too
      load_coords<D>(Wb + (size_t)r * in_features + (uint32_t)((ahead * 32 + n) * D), xn[r]);
    em_assign_whole<K, D>(cbs, Wb + (size_t)(4 * half) * in_features + (now * 32 + n) * D, in_features, h,
                          ab + (size_t)(4 * half) * (in_features / D) + (now * 32 + n));
  }
}

// Which codebooks take the filter; us at 4096 x 4096, loop over the centroids against filter (11008 x 4096 behind):
//                                        d = 2, k = 256, 8 rows     d = 4, k = 256, 256 rows    d = 4, k = 64, 16 rows
//   distinct centroids                   340, 109 (870, 283)        314, 84 (800, 220)          85, 40
//   vectors of the group, drawn with replacement (11, 1.5, 3 % of the centroids repeated, d = 2 with 8 rows most)
//                                        342, 269 (875, 623)        314, 94 (796, 237)          85, 64
//   half of W and a quarter of the centroids zero
//                                        332, 346                   308, 278 (786, 691)         82, 92
//   every centroid twice, or W far from zero: no vector is decided
//                                        340, 314                   310, 308 (794, 830)         85, 91
//   zero, negative or very uneven weights in every set of 32 vectors: no filter
//                                        338, 303                   309, 299 (794, 799)         85, 87
// Equal centroids cost so much because all vectors nearest to them are undecided; an M-step leaves the zero vector in
// the place of every empty cluster.  Not for d = 2, k = 64: 87, 82..110; d = 2, k = 32: 46, 62; d = 1, k = 64: 111, 170
// (scalars lie too close for the filter).  Waves of 16 rows, which would split the centroids' features over twice the
// vectors, were slower (144 for 124).
template <int K, int D> constexpr bool em_filtered() { return (D == 2 && K == 256) || (D == 4 && K >= 64); }
template <int K, int D> constexpr int em_threads() { return em_filtered<K, D>() ? 64 : 256; }
template <int K, int D> constexpr int em_waves() { return em_filtered<K, D>() ? 2 : 1; }   // per SIMD: 256 registers each

template <int K>
__global__ __launch_bounds__((em_threads<K, 2>()), (em_waves<K, 2>())) void em_assign_kernel(const float* __restrict__ W,
                                                        const float* __restrict__ hdiag,
                                                        const float* __restrict__ cb,
                                                        uint8_t* __restrict__ assign, int n_cb,
                                                        long long n_groups, int in_features) {
#pragma clang fp contract(off)
  if constexpr (em_filtered<K, 2>()) {
    em_assign_filtered<K, 2>(W, hdiag, cb, assign, n_cb, in_features, 8);
  } else {
  __shared__ __attribute__((aligned(16))) float2 cbs_all[4][K];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float2* cbs = cbs_all[wave];
  const long long g = (long long)blockIdx.x * 4 + wave;
  if (g >= n_groups) return;   // whole waves leave; no workgroup barrier below
  const long long rb = g / n_cb;
  const int c = (int)(g - rb * n_cb);

  const float2* cg = reinterpret_cast<const float2*>(cb) + g * K;
#pragma unroll
  for (int i = 0; i < (K + 63) / 64; ++i)
    if (i * 64 + lane < K) cbs[i * 64 + lane] = cg[i * 64 + lane];
  const float4 h = *reinterpret_cast<const float4*>(hdiag + (size_t)c * 256 + lane * 4);
  float4 x[8];
#pragma unroll
  for (int r = 0; r < 8; ++r)
    x[r] = *reinterpret_cast<const float4*>(W + (size_t)(rb * 8 + r) * in_features + (size_t)c * 256 + lane * 4);
  wave_lds_sync();

  float best[16];
  uint32_t arg[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    best[v] = __builtin_inff();
    arg[v] = 0;
  }
  for (int m = 0; m < K; ++m) {
    const float2 cm = cbs[m];   // the same address in every lane: one broadcast read
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float ea0 = x[r].x - cm.x, ea1 = x[r].y - cm.y;
      const float eb0 = x[r].z - cm.x, eb1 = x[r].w - cm.y;
      const float da = h.x * (ea0 * ea0) + h.y * (ea1 * ea1);
      const float db = h.z * (eb0 * eb0) + h.w * (eb1 * eb1);
      if (da < best[2 * r]) { best[2 * r] = da; arg[2 * r] = m; }
      if (db < best[2 * r + 1]) { best[2 * r + 1] = db; arg[2 * r + 1] = m; }
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r)
    *reinterpret_cast<uint16_t*>(assign + (size_t)(rb * 8 + r) * (in_features / 2) + (size_t)c * 128 + lane * 2) =
        (uint16_t)(arg[2 * r] | (arg[2 * r + 1] << 8));
  }
}

// ---- any dimensionality and group height ---------------------------------------------------
// E-step.  One wave per (8-row block, col-block); the codebook is that of the group the block
// lies in (NCB = 1), one codebook per row (NCB = 8: groups of one row) or one per 4 rows (NCB = 2).
// D values per centroid, 4 / D vectors per row and lane.  Same arithmetic as em_assign_kernel:
// unfused binary32, sum over t in order.
template <int K, int D, int NCB>
__global__ __launch_bounds__((NCB == 1 ? em_threads<K, D>() : 256), (NCB == 1 ? em_waves<K, D>() : 1)) void em_assign_any_kernel(const float* __restrict__ W,
                                                            const float* __restrict__ hdiag,
                                                            const float* __restrict__ cb,
                                                            uint8_t* __restrict__ assign, int n_cb,
                                                            long long n_blocks, int in_features,
                                                            int group_rows) {
#pragma clang fp contract(off)
  if constexpr (NCB == 1 && em_filtered<K, D>()) {
    em_assign_filtered<K, D>(W, hdiag, cb, assign, n_cb, in_features, group_rows);
  } else {
  constexpr int V = 4 / D;                 // vectors per row and lane
  constexpr int RPC = 8 / NCB;             // rows of the block that share a codebook
  __shared__ __attribute__((aligned(16))) float cbs_all[4][NCB * K * D];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* cbs = cbs_all[wave];
  const long long b = (long long)blockIdx.x * 4 + wave;
  if (b >= n_blocks) return;   // whole waves leave; no workgroup barrier below
  const long long rb = b / n_cb;
  const int c = (int)(b - rb * n_cb);

#pragma unroll
  for (int q = 0; q < NCB; ++q) {
    const long long g = ((rb * 8 + q * RPC) / group_rows) * n_cb + c;
    const float* cg = cb + g * (K * D);
    for (int i = lane; i < K * D; i += 64) cbs[q * K * D + i] = cg[i];
  }
  const float4 h4 = *reinterpret_cast<const float4*>(hdiag + (size_t)c * 256 + lane * 4);
  const float h[4] = {h4.x, h4.y, h4.z, h4.w};
  float x[8][4];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const float4 t = *reinterpret_cast<const float4*>(W + (size_t)(rb * 8 + r) * in_features + (size_t)c * 256 + lane * 4);
    x[r][0] = t.x; x[r][1] = t.y; x[r][2] = t.z; x[r][3] = t.w;
  }
  wave_lds_sync();

  float best[8 * V];
  uint32_t arg[8 * V];
#pragma unroll
  for (int v = 0; v < 8 * V; ++v) {
    best[v] = __builtin_inff();
    arg[v] = 0;
  }
  for (int m = 0; m < K; ++m) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float* cm = cbs + (r / RPC) * K * D + m * D;   // the same address in every lane: broadcast reads
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float e0 = x[r][v * D] - cm[0];
        float dist = h[v * D] * (e0 * e0);
#pragma unroll
        for (int t = 1; t < D; ++t) {
          const float e = x[r][v * D + t] - cm[t];
          dist = dist + h[v * D + t] * (e * e);
        }
        if (dist < best[r * V + v]) { best[r * V + v] = dist; arg[r * V + v] = m; }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    uint8_t* a = assign + (size_t)(rb * 8 + r) * (in_features / D) + (size_t)c * (256 / D) + lane * V;
    if constexpr (V == 4)
      *reinterpret_cast<uint32_t*>(a) = arg[4 * r] | (arg[4 * r + 1] << 8) | (arg[4 * r + 2] << 16) | (arg[4 * r + 3] << 24);
    else if constexpr (V == 2)
      *reinterpret_cast<uint16_t*>(a) = (uint16_t)(arg[2 * r] | (arg[2 * r + 1] << 8));
    else
      *a = (uint8_t)arg[r];
  }
  }
}

// M-step.  A wave walks 8-row blocks of one group (NG = 1) or owns one 8-row block that holds NG = 8 / n_rows
// groups (groups of 1 or 4 rows); WPG waves share a group and take its 8-row blocks in turn.  Every vector
// adds its weighted coordinates and its weights to its centroid's entries of the wave's own table in LDS,
// in binary64: W is read once, whatever k is.  The sums of the waves (and of the copies below) are then
// added in order, divided, and written.
//   Bound: the reads of W and LDS atomics (2 * D per vector, 22 clocks per wave and CU; binary32 atomics take
// 194).  us at 4096 x 4096, against a wave that kept 64 binary32 partial sums per lane and walked the group's
// rows once per 32 / D centroids: d = 4, k = 256, 64 rows 33 (1,081); d = 2, k = 256, 128 rows 30 (899), 8 rows
// 31 (181); k = 64, 32 rows 31 (81); 11008 x 4096, d = 4, k = 256, 256 rows: 86 (4,120).
//   Order: a wave's additions reach an entry in program order, lanes that meet in one instruction in the
// order in which the LDS serves them.  The terms are exact products of two binary32 numbers and the sums
// carry 29 more bits than the result, so even another order could only show where a sum lies within 2^-40 of
// a rounding boundary.
//   Small tables are kept in COPIES copies, lane L using copy L % COPIES, which bounds the lanes that meet
// in one entry; quantity-major order ([2 D][entries]) keeps the lanes of an addition on different banks.
typedef __attribute__((address_space(3))) double* lds_f64_ptr;

template <int K, int D, int NG, int WPG>
struct EmBins {
  static constexpr int kEntries = NG * K;
  static constexpr int kCopies = kEntries >= 64 ? 1 : 64 / kEntries;
  static constexpr int kStride = kEntries * kCopies;        // doubles per quantity
  // Counted: in tall groups with d = 4, k = 256 the weights' sums come from counts, 16 bits per centroid and vector
  // position of a row for the whole workgroup (at most 256 rows): one 32-bit atomic (8 clocks) in place of four
  // binary64 ones (22 to 31 each), and den[t] = sum over the positions of count * h, exact products, at the end.
  // M-step at 11008 x 4096, 256-row groups: 86.6 -> 65 us.  With d = 2 the counts are as large as the tables, which
  // leaves one workgroup on a CU where two fit: 29.9 -> 31.5 us at 4096 x 4096, not done.
  static constexpr bool kCounted = WPG == 8 && K == 256 && D == 4;
  static constexpr int kWords = 32;                         // dwords of counts per centroid: positions i and i + 32
  static constexpr int kTable = (kCounted ? 1 : 2) * D * kStride;   // doubles per wave
};

template <int K, int D, int NG, int WPG>
__global__ __launch_bounds__(WPG > 4 ? 64 * WPG : 256) void em_update_kernel(const float* __restrict__ W,
                                                                             const float* __restrict__ hdiag,
                                                                             const uint8_t* __restrict__ assign,
                                                                             float* __restrict__ cb_out, int n_cb,
                                                                             long long n_items, int in_features,
                                                                             int n_rows) {
  using Bins = EmBins<K, D, NG, WPG>;
  constexpr int V = 4 / D;                          // vectors per row and lane
  constexpr int WAVES = WPG > 4 ? WPG : 4;
  constexpr int RPG = 8 / NG;                       // rows of an 8-row block that share a codebook
  __shared__ __attribute__((aligned(16))) double tab_all[WAVES * Bins::kTable];
  constexpr int CW = Bins::kWords + 1;              // a gap spreads the centroids over the banks (108 KB in all)
  __shared__ uint32_t counts[Bins::kCounted ? K * CW : 1];
  __shared__ double h_all[Bins::kCounted ? 256 : 1], den_all[Bins::kCounted ? K * D : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave % WPG;                       // this wave's place among those that share its group
  double* tab = tab_all + wave * Bins::kTable;
  const long long item_raw = (long long)blockIdx.x * (WAVES / WPG) + wave / WPG;
  const bool present = item_raw < n_items;          // absent items repeat the last one and store nothing
  const long long item = present ? item_raw : n_items - 1;
  const long long ir = item / n_cb;                 // group row, or 8-row block where that holds several groups
  const int c = (int)(item - ir * n_cb);
  const int rows_item = NG > 1 ? 8 : n_rows;
  const long long row0 = ir * rows_item;

  for (int i = lane; i < Bins::kTable / 2; i += 64) reinterpret_cast<double2*>(tab)[i] = make_double2(0., 0.);
  const float4 h4 = *reinterpret_cast<const float4*>(hdiag + (size_t)c * 256 + lane * 4);
  const double h[4] = {h4.x, h4.y, h4.z, h4.w};
  const float* Wl = W + (size_t)row0 * in_features + (size_t)c * 256 + lane * 4;
  const uint8_t* al = assign + (size_t)row0 * (in_features / D) + (size_t)c * (256 / D) + lane * V;
  const int copy = Bins::kCopies > 1 ? lane % Bins::kCopies : 0;
  if constexpr (Bins::kCounted) {
    for (int i = threadIdx.x; i < K * CW; i += 64 * WPG) counts[i] = 0u;
    if (threadIdx.x < 256) h_all[threadIdx.x] = hdiag[(size_t)c * 256 + threadIdx.x];
    __syncthreads();
  } else {
    wave_lds_sync();
  }

  auto load = [&](int r0, float4 (&x)[8], uint32_t (&a)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      x[r] = *reinterpret_cast<const float4*>(Wl + (size_t)(r0 + r) * in_features);
      const uint8_t* ap = al + (size_t)(r0 + r) * (in_features / D);
      if constexpr (V == 4) a[r] = *reinterpret_cast<const uint32_t*>(ap);
      else if constexpr (V == 2) a[r] = *reinterpret_cast<const uint16_t*>(ap);
      else a[r] = *ap;
    }
  };
  auto add = [&](const float4 (&x)[8], const uint32_t (&a)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float xr[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const uint32_t m = (a[r] >> (8 * v)) & 0xffu;
        if (K == 256 || m < (uint32_t)K) {          // an assignment byte beyond the codebook counts nowhere
          double* e = tab + ((r / RPG) * K + m) * Bins::kCopies + copy;
#pragma unroll
          for (int t = 0; t < D; ++t) {
            __builtin_amdgcn_ds_atomic_fadd_f64((lds_f64_ptr)(e + t * Bins::kStride), h[v * D + t] * (double)xr[v * D + t]);
            if constexpr (!Bins::kCounted)
              __builtin_amdgcn_ds_atomic_fadd_f64((lds_f64_ptr)(e + (D + t) * Bins::kStride), h[v * D + t]);
          }
          if constexpr (Bins::kCounted)
            atomicAdd(counts + m * CW + (lane & 31), 1u << (16 * (lane >> 5)));
        }
      }
    }
  };

  // the next 8 rows are in flight while these are added
  float4 x0[8], x1[8];
  uint32_t a0[8], a1[8];
  int r0 = 8 * sub;
  if (r0 < rows_item) {
    load(r0, x0, a0);
    while (true) {
      const int r1 = r0 + 8 * WPG, r2 = r1 + 8 * WPG;
      if (r1 < rows_item) load(r1, x1, a1);
      add(x0, a0);
      if (r1 >= rows_item) break;
      if (r2 < rows_item) load(r2, x0, a0);
      add(x1, a1);
      if (r2 >= rows_item) break;
      r0 = r2;
    }
  }
  if constexpr (WPG > 1) __syncthreads();
  else wave_lds_sync();
  if constexpr (Bins::kCounted) {                   // one item per workgroup: all waves are here
    const int m = threadIdx.x >> 1, half = threadIdx.x & 1;   // two lanes per centroid
    const uint32_t* n = counts + m * CW + half * (Bins::kWords / 2);
    const double* hp = h_all + half * 4 * (Bins::kWords / 2);
    double den[D] = {};
#pragma unroll 4
    for (int i = 0; i < Bins::kWords / 2; ++i) {
      const double lo = n[i] & 0xffffu, hi = n[i] >> 16;
#pragma unroll
      for (int t = 0; t < D; ++t) den[t] += lo * hp[4 * i + t] + hi * hp[4 * i + 128 + t];
    }
#pragma unroll
    for (int t = 0; t < D; ++t) {
      if (den[t] != den[t]) {                       // 0 * infinity or NaN: such a weight counts only where it is used
        den[t] = 0.;
        for (int i = 0; i < Bins::kWords / 2; ++i) {
          if (n[i] & 0xffffu) den[t] += (double)(n[i] & 0xffffu) * hp[4 * i + t];
          if (n[i] >> 16) den[t] += (double)(n[i] >> 16) * hp[4 * i + 128 + t];
        }
      }
      den[t] += __shfl_xor(den[t], 1, 64);
      if (half == 0) den_all[m * D + t] = den[t];
    }
    __syncthreads();
  }
  if (!present) return;                             // no barrier below

  const double* group_tab = tab_all + (size_t)(wave - sub) * Bins::kTable;
  for (int i = sub * 64 + lane; i < NG * K * D; i += 64 * WPG) {
    const int e = i / D, t = i % D;
    double num = 0., den = 0.;
#pragma unroll
    for (int w = 0; w < WPG; ++w)
#pragma unroll
      for (int q = 0; q < Bins::kCopies; ++q) {
        const double* p = group_tab + w * Bins::kTable + e * Bins::kCopies + q;
        num += p[t * Bins::kStride];
        if constexpr (!Bins::kCounted) den += p[(D + t) * Bins::kStride];
      }
    if constexpr (Bins::kCounted) den = den_all[i];
    const long long g = NG > 1 ? (ir * NG + e / K) * n_cb + c : item;
    cb_out[(g * K + e % K) * D + t] = den != 0. ? (float)num / (float)den : 0.f;
  }
}

// M-step for small tables (NG * k * d <= 32) and groups of at most 32 rows: every lane has a table of its own,
// [entry][lane] in LDS, so a vector costs one 2 * D-wide read and write (22 clocks of LDS per wave) instead of
// 2 * D binary64 atomics (22..31 clocks each).  A lane sums its few vectors in binary32, the 64 lanes' sums are
// added in runs of 8, the runs in binary64: a fixed order.  us at 4096 x 4096: d = 2, k = 16, 8 rows 17 (27 with
// atomics); d = 1, k = 16, 8 rows 16 (28); d = 1, k = 4, 1 row 19 (53); d = 1, k = 8, 32 rows 20 (23).
template <int K, int D, int NG>
__global__ __launch_bounds__(64) void em_update_small_kernel(const float* __restrict__ W,
                                                             const float* __restrict__ hdiag,
                                                             const uint8_t* __restrict__ assign,
                                                             float* __restrict__ cb_out, int n_cb,
                                                             int in_features, int n_rows) {
  constexpr int V = 4 / D;
  constexpr int E = NG * K;                         // entries of 2 * D floats
  constexpr int RPG = 8 / NG;
  __shared__ __attribute__((aligned(16))) float tab[E * 64 * 2 * D];
  const int lane = threadIdx.x;
  const uint32_t ir = blockIdx.x / (uint32_t)n_cb;  // group row, or 8-row block where that holds several groups
  const int c = (int)(blockIdx.x - ir * (uint32_t)n_cb);
  const int rows_item = NG > 1 ? 8 : n_rows;

  const float4 h4 = *reinterpret_cast<const float4*>(hdiag + (size_t)c * 256 + lane * 4);
  const float h[4] = {h4.x, h4.y, h4.z, h4.w};
  const float* Wi = W + (size_t)ir * rows_item * in_features + (size_t)c * 256;
  const uint8_t* ai = assign + (size_t)ir * rows_item * (in_features / D) + (size_t)c * (256 / D);
  float* mine = tab + lane * 2 * D;

  auto load = [&](int r0, float4 (&x)[8], uint32_t (&a)[8]) {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      x[r] = *reinterpret_cast<const float4*>(Wi + (size_t)(r0 + r) * in_features + (uint32_t)(lane * 4));
      const uint8_t* ap = ai + (size_t)(r0 + r) * (in_features / D) + (uint32_t)(lane * V);
      if constexpr (V == 4) a[r] = *reinterpret_cast<const uint32_t*>(ap);
      else if constexpr (V == 2) a[r] = *reinterpret_cast<const uint16_t*>(ap);
      else a[r] = *ap;
    }
  };
  float4 x[8], xn[8];
  uint32_t a[8], an[8];
  load(0, x, a);
#pragma unroll
  for (int e = 0; e < E; ++e)
#pragma unroll
    for (int j = 0; j < 2 * D; ++j) mine[e * 128 * D + j] = 0.f;
  for (int r0 = 0;;) {
    const bool more = r0 + 8 < rows_item;
    if (more) load(r0 + 8, xn, an);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const float xr[4] = {x[r].x, x[r].y, x[r].z, x[r].w};
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const uint32_t m = (a[r] >> (8 * v)) & 0xffu;
        if (m < (uint32_t)K) {                      // an assignment byte beyond the codebook counts nowhere
          float* p = mine + ((r / RPG) * K + m) * 128 * D;
          float q[2 * D];
#pragma unroll
          for (int j = 0; j < 2 * D; ++j) q[j] = p[j];
#pragma unroll
          for (int t = 0; t < D; ++t) {
            q[t] += h[v * D + t] * xr[v * D + t];
            q[D + t] += h[v * D + t];
          }
#pragma unroll
          for (int j = 0; j < 2 * D; ++j) p[j] = q[j];
        }
      }
    }
    if (!more) break;
    r0 += 8;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      x[r] = xn[r];
      a[r] = an[r];
    }
  }
  wave_lds_sync();
  // lane q sums quantity q % (2 D) of entry q / (2 D) (d * E <= 32: at most one per lane), starting at another
  // lane for every entry so that the reads of a step hit different banks
  const int e = min(lane / (2 * D), E - 1), j = lane % (2 * D);
  double sum = 0.;
#pragma unroll
  for (int l0 = 0; l0 < 64; l0 += 8) {
    float part = 0.f;
#pragma unroll
    for (int l = 0; l < 8; ++l) part += tab[(e * 64 + ((l0 + l + e) & 63)) * 2 * D + j];
    sum += (double)part;
  }
  const double den = __shfl_down(sum, D, 64);
  if (lane < 2 * D * E && j < D) {
    const long long g = NG > 1 ? ((long long)ir * NG + e / K) * n_cb + c : (long long)blockIdx.x;
    cb_out[(g * K + e % K) * D + j] = den != 0. ? (float)sum / (float)den : 0.f;
  }
}

}  // namespace

// Calls F(K) for the codebook size k (4, 8, 16, 32, 64 or 256).
#define VQ_EM_K_SWITCH(k, F) \
  switch (k) {               \
    case 4: F(4); break;     \
    case 8: F(8); break;     \
    case 16: F(16); break;   \
    case 32: F(32); break;   \
    case 64: F(64); break;   \
    default: F(256); break;  \
  }

// Workgroups of one block each (filtered) or of four.
template <int K, int D> static unsigned em_grid(long long n_blocks) {
  return (unsigned)(em_filtered<K, D>() ? n_blocks : (n_blocks + 3) / 4);
}

hipError_t launch_em_assign(const vq_desc& d, const void* W, const void* hdiag, const void* cb, void* assign,
                            hipStream_t s) {
  const int k = d.k, out_features = d.out_features, in_features = d.in_features;
  const int n_cb = in_features / kGroupCols;
  const long long n_blocks = (long long)(out_features / kGroupRows) * n_cb;
  const unsigned grid = (unsigned)((n_blocks + 3) / 4);
  if (d.d == 2 && d.group_rows == kGroupRows && (k == 16 || k == 64 || k == 256)) {
#define VQ_EM(K)                                                                                   \
  hipLaunchKernelGGL(em_assign_kernel<K>, dim3((em_grid<K, 2>(n_blocks))), dim3((em_threads<K, 2>())), 0, s, (const float*)W, \
                     (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks, in_features)
    if (k == 16) VQ_EM(16);
    else if (k == 64) VQ_EM(64);
    else VQ_EM(256);
#undef VQ_EM
    return hipGetLastError();
  }
#define VQ_EM_ANY(K, D, NCB)                                                                             \
  hipLaunchKernelGGL((em_assign_any_kernel<K, D, NCB>), dim3((NCB == 1 ? em_grid<K, D>(n_blocks) : grid)), \
                     dim3((NCB == 1 ? em_threads<K, D>() : 256)), 0, s, (const float*)W,                   \
                     (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks, in_features, \
                     d.group_rows)
  if (d.group_rows == 1) {   // a codebook per row: k * d <= 64 (checked by the caller)
    if (d.d == 1) {
#define VQ_F(K) if constexpr (K <= 64) VQ_EM_ANY(K, 1, 8); else return hipErrorInvalidValue
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    } else if (d.d == 2) {
#define VQ_F(K) if constexpr (K <= 32) VQ_EM_ANY(K, 2, 8); else return hipErrorInvalidValue
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    } else {
#define VQ_F(K) if constexpr (K <= 16) VQ_EM_ANY(K, 4, 8); else return hipErrorInvalidValue
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    }
  } else if (d.group_rows == 4) {   // two codebooks per 8-row block (d = 1 or 2, checked by the caller)
    if (d.d == 1) {
#define VQ_F(K) VQ_EM_ANY(K, 1, 2)
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    } else {
#define VQ_F(K) VQ_EM_ANY(K, 2, 2)
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    }
  } else if (d.d == 1) {
#define VQ_F(K) VQ_EM_ANY(K, 1, 1)
    VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
  } else if (d.d == 2) {
#define VQ_F(K) VQ_EM_ANY(K, 2, 1)
    VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
  } else {
#define VQ_F(K) VQ_EM_ANY(K, 4, 1)
    VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
  }
#undef VQ_EM_ANY
  return hipGetLastError();
}

template <int K, int D, int NG, int WPG>
static void launch_update(const vq_desc& d, const void* W, const void* hdiag, const void* assign, void* cb_out,
                          hipStream_t s) {
  const int n_cb = d.in_features / kGroupCols;
  const long long n_items = (long long)(d.out_features / (NG > 1 ? kGroupRows : d.group_rows)) * n_cb;
  if constexpr (NG * K * D <= 32 && WPG == 1) {
    hipLaunchKernelGGL((em_update_small_kernel<K, D, NG>), dim3((unsigned)n_items), dim3(64), 0, s, (const float*)W,
                       (const float*)hdiag, (const uint8_t*)assign, (float*)cb_out, n_cb, d.in_features, d.group_rows);
  } else {
    constexpr int waves = WPG > 4 ? WPG : 4, items_per_wg = waves / WPG;
    hipLaunchKernelGGL((em_update_kernel<K, D, NG, WPG>), dim3((unsigned)((n_items + items_per_wg - 1) / items_per_wg)),
                       dim3(64 * waves), 0, s, (const float*)W, (const float*)hdiag, (const uint8_t*)assign,
                       (float*)cb_out, n_cb, n_items, d.in_features, d.group_rows);
  }
}

// Waves per group: one up to 16 rows (32 with a small table), 4 from 32 and 8 from 128 rows on.  A wave's table
// is 16 * k * d bytes, at most 16 KB, and half of it beside counts (d = 4, k = 256, from 128 rows on: 108 KB in all of the CU's 160 KB).
template <int K, int D>
static hipError_t launch_update_rows(const vq_desc& d, const void* W, const void* hdiag, const void* assign, void* cb_out,
                               hipStream_t s) {
  if (d.group_rows == 1) {
    if constexpr (K * D <= 64) launch_update<K, D, 8, 1>(d, W, hdiag, assign, cb_out, s);
    else return hipErrorInvalidValue;
  } else if (d.group_rows == 4) {
    if constexpr (D <= 2) launch_update<K, D, 2, 1>(d, W, hdiag, assign, cb_out, s);
    else return hipErrorInvalidValue;
  } else if (d.group_rows < 32 || (d.group_rows == 32 && K * D <= 32)) {
    launch_update<K, D, 1, 1>(d, W, hdiag, assign, cb_out, s);
  } else if (d.group_rows < 128) {
    launch_update<K, D, 1, 4>(d, W, hdiag, assign, cb_out, s);
  } else {
    launch_update<K, D, 1, 8>(d, W, hdiag, assign, cb_out, s);
  }
  return hipGetLastError();
}

hipError_t launch_em_update(const vq_desc& d, const void* W, const void* hdiag, const void* assign,
                            void* cb_out, hipStream_t s) {
#define VQ_F1(K) return launch_update_rows<K, 1>(d, W, hdiag, assign, cb_out, s)
#define VQ_F2(K) return launch_update_rows<K, 2>(d, W, hdiag, assign, cb_out, s)
#define VQ_F4(K) return launch_update_rows<K, 4>(d, W, hdiag, assign, cb_out, s)
  if (d.d == 1) {
    VQ_EM_K_SWITCH(d.k, VQ_F1)
  } else if (d.d == 2) {
    VQ_EM_K_SWITCH(d.k, VQ_F2)
  } else {
    VQ_EM_K_SWITCH(d.k, VQ_F4)
  }
#undef VQ_F1
#undef VQ_F2
#undef VQ_F4
  return hipErrorInvalidValue;   // not reached: the switch covers every k
}

}  // namespace vq
