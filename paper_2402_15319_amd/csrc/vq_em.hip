// Quantiser side: the E- and M-step of the Hessian-weighted EM that initialises a group's
// codebook (paragraph "Codebook Initialization": eq. "hessian_e_step" and the closed form
// below eq. "hessian_m_step"); the E-step is also the VQ_quant operation of Algorithm 2.
//
//   E-step:  a_i = argmin_m  sum_t h[c+t] * (x_i[t] - c_m[t])^2
//   M-step:  c_m[t] = sum_{i in I_m} h[c_i+t] * x_i[t] / sum_{i in I_m} h[c_i+t]   (0 if the sum of weights is 0)
//
// with x_i = W[r, c .. c+d-1] and h[c] = 1 / [H^-1]_cc, the diagonal weight of column c.
// em_assign_kernel (d = 2, groups of 8 x 256 weights) and em_assign_any_kernel (d = 1, 2 or 4 and groups of 1, 4, 8, 16,
// ... 256 rows x 256 columns: every group shape the decode formats use): large codebooks through em_assign_filtered,
// where the matrix cores leave 8 candidates of the k, the others through em_assign_loop.  em_update_small_kernel /
// em_update_kernel: the M-step with a table per lane or per group.
//
// The E-step is a decision taken in floating point, so its arithmetic is fixed: binary32,
// every operation rounded on its own (no fused multiply-add), in the order subtract, square,
// times weight, add; the smallest distance wins, the lowest m wins a tie.  The M-step's sums are
// deterministic (see there).
#include <type_traits>
#include "vq_device.h"
#include "vq_internal.h"

namespace vq {
namespace {

// E-step on the matrix cores.  The objective without the part that all centroids share,
//   s_m = sum_t h_t * c_m[t]^2 - 2 * (h_t * x_t) * c_m[t],
// is a product of 2 * D features of the vector (h_t, h_t x_t) with 2 * D features of the centroid.  Each
// feature is split into two fp16 halves and all four half products are taken (K = 16 for d = 2, twice 16
// for d = 4): v_mfma_f32_32x32x16_f16 gives the scores of 32 centroids x 32 vectors.
// Powers of two bring the largest coordinate of the codebook and the largest weight of each vector to
// [2^5, 2^6).  The scores are only a filter.  Per vector the smallest block of 8 centroids and the second
// smallest are kept (6.5 instructions per 8 scores, the block number in the low bits of the score); if the
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
//   Bound: vector instructions (80 % of the time with d = 4, k = 256), the minima first: 6.5 per 8 scores.  The loop over
// centroids that this replaces takes 18 (d = 4) or 10 (d = 2) instructions per centroid and vector.
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
  } else {
    const float2 t = *reinterpret_cast<const float2*>(p);
    v[0] = t.x; v[1] = t.y;
  }
}

// The q-th coordinate whose features a half-wave holds: d = 4: 2 * half + q; d = 2: half.
template <int D>
__device__ __forceinline__ float own_coord(const float (&v)[D], int q, int half) { return half ? v[D / 2 + q] : v[q]; }

// Where centroid m lies in LDS (floats): a gap after every eighth spreads the blocks that lanes read over the banks.
template <int D>
__device__ __forceinline__ int em_place(int m) { return D * (m + (m >> 3)); }

// The whole codebook for 2 * RR rows of 32 vectors: lanes L and L + 32 take RR rows each of the vectors in column
// place L, so that a read of a centroid serves RR vectors.  Per 8 centroids only the smallest distance is kept
// (the first block that has it), and its place is found in that block afterwards: 8 (d = 2) or 15 (d = 4)
// instructions per centroid and vector where keeping the place takes 10 or 18.  A NaN distance is never the smallest.
template <int K, int D, int RR>
__device__ __forceinline__ void em_assign_whole(const float* cbs, const float* __restrict__ Wl, int in_features,
                                                const float (&h)[D], uint8_t* __restrict__ out) {
#pragma clang fp contract(off)
  float x[RR][D], best[RR];
  uint32_t blk[RR];
#pragma unroll
  for (int r = 0; r < RR; ++r) {
    load_coords<D>(Wl + (size_t)r * in_features, x[r]);
    best[r] = __builtin_inff();
    blk[r] = 0;
  }
  // The same address in every lane, but in a vector register: from a scalar one the compiler makes an address of its own
  // for every coordinate (d = 4: 32 moves and 32 reads of 4 bytes per 8 centroids in place of 8 reads of 16).
  uint32_t place = 0;
  asm volatile("" : "+v"(place));
#pragma unroll 1
  for (uint32_t b = 0; b < K / 8; ++b, place += em_place<D>(8)) {
    float cm[8][D], low[RR];
#pragma unroll
    for (int j = 0; j < 8; ++j) load_coords<D>(cbs + place + j * D, cm[j]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const float dist = em_distance<D>(x[r], h, cm[j]);
        low[r] = j == 0 ? dist : __builtin_fminf(low[r], dist);
      }
    }
#pragma unroll
    for (int r = 0; r < RR; ++r)
      if (low[r] < best[r]) { best[r] = low[r]; blk[r] = b; }
  }
#pragma unroll
  for (int r = 0; r < RR; ++r) {
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

// Workgroups of four waves, one per (strip of 8, 16 or 32 rows, col-block).  A step is 32 vectors of one row: lanes L
// and L + 32 share vector L, and each scores half of every tile of 32 centroids.  A wave keeps to one place of 32
// vectors in the rows (its weights and their features are made once) and takes all rows of the strip (d = 2) or
// half of them (d = 4).  The centroids' features are made once per workgroup, in LDS, from where a wave reads those of
// a tile for R rows (64 registers and a prologue in every wave otherwise, which left two waves per SIMD).
//   Equal centroids: a vector nearest to one would see the same score in two blocks and be undecided.  Centroids are
// therefore compared through a table of their hashes; if some are equal, the filter works on the distinct ones (the
// lowest index of each), spread over the blocks, whose other places repeat the first of their block, and `origin`
// leads back.  Blocks list their centroids in the order of the codebook, so the lowest index still wins a tie.
template <int K, int D>
__device__ __forceinline__ void em_assign_filtered(const float* __restrict__ W, const float* __restrict__ hdiag,
                                                   const float* __restrict__ cb, uint8_t* __restrict__ assign,
                                                   int n_cb, int in_features, int group_rows, int strip_rows) {
#pragma clang fp contract(off)
  static_assert((D == 2 || D == 4) && K % 64 == 0 && K <= 256, "half-waves share the coordinates, lanes the centroids");
  constexpr int TILES = K / 32, NB = K / 8;
  constexpr int SETS = 8 / D;                 // places of 32 vectors in the 256 columns of a row
  constexpr int PARTS = 4 / SETS;             // waves that share a place
  constexpr int NM = D / 2;                   // coordinates per half-wave = matrix instructions of a tile's features
  constexpr uint32_t kBlockMask = 4 * TILES - 1;   // block number: tile, half-wave, upper or lower 8
  constexpr int R = 4;                        // steps filtered together
  // Undecided vectors of a step from which the whole codebook is faster, for its rows and those to come.  A vector taken by
  // itself costs 25, 17, 13 us per 4096 x 4096 and vector of a step (d = 2, d = 4 with k = 256, d = 4 with k = 64).
  constexpr int kMostUndecided = D == 2 ? (K == 256 ? 7 : 3) : K == 256 ? 13 : 3;
  __shared__ __attribute__((aligned(16))) float cbs[(K + K / 8) * D];
  __shared__ __attribute__((aligned(16))) float distinct[(K + K / 8) * D];
  __shared__ uint8_t origin[K];
  __shared__ int n_distinct[4];
  __shared__ __attribute__((aligned(16))) uint4 feat[TILES * NM * 64];
  static_assert(sizeof(feat) >= 8 * K * sizeof(uint32_t), "the hash tables lie where the features will");
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, n = lane & 31;
  const uint32_t strip = blockIdx.x / (uint32_t)n_cb;
  const int c = (int)(blockIdx.x - strip * (uint32_t)n_cb);
  const int rows = strip_rows / PARTS;        // of this wave
  const int set = wave % SETS, col = set * 32 + n;   // the vector's place in the row
  const long long row_strip = (long long)strip * strip_rows, row0 = row_strip + (wave / SETS) * rows;

  const float* Wb = W + (size_t)row0 * in_features + (size_t)c * 256 + col * D;
  uint8_t* ab = assign + (size_t)row0 * (in_features / D) + (size_t)c * (256 / D) + col;
  float xn[R][D], h[D];                       // the next R steps' vectors
#pragma unroll
  for (int r = 0; r < R; ++r) load_coords<D>(Wb + (size_t)r * in_features, xn[r]);
  load_coords<D>(hdiag + (size_t)c * 256 + col * D, h);

  // the codebook, and which of its centroids are the first of their value
  const float* fcb = cbs;                     // what the filter works on
  bool repeats, filter = true;
  {
    uint32_t* table = reinterpret_cast<uint32_t*>(feat);   // two of 4 K entries: a value that loses its place in both to others counts as distinct
    float v[D];
    uint32_t slot[2] = {0u, 4u * K};
    const bool mine = tid < K;
    for (int i = tid; i < 8 * K; i += 256) table[i] = K;
    if (mine) {
      const float* cg = cb + ((long long)((uint32_t)row_strip / (uint32_t)group_rows) * n_cb + c) * (K * D);
      load_coords<D>(cg + tid * D, v);
      uint32_t mix = 0;
#pragma unroll
      for (int t = 0; t < D; ++t) {
        cbs[em_place<D>(tid) + t] = v[t];
        mix = (mix ^ __builtin_bit_cast(uint32_t, v[t] + 0.f)) * 0x9e3779b1u;   // the two zeros are equal
        mix ^= mix >> 15;
      }
      slot[0] += mix % (4u * K);
      slot[1] += (mix >> 12) % (4u * K);
    }
    __syncthreads();
    if (mine) {
      atomicMin(table + slot[0], (uint32_t)tid);
      atomicMin(table + slot[1], (uint32_t)tid);
    }
    __syncthreads();
    bool first = mine;
    if (mine) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t m = table[slot[i]];
        if (m != (uint32_t)tid) {
          bool same = true;
#pragma unroll
          for (int t = 0; t < D; ++t) same = same && v[t] == cbs[em_place<D>(m) + t];
          first = first && !same;
        }
      }
    }
    const unsigned long long firsts = __ballot(first);
    if (lane == 0) n_distinct[wave] = __builtin_popcountll(firsts);
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int nw = n_distinct[w];
      before += w < wave ? nw : 0;
      all += nw;
    }
    all = __builtin_amdgcn_readfirstlane(all);
    repeats = all < K;
    if (repeats) {
      if (all < NB) {                         // a block for each would leave some empty
        filter = false;
      } else {
        const int rank = before + __builtin_popcountll(firsts & ((1ull << lane) - 1ull));
        if (first) {
          const int m = 8 * (rank % NB) + rank / NB;
#pragma unroll
          for (int t = 0; t < D; ++t) distinct[em_place<D>(m) + t] = v[t];
          origin[m] = (uint8_t)tid;
        }
        __syncthreads();
        if (mine && (tid & 7) * NB + (tid >> 3) >= all) {   // a place that no distinct centroid has
          const int m = tid & ~7;
#pragma unroll
          for (int t = 0; t < D; ++t) distinct[em_place<D>(tid) + t] = distinct[em_place<D>(m) + t];
          origin[tid] = origin[m];
        }
        __syncthreads();
        fcb = distinct;
      }
    }
  }

  // Centroid features: row j of a tile is given centroid 16 * ((j >> 2) & 1) + 4 * (j >> 3) + (j & 3), so that a
  // lane's 16 scores of a tile are those of centroids 16 * half .. + 15, in order.  K slots of a half-wave, per
  // coordinate: (h hi, h hi, h lo, h lo, hx hi, hx hi, hx lo, hx lo) against (c^2 hi, c^2 lo, twice; -2c hi, -2c lo, twice).
  // d = 2: both in one matrix instruction; d = 4: the first four of the half-wave's two coordinates in one, which serves
  // the R rows, the last four in another.
  float top = 0.f;                            // largest coordinate of the codebook (NaN if there is one)
#pragma unroll
  for (int i = 0; i < K / 64; ++i)
#pragma unroll
    for (int t = 0; t < D; ++t) top = max_nn(top, __builtin_fabsf(cbs[em_place<D>(i * 64 + lane) + t]));
  const bool nan_c = __any(!(top >= 0.f));
  top = -wave_min(nan_c ? 0.f : -top);
  const bool ok_c = !nan_c && top >= 0x1p-40f && top <= 0x1p20f;
  const float c_scale = ok_c ? scale_to_32(top) : 1.f;
  const float margin_x = EmMargin<D>::kX * c_scale, max_norm = kMaxNorm * power_inverse(c_scale);   // X below lacks one factor c_scale
  const int row_centroid = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  for (int t = wave; t < TILES; t += 4) {
    uint32_t sq[NM], mul[NM];
#pragma unroll
    for (int q = 0; q < NM; ++q) {
      const float cv = c_scale * fcb[em_place<D>(32 * t + row_centroid) + NM * half + q];
      sq[q] = split_once(cv * cv);
      mul[q] = split_once(-2.f * cv);
    }
    if constexpr (D == 2) {
      feat[t * 64 + lane] = make_uint4(sq[0], sq[0], mul[0], mul[0]);
    } else {
      feat[(2 * t) * 64 + lane] = make_uint4(sq[0], sq[0], sq[1], sq[1]);
      feat[(2 * t + 1) * 64 + lane] = make_uint4(mul[0], mul[0], mul[1], mul[1]);
    }
  }
  __syncthreads();                            // the last one: waves leave at different times

  uint4 Bh = make_uint4(0, 0, 0, 0);          // the weights' halves (d = 2: .x and .y of the operand)
  float hs[D];                                // weights times both scales
  {
    float h_top = h[0], h_low = h[0];
#pragma unroll
    for (int t = 1; t < D; ++t) {
      h_top = max_nn(h_top, h[t]);
      h_low = min_nn(h_low, h[t]);
    }
    // with h_low >= 2^-20 h_top the bound on h x below is one on x
    const bool good = h_low >= 0x1p-30f && h_top <= 0x1p30f && h_low >= 0x1p-20f * h_top;
    filter = filter && ok_c && __all(good);
    const float h_scale = good ? scale_to_32(h_top) : 1.f;
    float hq[D];
#pragma unroll
    for (int t = 0; t < D; ++t) {
      hq[t] = h[t] * h_scale;
      hs[t] = hq[t] * c_scale;
    }
    split_twice(own_coord<D>(hq, 0, half), Bh.x, Bh.y);
    if constexpr (D == 4) split_twice(own_coord<D>(hq, 1, half), Bh.z, Bh.w);
  }
  // The filter decides hardly any of the vectors far from zero beside the distances between centroids: its margin is that
  // share of their norm.  With K centroids drawn from a normal distribution, 95 % are undecided if the margin is the distance of
  // two centroids times 2 / K (d = 2) or 0.5 / sqrt(K) (d = 4); each lane asks that of its first vector and two distinct
  // centroids, and the wave follows the majority.  A rule of speed alone.
  {
    float a[D], norm = 0.f;
    load_coords<D>(fcb + em_place<D>(8) * (n % NB), a);
#pragma unroll
    for (int t = 0; t < D; ++t) norm += h[t] * xn[0][t] * xn[0][t];
    const float apart = em_distance<D>(a, h, fcb + em_place<D>(8) * ((n + 1) % NB));
    const float share = D == 2 ? 2.f / K : K == 256 ? 0.5f / 16 : 0.5f / 8;
    filter = filter && __builtin_popcountll(__ballot(EmMargin<D>::kX * norm > share * apart)) <= 32;
  }
#pragma unroll 1
  for (int row = 0; row < rows;) {            // R steps each
    float xs[R][D];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < D; ++t) xs[r][t] = xn[r][t];
    const int row_now = row;
    row += R;
    {   // past the end: a harmless re-read
      const int ahead = row < rows ? row : 0;
#pragma unroll
      for (int r = 0; r < R; ++r) load_coords<D>(Wb + (size_t)(ahead + r) * in_features, xn[r]);
    }
    uint32_t args[R], unsures[R];
    bool in_upper[R];                         // which of lanes L and L + 32 holds the result
    if (filter) {     // R steps' filters, without a branch between them
      uint4 Bx[R];
      float X[R], m1[R], m2[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float hx[D];
#pragma unroll
        for (int t = 0; t < D; ++t) {
          hx[t] = hs[t] * xs[r][t];
          X[r] = t == 0 ? hx[t] * xs[r][t] : X[r] + hx[t] * xs[r][t];
        }
        if constexpr (D == 2) {
          Bx[r].x = Bh.x;
          Bx[r].y = Bh.y;
          split_twice(own_coord<D>(hx, 0, half), Bx[r].z, Bx[r].w);
        } else {
          split_twice(own_coord<D>(hx, 0, half), Bx[r].x, Bx[r].y);
          split_twice(own_coord<D>(hx, 1, half), Bx[r].z, Bx[r].w);
        }
        m1[r] = m2[r] = __builtin_inff();
      }
      // One tile after the other, R rows each.
#pragma unroll
      for (int i = 0; i < TILES; ++i) {
        f16v_t sc[R], zero;
#pragma unroll
        for (int j = 0; j < 16; ++j) zero[j] = 0.f;
        if constexpr (D == 4) {
          const f16v_t base = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8v_t, feat[2 * i * 64 + lane]),
                                                                     __builtin_bit_cast(h8v_t, Bh), zero, 0, 0, 0);
          const h8v_t a = __builtin_bit_cast(h8v_t, feat[(2 * i + 1) * 64 + lane]);
#pragma unroll
          for (int r = 0; r < R; ++r) sc[r] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, __builtin_bit_cast(h8v_t, Bx[r]), base, 0, 0, 0);
        } else {
          const h8v_t a = __builtin_bit_cast(h8v_t, feat[i * 64 + lane]);
#pragma unroll
          for (int r = 0; r < R; ++r) sc[r] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, __builtin_bit_cast(h8v_t, Bx[r]), zero, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float e[2];
#pragma unroll
          for (int k8 = 0; k8 < 2; ++k8) {
            const f16v_t& v = sc[r];
            float m = min_nn(min_nn(v[8 * k8], v[8 * k8 + 1]), v[8 * k8 + 2]);
            m = min_nn(min_nn(m, v[8 * k8 + 3]), v[8 * k8 + 4]);
            m = min_nn(min_nn(m, v[8 * k8 + 5]), v[8 * k8 + 6]);
            m = min_nn(m, v[8 * k8 + 7]);
            e[k8] = __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, m) & ~kBlockMask) | (uint32_t)(4 * i + k8));
          }
          // m1 <= m2: of the four the second smallest is the middle one of m1 and the new ones, unless m2 is below it
          m2[r] = min_nn(m2[r], __builtin_amdgcn_fmed3f(m1[r], e[0], e[1]));
          m1[r] = min_nn(min_nn(m1[r], e[0]), e[1]);
        }
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
        const float* cand = fcb + em_place<D>(8) * (int)blk + 4 * D * half;
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
      if (repeats) {
#pragma unroll
        for (int r = 0; r < R; ++r) args[r] = origin[args[r]];
      }
      uint32_t any = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) any |= unsures[r];
      if (any != 0) {
        int undecided = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) undecided += __builtin_popcount(unsures[r]);
        if (undecided > kMostUndecided * R) {
          filter = false;                     // the rows to come will be no better
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
        if (in_upper[r] == (half != 0)) ab[(size_t)(row_now + r) * (in_features / D)] = (uint8_t)arg;
      }
      continue;
    }
  whole_codebook:
    const bool eight = rows - row_now >= 8;   // else 4
    row = row_now + (eight ? 8 : 4);
    const int ahead = row < rows ? row : 0;
#pragma unroll
    for (int r = 0; r < R; ++r)   // before the stores, as on the way past this: a wait for them is one for these too
      load_coords<D>(Wb + (size_t)(ahead + r) * in_features, xn[r]);
    const size_t mine = (size_t)(row_now + (eight ? 4 : 2) * half);
    if (eight)
      em_assign_whole<K, D, 4>(cbs, Wb + mine * in_features, in_features, h, ab + mine * (in_features / D));
    else
      em_assign_whole<K, D, 2>(cbs, Wb + mine * in_features, in_features, h, ab + mine * (in_features / D));
  }
}

// Which codebooks take the filter; us at 4096 x 4096, loop over the centroids against filter (11008 x 4096 behind):
//                               d = 2, k = 64, 8 rows  d = 2, k = 256, 8 rows   d = 4, k = 256, 256 rows  d = 4, k = 64, 16 rows
//   distinct centroids                    88, 50             340, 107 (870, 286)      314, 67 (800, 178)       85, 38
//   vectors of the group, drawn with replacement (11, 1.5, 3 % of the centroids repeated, d = 2 with 8 rows most)
//                                         88, 52             342, 116 (875, 305)      314, 69 (796, 185)       85, 40
//   half of W and a quarter of the centroids zero
//                                         86, 49             332, 110                 308, 72 (786, 186)       82, 37
//   every centroid twice                  89, 57             340, 117 (-, 300)        310, 79 (794, 194)       85, 45
//   W far from zero: not tried            88, 89             338, 292                 309, 275                 85, 86
//   zero, negative or very uneven weights in every set of 32 vectors: no filter
//                                         88, 89             338, 289                 309, 279                 85, 86
//   rows 4 to 7 of every 8 far from zero: found out by the filter
//                                         86, 111              -, 333                   -, 352                   -, 106
// Not for d = 2, k = 32 and d = 1 (scalars lie too close for the filter).  Against a wave to 8 rows alone, the features of all
// centroids in its registers and equal centroids undecided: d = 4, k = 256, 256 rows 11008 x 4096 223 -> 178; d = 2, k = 256, 8 rows with
// centroids drawn from the vectors 267 -> 116, 512 x 512 81 -> 10; d = 4 in groups of 8 rows, whose waves have four, 74 -> 82 and 24 -> 26
// (2048 x 2048, far from zero, k = 256 and 64).
template <int K, int D> constexpr bool em_filtered() { return (D == 2 || D == 4) && K >= 64; }
template <int K, int D> constexpr int em_waves() { return em_filtered<K, D>() ? (D == 4 && K == 256 ? 3 : 4) : 1; }   // per SIMD

// Centroids to an iteration of the loop below; with a codebook per row four waves per SIMD, and twice the loop where those have
// the registers.  us with one, two, all, groups of one row: d = 1, k = 4 4096 x 4096 20.0, 22.8, 19.1, 512 x 512 5.4, 5.0, 4.4;
// d = 1, k = 8 26.2, 27.3, 46.8, 8.2, 7.5, 9.2; d = 2, k = 16 33.4, 33.9, -, 11.9, 9.3, -; groups of 32 rows d = 1, k = 8
// 2048 x 2048 -, 6.9, 6.0; d = 4, k = 4 -, 3.7, 3.6; groups of 4 rows, d = 2, k = 8 4096 x 4096 -, 17.8, 18.7.
template <int K, int D, int NCB> constexpr int em_unroll() {
  return NCB == 8 ? (K == 4 ? 4 : K == 8 && D == 1 ? 1 : 2) : NCB == 1 && K <= 8 ? K : 2;
}

// The loop over the centroids, for ROWS rows (8, or 2 where a launch has few blocks) of one 8-row block and col-block per
// wave; the codebook is that of the group the block lies in (NCB = 1), one codebook per row (NCB = 8: groups of one
// row) or one per 4 rows (NCB = 2).  D values per centroid, 4 / D vectors per row and lane: lane L owns columns
// 4L .. 4L+3, exactly as in the matrix-vector kernels.  Unfused binary32, sum over t in order.
template <int K, int D, int NCB, int ROWS>
__device__ __forceinline__ void em_assign_loop(const float* __restrict__ W, const float* __restrict__ hdiag,
                                               const float* __restrict__ cb, uint8_t* __restrict__ assign, int n_cb,
                                               int in_features, int group_rows, long long b, int part, float* cbs) {
#pragma clang fp contract(off)
  static_assert(ROWS == 8 || NCB == 1, "parts of a block share its codebook");
  constexpr int V = 4 / D;                 // vectors per row and lane
  constexpr int RPC = 8 / NCB;             // rows of the block that share a codebook
  const int lane = threadIdx.x & 63;
  const long long rb = b / n_cb;
  const int c = (int)(b - rb * n_cb);
  const long long row0 = rb * 8 + part * ROWS;

#pragma unroll
  for (int q = 0; q < NCB; ++q) {
    const long long g = ((rb * 8 + q * RPC) / group_rows) * n_cb + c;
    const float* cg = cb + g * (K * D);
    for (int i = lane; i < K * D; i += 64) cbs[q * K * D + i] = cg[i];
  }
  const float4 h4 = *reinterpret_cast<const float4*>(hdiag + (size_t)c * 256 + lane * 4);
  const float h[4] = {h4.x, h4.y, h4.z, h4.w};
  float x[ROWS][4];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const float4 t = *reinterpret_cast<const float4*>(W + (size_t)(row0 + r) * in_features + (size_t)c * 256 + lane * 4);
    x[r][0] = t.x; x[r][1] = t.y; x[r][2] = t.z; x[r][3] = t.w;
  }
  wave_lds_sync();

  float best[ROWS * V];
  uint32_t arg[ROWS * V];
#pragma unroll
  for (int v = 0; v < ROWS * V; ++v) {
    best[v] = __builtin_inff();
    arg[v] = 0;
  }
#pragma unroll (em_unroll<K, D, NCB>())
  for (int m = 0; m < K; ++m) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
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
  for (int r = 0; r < ROWS; ++r) {
    uint8_t* a = assign + (size_t)(row0 + r) * (in_features / D) + (size_t)c * (256 / D) + lane * V;
    if constexpr (V == 4)
      *reinterpret_cast<uint32_t*>(a) = arg[4 * r] | (arg[4 * r + 1] << 8) | (arg[4 * r + 2] << 16) | (arg[4 * r + 3] << 24);
    else if constexpr (V == 2)
      *reinterpret_cast<uint16_t*>(a) = (uint16_t)(arg[2 * r] | (arg[2 * r + 1] << 8));
    else
      *a = (uint8_t)arg[r];
  }
}

// The E-step's kernels, workgroups of four waves.  strip_rows: filtered codebooks: the rows of a workgroup; the
// others: 8 (a wave to a block) or 2 (a workgroup to a block).
template <int K, int D, int NCB>
__device__ __forceinline__ void em_assign(const float* __restrict__ W, const float* __restrict__ hdiag,
                                          const float* __restrict__ cb, uint8_t* __restrict__ assign, int n_cb,
                                          long long n_blocks, int in_features, int group_rows, int strip_rows) {
  if constexpr (NCB == 1 && em_filtered<K, D>()) {
    em_assign_filtered<K, D>(W, hdiag, cb, assign, n_cb, in_features, group_rows, strip_rows);
  } else {
    __shared__ __attribute__((aligned(16))) float cbs_all[4][NCB * K * D];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (NCB == 1) {
      if (strip_rows == 2) {
        em_assign_loop<K, D, 1, 2>(W, hdiag, cb, assign, n_cb, in_features, group_rows, blockIdx.x, wave, cbs_all[wave]);
        return;
      }
    }
    const long long b = (long long)blockIdx.x * 4 + wave;
    if (b >= n_blocks) return;   // whole waves leave; no workgroup barrier in the loop
    em_assign_loop<K, D, NCB, 8>(W, hdiag, cb, assign, n_cb, in_features, group_rows, b, 0, cbs_all[wave]);
  }
}

template <int K>
__global__ __launch_bounds__(256, (em_waves<K, 2>())) void em_assign_kernel(
    const float* __restrict__ W, const float* __restrict__ hdiag, const float* __restrict__ cb, uint8_t* __restrict__ assign,
    int n_cb, long long n_blocks, int in_features, int strip_rows) {
  em_assign<K, 2, 1>(W, hdiag, cb, assign, n_cb, n_blocks, in_features, 8, strip_rows);
}

// any dimensionality and group height
template <int K, int D, int NCB>
__global__ __launch_bounds__(256, (NCB == 1 ? em_waves<K, D>() : NCB == 8 ? 4 : 1)) void em_assign_any_kernel(
    const float* __restrict__ W, const float* __restrict__ hdiag, const float* __restrict__ cb, uint8_t* __restrict__ assign,
    int n_cb, long long n_blocks, int in_features, int group_rows, int strip_rows) {
  em_assign<K, D, NCB>(W, hdiag, cb, assign, n_cb, n_blocks, in_features, group_rows, strip_rows);
}

// M-step.  An item is a group (NG = 1) or an 8-row block that holds NG = 8 / n_rows groups (groups of 1 or 4 rows);
// a wave holds RB 8-row blocks of it in registers (of 256 rows half at a time), and the waves of an item share its
// tables in LDS: per centroid and coordinate the sum of h x, and that of h.
//   Order: which of the vectors of a centroid arrives first is for the LDS to say, so the sums are in fixed point, where
// order makes no difference.  A first pass over the registers finds the largest |x| of every entry (a maximum has no
// order either); in the second the products h x, exact in binary64, are rounded to 2^-kBits of the power of two above
// that |x| times the col-block's largest weight, and added as 64-bit integers, which cannot overflow.  The weights'
// sums are exact.  That holds while the weights of the col-block (256 columns) are finite and within 2^kSpread of each
// other, zeros aside; otherwise (kAny) both sums are scaled by an entry's own largest |h x| and |h|.  Either way a sum
// is off by at most n * 2^(kSpread - kBits) = n * 2^-36 of its largest term, by n * 2^-41 or less for weights within 2^5.
//   Skew: lanes that meet in one entry are served one after the other (64 of them: 130 clocks an atomic, 8 to 13 where
// they spread).  A wave therefore picks the centroid that most lanes share, if 12 do, and keeps its sums in registers,
// a binary64 sum per lane, added up over the lanes and then over the waves in a fixed order.
//   Bound: the reads of W and the LDS (clocks a wave and CU: maximum 8, addition 13, gather 7; binary64 additions,
// which depend on order, take 22 .. 31, binary32 ones 194).  us at 11008 x 4096, uniform assignments, one centroid for
// all, and in brackets both with binary64 additions: d = 2, k = 64, 32 rows 67, 32 (75, 456); d = 2, k = 256, 8 rows 77,
// 45 (72, 459), 128 rows 73, 39 (77, 501); d = 4, k = 256, 64 rows 69, 40 (81, 469).  Weights further apart than 2^kSpread:
// 35 .. 64 for 28 .. 36 at 4096 x 4096.
// SHARED: 0, or for the workgroups of a coordinate (see below) log2 of the weights of their groups at most.
template <int K, int D, int NG, int GPW, int RB, int SHARED>
struct EmTables {
  static constexpr int kEntries = NG * K;
  static constexpr int kCopies = kEntries >= 64 ? 1 : 64 / kEntries;
  static constexpr int kStride = kEntries * kCopies;        // entries per quantity
  static constexpr int kQuantities = SHARED ? 2 : 2 * D;
  static constexpr int kTable = kQuantities * kStride;      // entries per item
  static constexpr int kMaxWaves = GPW > 1 ? GPW : SHARED > 14 ? 16 : 8;
  // an item has at most 2^kLog2N vectors; 51 bits are what the conversion below takes
  static constexpr int kLog2N = (GPW > 1 ? 11 : SHARED ? SHARED : RB > 1 ? 16 : 14) - (D == 4 ? 2 : D == 2 ? 1 : 0);
  static constexpr int kBits = 62 - kLog2N < 51 ? 62 - kLog2N : 51;
  static constexpr int kSpread = kBits - 36;
};

__device__ __forceinline__ uint32_t high_magnitude(double v) {
  return (uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32) & 0x7fffffffu;
}
// v * 2^(scale - 1023) + 1.5 * 2^52, rounded once: its low bits are that product as an integer (below 2^51).
__device__ __forceinline__ unsigned long long to_fixed(double v, uint32_t scale_high) {
  const double scale = __builtin_bit_cast(double, (uint64_t)scale_high << 32);
  return __builtin_bit_cast(uint64_t, __builtin_fma(v, scale, 0x1.8p52)) - 0x4338000000000000ull;
}
__device__ __forceinline__ double from_fixed(unsigned long long sum, int scale) {
  return (double)(long long)sum * __builtin_bit_cast(double, (uint64_t)scale << 52);
}
// h * x + 1.5 * 2^52, rounded once, as above (h holds the scale).
__device__ __forceinline__ unsigned long long fixed_product(double h, double x) {
  return __builtin_bit_cast(uint64_t, __builtin_fma(h, x, 0x1.8p52)) - 0x4338000000000000ull;
}
// An entry that has met infinities or NaN holds what it has met: 1 +inf, 2 -inf, 4 NaN.
__device__ __forceinline__ void add_nonfinite(unsigned long long* sum, double v) {
  if (!(__builtin_fabs(v) < __builtin_inf())) atomicOr(sum, v != v ? 4ull : v > 0. ? 1ull : 2ull);
}
__device__ __forceinline__ double from_nonfinite(unsigned long long sum) {
  return sum == 1 ? __builtin_inf() : sum == 2 ? -__builtin_inf() : __builtin_nan("");
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// Sum over the 64 lanes, in lane 63 (as wave_min).
__device__ __forceinline__ double wave_sum63(double v) {
  v += dpp_or_zero<0x111, 0xf>(v);
  v += dpp_or_zero<0x112, 0xf>(v);
  v += dpp_or_zero<0x114, 0xf>(v);
  v += dpp_or_zero<0x118, 0xf>(v);
  v += dpp_or_zero<0x142, 0xa>(v);
  v += dpp_or_zero<0x143, 0xc>(v);
  return v;
}

//   SHARED: few groups.  D workgroups take a group, a coordinate each, with up to 16 waves: what takes the time then is the
// chain of a wave's vectors, one after the other (figures at em_shared; shares of the codebook instead of coordinates
// leave every wave its chain: 24.6 us for 12.4 at 512 x 512, 256 rows, and 41 for 28 at 2048 x 2048).
template <int K, int D, int NG, int GPW, int RB, int SHARED>
__global__ __launch_bounds__((64 * EmTables<K, D, NG, GPW, RB, SHARED>::kMaxWaves), (GPW > 1 ? 1 : 4)) void em_update_kernel(
    const float* __restrict__ W, const float* __restrict__ hdiag, const uint8_t* __restrict__ assign,
    float* __restrict__ cb_out, int n_cb, long long n_items, int in_features, int n_rows) {
  static_assert(!SHARED || (GPW == 1 && NG == 1), "a workgroup has one group");
  using Tab = EmTables<K, D, NG, GPW, RB, SHARED>;
  constexpr int DT = SHARED ? 1 : D;                // coordinates of this workgroup
  constexpr int V = 4 / D;                          // vectors per row and lane
  constexpr int N = V * DT;                         // values of a row and lane: DT of each vector
  constexpr int RPG = 8 / NG;                       // rows of an 8-row block that share a codebook
  constexpr uint32_t kNone = 0x100;
  __shared__ __attribute__((aligned(16))) unsigned long long sum_all[GPW * Tab::kTable];
  __shared__ uint32_t top_all[GPW * Tab::kTable];
  __shared__ double hot_sums[Tab::kMaxWaves][NG][2 * DT];
  __shared__ uint32_t hot_of[Tab::kMaxWaves][NG];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = GPW > 1 ? 1 : (int)blockDim.x / 64;   // of this item
  const int parts = RB > 1 ? n_rows / (8 * RB * waves) : 1;   // what a wave takes one after the other, 8 * RB rows each
  const int sub = GPW > 1 ? 0 : wave;               // this wave's place among them
  const int slot = GPW > 1 ? wave : 0;
  const int t_item = sub * 64 + lane, t_count = waves * 64;
  unsigned long long* sums = sum_all + slot * Tab::kTable;
  uint32_t* tops = top_all + slot * Tab::kTable;
  const long long item = SHARED ? (long long)(blockIdx.x / D) : (long long)blockIdx.x * GPW + slot;
  const int t0 = SHARED ? (int)(blockIdx.x % D) : 0;   // the first of its coordinates
  if (GPW > 1 && item >= n_items) return;           // whole waves leave; no workgroup barrier with GPW > 1
  const long long ir = item / n_cb;                 // group row, or 8-row block where that holds several groups
  const int c = (int)(item - ir * n_cb);
  const long long row0 = ir * (NG > 1 ? 8 : n_rows) + sub * 8 * RB;
  auto item_sync = [] {
    if constexpr (GPW > 1) wave_lds_sync();
    else __syncthreads();
  };

  float h[N];
  auto load_values = [&](const float* p, float (&v)[N]) {
    if constexpr (SHARED) {
#pragma unroll
      for (int i = 0; i < V; ++i) v[i] = p[i * D];
    } else {
      const float4 t = *reinterpret_cast<const float4*>(p);
      v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }
  };
  load_values(hdiag + (size_t)c * 256 + lane * 4 + t0, h);
  const float* Wl = W + (size_t)row0 * in_features + (size_t)c * 256 + lane * 4 + t0;
  const uint8_t* al = assign + (size_t)row0 * (in_features / D) + (size_t)c * (256 / D) + lane * V;
  auto load = [&](int r, float (&xr)[N], uint32_t& ar) {
    load_values(Wl + (size_t)r * in_features, xr);
    const uint8_t* ap = al + (size_t)r * (in_features / D);
    if constexpr (V == 4) ar = *reinterpret_cast<const uint32_t*>(ap);
    else if constexpr (V == 2) ar = *reinterpret_cast<const uint16_t*>(ap);
    else ar = *ap;
  };
  float x[8 * RB][N];
  uint32_t a[8 * RB];
  auto load_part = [&](int p) {
#pragma unroll
    for (int r = 0; r < 8 * RB; ++r) load(p * waves * 8 * RB + r, x[r], a[r]);
  };
  load_part(0);
  for (int i = t_item; i < Tab::kTable; i += t_count) {
    sums[i] = 0ull;
    tops[i] = 0u;
  }
  item_sync();

  const int copy = Tab::kCopies > 1 ? lane % Tab::kCopies : 0;
  // the centroid of each group that the most lanes of a row share, among a few that are asked
  uint32_t hot[NG];
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    hot[g] = kNone;
    int most = 11;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t m = (a[g * RPG + j % RPG] & 0xffu);
      const uint32_t asked = (uint32_t)__builtin_amdgcn_readlane((int)m, 8 * j + 3);
      const int n = __builtin_popcountll(__ballot(m == asked));
      if (n > most && (K == 256 || asked < (uint32_t)K)) { most = n; hot[g] = asked; }
    }
  }

  // are the weights of the col-block finite and near each other (every wave of the item sees the same ones)
  uint32_t h_exp;                                   // exponent field of the largest
  bool any_h;
  {
    float big = 0.f, small = __builtin_inff();
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const float v = __builtin_fabsf(h[t]);
      big = max_nn(big, v);
      small = __builtin_fminf(small, v == 0.f ? __builtin_inff() : v);
    }
    const bool finite = !__any(!(big < __builtin_inff()));
    big = -wave_min(finite ? -big : 0.f);
    small = wave_min(finite ? small : 0.f);
    h_exp = __builtin_bit_cast(uint32_t, big) >> 23;
    any_h = !finite || h_exp < 32 || __builtin_bit_cast(uint32_t, small) >> 23 < h_exp - Tab::kSpread;
  }
  constexpr int P = Tab::kBits;
  auto finish = [&](int g, const double (&own)[2 * DT]) {   // the wave's sums of the centroid kept in registers
    if (hot[g] != kNone) {
#pragma unroll
      for (int q = 0; q < 2 * DT; ++q) {
        const double sum = wave_sum63(own[q]);
        if (lane == 63) hot_sums[wave][g][q] = sum;
      }
    }
    if (lane == 63) hot_of[wave][g] = hot[g];
  };
  if (any_h) {
    // Entries scaled by their largest |h x| and |h|, as high words of binary64 (|term| < 2^(field - 1022)).  Rare: rows are read
    // again one by one.
    if constexpr (NG > 1) {
#pragma unroll
      for (int g = 0; g < NG; ++g) hot[g] = kNone;
    }
    double own[2 * DT] = {};
    auto pass = [&](auto second) {
#pragma unroll 1
      for (int r = 0; r < 8 * RB * parts; ++r) {
        float xr[N];
        uint32_t ar;
        load(RB > 1 ? r / (8 * RB) * waves * 8 * RB + r % (8 * RB) : r, xr, ar);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const uint32_t m = ((ar >> (8 * v)) & 0xffu);
          if (K < 256 && m >= (uint32_t)K) continue;
          const bool kept = NG == 1 && m == hot[0];
          const int e = ((NG > 1 ? r / RPG : 0) * K + m) * Tab::kCopies + copy;
#pragma unroll
          for (int q = 0; q < Tab::kQuantities; ++q) {
            const double hv = h[v * DT + q % DT], term = q < DT ? hv * (double)xr[v * DT + q % DT] : hv;
            const int i = e + q * Tab::kStride;
            if constexpr (!decltype(second)::value) {
              if (!kept) atomicMax(tops + i, high_magnitude(term));
            } else if (kept) {
              own[q] += term;
            } else {
              const uint32_t top = tops[i];
              if (top >= 0x7ff00000u) add_nonfinite(sums + i, term);
              else atomicAdd(sums + i, to_fixed(term, ((P + 2045u) << 20) - (top & 0x7ff00000u)));
            }
          }
        }
      }
    };
    pass(std::false_type{});
    item_sync();
    pass(std::true_type{});
#pragma unroll
    for (int g = 0; g < NG; ++g) finish(g, own);
  } else {
    // Entries scaled by their largest |x|, as binary32 (|x| < 2^(field - 126)), and all by the largest weight.
#pragma unroll 1
    for (int p = 0; p < parts; ++p) {
      if (p > 0) load_part(p);
#pragma unroll
      for (int r = 0; r < 8 * RB; ++r) {
        const int g = NG > 1 ? r / RPG : 0;
        const float (&xr)[N] = x[r];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const uint32_t m = ((a[r] >> (8 * v)) & 0xffu);
          if (m != hot[g] && (K == 256 || m < (uint32_t)K)) {
            uint32_t* e = tops + (g * K + m) * Tab::kCopies + copy;
#pragma unroll
            for (int t = 0; t < DT; ++t) atomicMax(e + t * Tab::kStride, __builtin_bit_cast(uint32_t, xr[v * DT + t]) & 0x7fffffffu);
          }
        }
      }
    }
    item_sync();
    unsigned long long h_fixed[N];                  // |h| < 2^(h_exp - 126)
#pragma unroll
    for (int t = 0; t < N; ++t) h_fixed[t] = to_fixed((double)h[t], (P + 1149u - h_exp) << 20);
    double own[2 * DT] = {};
#pragma unroll 1
    for (int p = parts - 1; p >= 0; --p) {          // the part at hand first
      if (p < parts - 1) load_part(p);
      // what this pass needs is computed again: kept from the first, it would not fit the registers
#pragma unroll
      for (int r = 0; r < 8 * RB; ++r)
      {
#pragma unroll
        for (int t = 0; t < N; ++t) asm volatile("" : "+v"(x[r][t]));
        asm volatile("" : "+v"(a[r]));
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        constexpr int ROWS = NG > 1 ? RPG : 8 * RB;
#pragma unroll
        for (int r = g * ROWS; r < (g + 1) * ROWS; ++r) {
          const float (&xr)[N] = x[r];
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const uint32_t m = ((a[r] >> (8 * v)) & 0xffu);
            if (m == hot[g]) {
#pragma unroll
              for (int t = 0; t < DT; ++t) {
                own[t] += (double)h[v * DT + t] * (double)xr[v * DT + t];
                own[DT + t] += (double)h[v * DT + t];
              }
            } else if (K == 256 || m < (uint32_t)K) {
              const int e = (g * K + m) * Tab::kCopies + copy;
#pragma unroll
              for (int t = 0; t < DT; ++t) {
                const int i = e + t * Tab::kStride;
                const uint32_t top = tops[i];
                const double hx = (double)h[v * DT + t] * (double)xr[v * DT + t];
                if (top >= 0x7f800000u) add_nonfinite(sums + i, hx);
                else atomicAdd(sums + i, to_fixed(hx, ((P + 1275u - h_exp) << 20) - ((top >> 3) & 0x0ff00000u)));
                atomicAdd(sums + i + DT * Tab::kStride, h_fixed[v * DT + t]);
              }
            }
          }
        }
        if constexpr (NG > 1) {                       // one part
          finish(g, own);
#pragma unroll
          for (int q = 0; q < 2 * DT; ++q) own[q] = 0.;
        }
      }
    }
    if constexpr (NG == 1) finish(0, own);
  }
  item_sync();
  for (int i = t_item; i < NG * K * DT; i += t_count) {
    const int e = i / DT, t = i % DT, g = e / K;
    double num = 0., den = 0.;
#pragma unroll
    for (int q = 0; q < Tab::kCopies; ++q) {
      const int p = t * Tab::kStride + e * Tab::kCopies + q, p_h = p + DT * Tab::kStride;
      const uint32_t top = tops[p];
      if (any_h) {
        if (top != 0) num += top >= 0x7ff00000u ? from_nonfinite(sums[p]) : from_fixed(sums[p], (int)(top >> 20) + 1 - P);
        const uint32_t top_h = tops[p_h];
        if (top_h != 0) den += top_h >= 0x7ff00000u ? from_nonfinite(sums[p_h]) : from_fixed(sums[p_h], (int)(top_h >> 20) + 1 - P);
      } else {
        num += top >= 0x7f800000u ? from_nonfinite(sums[p]) : from_fixed(sums[p], (int)(top >> 23) + (int)h_exp + 771 - P);
        den += from_fixed(sums[p_h], (int)h_exp + 897 - P);
      }
    }
    for (int w = 0; w < waves; ++w) {
      if (hot_of[wave - sub + w][g] == (uint32_t)(e % K)) {
        num += hot_sums[wave - sub + w][g][t];
        den += hot_sums[wave - sub + w][g][DT + t];
      }
    }
    const long long gi = NG > 1 ? (ir * NG + g) * n_cb + c : item;
    cb_out[(gi * K + e % K) * D + t0 + t] = den != 0. ? (float)num / (float)den : 0.f;
  }
}

// M-step of tall groups (128 or 256 rows) with d = 4, k = 256, a workgroup of eight waves to a group.  As em_update_kernel, but:
//   Counts: the weights' sums come from counts, 16 bits per centroid and vector position of a row for the whole group: one
// 32-bit atomic in place of eight, and den[t] = sum over the positions of count * h, exact products, at the end.
//   One scale for the whole group, from the largest |x| of the rows that are read first, every other one of the first 64
// (up to four times that may follow, see below), instead of a maximum and a look at it for every vector and
// entry (52 + 8 clocks of LDS a wave's vectors for 120), and each row is read once, four rows a wave ahead, in 80 registers
// without spills for three workgroups per CU.
//   A numerator formed so is the exact sum's, rounded to binary32: whatever the sum may be off by, half a unit per vector, changes
// nothing.  Where it might (the sum cancels, or its members are small beside the group's largest, or so many that they could
// overflow) the centroid is formed again from its members alone, at their own scale: the assignment is read again, and of W those, the next
// eight of a lane's at a time (one chain of memory round trips; row by row in chunks it took 13 us of a group).  A margin of the error
// that this has too makes both agree, so neither the scale nor the order of the rows shows, but for a centroid that many lanes
// share.  A vector beyond the scale, an infinity or a NaN has its centroid formed again; where more than 16 lanes of a wave meet
// such ones in four rows, the group is taken once more with the scale of all its rows.  Weights further apart: entry by entry.
//   us, two passes of em_update_kernel before, this kernel, at 11008 x 4096, 256 rows; 128 rows; 4096 x 4096, 256 rows; 128 rows:
// uniform assignments 81, 51; 81, 54; 34, 25; 36, 27; of the E-step 81, 50; 81, 51; 34, 24; 36, 26; a few values 30 times as
// large 81, 55; 80, 63; 37, 28; 36, 28; half of W zero, of the E-step 86, 62; 85, 71; 37, 36; 37, 32; odd rows 400 times the even
// ones (twice taken) 81, 75; 80, 84; 36, 34; 35, 41; all sums zero (all formed again) 81, 117; 80, 118; 37, 57; 35, 49.
//   A kernel of its own, since the code of
// em_update_kernel changed for every other instance where it had both (72 to 73 registers with d = 1, k = 64).
__global__ __launch_bounds__(512, 6) void em_update_counted_kernel(
    const float* __restrict__ W, const float* __restrict__ hdiag, const uint8_t* __restrict__ assign,
    float* __restrict__ cb_out, int n_cb, int in_features, int n_rows) {
  constexpr int K = 256, D = 4, WAVES = 8;
  constexpr int kWords = 32;                        // dwords of counts per centroid: positions i and i + 32
  constexpr int CW = kWords + 1;                    // a gap spreads the centroids over the banks
  constexpr int QR = 4;                             // rows that a wave reads ahead
  constexpr int P = EmTables<K, D, 1, 1, 2, 0>::kBits, kSpread = EmTables<K, D, 1, 1, 2, 0>::kSpread;
  constexpr int PQ = 51;                            // of the quick pass, for entries of up to kMost vectors
  constexpr uint32_t kMost = 4095, kRoom = 2;       // kRoom: binades that later rows may lie above the first ones
  constexpr uint32_t kNone = 0x100;
  __shared__ __attribute__((aligned(16))) unsigned long long sums[D * K];
  __shared__ uint32_t tops[D * K];
  __shared__ uint32_t counts[K * CW];
  __shared__ double h_all[256];
  __shared__ double hot_sums[WAVES][D];
  __shared__ uint32_t hot_of[WAVES], wave_top[WAVES], weak[K / 32], over;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int item = blockIdx.x;
  const int ir = item / n_cb;
  const int c = item - ir * n_cb;
  const long long row0 = (long long)ir * n_rows + wave * 8;   // of each 64 rows a wave has eight
  const float* Ww = W + (size_t)row0 * in_features + (size_t)c * 256;   // the wave's (all of an address but the lane's part is uniform)
  const uint8_t* aw = assign + (size_t)row0 * (in_features / D) + (size_t)c * 64;
  // What is made of the lane is not to be kept: an address of 64 bits per row, for one, would not fit the registers.
  auto not_kept = [](uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto thread = [&] { return (int)not_kept(lane) + wave * 64; };
  auto weights = [&](int row) {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const uint8_t*>(Ww + (size_t)row * in_features) + not_kept(lane * 16));
  };
  auto centroid = [&](int row) { return (uint32_t)*(aw + (size_t)row * (in_features / D) + not_kept(lane)); };
  const float4 h4 = reinterpret_cast<const float4*>(hdiag + (size_t)c * 256)[lane];
  float xq[2][QR][4];
  uint32_t mq[2][QR];
  auto load = [&](int p, float (&xr)[QR][4], uint32_t (&mr)[QR]) {   // every other one of the wave's rows in 64
#pragma unroll
    for (int r = 0; r < QR; ++r) {
      const int row = (p >> 1) * 64 + 2 * r + (p & 1);
      const float4 t = weights(row);
      xr[r][0] = t.x; xr[r][1] = t.y; xr[r][2] = t.z; xr[r][3] = t.w;
      mr[r] = centroid(row);
    }
  };
  auto clear = [&] {
    const int t = thread();
    if (t < K / 32) weak[t] = 0u;
    for (int i = t; i < D * K; i += 512) sums[i] = 0ull;
    for (int i = t; i < K * CW; i += 512) counts[i] = 0u;
    if (t == 0) over = 0u;
  };
  auto clear_tops = [&] {
    for (int i = thread(); i < D * K; i += 512) tops[i] = 0u;
  };
  load(0, xq[0], mq[0]);
  const float h[4] = {h4.x, h4.y, h4.z, h4.w};
  if (wave < 4) h_all[wave * 64 + lane] = hdiag[(size_t)c * 256 + wave * 64 + lane];
  clear();

  // the centroid that the most lanes of a row share, among a few that are asked
  uint32_t hot = kNone;
  int most = 11;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t m = mq[0][j % QR];
    const uint32_t asked = (uint32_t)__builtin_amdgcn_readlane((int)m, 8 * j + 3);
    const int n = __builtin_popcountll(__ballot(m == asked));
    if (n > most) { most = n; hot = asked; }
  }
  if (lane == 0) hot_of[wave] = hot;

  // are the weights of the col-block finite and near each other (every wave sees the same ones)
  uint32_t h_exp;                                   // exponent field of the largest
  bool any_h;
  {
    float big = 0.f, small = __builtin_inff();
#pragma unroll
    for (int t = 0; t < D; ++t) {
      const float v = __builtin_fabsf(h[t]);
      big = max_nn(big, v);
      small = __builtin_fminf(small, v == 0.f ? __builtin_inff() : v);
    }
    const bool finite = !__any(!(big < __builtin_inff()));
    big = -wave_min(finite ? -big : 0.f);
    small = wave_min(finite ? small : 0.f);
    h_exp = __builtin_bit_cast(uint32_t, big) >> 23;
    any_h = !finite || h_exp < 32 || __builtin_bit_cast(uint32_t, small) >> 23 < h_exp - kSpread;
  }
  auto largest = [&](const float (&xr)[QR][4]) {    // NaN if there is one
    float top = 0.f;
#pragma unroll
    for (int r = 0; r < QR; ++r)
#pragma unroll
      for (int t = 0; t < D; ++t) top = max_nn(top, __builtin_fabsf(xr[r][t]));
    return top;
  };
  // The exponent field of the largest of the workgroup's lanes', of those that are below 2^127.
  auto exponent_of_all = [&](float top) {
    top = -wave_min(top < 0x1p127f ? -top : 0.f);
    if (lane == 0) wave_top[wave] = __builtin_bit_cast(uint32_t, top);
    __syncthreads();
    uint32_t all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) all = max(all, wave_top[w]);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(all >> 23));
  };
  auto count = [&](uint32_t m) { atomicAdd(counts + m * CW + (lane & 31), 1u << (16 * (lane >> 5))); };
  auto finish = [&](const double (&own)[D], double scale) {   // the wave's sums of the centroid kept in registers
    if (hot != kNone) {
#pragma unroll
      for (int t = 0; t < D; ++t) {
        const double sum = wave_sum63(own[t]);
        if (lane == 63) hot_sums[wave][t] = sum * scale;
      }
    }
  };

  __syncthreads();
  uint32_t x_exp = exponent_of_all(largest(xq[0])) + kRoom;   // |x| < 2^(x_exp - 126)
  bool again = false;
  while (!any_h) {                                  // once, or twice
    float limit = __builtin_bit_cast(float, min(x_exp + 1u, 254u) << 23), seen = 0.f;
    double hs[D], own[D] = {};
    const double scale = __builtin_bit_cast(double, (uint64_t)(PQ + 1275u - h_exp - x_exp) << 52);
#pragma unroll
    for (int t = 0; t < D; ++t) hs[t] = h_all[4 * lane + t] * scale;
    auto add = [&](float (&xr)[QR][4], const uint32_t (&mr)[QR]) {
      const float top = largest(xr);
      seen = max_nn(seen, top);
      if (__any(!(top < limit))) {                  // rare: such a vector's centroid is formed again
        if (!again && __builtin_popcountll(__ballot(!(top < limit))) > 16) over = 1u;   // ... all of them, if they are many
#pragma unroll
        for (int r = 0; r < QR; ++r) {
          const float v = max_nn(max_nn(__builtin_fabsf(xr[r][0]), __builtin_fabsf(xr[r][1])),
                                 max_nn(__builtin_fabsf(xr[r][2]), __builtin_fabsf(xr[r][3])));
          if (!(v < limit) && mr[r] != hot) {
            atomicOr(weak + (mr[r] >> 5), 1u << (mr[r] & 31));
#pragma unroll
            for (int t = 0; t < D; ++t) xr[r][t] = 0.f;
          }
        }
      }
#pragma unroll
      for (int r = 0; r < QR; ++r) {
        const uint32_t m = mr[r];
        count(m);
        if (m == hot) {
#pragma unroll
          for (int t = 0; t < D; ++t) own[t] += hs[t] * (double)xr[r][t];
        } else {
#pragma unroll
          for (int t = 0; t < D; ++t) atomicAdd(sums + t * K + m, fixed_product(hs[t], (double)xr[r][t]));
        }
      }
    };
    const int n_parts = n_rows / 32;                // an even number
    int p = 0;
#pragma unroll 1
    for (; p < n_parts; p += 2) {
      load(p + 1, xq[1], mq[1]);
      add(xq[0], mq[0]);
      if (p + 2 < n_parts) load(p + 2, xq[0], mq[0]);
      add(xq[1], mq[1]);
      if (__hip_atomic_load(&over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0u) break;   // in any wave
    }
    finish(own, __builtin_bit_cast(double, (uint64_t)(771u - PQ + h_exp + x_exp) << 52));
    __syncthreads();
    if (over == 0u) break;
    again = true;                                   // once more, with the largest of all rows
#pragma unroll 1
    for (p += 2; p < n_parts; p += 2) {
      load(p, xq[0], mq[0]);
      load(p + 1, xq[1], mq[1]);
      seen = max_nn(seen, max_nn(largest(xq[0]), largest(xq[1])));
    }
    x_exp = exponent_of_all(seen);
    clear();
    load(0, xq[0], mq[0]);
    __syncthreads();
  }
  if (any_h) {
    // Entries scaled by their largest |h x|, as high words of binary64 (|term| < 2^(field - 1022)).  Rare: rows are read
    // again one by one.
    clear();
    clear_tops();
    __syncthreads();
    double own[D] = {};
    auto pass = [&](auto second) {
#pragma unroll 1
      for (int r = 0; r < n_rows / WAVES; ++r) {
        const int row = (r >> 3) * 64 + (r & 7);
        const float4 x4 = weights(row);
        const float xr[4] = {x4.x, x4.y, x4.z, x4.w};
        const uint32_t m = centroid(row);
        if constexpr (!decltype(second)::value) count(m);
#pragma unroll
        for (int t = 0; t < D; ++t) {
          const double term = h_all[4 * lane + t] * (double)xr[t];
          const int e = t * K + m;
          if constexpr (!decltype(second)::value) {
            if (m != hot) atomicMax(tops + e, high_magnitude(term));
          } else if (m == hot) {
            own[t] += term;
          } else {
            const uint32_t top = tops[e];
            if (top >= 0x7ff00000u) add_nonfinite(sums + e, term);
            else atomicAdd(sums + e, to_fixed(term, ((P + 2045u) << 20) - (top & 0x7ff00000u)));
          }
        }
      }
    };
    pass(std::false_type{});
    __syncthreads();
    pass(std::true_type{});
    finish(own, 1.);
    __syncthreads();
  }

  // Two lanes per centroid: the weights' sums of half the positions each, then two coordinates each.
  const int i_thread = thread(), m = i_thread >> 1, half = i_thread & 1;
  double den[2];
  uint32_t members = 0;
  {
    const uint32_t* n = counts + m * CW + half * (kWords / 2);
    const double* hp = h_all + half * 4 * (kWords / 2);
    double part[D] = {};
#pragma unroll 4
    for (int w = 0; w < kWords / 2; ++w) {
      const double lo = n[w] & 0xffffu, hi = n[w] >> 16;
      members += (n[w] & 0xffffu) + (n[w] >> 16);
#pragma unroll
      for (int t = 0; t < D; ++t) part[t] += lo * hp[4 * w + t] + hi * hp[4 * w + 128 + t];
    }
#pragma unroll
    for (int t = 0; t < D; ++t) {
      if (part[t] != part[t]) {                     // 0 * infinity or NaN: such a weight counts only where it is used
        part[t] = 0.;
        for (int w = 0; w < kWords / 2; ++w) {
          if (n[w] & 0xffffu) part[t] += (double)(n[w] & 0xffffu) * hp[4 * w + t];
          if (n[w] >> 16) part[t] += (double)(n[w] >> 16) * hp[4 * w + 128 + t];
        }
      }
      part[t] += __shfl_xor(part[t], 1, 64);
    }
    members += __shfl_xor(members, 1, 64);
    den[0] = half ? part[2] : part[0];
    den[1] = half ? part[3] : part[1];
  }
  // num: of its two coordinates, the sums in the tables, each within `off` of what it stands for.  Returns whether the
  // numerators are the same for all that they may stand for.
  auto write = [&](const double (&num)[2], double off) {
    double total[2] = {num[0], num[1]};
    int kept = 0;                                   // waves that have their part of it in registers
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      if (hot_of[w] == (uint32_t)m) {
        ++kept;
        total[0] += hot_sums[w][2 * half];
        total[1] += hot_sums[w][2 * half + 1];
      }
    }
    float2 out;
    out.x = den[0] != 0. ? (float)total[0] / (float)den[0] : 0.f;
    out.y = den[1] != 0. ? (float)total[1] / (float)den[1] : 0.f;
    *reinterpret_cast<float2*>(cb_out + ((long long)item * K + m) * D + 2 * half) = out;
    bool certain = true;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const double d = off + __builtin_fabs(num[j]) * 0x1p-50;   // (the conversions to binary64 and the additions above)
      certain = certain && (float)(total[j] - d) == (float)(total[j] + d);
    }
    return kept == WAVES || (certain && members <= kMost);
  };
  const int e0 = 2 * half * K + m;                  // of its first coordinate; the second follows K entries later
  const double unit = __builtin_bit_cast(double, (uint64_t)((int)x_exp + (int)h_exp + 771 - PQ) << 52);
  double num[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int e = e0 + j * K;
    if (!any_h) {
      num[j] = (double)(long long)sums[e] * unit;
    } else {
      const uint32_t top = tops[e];
      num[j] = top == 0 ? 0. : top >= 0x7ff00000u ? from_nonfinite(sums[e]) : from_fixed(sums[e], (int)(top >> 20) + 1 - P);
    }
  }
  const bool certain = write(num, unit * (double)members);   // half a unit per vector, twice
  if (any_h) return;
  if (!certain) atomicOr(weak + (m >> 5), 1u << (m & 31));
  __syncthreads();
  uint32_t some = 0;
#pragma unroll
  for (int w = 0; w < K / 32; ++w) some |= weak[w];
  if (some == 0) return;

  // Those that are not are formed again, at the scale of their own members.
  const uint32_t bits = members <= kMost ? PQ : P;
  auto is_weak = [&](uint32_t v) { return (weak[v >> 5] >> (v & 31) & 1u) != 0; };
  if (is_weak(m)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      sums[e0 + j * K] = 0ull;
      tops[e0 + j * K] = 0u;
    }
    counts[m * CW + kWords] = bits;
  }
  uint32_t rows = 0;                                // the wave's rows with a vector of theirs in this lane
  {
    uint32_t v[32];
#pragma unroll
    for (int r = 0; r < 32; ++r)
      if (r < n_rows / WAVES) v[r] = centroid((r >> 3) * 64 + (r & 7));
#pragma unroll
    for (int r = 0; r < 32; ++r)
      if (r < n_rows / WAVES && v[r] != hot && is_weak(v[r])) rows |= 1u << r;
  }
  // The next eight of a lane's, all at a time.
  float4 x[8];
  uint32_t v[8];
  auto fetch = [&](uint32_t left) {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      v[b] = kNone;
      if (left != 0) {
        const int r = __builtin_ctz(left), row = (r >> 3) * 64 + (r & 7);
        x[b] = *reinterpret_cast<const float4*>(Ww + (size_t)row * in_features + 4 * lane);
        v[b] = aw[(size_t)row * (in_features / D) + lane];
        left &= left - 1;
      }
    }
    return left;
  };
  auto all_of = [&](auto f) {
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      if (v[b] != kNone) {
        f(v[b], 0, x[b].x);
        f(v[b], 1, x[b].y);
        f(v[b], 2, x[b].z);
        f(v[b], 3, x[b].w);
      }
    }
  };
  __syncthreads();
  uint32_t todo = rows, left;
  while (true) {
    left = fetch(todo);
    all_of([&](uint32_t v, int t, float xv) { atomicMax(tops + t * K + v, __builtin_bit_cast(uint32_t, xv) & 0x7fffffffu); });
    if (!__any(left != 0)) break;
    todo = left;
  }
  todo = rows & ~todo;                              // (the last ones are at hand)
  __syncthreads();
  while (true) {
    all_of([&](uint32_t v, int t, float xv) {
      const uint32_t top = tops[t * K + v];
      const double hx = h_all[4 * lane + t] * (double)xv;
      if (top >= 0x7f800000u) add_nonfinite(sums + t * K + v, hx);
      else atomicAdd(sums + t * K + v, to_fixed(hx, ((counts[v * CW + kWords] + 1275u - h_exp) << 20) - ((top >> 3) & 0x0ff00000u)));
    });
    if (!__any(todo != 0)) break;
    todo = fetch(todo);
  }
  __syncthreads();
  if (is_weak(m)) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t top = tops[e0 + j * K];
      num[j] = top >= 0x7f800000u ? from_nonfinite(sums[e0 + j * K]) : from_fixed(sums[e0 + j * K], (int)(top >> 23) + (int)h_exp + 771 - (int)bits);
    }
    write(num, 0.);
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

// Rows of a strip.  Filtered: a workgroup to 8 rows in small launches and low groups, else to 16 or 32, which make the
// centroids' features fewer times and, with d = 4, read a centroid for four vectors in place of two where they are undecided.
// us with strips of 8, 16, 32, groups of 32 or 64 rows, and with weights of zero in every set of 32 vectors behind:
//                       512 blocks                        1,024                             1,536
//   d = 2, k = 64       7.2, 9.3, 14.8; 9.3, 13.7, 23.4   10.1, 10.7, 15.1; 15.4, 14.1, 23  12.9, 13.0, 17.5; 20.8, 20.6, 23.7
//   d = 2, k = 256      12.5, 15.8, 26.5; 23, 36, 69      18.4, 18.6, 26.9; 40, 38, 69      24.4, 24.2, 32.1; 57, 66, 72
//   d = 4, k = 64       6.0, 7.0, 10.4; 9.1, 12.6, 21     8.3, 8.4, 10.5; 14.9, 12.8, 21    10.6, 9.7, 12.3; 20.1, 20.9, 21.3
//   d = 4, k = 256      8.9, 10.3, 16.0; 23, 36, 67       14.2, 12.8, 15.8; 47, 37, 67      17.9, 16.1, 19.6; 62, 66, 67
//                       2,048                             3,072                             4,096
//   d = 2, k = 64       15.6, 15.5, 17.6; 25.8, 24.6, 24  21.5, 21.0, 22.5; 37, 35, 38      27.6, 26.2, 27.5; 48, 46, 46
//   d = 2, k = 256      30.8, 29.9, 32.3; 75, 73, 73      43.3, 42.1, 43.7; 113, 108, 124   57.3, 54.6, 56.3; 149, 143, 143
//   d = 4, k = 64       12.9, 11.5, 12.5; 25.7, 23.3, 22  18.0, 16.0, 15.8; 37, 34, 37      23.3, 20.5, 19.5; 49, 44, 42
//   d = 4, k = 256      21.5, 20.2, 20.2; 82, 73, 69      31.1, 28.5, 27.7; 122, 109, 124   40.7, 36.8, 36.2; 162, 144, 141
// and 8,192 blocks 51.9, 48.1, 48.3; 108, 103, 103; 43.4, 37.9, 35.8; 76.9, 70.5, 66.8.
//   Loops: a wave to 8 rows, or to 2 where the blocks would leave SIMDs idle and a codebook is long enough to be fetched
// by four waves.  us with 8, 2:    128 blocks   512         1,024       1,536       1,792       2,048
//   d = 1, k = 4                   3.6, 2.5     3.7, 2.8    3.9, 3.8    4.5, 4.7    4.6, 5.2    4.7, 5.7     1,280 4.4, 4.3
//   d = 1, k = 8                   5.0, 2.9     5.1, 3.4    5.3, 4.7    6.0, 6.0    6.1, 6.5    6.3, 7.1
//   d = 1, k = 16                  9.6, 3.8     10.0, 4.3   10.1, 6.7   10.7, 8.8   10.7, 9.8   10.9, 10.8
//   d = 1, k = 64                  26.5, 9.0    27.2, 10.4  27.4, 17.7  33.5, 23.6  33.5, 26.6  33.7, 29.3   k = 32, 256 alike
//   d = 2, k = 4                   3.3, 2.5     3.4, 2.8    3.6, 3.6    3.9, 4.2    4.0, 4.5    4.1, 4.9     d = 4 alike
//   d = 2, k = 8                   4.4, 2.7     4.6, 3.0    4.8, 4.0    5.2, 4.9    5.2, 5.6    5.3, 6.1     d = 4 alike
//   d = 2, k = 16                  6.9, 3.5     7.2, 3.9    7.3, 5.4    7.8, 7.0    7.8, 8.0    7.9, 8.4
//   d = 2, k = 32                  11.6, 5.0    11.9, 5.5   12.1, 8.7   12.6, 11.9  12.7, 14.7  12.8, 15.0
//   d = 4, k = 16                  6.4, 3.4     6.5, 3.7    6.7, 5.4    7.0, 6.9    7.1, 8.3    7.2, 8.7     k = 32 alike
template <int K, int D, int NCB> static int em_strip_rows(const vq_desc& d, long long n_blocks) {
  const long long cus = device_cus();
  if (NCB == 1 && em_filtered<K, D>()) {
    const int rows = n_blocks < (D == 4 ? 4 : 8) * cus ? kGroupRows : n_blocks < (D == 4 ? 12 : 16) * cus ? 16 : 32;
    return d.group_rows <= kGroupRows ? kGroupRows : d.group_rows < rows ? d.group_rows : rows;
  }
  return NCB == 1 && n_blocks <= (D == 1 && K >= 16 ? 8 : K == 4 ? 5 : 6) * cus ? 2 : 8;
}
template <int K, int D, int NCB> static unsigned em_grid(long long n_blocks, int strip_rows) {
  if (NCB == 1 && em_filtered<K, D>()) return (unsigned)(n_blocks / (strip_rows / kGroupRows));
  return (unsigned)(strip_rows == 2 ? n_blocks : (n_blocks + 3) / 4);
}
constexpr long long kMostEmBlocks = 1ll << 23;   // of a launch: fewer than 2^32 threads

hipError_t launch_em_assign(const vq_desc& d, const void* W, const void* hdiag, const void* cb, void* assign,
                            hipStream_t s) {
  const int k = d.k, out_features = d.out_features, in_features = d.in_features;
  const int n_cb = in_features / kGroupCols;
  const long long n_blocks = (long long)(out_features / kGroupRows) * n_cb;
  if (n_blocks > kMostEmBlocks) {       // in parts of whole groups
    const int unit = d.group_rows > kGroupRows ? d.group_rows : kGroupRows;
    const long long fit = kMostEmBlocks / n_cb * kGroupRows / unit * unit;
    const int rows = fit < unit ? unit : (int)fit;   // a single row of groups: filtered ones take strips of up to 32 rows
    for (int at = 0; rows < out_features && at < out_features; at += rows) {
      vq_desc p = d;
      p.out_features = rows < out_features - at ? rows : out_features - at;
      const hipError_t e =
          launch_em_assign(p, (const float*)W + (size_t)at * in_features, hdiag,
                           (const float*)cb + (size_t)(at / d.group_rows) * n_cb * k * d.d,
                           (uint8_t*)assign + (size_t)at * (in_features / d.d), s);
      if (e != hipSuccess) return e;
    }
    if (rows < out_features) return hipSuccess;
  }
  if (d.d == 2 && d.group_rows == kGroupRows && (k == 16 || k == 64 || k == 256)) {
#define VQ_EM(K)                                                                                                   \
  do {                                                                                                             \
    const int strip_rows = em_strip_rows<K, 2, 1>(d, n_blocks);                                                    \
    hipLaunchKernelGGL(em_assign_kernel<K>, dim3((em_grid<K, 2, 1>(n_blocks, strip_rows))), dim3(256), 0, s,       \
                       (const float*)W, (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks,   \
                       in_features, strip_rows);                                                                   \
  } while (0)
    if (k == 16) VQ_EM(16);
    else if (k == 64) VQ_EM(64);
    else VQ_EM(256);
#undef VQ_EM
    return hipGetLastError();
  }
#define VQ_EM_ANY(K, D, NCB)                                                                                        \
  do {                                                                                                             \
    const int strip_rows = em_strip_rows<K, D, NCB>(d, n_blocks);                                                  \
    hipLaunchKernelGGL((em_assign_any_kernel<K, D, NCB>), dim3((em_grid<K, D, NCB>(n_blocks, strip_rows))), dim3(256), 0, s, \
                       (const float*)W, (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks,   \
                       in_features, d.group_rows, strip_rows);                                                     \
  } while (0)
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

// Whether D workgroups share a group of 16 rows or more in the M-step: up to two workgroups per CU, and up to one where
// they have eight waves and more and both coordinates are needed for a line of W.  us with one, D, by groups:
//                             8           64          96          128         192         256
//   d = 4, k = 256, 256 rows  14.7, 12.5  20.2, 18.6  20.4, 24.4  21.0, 28.7  24.9, 38.9  28.6, 49.9   of the E-step one: 14.7, 14.7, 14.8, 21.2
//                   128 rows  10.8, 8.2   15.7, 10.2  11.0, 14.5  15.3, 16.5  15.8, 22.0  16.4, 26.9   .. 10.8, 10.9, 15.3, 15.4
//                   64 rows   9.8, 5.7    10.0, 6.1   10.1, 7.8   10.1, 10.2              k = 16 and 64 alike
//                   16 rows   9.9, 4.6    10.0, 4.8   10.0, 5.5   10.0, 5.6
//   d = 2, k = 256, 256 rows  26.9, 21.1  27.2, 21.8  27.3, 22.4  28.1, 26.7  31.9, 44.8  35.2, 48.7
//                   128 rows  15.4, 12.5  15.6, 12.8  15.7, 13.0  16.1, 14.0  18.1, 22.2  19.4, 22.9   k = 64 alike
//                   64 rows   9.3, 7.9    9.4, 8.2    9.5, 8.4    9.7, 8.3    9.8, 11.1   11.2, 11.9
//                   32 rows   8.4, 6.2    8.5, 6.3    8.5, 6.4    8.6, 6.4    8.7, 7.9    8.7, 8.0     k = 64 8.4, 8.4 from 192 on
//                   16 rows   8.4, 5.7    8.6, 5.9    8.6, 5.9    8.6, 5.9    8.7, 6.8    8.7, 6.9
// (em_update_counted_kernel, the one of the first two rows, has cut its side since the line was drawn at two: there it would now
// lie at one, between 64 and 72 groups: 20.2, 18.6 and 19.9, 23.7.)
static bool em_shared(const vq_desc& d, long long n_items) {
  return n_items * d.d <= (d.d == 2 && d.group_rows >= 64 ? 1 : 2) * (long long)device_cus();
}

template <int K, int D, int NG, int GPW, int RB>
static void launch_update(const vq_desc& d, const void* W, const void* hdiag, const void* assign, void* cb_out,
                          hipStream_t s) {
  const int n_cb = d.in_features / kGroupCols;
  const long long n_items = (long long)(d.out_features / (NG > 1 ? kGroupRows : d.group_rows)) * n_cb;
  if constexpr (NG * K * D <= 32) {
    if (d.group_rows <= 32) {
      hipLaunchKernelGGL((em_update_small_kernel<K, D, NG>), dim3((unsigned)n_items), dim3(64), 0, s, (const float*)W,
                         (const float*)hdiag, (const uint8_t*)assign, (float*)cb_out, n_cb, d.in_features, d.group_rows);
      return;
    }
  }
  const int waves = GPW > 1 ? GPW : RB > 1 ? 8 : d.group_rows / kGroupRows;
  if constexpr (GPW == 1 && NG == 1 && D > 1) {
    if (em_shared(d, n_items)) {
#define VQ_SHARED(RBS, WAVES, LOG2)                                                                                              \
  hipLaunchKernelGGL((em_update_kernel<K, D, 1, 1, RBS, LOG2>), dim3((unsigned)(n_items * D)), dim3(64 * (WAVES)), 0, s,   \
                     (const float*)W, (const float*)hdiag, (const uint8_t*)assign, (float*)cb_out, n_cb, n_items,          \
                     d.in_features, d.group_rows)
      if constexpr (RB > 1) {
        if (d.group_rows == 256) VQ_SHARED(2, 16, 16);
        else VQ_SHARED(1, 16, 15);
      } else {
        VQ_SHARED(1, d.group_rows / kGroupRows, 14);
      }
#undef VQ_SHARED
      return;
    }
  }
  if constexpr (K == 256 && D == 4 && RB > 1) {
    hipLaunchKernelGGL(em_update_counted_kernel, dim3((unsigned)n_items), dim3(512), 0, s, (const float*)W, (const float*)hdiag,
                       (const uint8_t*)assign, (float*)cb_out, n_cb, d.in_features, d.group_rows);
  } else {
    hipLaunchKernelGGL((em_update_kernel<K, D, NG, GPW, RB, 0>), dim3((unsigned)((n_items + GPW - 1) / GPW)), dim3(64 * waves), 0, s,
                       (const float*)W, (const float*)hdiag, (const uint8_t*)assign, (float*)cb_out, n_cb, n_items,
                       d.in_features, d.group_rows);
  }
}

// Up to 8 rows a group to a wave and four waves to a workgroup; beyond that a workgroup to a group, a wave to 8 rows up to
// 64 rows, then eight waves.
template <int K, int D>
static hipError_t launch_update_rows(const vq_desc& d, const void* W, const void* hdiag, const void* assign, void* cb_out,
                               hipStream_t s) {
  if (d.group_rows == 1) {
    if constexpr (K * D <= 64) launch_update<K, D, 8, 4, 1>(d, W, hdiag, assign, cb_out, s);
    else return hipErrorInvalidValue;
  } else if (d.group_rows == 4) {
    if constexpr (D <= 2) launch_update<K, D, 2, 4, 1>(d, W, hdiag, assign, cb_out, s);
    else return hipErrorInvalidValue;
  } else if (d.group_rows == 8) {
    launch_update<K, D, 1, 4, 1>(d, W, hdiag, assign, cb_out, s);
  } else if (d.group_rows <= 64) {
    launch_update<K, D, 1, 1, 1>(d, W, hdiag, assign, cb_out, s);
  } else {
    launch_update<K, D, 1, 1, 2>(d, W, hdiag, assign, cb_out, s);
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
