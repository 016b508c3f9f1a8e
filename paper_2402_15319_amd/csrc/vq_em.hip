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
// shape the decode formats use), the same lane ownership.  em_update_small_kernel /
// em_update_kernel: the M-step with a table per lane or per wave.
//
// The E-step is a decision taken in floating point, so its arithmetic is fixed: binary32,
// every operation rounded on its own (no fused multiply-add), in the order subtract, square,
// times weight, add; the smallest distance wins, the lowest m wins a tie.  The M-step's sums are
// deterministic (see there).
#include "vq_device.h"
#include "vq_internal.h"

namespace vq {
namespace {

template <int K>
__global__ __launch_bounds__(256) void em_assign_kernel(const float* __restrict__ W,
                                                        const float* __restrict__ hdiag,
                                                        const float* __restrict__ cb,
                                                        uint8_t* __restrict__ assign, int n_cb,
                                                        long long n_groups, int in_features) {
#pragma clang fp contract(off)
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

// ---- any dimensionality and group height ---------------------------------------------------
// E-step.  One wave per (8-row block, col-block); the codebook is that of the group the block
// lies in (NCB = 1), one codebook per row (NCB = 8: groups of one row) or one per 4 rows (NCB = 2).
// D values per centroid, 4 / D vectors per row and lane.  Same arithmetic as em_assign_kernel:
// unfused binary32, sum over t in order.
template <int K, int D, int NCB>
__global__ __launch_bounds__(256) void em_assign_any_kernel(const float* __restrict__ W,
                                                            const float* __restrict__ hdiag,
                                                            const float* __restrict__ cb,
                                                            uint8_t* __restrict__ assign, int n_cb,
                                                            long long n_blocks, int in_features,
                                                            int group_rows) {
#pragma clang fp contract(off)
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
  static constexpr int kTable = 2 * D * kStride;            // doubles per wave
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
  wave_lds_sync();

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
            __builtin_amdgcn_ds_atomic_fadd_f64((lds_f64_ptr)(e + (D + t) * Bins::kStride), h[v * D + t]);
          }
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
        den += p[(D + t) * Bins::kStride];
      }
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

// Calls F(K) for the codebook size k (4, 8, 16, 64 or 256).
#define VQ_EM_K_SWITCH(k, F) \
  switch (k) {               \
    case 4: F(4); break;     \
    case 8: F(8); break;     \
    case 16: F(16); break;   \
    case 32: F(32); break;   \
    case 64: F(64); break;   \
    default: F(256); break;  \
  }

hipError_t launch_em_assign(const vq_desc& d, const void* W, const void* hdiag, const void* cb, void* assign,
                            hipStream_t s) {
  const int k = d.k, out_features = d.out_features, in_features = d.in_features;
  const int n_cb = in_features / kGroupCols;
  const long long n_blocks = (long long)(out_features / kGroupRows) * n_cb;
  const unsigned grid = (unsigned)((n_blocks + 3) / 4);
  if (d.d == 2 && d.group_rows == kGroupRows && (k == 16 || k == 64 || k == 256)) {
#define VQ_EM(K)                                                                                   \
  hipLaunchKernelGGL(em_assign_kernel<K>, dim3(grid), dim3(256), 0, s, (const float*)W,            \
                     (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks, in_features)
    if (k == 16) VQ_EM(16);
    else if (k == 64) VQ_EM(64);
    else VQ_EM(256);
#undef VQ_EM
    return hipGetLastError();
  }
#define VQ_EM_ANY(K, D, NCB)                                                                             \
  hipLaunchKernelGGL((em_assign_any_kernel<K, D, NCB>), dim3(grid), dim3(256), 0, s, (const float*)W,     \
                     (const float*)hdiag, (const float*)cb, (uint8_t*)assign, n_cb, n_blocks, in_features, \
                     d.group_rows)
  if (d.group_rows == 1) {   // a codebook per row: k * d <= 64 (checked by the caller)
    if (d.d == 1) {
#define VQ_F(K) if constexpr (K <= 64) VQ_EM_ANY(K, 1, 8)
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    } else if (d.d == 2) {
#define VQ_F(K) if constexpr (K <= 16) VQ_EM_ANY(K, 2, 8)
      VQ_EM_K_SWITCH(k, VQ_F)
#undef VQ_F
    } else {
#define VQ_F(K) if constexpr (K <= 16) VQ_EM_ANY(K, 4, 8)
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
// is 16 * k * d bytes, at most 16 KB (the 8 waves of a group with d = 4, k = 256 fill 128 KB of the CU's 160 KB).
template <int K, int D>
static void launch_update_rows(const vq_desc& d, const void* W, const void* hdiag, const void* assign, void* cb_out,
                               hipStream_t s) {
  if (d.group_rows == 1) {
    if constexpr (K * D <= 64) launch_update<K, D, 8, 1>(d, W, hdiag, assign, cb_out, s);
  } else if (d.group_rows == 4) {
    if constexpr (D <= 2) launch_update<K, D, 2, 1>(d, W, hdiag, assign, cb_out, s);
  } else if (d.group_rows < 32 || (d.group_rows == 32 && K * D <= 32)) {
    launch_update<K, D, 1, 1>(d, W, hdiag, assign, cb_out, s);
  } else if (d.group_rows < 128) {
    launch_update<K, D, 1, 4>(d, W, hdiag, assign, cb_out, s);
  } else {
    launch_update<K, D, 1, 8>(d, W, hdiag, assign, cb_out, s);
  }
}

hipError_t launch_em_update(const vq_desc& d, const void* W, const void* hdiag, const void* assign,
                            void* cb_out, hipStream_t s) {
#define VQ_F1(K) launch_update_rows<K, 1>(d, W, hdiag, assign, cb_out, s)
#define VQ_F2(K) launch_update_rows<K, 2>(d, W, hdiag, assign, cb_out, s)
#define VQ_F4(K) launch_update_rows<K, 4>(d, W, hdiag, assign, cb_out, s)
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
  return hipGetLastError();
}

}  // namespace vq
