// Batch-1 product y = W x for four-dimensional vector quantisation (Sec. 2.1 with d = 4; the
// 4D rows of the appendix table of VQ configurations): k = 256, one index byte per 4 weights,
// int8 tables with a scale (Sec. 3.1), groups of 64, 128 or 256 rows x 256 columns; also with fp16
// tables, and with blockwise normalisation on top of the int8 tables.
//
// A table is 256 entries x 4 values, far too large to rebuild per 8-row strip (a strip holds
// 512 bytes of indices per col-block, the table is 1 KB), so the unit of work is a workgroup of
// 8 waves that owns 64 consecutive rows (8 row-blocks of ONE group row): per pair of col-blocks
// the 512 threads dequantise the two tables once (one entry each: int8 x 4 -> fp16 x 4, times
// the scale, 8 bytes into LDS), a barrier, and every wave does its 16 lookups per lane (one
// 8-byte LDS read returns the four weights of a vector) and 32 dot2 steps.  The tables are
// double-buffered, so one barrier per pair of col-blocks is enough; indices, activations and
// the next table entry are loaded one step ahead.  A lane owns columns 4L .. 4L+3 of a
// col-block and keeps 8 row accumulators, reduced over the wave at the end exactly as in the
// other GEMV kernels.
//
// KS > 1 (launches of few 64-row items): KS workgroups share an item, each owns 8 / KS of its row-blocks, and
// KS groups of 8 / KS waves split the col-block pairs between them, each with tables of its own; the partial
// sums meet in LDS in a fixed order.  A 4096-row matrix is 64 items, a quarter of the CUs (rule and figures:
// wide_splits below).
//
// What bounds it: the LDS, whose random 8-byte lookups of uniform indices take 7.4 clocks a wave (2.9 without
// conflicts).  8 decoder layers in one launch (433 MB, d = 4): 119 -> 98 us, k = 256 int8 113 -> 91 us for 4 layers.
// What that took: the widest products first (widest_first in vq_api.hip; CUs stood idle for a fifth of the launch, 108.9),
// and two steps to a loop turn, whose loads are all unconditional and whose table buffers are constants: with a branch
// around one load, or the next step's registers copied, the compiler waited for the new loads of a step before it used
// the old ones (100), and half of the address instructions of the lookups go (98).  Not faster: a table of the 256 x 64
// products c.x (conflict-free lookups of 3.0 clocks, but 3.2 more to write the table for 256 rows), 16 or 32 copies of
// the table (5.0 + 1.6 and 3.1 + 3.2), 4-byte lookups of the int8 entries (7.0).
#include <type_traits>
#include "vq_gemv_impl.h"

namespace vq {
namespace {

// The 64-row item of a workgroup.  Workgroups go to the eight XCDs in turn; the four items of a 256-row group read the same
// tables, so each aligned 32 workgroups put four neighbouring items on one XCD, whose L2 then serves three of the four reads.
// 4 layers of 4096 / 11008 in one launch, d = 4, in the order of the workgroups and in this one: what the L2s fetch, by
// counter, 145 -> 109 MiB with fp16 tables and 121 -> 103 with int8 (of 2 KB and 1 KB a group), us 50.2 -> 45.3 and 48.8 -> 48.6; 32000 x
// 4096 11.8 -> 10.6 and 11.7 -> 10.4, with block scales 15.7 -> 14.9; 16 products of 11008 x 4096 45.2 -> 41.7 and 43.3 -> 43.4.  Where
// fewer rows share a table it only spreads the reads over memory differently: 64 rows, 512 items of 2048 columns 5.8 -> 6.4
// (fp16 tables 5.8 -> 7.0), 1024 of 8192 30.8 -> 35.2, 128 rows 5.8 -> 6.3; so it does for k = 256, d = 2, whose tables are 512 bytes (205
// -> 196 MiB): 256 rows, 32000 x 4096 17.5 -> 19.2, 16 of 4096 x 4096 31.0 -> 32.4.
__device__ __forceinline__ int item_of_workgroup(int b, int total) {
  return (b | 31) < total ? (b & ~31) | (b & 7) << 2 | ((b >> 3) & 3) : b;
}

// Table duty.  The waves that share tables write 512 entries, KS per thread: entry e0 + lane of table h (of the pair's first or
// second col-block).  From KS = 4 on the first half of them is of table 0 and the rest of table 1, and a scale and a
// level are held per table, not per entry: with KS = 4 k = 256 with block scales has 78 registers for 81, which makes room
// for a third workgroup per CU (us, 4096, 11008 and 3 x 4096 rows of 4096 columns: 6.43, 12.43, 12.67 -> 6.45, 11.92, 12.04), and
// d = 4 with an adapter 62, where a limit of 64 made it spill (7.90, 11.92, 12.11 -> 7.15, 10.88, 10.77).
template <int KS>
struct Duty {
  static constexpr int THREADS = 512 / KS;                          // threads that share tables
  static constexpr int TABLES = KS == 1 ? 1 : 2;                    // of a thread's entries
  static constexpr int PER_TABLE = KS / TABLES;
  // st: the first entry of the wave
  static __device__ __forceinline__ int h(int st, int i) { return PER_TABLE == 1 ? (st + i * THREADS) >> 8 : i / PER_TABLE; }
  static __device__ __forceinline__ int e0(int st, int i) { return (st + i * THREADS) & 255; }
};

template <int KS>
struct D4Step {
  uint4 w;        // the lane's 8 + 8 index bytes of the pair
  uint2 xa, xb;   // its activations in the two col-blocks
  uint2 q[KS];                   // this thread's table entries: 4 int8 in .x, or 4 fp16
  uint32_t sc[Duty<KS>::TABLES]; // int8 tables: the fp16 scales of their tables
  uint2 cw;       // blockwise normalisation: the lane's block codes in the two col-blocks (row r in bits [4r, 4r+4))
  uint32_t lv[Duty<KS>::TABLES]; // ... and level (lane & 15) of their tables (fp16)
};

// MODE 1 (F16): the tables are fp16 (2 KB per group, copied to LDS as they are) instead of int8
// with a scale.  MODE 2 (BN): int8 tables with blockwise normalisation (appendix "Blockwise data
// normalization"): the group's 16 block-scale levels sit next to its table in LDS, and per row
// the looked-up vector is multiplied by the scale of the lane's 32-weight block before the dot2.
template <bool LORA, int MODE, int CAP, int KS, bool XCD>
__global__ __launch_bounds__(512) void gemv_d4_kernel(const typename BatchOf<LORA, CAP>::type arg) {
  constexpr bool F16 = MODE == 1, BN = MODE == 2;
  const auto& batch = base_of(arg);
  constexpr int RBW = 8 / KS;                       // row-blocks of a workgroup
  __shared__ __attribute__((aligned(16))) uint2 tabs_all[KS][2][2][256];   // [buffer][col-block of the pair][entry]
  __shared__ uint32_t levs_all[KS][2][2][16];                               // BN: the tables' levels, the value in both halves
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int item = XCD ? item_of_workgroup((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x / KS;
  const int pi = find_problem(batch, item);
  const GemvItem P = item_of(batch, pi);
  const int oct = item - P.wg_begin;                // which 64 rows
  const int split = KS == 1 ? 0 : wave / RBW;       // which pairs of col-blocks
  auto& tabs = tabs_all[split];
  auto& levs = levs_all[split];
  const int n_cb = P.n_cb, n_pairs = (n_cb + 1) >> 1;
  const int rb = oct * 8 + (KS == 1 ? wave : ((int)blockIdx.x - item * KS) * RBW + wave % RBW);   // n_rb is a multiple of 8 (groups are >= 64 rows)
  const long long grow = (oct * 8) >> P.cb_log2;
  const uint8_t* tab = reinterpret_cast<const uint8_t*>(P.cb);
  const long long n_groups = (long long)(P.n_rb >> P.cb_log2) * n_cb;
  const uint16_t* scales = reinterpret_cast<const uint16_t*>(tab + n_groups * 1024);   // int8 tables only
  const uint16_t* levels = reinterpret_cast<const uint16_t*>(tab + wide_bn_level_offset((size_t)n_groups, 1024));
  const uint8_t* codes_lane = tab + wide_bn_code_offset((size_t)n_groups, 1024) + (size_t)rb * n_pairs * 64 + (lane >> 3) * 8;
  (void)levels; (void)codes_lane;
  const uint8_t* idx_rb = P.idx + (size_t)rb * n_pairs * 1024;
  using duty = Duty<KS>;
  const int st = wave % (duty::THREADS / 64) * 64;  // table duty of this wave: entries st + lane, st + lane + THREADS, .. of the two
  const int p_begin = n_pairs * split / KS, p_end = n_pairs * (split + 1) / KS;
  const int steps = (n_pairs + KS - 1) / KS;        // of the longest split: all take as many barriers

  auto load = [&](int p, D4Step<KS>& s) {           // (tables first: they are needed first; all of an address but the lane's part is wave-uniform)
    const int c0 = 2 * p, c1_ld = KS == 1 ? min(c0 + 1, n_cb - 1) : c0 + 1 < n_cb ? c0 + 1 : c0;   // an absent second col-block re-reads the first (not used)
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const int h = duty::h(st, i);
      const long long g = grow * n_cb + (KS == 1 ? min(c0 + h, n_cb - 1) : h == 0 ? c0 : c1_ld);   // (KS = 1: h is not a constant)
      if constexpr (F16) s.q[i] = reinterpret_cast<const uint2*>(tab + g * 2048 + duty::e0(st, i) * 8)[lane];
      else s.q[i] = make_uint2(reinterpret_cast<const uint32_t*>(tab + g * 1024 + duty::e0(st, i) * 4)[lane], 0u);
      if (i % duty::PER_TABLE == 0) {
        s.sc[i / duty::PER_TABLE] = F16 ? 0 : scales[g];
        if constexpr (BN) s.lv[i / duty::PER_TABLE] = levels[g * 16 + (lane & 15)];
      }
    }
    s.w = reinterpret_cast<const uint4*>(idx_rb + (size_t)p * 1024)[lane];
    s.xa = reinterpret_cast<const uint2*>(P.x + (size_t)c0 * 256)[lane];
    s.xb = reinterpret_cast<const uint2*>(P.x + (size_t)c1_ld * 256)[lane];
    if constexpr (BN) s.cw = *reinterpret_cast<const uint2*>(codes_lane + (size_t)p * 64);
  };

  float acc[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) acc[r] = 0.f;
  float tv[8];
  uint4 lb = make_uint4(0, 0, 0, 0);
  (void)tv; (void)lb; (void)pi;
  if constexpr (LORA) {      // issued ahead of the main loop, used after the reduction
    lora_load_t(arg.l[pi], P.x, lane, tv);
    lb = lora_load_b(arg.l[pi], P.x, rb, lane);
  }

  D4Step<KS> even, odd;
  const int p_last = p_end > p_begin ? p_end - 1 : 0;
  // One step: the next one's loads, this one's tables into buffer `buf`, a barrier, the lookups.
  auto run_step = [&](auto buf, auto ahead, int p, const D4Step<KS>& cur, D4Step<KS>& nxt) {
    if constexpr (ahead) load(min(p + 1, p_last), nxt);   // (a harmless re-read at the end)
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const int h = duty::h(st, i), e = duty::e0(st, i) + lane;
      const bool mine = h == 0 || 2 * p + 1 < n_cb; // the absent col-block of an odd matrix gets a zero table
      tabs[buf][h][e] = zero_unless(mine, F16 ? cur.q[i] : d4_dequant_entry(cur.q[i].x, __builtin_bit_cast(_Float16, (uint16_t)cur.sc[i / duty::PER_TABLE])));
      if constexpr (BN) {
        if (i % duty::PER_TABLE == 0 && e < 16) levs[buf][h][e] = mine ? cur.lv[i / duty::PER_TABLE] * 0x10001u : 0u;
      }
    }
    __syncthreads();   // tables of this step complete; the other buffer is free again (see header)
    if (KS > 1 && p >= p_end) return;               // the longest splits' last step
    const uint2 xb = zero_unless(2 * p + 1 < n_cb, cur.xb);
    const uint2* T0 = tabs[buf][0];
    const uint2* T1 = tabs[buf][1];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t j0 = ((r < 4 ? cur.w.x : cur.w.y) >> (8 * (r & 3))) & 0xffu;
      const uint32_t j1 = ((r < 4 ? cur.w.z : cur.w.w) >> (8 * (r & 3))) & 0xffu;
      uint2 t0 = T0[j0], t1 = T1[j1];
      if constexpr (BN) {
        const uint32_t s0 = levs[buf][0][(cur.cw.x >> (4 * r)) & 15u], s1 = levs[buf][1][(cur.cw.y >> (4 * r)) & 15u];
        t0 = make_uint2(scale_pair(t0.x, s0), scale_pair(t0.y, s0));
        t1 = make_uint2(scale_pair(t1.x, s1), scale_pair(t1.y, s1));
      }
      acc[r] = dot2(t0.x, cur.xa.x, acc[r]);
      acc[r] = dot2(t0.y, cur.xa.y, acc[r]);
      acc[r] = dot2(t1.x, xb.x, acc[r]);
      acc[r] = dot2(t1.y, xb.y, acc[r]);
    }
  };
  // A single step looks no further: one or two col-blocks (in two workgroups: up to four), which waited at the end for what nothing
  // uses.  1408 x 256, fp16 tables 2.61 -> 2.49 us, 16 of 2688 x 256 3.95 -> 3.57, int8 4352 x 256 2.70 -> 2.57.  Not in the kernels
  // whose registers it would take beyond what lets four workgroups share a CU.
  constexpr bool kAlone = !BN && (KS == 1 || (KS == 2 && !LORA));
  load(min(p_begin, p_last), even);
  const int p_stop = p_begin + steps;
  if (kAlone && steps == 1) run_step(std::integral_constant<int, 0>(), std::false_type(), p_begin, even, odd);
  else for (int p = p_begin;;) {   // (two exits: at a merge the compiler would wait for all loads)
    run_step(std::integral_constant<int, 0>(), std::true_type(), p, even, odd);
    if (++p >= p_stop) break;
    run_step(std::integral_constant<int, 1>(), std::true_type(), p, odd, even);
    if (++p >= p_stop) break;
  }

  float v = wave_reduce8(acc, lane);   // every lane: the total of row (lane >> 3) & 7
  if constexpr (KS > 1) {              // the splits' sums in order, by the waves of split 0
    __shared__ float part[8][8];
    if ((lane & 7) == 0) part[wave][lane >> 3] = v;
    __syncthreads();
    if (split > 0) return;
    v = 0.f;
#pragma unroll
    for (int q = 0; q < KS; ++q) v += part[q * RBW + wave][lane >> 3];
  }
  if constexpr (LORA) v += lora_term(lb, tv);
  if ((lane & 7) == 0) {
    const size_t o = (size_t)rb * 8 + (lane >> 3);
    if (P.y_f32) reinterpret_cast<float*>(P.y)[o] = v;
    else reinterpret_cast<_Float16*>(P.y)[o] = (_Float16)v;
  }
}

// ---- d = 2, k = 256, int8 tables with a scale, groups of 64, 128 or 256 rows ---------------
// The 4-bits-per-dimension 2D setting of the appendix table of VQ configurations: a 256-entry
// table is worth its bytes only when many rows share it, so the work is cut as above: 8 waves
// own 64 rows of one group row, per pair of col-blocks the 512 threads dequantise the two
// tables once (one entry each: two int8 times the scale, one dword into LDS), a barrier, and
// every wave runs the k = 256 inner block (16 lookups and 16 dot2 per col-block and lane) on
// its own 8 rows.  Indices are laid out as for k = 256 with fp16 codebooks (1 KB per 8-row
// block and col-block); the tables keep the canonical order (512 bytes per group, then scales).
template <int KS>
struct K256Step {
  uint4 w0, w1;   // the lane's 16 index bytes in the two col-blocks of the pair
  uint2 xa, xb;   // its activations there
  uint32_t q[KS];   // this thread's table entries (2 int8)
  uint32_t sc[Duty<KS>::TABLES];   // the fp16 scales of their tables
  uint2 cw;       // blockwise normalisation: the lane's block codes in the two col-blocks
  uint32_t lv[Duty<KS>::TABLES];   // ... and level (lane & 15) of their tables (fp16)
};

// BN: with blockwise normalisation; the plain C++ inner block replaces the hand-scheduled one.
template <bool LORA, bool BN, int CAP, int KS, bool = false>
__global__ __launch_bounds__(512) void gemv_k256i8_kernel(const typename BatchOf<LORA, CAP>::type arg) {
  const auto& batch = base_of(arg);
  constexpr int RBW = 8 / KS;                       // row-blocks of a workgroup
  __shared__ __attribute__((aligned(16))) uint32_t tabs_all[KS][2][2][256];   // [buffer][col-block of the pair][entry]
  __shared__ uint32_t levs_all[KS][2][2][16];                                  // BN: the tables' levels, the value in both halves
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int item = (int)blockIdx.x / KS;
  const int pi = find_problem(batch, item);
  const GemvItem P = item_of(batch, pi);
  const int oct = item - P.wg_begin;                // which 64 rows
  const int split = KS == 1 ? 0 : wave / RBW;       // which pairs of col-blocks
  auto& tabs = tabs_all[split];
  auto& levs = levs_all[split];
  const int n_cb = P.n_cb, n_pairs = (n_cb + 1) >> 1;
  const int rb = oct * 8 + (KS == 1 ? wave : ((int)blockIdx.x - item * KS) * RBW + wave % RBW);   // n_rb is a multiple of 8 (groups are >= 64 rows)
  const long long grow = (oct * 8) >> P.cb_log2;
  const uint8_t* tab = reinterpret_cast<const uint8_t*>(P.cb);
  const long long n_groups = (long long)(P.n_rb >> P.cb_log2) * n_cb;
  const uint16_t* scales = reinterpret_cast<const uint16_t*>(tab + n_groups * 512);
  const uint16_t* levels = reinterpret_cast<const uint16_t*>(tab + wide_bn_level_offset((size_t)n_groups, 512));
  const uint8_t* codes_lane = tab + wide_bn_code_offset((size_t)n_groups, 512) + (size_t)rb * n_pairs * 64 + (lane >> 3) * 8;
  (void)levels; (void)codes_lane;
  const uint8_t* idx_rb = P.idx + (size_t)rb * n_cb * 1024;
  using duty = Duty<KS>;
  const int st = wave % (duty::THREADS / 64) * 64;  // table duty of this wave: entries st + lane, st + lane + THREADS, .. of the two
  const int p_begin = n_pairs * split / KS, p_end = n_pairs * (split + 1) / KS;
  const int steps = (n_pairs + KS - 1) / KS;        // of the longest split: all take as many barriers

  auto load = [&](int p, K256Step<KS>& s) {         // (tables first: they are needed first; all of an address but the lane's part is wave-uniform)
    const int c0 = 2 * p, c1 = 2 * p + 1;
    const int c1_ld = c1 < n_cb ? c1 : c0;          // an absent second col-block re-reads the first (not used)
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const long long g = grow * n_cb + (duty::h(st, i) == 0 ? c0 : c1_ld);
      s.q[i] = reinterpret_cast<const uint16_t*>(tab + g * 512 + duty::e0(st, i) * 2)[lane];
      if (i % duty::PER_TABLE == 0) {
        s.sc[i / duty::PER_TABLE] = scales[g];
        if constexpr (BN) s.lv[i / duty::PER_TABLE] = levels[g * 16 + (lane & 15)];
      }
    }
    s.w0 = reinterpret_cast<const uint4*>(idx_rb + (size_t)c0 * 1024)[lane];
    s.w1 = reinterpret_cast<const uint4*>(idx_rb + (size_t)c1_ld * 1024)[lane];
    s.xa = reinterpret_cast<const uint2*>(P.x + (size_t)c0 * 256)[lane];
    s.xb = reinterpret_cast<const uint2*>(P.x + (size_t)c1_ld * 256)[lane];
    if constexpr (BN) s.cw = *reinterpret_cast<const uint2*>(codes_lane + (size_t)p * 64);
  };

  float acc[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) acc[r] = 0.f;
  float tv[8];
  uint4 lb = make_uint4(0, 0, 0, 0);
  (void)tv; (void)lb; (void)pi;
  if constexpr (LORA) {      // issued ahead of the main loop, used after the reduction
    lora_load_t(arg.l[pi], P.x, lane, tv);
    lb = lora_load_b(arg.l[pi], P.x, rb, lane);
  }

  K256Step<KS> even, odd;
  const int p_last = p_end > p_begin ? p_end - 1 : 0;
  auto run_step = [&](auto buf, int p, const K256Step<KS>& cur, K256Step<KS>& nxt) {   // as in gemv_d4_kernel
    load(min(p + 1, p_last), nxt);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      const int h = duty::h(st, i), e = duty::e0(st, i) + lane;
      const bool mine = h == 0 || 2 * p + 1 < n_cb; // the absent col-block of an odd matrix gets a zero table
      tabs[buf][h][e] = mine ? k64_dequant_pair(cur.q[i], __builtin_bit_cast(_Float16, (uint16_t)cur.sc[i / duty::PER_TABLE])) : 0u;
      if constexpr (BN) {
        if (i % duty::PER_TABLE == 0 && e < 16) levs[buf][h][e] = mine ? cur.lv[i / duty::PER_TABLE] * 0x10001u : 0u;
      }
    }
    __syncthreads();   // tables of this step complete; the other buffer is free again
    if (KS > 1 && p >= p_end) return;               // the longest splits' last step
    const uint2 xb = zero_unless(2 * p + 1 < n_cb, cur.xb);
    if constexpr (BN) {
      k256_group_scaled(cur.w0.x, cur.w0.y, cur.w0.z, cur.w0.w, cur.cw.x, tabs[buf][0], levs[buf][0], cur.xa.x, cur.xa.y, acc);
      k256_group_scaled(cur.w1.x, cur.w1.y, cur.w1.z, cur.w1.w, cur.cw.y, tabs[buf][1], levs[buf][1], xb.x, xb.y, acc);
    } else {
      const uint32_t base = lds_addr(&tabs[buf][0][0]);
      k256_group<0>(cur.w0.x, cur.w0.y, cur.w0.z, cur.w0.w, base, cur.xa.x, cur.xa.y, acc);
      k256_group<1024>(cur.w1.x, cur.w1.y, cur.w1.z, cur.w1.w, base, xb.x, xb.y, acc);
      acc_hazard_fence();
    }
  };
  load(min(p_begin, p_last), even);
  const int p_stop = p_begin + steps;
  for (int p = p_begin;;) {
    run_step(std::integral_constant<int, 0>(), p, even, odd);
    if (++p >= p_stop) break;
    run_step(std::integral_constant<int, 1>(), p, odd, even);
    if (++p >= p_stop) break;
  }

  float v = wave_reduce8(acc, lane);   // every lane: the total of row (lane >> 3) & 7
  if constexpr (KS > 1) {              // the splits' sums in order, by the waves of split 0
    __shared__ float part[8][8];
    if ((lane & 7) == 0) part[wave][lane >> 3] = v;
    __syncthreads();
    if (split > 0) return;
    v = 0.f;
#pragma unroll
    for (int q = 0; q < KS; ++q) v += part[q * RBW + wave][lane >> 3];
  }
  if constexpr (LORA) v += lora_term(lb, tv);
  if ((lane & 7) == 0) {
    const size_t o = (size_t)rb * 8 + (lane >> 3);
    if (P.y_f32) reinterpret_cast<float*>(P.y)[o] = v;
    else reinterpret_cast<_Float16*>(P.y)[o] = (_Float16)v;
  }
}

}  // namespace

// Workgroups per 64-row item.  us per launch at 1, 2, 4, 8 splits on 256 CUs (a pair: two col-blocks), 64-row groups, d = 4 with
// int8 tables / d = 2, k = 256:
//   32 items, 16 pairs 11.0, 7.5, 5.1, 4.2 / 16.9, 10.1, 6.5, 4.8
//   64, 8 pairs 6.4, 4.9, 3.9, 4.4 / 9.3, 6.1, 4.4, 4.6; 16 pairs 11.0, 7.6, 5.3, 6.0 / 17.0, 10.6, 7.4, 6.6; 22 pairs 14.6, 9.6, 6.7, 8.1 /
//     22.5, 13.4, 8.8, 8.7
//   128, 2 pairs 3.1, 3.0, 3.6 / 4.0, 3.4, 4.0; 8 pairs 6.6, 5.1, 5.1, 6.4 / 9.9, 7.1, 6.2, 6.5
//   192, 2 pairs 3.1, 3.4 / 4.0, 4.2 (block scales 5.1, 5.3); 4 pairs 4.3, 4.6, 4.4 / 5.8, 5.8, 5.1; 8 pairs 6.6, 6.8, 6.3 / 10.1, 10.3, 8.0
//   256, 4 pairs 4.3, 4.7 / 6.2, 5.9; 8 pairs 6.6, 6.8, 7.5 / 10.2, 10.5, 10.9
//   320, 2 pairs 4.0, 4.0 / 5.4, 4.9; 4 pairs 5.8, 5.6 / 8.8, 7.3, 6.6; 16 pairs 17.0, 15.8, 16.6 / 28.6, 23.5, 21.9
//   448, 4 pairs 5.8, 6.4 / 9.2, 9.1; 16 pairs 17.3, 19.8 / 29.4, 29.9; 512, 8 pairs 10.6, 11.7 / 16.4, 18.0
// d = 4 with fp16 tables stages twice the bytes: 192 items, 8 pairs 6.6, 6.5, 7.8; 320, 4 pairs 5.7, 5.4, 8 pairs 9.5, 9.5, 16 pairs 16.9,
// 17.4; 64 items, 16 pairs at 4 and 8 splits 5.3, 9.0, 32 items 5.1, 4.5.  So d = 4 splits less than d = 2 and neither much
// beyond one and a half items per CU.  The widest product of a launch decides, as a narrow one beside it costs
// little: 3 x 1024 x 256 + 64 x 11008 14.2, 9.4, 6.4, 5.1 / 21.9, 12.9, 8.2, 5.8; 11008 x 256 + 1024 x 11008 14.5, 9.5, 6.9, 8.9 / 22.4, 13.4,
// 8.8, 8.2, with fp16 tables 13.7, 9.1, 7.1, 10.6.  (The lines were drawn with a loop of one step to a turn.  With the loop
// above they would lie elsewhere for 64 items of d = 4 with int8 tables, four splits, and for d = 2 at 320 items of 4 and of 16
// pairs, four: 5.9, 5.3 / 7.2, 6.6 and 23.5, 21.9.)
static int wide_splits(const GemvBatch& b, int fmt) {
  int pairs = 1;
  for (int i = 0; i < b.count; ++i) pairs = max(pairs, (b.p[i].n_cb + 1) / 2);
  const long long items = b.total_wgs, cus = device_cus();
  long long work = 0;
  for (int i = 0; i < b.count; ++i) work += (long long)(b.p[i].n_rb / 8) * ((b.p[i].n_cb + 1) / 2);
  const long long full = work / pairs;              // items of full width with the same work
  if (b.count > kFewProblems || pairs < 2 || items > 2 * cus) return 1;
  const bool d2 = fmt == kFmtK256I8 || fmt == kFmtK256I8BN, f16 = fmt == kFmtD4F16;
  if (4 * items <= cus && pairs >= 16 && (!f16 || 8 * full <= cus)) return 8;
  if (2 * items <= cus) return pairs >= 4 ? 4 : 2;
  if (d2 && items <= cus && pairs < 4) return 1;
  if (d2 && 4 * items <= 3 * cus) return 4;
  if (d2) return 2 * items <= 3 * cus || pairs >= 16 || (pairs >= 4 && pairs < 8) ? 2 : 1;
  if (2 * items > 3 * cus) return 1;
  if (4 * items <= 3 * cus && pairs >= 8) return f16 && 2 * full > cus ? 2 : 4;
  if (items <= cus) return pairs >= 8 ? 2 : 1;
  return pairs >= 4 && !(f16 && pairs >= 8 && pairs < 16) ? 2 : 1;
}

// Whether neighbouring items go to one XCD (figures at item_of_workgroup): where all groups have 256 rows, but not up to two
// items of 2048 columns per CU (512: 5.8 -> 6.3 us, fp16 tables 5.8 -> 6.2; 640 of 2304 9.8 -> 9.2, 512 of 4096 10.7 -> 10.0).
static bool neighbours_by_xcd(const GemvBatch& b) {
  int widest = 0;
  for (int i = 0; i < b.count; ++i) {
    if (b.p[i].rb_per_cb != 32) return false;
    widest = max(widest, b.p[i].n_cb);
  }
  return widest > 8 || b.total_wgs > 2 * (long long)device_cus();
}

// (kernel, whether it has a variant for neighbours_by_xcd, template arguments before CAP)
#define VQ_LAUNCH_WIDE(KERNEL, XCD, ...)                                                                         \
  do {                                                                                                           \
    const int ks = wide_splits(base_of_host(batch), fmt);                                                        \
    const dim3 grid((unsigned)(total_wgs * ks));                                                                 \
    const bool xcd = XCD && neighbours_by_xcd(base_of_host(batch));                                              \
    if (base_of_host(batch).count > kFewProblems) {                                                              \
      if (xcd) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kMaxProblemsPerLaunch, 1, XCD>), grid, dim3(512), 0, s, batch); \
      else hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kMaxProblemsPerLaunch, 1, false>), grid, dim3(512), 0, s, batch); \
    } else if (ks == 8) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFewProblems, 8, false>), grid, dim3(512), 0, s, few_problems(batch)); \
    else if (ks == 4) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFewProblems, 4, false>), grid, dim3(512), 0, s, few_problems(batch)); \
    else if (ks == 2) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFewProblems, 2, false>), grid, dim3(512), 0, s, few_problems(batch)); \
    else if (xcd) hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFewProblems, 1, XCD>), grid, dim3(512), 0, s, few_problems(batch)); \
    else hipLaunchKernelGGL((KERNEL<__VA_ARGS__, kFewProblems, 1, false>), grid, dim3(512), 0, s, few_problems(batch)); \
  } while (0)

hipError_t launch_gemv_k256i8(const GemvBatch& batch, int total_wgs, hipStream_t s, int fmt) {
  if (fmt == kFmtK256I8BN) VQ_LAUNCH_WIDE(gemv_k256i8_kernel, false, false, true);
  else if (fmt == kFmtK256I8) VQ_LAUNCH_WIDE(gemv_k256i8_kernel, false, false, false);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_gemv_d4(const GemvBatch& batch, int total_wgs, hipStream_t s, int fmt) {
  if (fmt == kFmtD4F16) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, false, 1);
  else if (fmt == kFmtD4BN) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, false, 2);
  else if (fmt == kFmtD4) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, false, 0);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// The same kernels with the low-rank adapter term added to every row before it is stored.
hipError_t launch_gemv_k256i8_lora(const GemvBatchLora& batch, int total_wgs, hipStream_t s, int fmt) {
  if (fmt == kFmtK256I8BN) VQ_LAUNCH_WIDE(gemv_k256i8_kernel, false, true, true);
  else if (fmt == kFmtK256I8) VQ_LAUNCH_WIDE(gemv_k256i8_kernel, false, true, false);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_gemv_d4_lora(const GemvBatchLora& batch, int total_wgs, hipStream_t s, int fmt) {
  if (fmt == kFmtD4F16) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, true, 1);
  else if (fmt == kFmtD4BN) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, true, 2);
  else if (fmt == kFmtD4) VQ_LAUNCH_WIDE(gemv_d4_kernel, true, true, 0);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
#undef VQ_LAUNCH_WIDE

}  // namespace vq
