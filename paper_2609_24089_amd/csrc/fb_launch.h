// Host side of libflashbob.so shared by its translation units: launch shapes,
// problem validation and the per-(dtype, head dim) launchers.  flashbob.hip
// holds the C ABI; fb_passes_d128.hip holds the bf16 d = 128 instances of the
// two BoB pass launchers, which are built with a different instruction
// scheduler (see that file), and every other unit refers to them through the
// extern template declarations at the end.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <initializer_list>

#include "../../include/flashbob.h"
#include "fb_forms.h"
#include "fb_kernels.h"

namespace fb {

// Launch shapes per (element type, head dim) and kernel: MR = 16-row MFMA
// blocks per wave, NW = waves per workgroup (a workgroup owns 16*MR*NW
// stationary rows), OCC = waves per SIMD the register budget is held to, ST =
// LDS pipeline stages (tiles in flight + 1), DS = workgroups that share one
// row block, each accumulating 1/DS of the head dims (Pass 1 only), PF = 1 to
// read the accumulate operands one block ahead (Pass 1 and Pass 2; Pass 2
// then also reads its score operands one step ahead), 2 to also read Pass 1's
// score operands one step ahead.  KL = 1 keeps the first backward column
// kernel's stationary K rows in LDS instead of registers.
// kColsF and kP2F are the shapes of the column kernels' two-level
// (sectioned) accumulation for long streams (SectionSums), which holds a
// second set of key-side sums; mr = 0 where that form is not built.  kP2W
// is Pass 2 in wide workgroups (more waves sharing one copy of each streamed
// tile, one workgroup per CU), run on grids that fill the device without
// wave sets, parts or sections; mr = 0 where it is not built.  kP2P is Pass
// 2 in wave pairs that split the head dims (bob_pass2_pair_kernel, nw waves
// = nw / 2 pairs of 16 key rows), for head dims whose one-wave form holds
// one wave per SIMD; run where kP2W would be, dense or causal.
struct Shape {
  int mr, nw, occ, st, ds = 1, pf = 0, kl = 0;
};
constexpr Shape kNoForm{0, 1, 1, 2};
template <typename T, int D> struct Cfg;
template <> struct Cfg<bf16, 32> {
  static constexpr Shape kFwd{2, 4, 2, 2}, kRows{2, 4, 2, 2}, kCols{2, 4, 2, 2};
  static constexpr Shape kP1{1, 4, 3, 2}, kP1Six{2, 4, 2, 2}, kP2{2, 2, 2, 2};
  static constexpr Shape kAlpha{2, 4, 2, 2};
  static constexpr Shape kColsF{2, 4, 2, 2}, kP2F{2, 2, 2, 2}, kP2W = kNoForm, kP2P = kNoForm;
};
template <> struct Cfg<bf16, 64> {
  static constexpr Shape kFwd{2, 4, 4, 2}, kRows{2, 4, 2, 2}, kCols{2, 4, 2, 2, 1, 0, 1};
  static constexpr Shape kP1{1, 4, 2, 2}, kP1Six{1, 4, 2, 2}, kP2{2, 4, 2, 2};
  static constexpr Shape kAlpha{2, 4, 2, 2};
  static constexpr Shape kColsF{1, 4, 2, 2}, kP2F{1, 4, 3, 2}, kP2W = kNoForm, kP2P = kNoForm;
};
template <> struct Cfg<bf16, 128> {
  static constexpr Shape kFwd{2, 4, 3, 2}, kRows{2, 4, 2, 2}, kCols{2, 4, 2, 2, 1, 0, 1};
  static constexpr Shape kP1{1, 8, 2, 2, 1, 1}, kP1Six{1, 4, 1, 2}, kP2{1, 4, 2, 2, 1, 1};
  static constexpr Shape kAlpha{2, 4, 2, 2};
  static constexpr Shape kColsF{1, 4, 2, 2}, kP2F{1, 4, 1, 2, 1, 1}, kP2W{1, 8, 2, 2, 1, 1}, kP2P = kNoForm;
};
template <> struct Cfg<bf16, 256> {
  static constexpr Shape kFwd{1, 4, 2, 2}, kRows{1, 4, 2, 2}, kCols{1, 8, 2, 2, 1, 0, 1};
  static constexpr Shape kP1{1, 4, 1, 2}, kP1Six{1, 4, 1, 2, 2}, kP2{1, 4, 1, 2};
  static constexpr Shape kAlpha{1, 4, 2, 2};
  static constexpr Shape kColsF = kNoForm, kP2F = kNoForm, kP2W = kNoForm, kP2P{1, 8, 2, 2};
};
template <> struct Cfg<float, 32> {
  static constexpr Shape kFwd{1, 4, 1, 2}, kRows{1, 4, 1, 2}, kCols{1, 4, 1, 2};
  static constexpr Shape kP1{1, 4, 1, 2}, kP1Six{1, 4, 1, 2}, kP2{1, 4, 2, 2};
  static constexpr Shape kAlpha{1, 4, 1, 2};
  static constexpr Shape kColsF = kNoForm, kP2F = kNoForm, kP2W = kNoForm, kP2P = kNoForm;
};
template <> struct Cfg<float, 64> {
  static constexpr Shape kFwd{1, 4, 1, 2}, kRows{1, 4, 1, 2}, kCols{1, 4, 1, 2};
  static constexpr Shape kP1{1, 4, 1, 2}, kP1Six{1, 4, 1, 2}, kP2{1, 4, 2, 2};
  static constexpr Shape kAlpha{1, 4, 1, 2};
  static constexpr Shape kColsF = kNoForm, kP2F = kNoForm, kP2W = kNoForm, kP2P = kNoForm;
};
template <> struct Cfg<float, 128> {
  static constexpr Shape kFwd{1, 4, 1, 2}, kRows{1, 4, 1, 2}, kCols{1, 4, 1, 2};
  static constexpr Shape kP1{1, 4, 1, 2}, kP1Six{1, 4, 1, 2}, kP2{1, 4, 1, 2};
  static constexpr Shape kAlpha{1, 4, 1, 2};
  static constexpr Shape kColsF = kNoForm, kP2F = kNoForm, kP2W = kNoForm, kP2P = kNoForm;
};

constexpr int64_t kMaxN = int64_t(1) << 30;

inline bool aligned16(const void* p) { return p != nullptr && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// H query heads per batch entry; Hkv key/value heads (H for multi-head
// attention, a divisor of H for grouped-query attention).
struct Problem {
  int32_t dtype;
  int64_t B, H, N, d;
  float scale;
  int32_t causal;
  int64_t Hkv;
};
inline int group(const Problem& p) { return (int)(p.H / p.Hkv); }

// (dtype, head dim) pairs built into the library: bf16 d = 32, 64, 128, 256;
// fp32 d = 32, 64, 128 (fp32 d = 256 would need twice the registers of bf16).
inline bool supported(int32_t dtype, int64_t d) {
  if (dtype == BOB_BF16) return d == 32 || d == 64 || d == 128 || d == 256;
  if (dtype == BOB_F32) return d == 32 || d == 64 || d == 128;
  return false;
}

// Returns BOB_OK to proceed, or an error; sets *empty for B*H*N == 0.
inline int32_t check_problem(const Problem& p, bool* empty) {
  *empty = false;
  if (p.dtype != BOB_F32 && p.dtype != BOB_BF16) return BOB_EINVAL;
  if (p.B < 0 || p.H < 0 || p.N < 0 || p.d < 1) return BOB_EINVAL;
  if (!std::isfinite(p.scale)) return BOB_EINVAL;
  if (p.causal != 0 && p.causal != 1) return BOB_EINVAL;
  if (p.Hkv < 0 || (p.H > 0 && (p.Hkv < 1 || p.H % p.Hkv != 0))) return BOB_EINVAL;
  if (!supported(p.dtype, p.d)) return BOB_EUNSUPPORTED;
  if (p.B == 0 || p.H == 0 || p.N == 0) {
    *empty = true;
    return BOB_OK;
  }
  if (p.N > kMaxN) return BOB_EINVAL;
  // 32-bit grid and loop counts: heads x row blocks sizes the grid (the whole block
  // shapes have 64 rows or more; pick_form() takes no narrower one whose grid is too
  // large), and a column kernel streams up to H/Hkv heads of ceil(N/32) tiles in one
  // loop, so heads x 32-row tiles must fit an int
  const int64_t heads = p.B * p.H;
  if (p.B > INT32_MAX || p.H > INT32_MAX || heads > INT32_MAX) return BOB_EINVAL;
  if (heads * ((p.N + 31) / 32) > INT32_MAX) return BOB_EINVAL;
  return BOB_OK;
}

inline int32_t check_ptrs(std::initializer_list<const void*> ptrs) {
  for (const void* q : ptrs)
    if (!aligned16(q)) return BOB_EINVAL;
  return BOB_OK;
}

inline int32_t finish_launch() { return hipGetLastError() == hipSuccess ? BOB_OK : BOB_ELAUNCH; }

struct Grid {
  int nRB, total;
};
// Row kernels run over the query heads, column kernels over the key/value heads.
inline Grid grid_for(const Problem& p, int rows_per_block, bool kv_heads = false) {
  Grid g;
  g.nRB = (int)((p.N + rows_per_block - 1) / rows_per_block);
  g.total = (int)(p.B * (kv_heads ? p.Hkv : p.H) * g.nRB);
  return g;
}

// Compute units of the current device (0 if it cannot be read).
int device_cus();

// Workgroups of kKernel that fit one CU (1 if the runtime cannot tell), read
// once per kernel: a property of its code object.
template <auto kKernel> int resident_blocks(int threads) {
  static std::atomic<int> known;
  return std::max(1, read_once(known, [&] {
    int n = 0;
    const hipError_t rc = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void*)kKernel, threads, 0);
    return rc == hipSuccess ? n : 0;
  }));
}

// The `resident` argument of a launch of kKernel (balanced_order()).
template <auto kKernel> int causal_resident(const Problem& p, const Grid& g, int threads) {
  return p.causal == 0 ? 0 : balanced_order(g.total, resident_blocks<kKernel>(threads), device_cus());
}

// What a step of each kernel costs: base, per 16-row block, and what a block of the
// narrow forms weighs (csrc/fb_forms.h; the figures' origin is beside pick_form()).
template <typename T> constexpr bool kBf = sizeof(T) == 2;
template <typename T> constexpr StepCost kFwdStep = kBf<T> ? StepCost{7.0, 0.36, 2.1} : StepCost{5.0, 1.2, 1.0};
template <typename T> constexpr StepCost kRowsStep = kBf<T> ? StepCost{4.6, 0.62, 1.2} : StepCost{2.8, 1.2, 1.1};
template <typename T> constexpr StepCost kP1Step = kBf<T> ? StepCost{7.7, 0.38, 1.55} : StepCost{4.5, 0.45, 1.0};
template <typename T> constexpr StepCost kColsStep = kBf<T> ? StepCost{8.6, 0.48, 1.8} : StepCost{3.3, 0.39, 1.6};
template <typename T> constexpr StepCost kP2Step = kBf<T> ? StepCost{7.2, 0.48, 1.55} : StepCost{5.3, 0.38, 1.0};
// Row kernels leave their whole blocks only for an estimated gain of a tenth.
constexpr double kRowMargin = 1.1;
// The wave pairs of Pass 2 at bf16 d = 256 (two waves per SIMD) against the one-wave
// form that its splits run.
constexpr double kPairWeight = 0.2;

// Adding one more wave set's `sums` accumulators of one 16-row block through LDS: 1.5 us
// per 64 KB where a block's sums are large; with narrower heads it does not show
// beside the rest of a round.
inline double merge_us(int sums, int64_t d) { return d < 256 ? 0.0 : 1.5 * sums * (double)d / 1024; }

// Time of `contractions` tile contractions of one 16-row block, in us at 85% of the
// rate that a large matrix product reached on one CU (1366 TFLOP/s bf16, 154 fp32,
// on 256 CUs).
template <typename T> double block_us(int contractions, int64_t d) {
  constexpr double kRate = (sizeof(T) == 2 ? 1366e6 : 154e6) * 0.85 / 256;  // FLOP per us
  return 2.0 * contractions * 16 * kBS * (double)d / kRate;
}

// ---------------------------------------------------------------------------
// Small grids: blocks of 16 nw stationary rows (nw = 4, 2, 1), with as many wave
// sets as the LDS holds, which share the streamed tiles.  The structs below name
// their kernel in kernel() alone, which only form() and launch() call, and those are
// defined out of class: a unit compiles the kernels of the structs that it
// instantiates and no others (an address in a class-level constant compiled every
// kernel in every unit).
// ---------------------------------------------------------------------------
struct SetShape {
  int nw, ks, occ;
};
// The wave sets of a kernel that streams `tensors` tensors and keeps `extra`
// bytes of LDS beside each ring: a power of two whose two-stage rings fit 160 KB,
// in at most `max_waves` waves.
template <typename T, int D> constexpr SetShape set_shape(int nw, int tensors, int extra, int max_waves, int occ) {
  const int ring = 2 * tensors * Geo<T, D>::kTileElems * (int)sizeof(T);
  int ks = 1;
  while (2 * ks * nw <= max_waves && 2 * ks * (ring + extra) <= 160 * 1024) ks *= 2;
  return {nw, ks, std::max(occ, ks * nw / 4)};
}
// Whether blocks of nw waves are worth building beside those of twice as many, the
// next wider form: not where those have the same sets and need no more than a CU's four
// SIMDs, so that a step takes them as long and they hold twice the rows (a gain of half
// a merge, under 0.5 us, on problems of one such block a head).
constexpr bool worth_building(SetShape s, SetShape twice) { return s.ks != twice.ks || 2 * s.nw * s.ks > 4; }

// ---------------------------------------------------------------------------
// Column kernels (the first backward's dK, dV and Pass 2's Kt, Vt): how one
// problem's column blocks are laid out over workgroups.
//  * parts: workgroups per column block (kParts forms; 1 = unsplit).  Split,
//    each part stores fp32 partial sums to a caller's workspace and
//    bob_column_parts_reduce_kernel adds them.
//  * sets: wave sets per workgroup (KS = 2 fills a CU with one workgroup when
//    the grid has no more workgroups than the device has CUs; shapes held to
//    two waves per SIMD whose two LDS rings fit 160 KB and hold the merge
//    buffer), or narrow blocks in two or more sets where pick_form() expects
//    them to be faster; a request for two sets means either.
//  * flush_tiles: streamed tiles per MFMA accumulation section (SectionSums;
//    0 = one chain over the whole stream), with the kColsF / kP2F shape.
// The caller's requests (bob_column_opts; 0 = automatic) are resolved here,
// deterministically from the problem and the device's CU count, so the
// workspace query and the call that uses the workspace agree.
// ---------------------------------------------------------------------------
constexpr int kMaxParts = 8;
// Automatic sections: a stream longer than kLongChain tiles per accumulator
// chain is cut into sections of kSectionTiles.  Measured on the zero column
// sums (B1 H1 d64 bf16): at chains of 16384 tiles the residual stays at the
// bf16 rounding floor (about 3e-3), at 32768 it is 8.8e-3 and at 65536
// 2.9e-2; in sections of 1024 it stays at the floor up to N = 2^22.
constexpr int64_t kLongChain = 16384;
constexpr int kSectionTiles = 1024;

// Automatic part counts of column blocks of at least kLongBlock streamed
// iterations follow resolve_parts(), those of shorter ones (of min_iters or more)
// pick_form().
constexpr int64_t kLongBlock = 1024;
struct ColumnOpts {
  int parts = 0, wave_sets = 0, flush_tiles = 0;
  int64_t min_iters = 0;
};
struct ColumnPlan {
  Grid g{0, 0};
  int parts = 1, sets = 1, flush_tiles = 0;
  int narrow = 0;      // 4, 2 or 1: blocks of 16 times that many key rows in wave sets (ColsSmall, Pass2Small)
  bool wide = false;   // Pass 2 in the kP2W shape
  bool pairs = false;  // Pass 2 in wave pairs (kP2P)
};

// Automatic part count for a column grid of `workgroups` with at least
// kLongBlock streamed iterations per block.
int resolve_parts(int workgroups, bool causal, bool pass2);


// Automatic (requested = 0: two sets when the grid has no more workgroups
// than the device has CUs) or forced (1, 2) wave sets.
inline bool resolve_two_sets(int requested, int workgroups) {
  if (requested == 1) return false;
  if (requested == 2) return true;
  return workgroups <= device_cus();
}

template <typename T, int D, int MC, int NW, int OCC, int NSTAGE, int NTENS, int NSCAL, bool KL = false>
constexpr bool two_sets_fit() {
  constexpr size_t ring = (size_t)NSTAGE * NTENS * Geo<T, D>::kTileElems * sizeof(T);
  constexpr size_t scal = (size_t)(NSTAGE + 2) * NSCAL * kBS * sizeof(float);
  constexpr size_t kst = KL ? (size_t)NW * Geo<T, D>::kTileElems * sizeof(T) : 0;  // shared by both sets
  return OCC == 2 && NW <= 4 && 2 * (ring + scal) + kst <= 160 * 1024 &&
         2 * ring >= (size_t)NW * Geo<T, D>::kNB * MC * 1024;
}

// Streamed iterations of one column block: its group's query heads times
// 32-row query tiles (the first block under the causal mask streams them all).
inline int64_t column_iters(const Problem& p) { return (int64_t)group(p) * ((p.N + 31) / 32); }

// fp32 workspace of a split column kernel: parts x {Kt, Vt} (or {dK, dV})
// x B*Hkv*N*d.
inline int64_t column_workspace_bytes(const Problem& p, int parts) {
  return parts > 1 ? (int64_t)parts * 2 * p.B * p.Hkv * p.N * p.d * (int64_t)sizeof(float) : 0;
}

template <typename T, int D, bool kPass2, bool kF>
struct ColumnShape {
  static constexpr Shape kS =
      kPass2 ? (kF ? Cfg<T, D>::kP2F : Cfg<T, D>::kP2) : (kF ? Cfg<T, D>::kColsF : Cfg<T, D>::kCols);
  static constexpr bool kTwoFit =
      kS.mr > 0 && two_sets_fit<T, D, kS.mr, kS.nw, kS.occ, kS.st, kPass2 ? 3 : 2, kPass2 ? 4 : 2, kS.kl != 0>();
};

// The split form of a column kernel.
template <typename T, int D, bool kPass2, bool kF> constexpr auto parts_kernel() {
  constexpr Shape s = ColumnShape<T, D, kPass2, kF>::kS;
  if constexpr (kPass2)
    return &bob_pass2_kernel<T, D, s.mr, s.nw, s.occ, s.st, true, 1, s.pf != 0, true, kF>;
  else
    return &attn_bwd_cols_kernel<T, D, s.mr, s.nw, s.occ, s.st, true, 1, true, kF, s.kl != 0>;
}

// Workgroups of a column kernel that fit one CU, in its split or its (one wave
// set) unsplit form.
template <typename T, int D, bool kPass2, bool kF> int columns_resident(bool split) {
  constexpr Shape s = ColumnShape<T, D, kPass2, kF>::kS;
  if (split) return resident_blocks<parts_kernel<T, D, kPass2, kF>()>(64 * s.nw);
  if constexpr (kPass2)
    return resident_blocks<&bob_pass2_kernel<T, D, s.mr, s.nw, s.occ, s.st, true, 1, s.pf != 0, false, kF>>(64 * s.nw);
  else
    return resident_blocks<&attn_bwd_cols_kernel<T, D, s.mr, s.nw, s.occ, s.st, true, 1, false, kF, s.kl != 0>>(64 *
                                                                                                             s.nw);
}
extern template int columns_resident<bf16, 128, true, false>(bool);  // built in fb_passes_d128.hip, with their kernels
extern template int columns_resident<bf16, 128, true, true>(bool);

// The column kernels in narrow blocks of 16 NW key rows with wave sets, for
// grids with fewer column blocks than the device has CUs.  Built on the grouped
// loop, which also runs multi-head problems.
template <typename T, int D, int NW> struct ColsSmall {
  static constexpr int kExtra = 4 * 2 * kBS * (int)sizeof(float);  // raw and transformed L, D
  // K, V and two accumulators of 16 rows fit four waves per SIMD up to 128-byte rows
  static constexpr SetShape shape(int nw) {
    return set_shape<T, D>(nw, 2, kExtra, D * (int)sizeof(T) <= 128 ? 16 : 8, Cfg<T, D>::kCols.occ);
  }
  static constexpr SetShape kS = shape(NW);
  static constexpr bool kBuilt = kS.ks > 1 && worth_building(kS, shape(2 * NW));
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt)
      return &attn_bwd_cols_kernel<T, D, 1, NW, kS.occ, 2, true, kS.ks, false, false, false>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, const void* dO, const float* L,
                        const float* Dv, void* dK, void* dV, hipStream_t s);
};
template <typename T, int D, int NW> struct Pass2Small {
  static constexpr int kExtra = 4 * 4 * kBS * (int)sizeof(float);  // raw and transformed L, D, alpha, E
  static constexpr SetShape shape(int nw) { return set_shape<T, D>(nw, 3, kExtra, 8, Cfg<T, D>::kP2.occ); }
  static constexpr SetShape kS = shape(NW);
  // three tensors of two 1 KB blocks (bf16 d = 32) do not deal out over four waves;
  // where four blocks in two sets are the whole shape's two sets, those run
  static constexpr bool kSameAsWhole = Cfg<T, D>::kP2.mr == 1 && Cfg<T, D>::kP2.nw == NW && kS.ks == 2 &&
                                       ColumnShape<T, D, true, false>::kTwoFit;
  static constexpr bool kBuilt = kS.ks > 1 && !kSameAsWhole && !(sizeof(T) == 2 && D == 32 && NW == 4) &&
                                 worth_building(kS, shape(2 * NW));
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt)
      return &bob_pass2_kernel<T, D, 1, NW, kS.occ, 2, true, kS.ks, Cfg<T, D>::kP2.pf != 0, false, false>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, const void* dO, const void* UQ,
                        const void* UK, const void* UV, const float* L, const float* Dv, const float* alpha,
                        const float* E, void* Kt, void* Vt, hipStream_t s);
};
template <typename T, int D, int NW> Form ColsSmall<T, D, NW>::form() {
  constexpr int kThreads = 64 * NW * kS.ks;
  if constexpr (kBuilt) return {NW, kS.ks, resident_blocks<kernel()>(kThreads), kThreads, 1, 0.0, kColsStep<T>.narrow};
  else return {};
}
template <typename T, int D, int NW>
int32_t ColsSmall<T, D, NW>::launch(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                                    const float* L, const float* Dv, void* dK, void* dV, hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * NW, true);
    const int res = causal_resident<kernel()>(p, g, 64 * NW * kS.ks);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(64 * NW * kS.ks), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (const T*)dO, L, Dv, (T*)dK, (T*)dV, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p),
                       (float*)nullptr, 1, 0);
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}
template <typename T, int D, int NW> Form Pass2Small<T, D, NW>::form() {
  constexpr int kThreads = 64 * NW * kS.ks;
  if constexpr (kBuilt) return {NW, kS.ks, resident_blocks<kernel()>(kThreads), kThreads, 1, 0.0, kP2Step<T>.narrow};
  else return {};
}
template <typename T, int D, int NW>
int32_t Pass2Small<T, D, NW>::launch(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                                     const void* UQ, const void* UK, const void* UV, const float* L, const float* Dv,
                                     const float* alpha, const float* E, void* Kt, void* Vt, hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * NW, true);
    const int res = causal_resident<kernel()>(p, g, 64 * NW * kS.ks);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(64 * NW * kS.ks), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, alpha, E, (T*)Kt, (T*)Vt,
                       (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p), (float*)nullptr, 1, 0);
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}
template <typename T, int D, bool kPass2, int NW> Form narrow_form() {
  if constexpr (kPass2) return Pass2Small<T, D, NW>::form();
  else return ColsSmall<T, D, NW>::form();
}
// Built in fb_cols_small.hip and (Pass 2 at bf16 d = 128) fb_passes_d128.hip.
#define FB_COLS_SMALL(EXT, T, D) \
  EXT template struct ColsSmall<T, D, 4>; EXT template struct ColsSmall<T, D, 2>; EXT template struct ColsSmall<T, D, 1>;
#define FB_PASS2_SMALL(EXT, T, D) \
  EXT template struct Pass2Small<T, D, 4>; EXT template struct Pass2Small<T, D, 2>; EXT template struct Pass2Small<T, D, 1>;
#define FB_EACH_BUT_BF16_128(M, EXT) \
  M(EXT, bf16, 32) M(EXT, bf16, 64) M(EXT, bf16, 256) M(EXT, float, 32) M(EXT, float, 64) M(EXT, float, 128)
FB_EACH_BUT_BF16_128(FB_COLS_SMALL, extern)
FB_COLS_SMALL(extern, bf16, 128)
FB_EACH_BUT_BF16_128(FB_PASS2_SMALL, extern)
FB_PASS2_SMALL(extern, bf16, 128)

// Plan of a validated, non-empty, supported problem.  BOB_EINVAL for a
// request out of range, BOB_EUNSUPPORTED for sections requested where the
// sectioned form is not built.
template <typename T, int D, bool kPass2>
int32_t plan_columns(const Problem& p, const ColumnOpts& o, ColumnPlan* out) {
  if (o.parts < 0 || o.parts > kMaxParts || o.wave_sets < 0 || o.wave_sets > 2 || o.flush_tiles < -1)
    return BOB_EINVAL;
  using S0 = ColumnShape<T, D, kPass2, false>;
  using SF = ColumnShape<T, D, kPass2, true>;
  const int cus = device_cus();
  auto fill = [&](auto shape, auto f) {
    constexpr Shape s = decltype(shape)::kS;
    constexpr bool two_fit = decltype(shape)::kTwoFit;
    ColumnPlan c;
    c.g = grid_for(p, 16 * s.mr * s.nw, true);
    const int64_t iters = column_iters(p);
    const bool two = two_fit && resolve_two_sets(o.wave_sets, c.g.total);
    if (o.parts > 0)
      c.parts = o.parts;
    else if (iters >= kLongBlock)
      c.parts = resolve_parts(c.g.total, p.causal != 0, kPass2);
    int narrow = 0;
    if (c.parts == 1 && cus > 0) {
      constexpr bool kSection = decltype(f)::value;
      Form whole{s.mr * s.nw, 1, 1, 64 * s.nw}, n4, n2, n1, split[kMaxParts + 1];
      if (two)
        whole.sets = 2;
      else if constexpr (!kSection)
        whole.resident = columns_resident<T, D, kPass2, false>(false);
      // what an unsplit Pass 2 runs in (below): wide blocks, wave pairs
      if constexpr (!kSection && kPass2 && Cfg<T, D>::kP2W.mr > 0)
        if (constexpr Shape w = Cfg<T, D>::kP2W; !two && o.wave_sets == 0 && !p.causal && o.flush_tiles <= 0 &&
            grid_for(p, 16 * w.mr * w.nw, true).total >= cus)
          whole = {w.mr * w.nw, 1, 1, 64 * w.nw};
      if constexpr (!kSection && kPass2 && Cfg<T, D>::kP2P.mr > 0)
        if (constexpr Shape q = Cfg<T, D>::kP2P; o.wave_sets == 0 && o.flush_tiles <= 0)
          whole = {q.nw / 2, 1, 1, 64 * q.nw, 1, 0.0, kPairWeight};
      // narrow blocks: on grids with no more whole blocks than CUs, where wave
      // sets may be chosen and the whole block does not run in wave pairs
      if constexpr (!kSection && !(kPass2 && Cfg<T, D>::kP2P.mr > 0))
        if (o.wave_sets != 1 && o.flush_tiles <= 0 && c.g.total <= cus) {
          n4 = narrow_form<T, D, kPass2, 4>();
          n2 = narrow_form<T, D, kPass2, 2>();
          n1 = narrow_form<T, D, kPass2, 1>();
        }
      // parts: 16 bytes an output element and part, written and read at 6 TB/s,
      // and a launch (4 us in a trace, 6 with its gap); not where wave sets are asked
      // for, which a split has none of
      if (o.parts == 0 && o.wave_sets == 0 && iters < kLongBlock && iters >= o.min_iters)
        for (int n = 2; n <= kMaxParts; ++n)
          split[n] = {s.mr * s.nw, 1, columns_resident<T, D, kPass2, kSection>(true), 64 * s.nw, n,
                      6.2 + 16.0 * n * (double)(p.B * p.Hkv * p.N * p.d) / 6e6};
      const int form = pick_form(
          {cus, p.B * p.Hkv, p.N, iters, p.causal != 0, block_us<T>(kPass2 ? 8 : 4, p.d),
           kPass2 ? kP2Step<T> : kColsStep<T>, merge_us(2, p.d)},
          {whole, n4, n2, n1, split[2], split[3], split[4], split[5], split[6], split[7], split[8]});
      if (form >= 4) c.parts = form - 2;
      else if (form >= 1) narrow = 8 >> form;
    }
    if ((int64_t)c.g.total * c.parts > INT32_MAX) c.parts = 1;
    c.sets = c.parts == 1 && two ? 2 : 1;
    if (c.parts == 1 && narrow != 0) {
      c.narrow = narrow;
      c.sets = 2;
      c.g = grid_for(p, 16 * narrow, true);
    }
    return c;
  };
  ColumnPlan c = fill(S0{}, std::false_type{});
  int ft = o.flush_tiles;
  if (ft == 0) {
    const int64_t per = (int64_t)c.parts * c.sets;  // narrow blocks have two sets or more
    const int64_t chain = (column_iters(p) + per - 1) / per;
    ft = (SF::kS.mr > 0 && chain > kLongChain) ? kSectionTiles : -1;
  }
  if (ft > 0) {
    if constexpr (SF::kS.mr == 0) return BOB_EUNSUPPORTED;
    else c = fill(SF{}, std::true_type{});
    c.flush_tiles = ft;
  }
  // Wide Pass 2 workgroups on dense grids that fill every CU with them
  // (under the causal mask the larger blocks balance worse), when the wave
  // sets are automatic: 3-4% faster at N = 16384, d = 128 with 16 and with 4
  // key/value heads, outputs bit for bit those of the narrow form (each wave
  // does the same arithmetic), which a forced wave_sets = 1 still runs.
  if constexpr (kPass2 && Cfg<T, D>::kP2W.mr > 0) {
    constexpr Shape w = Cfg<T, D>::kP2W;
    if (o.wave_sets == 0 && !p.causal && c.parts == 1 && c.sets == 1 && c.flush_tiles <= 0 && cus > 0) {
      const Grid gw = grid_for(p, 16 * w.mr * w.nw, true);
      if (gw.total >= cus) {
        c.g = gw;
        c.wide = true;
      }
    }
  }
  // Wave pairs where the one-wave Pass 2 holds one wave per SIMD, on the
  // same unsplit, single-set, one-section layouts (the pairs' column blocks
  // have the one-wave form's 16 key rows per pair).
  if constexpr (kPass2 && Cfg<T, D>::kP2P.mr > 0) {
    constexpr Shape q = Cfg<T, D>::kP2P;
    if (o.wave_sets == 0 && c.parts == 1 && c.sets == 1 && c.flush_tiles <= 0) {
      c.g = grid_for(p, 16 * (q.nw / 2), true);
      c.pairs = true;
    }
  }
  *out = c;
  return BOB_OK;
}

// The query of a row kernel's launch.
template <typename T> FormQuery row_query(const Problem& p, int contractions, int sums, const StepCost& step) {
  return {device_cus(), p.B * p.H, p.N, (p.N + kBS - 1) / kBS, p.causal != 0, block_us<T>(contractions, p.d), step,
          merge_us(sums, p.d), kRowMargin};
}

template <typename T, int D, int NW> struct FwdSmall {
  static constexpr SetShape shape(int nw) { return set_shape<T, D>(nw, 2, 128 * nw, 16, Cfg<T, D>::kFwd.occ); }
  static constexpr SetShape kS = shape(NW);
  static constexpr bool kBuilt = worth_building(kS, shape(2 * NW));
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt) return &attn_fwd_kernel<T, D, 1, NW, kS.occ, 2, kS.ks>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* L,
                        hipStream_t s);
};
template <typename T, int D, int NW> Form FwdSmall<T, D, NW>::form() {
  constexpr int kThreads = 64 * NW * kS.ks;
  if constexpr (kBuilt) return {NW, kS.ks, resident_blocks<kernel()>(kThreads), kThreads, 1, 0.0, kFwdStep<T>.narrow};
  else return {};
}
template <typename T, int D, int NW>
int32_t FwdSmall<T, D, NW>::launch(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* L,
                                   hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * NW);
    const int res = causal_resident<kernel()>(p, g, 64 * NW * kS.ks);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(64 * NW * kS.ks), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (T*)O, L, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p));
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}

// The whole block shape (32 rows per wave) in two wave sets, for grids that leave
// a CU's slots empty or, causal, its last blocks alone.  Forward, whole -> two
// sets (us): bf16 B2 H8 N4096 d64 93 -> 81, B1 H16 N4096 d64 causal 73 -> 54, B1
// H8 N4096 d128 93 -> 79, B1 H1 N65536 d64 1489 -> 1215.
template <typename T, int D> struct FwdWide {
  static constexpr Shape kS = Cfg<T, D>::kFwd;
  static constexpr bool kBuilt = kS.mr == 2;
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt) return &attn_fwd_kernel<T, D, kS.mr, kS.nw, kS.occ, kS.st, 2>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* L,
                        hipStream_t s);
};
template <typename T, int D> Form FwdWide<T, D>::form() {
  if constexpr (kBuilt) return {kS.mr * kS.nw, 2, resident_blocks<kernel()>(128 * kS.nw), 128 * kS.nw};
  else return {};
}
template <typename T, int D>
int32_t FwdWide<T, D>::launch(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* L,
                              hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * kS.mr * kS.nw);
    const int res = causal_resident<kernel()>(p, g, 128 * kS.nw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(128 * kS.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (T*)O,
                       L, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p));
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}
template <typename T, int D> struct RowsWide {
  static constexpr Shape kS = Cfg<T, D>::kRows;
  // at d = 128 one workgroup of 16 block-sets fits a CU, as two of RowsSmall<4>'s do
  // in the same step and finer grain
  static constexpr bool kBuilt = kS.mr == 2 && D < 128;
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt) return &attn_bwd_rows_kernel<T, D, kS.mr, kS.nw, kS.occ, kS.st, 2>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* L, void* dQ, float* Dv, hipStream_t s);
};
template <typename T, int D> Form RowsWide<T, D>::form() {
  if constexpr (kBuilt) return {kS.mr * kS.nw, 2, resident_blocks<kernel()>(128 * kS.nw), 128 * kS.nw};
  else return {};
}
template <typename T, int D>
int32_t RowsWide<T, D>::launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                               const void* dO, const float* L, void* dQ, float* Dv, hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * kS.mr * kS.nw);
    const int res = causal_resident<kernel()>(p, g, 128 * kS.nw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(128 * kS.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (const T*)O, (const T*)dO, L, (T*)dQ, Dv, (int)p.N, g.nRB, g.total, p.scale, p.causal, res,
                       group(p));
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}

template <typename T, int D, int NW> struct RowsSmall {
  // two operands and an accumulator of 16 rows fit four waves per SIMD up to 128-byte rows
  static constexpr SetShape shape(int nw) {
    return set_shape<T, D>(nw, 2, 128 * nw, D * (int)sizeof(T) <= 128 ? 16 : 8, Cfg<T, D>::kRows.occ);
  }
  static constexpr SetShape kS = shape(NW);
  static constexpr bool kBuilt = worth_building(kS, shape(2 * NW));
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt) return &attn_bwd_rows_kernel<T, D, 1, NW, kS.occ, 2, kS.ks>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* L, void* dQ, float* Dv, hipStream_t s);
};
template <typename T, int D, int NW> Form RowsSmall<T, D, NW>::form() {
  constexpr int kThreads = 64 * NW * kS.ks;
  if constexpr (kBuilt) return {NW, kS.ks, resident_blocks<kernel()>(kThreads), kThreads, 1, 0.0, kRowsStep<T>.narrow};
  else return {};
}
template <typename T, int D, int NW>
int32_t RowsSmall<T, D, NW>::launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                                    const void* dO, const float* L, void* dQ, float* Dv, hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * NW);
    const int res = causal_resident<kernel()>(p, g, 64 * NW * kS.ks);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(64 * NW * kS.ks), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (const T*)O, (const T*)dO, L, (T*)dQ, Dv, (int)p.N, g.nRB, g.total, p.scale, p.causal, res,
                       group(p));
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}

template <typename T, int D, int NW> struct Pass1Small {
  static constexpr SetShape shape(int nw) { return set_shape<T, D>(nw, 4, 128 * nw, 8, Cfg<T, D>::kP1.occ); }
  static constexpr SetShape kS = shape(NW);
  // where no second set fits, four blocks are the whole-block shape itself and
  // not built here again
  static constexpr bool kBuilt = (NW != 4 || kS.ks > 1) && worth_building(kS, shape(2 * NW));
  static __host__ constexpr auto kernel() {
    if constexpr (kBuilt) return &bob_pass1_kernel<T, D, 1, NW, kS.occ, 2, kWithDQ, 1, Cfg<T, D>::kP1.pf, kS.ks>;
  }
  static Form form();
  static int32_t launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const void* UQ, const void* UK, const void* UV, const float* L, const float* Dv,
                        const void* dQ, void* Qt, void* dOt, float* alpha, float* E, hipStream_t s);
};
template <typename T, int D, int NW> Form Pass1Small<T, D, NW>::form() {
  constexpr int kThreads = 64 * NW * kS.ks;
  if constexpr (kBuilt) return {NW, kS.ks, resident_blocks<kernel()>(kThreads), kThreads, 1, 0.0, kP1Step<T>.narrow};
  else return {};
}
template <typename T, int D, int NW>
int32_t Pass1Small<T, D, NW>::launch(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                                     const void* dO, const void* UQ, const void* UK, const void* UV, const float* L,
                                     const float* Dv, const void* dQ, void* Qt, void* dOt, float* alpha, float* E,
                                     hipStream_t s) {
  if constexpr (kBuilt) {
    const Grid g = grid_for(p, 16 * NW);
    const int res = causal_resident<kernel()>(p, g, 64 * NW * kS.ks);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel(), dim3(g.total), dim3(64 * NW * kS.ks), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                       (const T*)O, (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, (const T*)dQ,
                       (const float*)nullptr, (T*)Qt, (T*)dOt, alpha, E, (int)p.N, g.nRB, g.total, p.scale, p.causal,
                       res, group(p));
    return finish_launch();
  }
  return BOB_EUNSUPPORTED;
}

// Built in fb_rows_small.hip, fb_pass1_small.hip and (Pass 1 at bf16 d = 128)
// fb_passes_d128.hip.
#define FB_ROWS_SMALL(EXT, T, D) \
  EXT template struct FwdWide<T, D>; EXT template struct RowsWide<T, D>; \
  EXT template struct FwdSmall<T, D, 4>; EXT template struct FwdSmall<T, D, 2>; EXT template struct FwdSmall<T, D, 1>; \
  EXT template struct RowsSmall<T, D, 4>; EXT template struct RowsSmall<T, D, 2>; EXT template struct RowsSmall<T, D, 1>;
#define FB_PASS1_SMALL(EXT, T, D) \
  EXT template struct Pass1Small<T, D, 4>; EXT template struct Pass1Small<T, D, 2>; EXT template struct Pass1Small<T, D, 1>;
FB_EACH_BUT_BF16_128(FB_ROWS_SMALL, extern)
FB_ROWS_SMALL(extern, bf16, 128)
FB_EACH_BUT_BF16_128(FB_PASS1_SMALL, extern)
FB_PASS1_SMALL(extern, bf16, 128)

// The form that each row kernel's launch takes (its place in the list; *chosen, may
// be null: the form).
template <typename T, int D> int fwd_form(const Problem& p, Form* chosen = nullptr) {
  constexpr Shape c = Cfg<T, D>::kFwd;
  constexpr auto whole = &attn_fwd_kernel<T, D, c.mr, c.nw, c.occ, c.st>;
  return pick_form(row_query<T>(p, 2, 1, kFwdStep<T>),
                   {{c.mr * c.nw, 1, resident_blocks<whole>(64 * c.nw), 64 * c.nw}, FwdSmall<T, D, 4>::form(),
                    FwdSmall<T, D, 2>::form(), FwdSmall<T, D, 1>::form(), FwdWide<T, D>::form()}, chosen);
}
template <typename T, int D> int bwd_rows_form(const Problem& p, Form* chosen = nullptr) {
  constexpr Shape c = Cfg<T, D>::kRows;
  constexpr auto whole = &attn_bwd_rows_kernel<T, D, c.mr, c.nw, c.occ, c.st>;
  return pick_form(row_query<T>(p, 3, 1, kRowsStep<T>),
                   {{c.mr * c.nw, 1, resident_blocks<whole>(64 * c.nw), 64 * c.nw}, RowsSmall<T, D, 4>::form(),
                    RowsSmall<T, D, 2>::form(), RowsSmall<T, D, 1>::form(), RowsWide<T, D>::form()}, chosen);
}
template <typename T, int D> int pass1_form(const Problem& p, Form* chosen) {  // the dQ form
  constexpr Shape c = Cfg<T, D>::kP1;
  constexpr auto whole = &bob_pass1_kernel<T, D, c.mr, c.nw, c.occ, c.st, kWithDQ, c.ds, c.pf>;
  return pick_form(row_query<T>(p, 10, 3, kP1Step<T>),
                   {{c.mr * c.nw, 1, resident_blocks<whole>(64 * c.nw), 64 * c.nw}, Pass1Small<T, D, 4>::form(),
                    Pass1Small<T, D, 2>::form(), Pass1Small<T, D, 1>::form()}, chosen);
}
extern template int pass1_form<bf16, 128>(const Problem&, Form*);  // built in fb_passes_d128.hip, with its kernel

template <typename T, int D>
int32_t launch_fwd(const Problem& p, const void* Q, const void* K, const void* V, void* O, float* L,
                   hipStream_t s) {
  constexpr Shape c = Cfg<T, D>::kFwd;
  constexpr auto kernel = &attn_fwd_kernel<T, D, c.mr, c.nw, c.occ, c.st>;
  switch (fwd_form<T, D>(p)) {
    case 1: return FwdSmall<T, D, 4>::launch(p, Q, K, V, O, L, s);
    case 2: return FwdSmall<T, D, 2>::launch(p, Q, K, V, O, L, s);
    case 3: return FwdSmall<T, D, 1>::launch(p, Q, K, V, O, L, s);
    case 4: return FwdWide<T, D>::launch(p, Q, K, V, O, L, s);
  }
  const Grid g = grid_for(p, 16 * c.mr * c.nw);
  const int res = causal_resident<kernel>(p, g, 64 * c.nw);
  (void)hipGetLastError();
  hipLaunchKernelGGL(kernel, dim3(g.total), dim3(64 * c.nw), 0, s,
                     (const T*)Q, (const T*)K, (const T*)V, (T*)O, L, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p));
  return finish_launch();
}

// Adds the parts of a split column kernel: x times p.scale and y times y_scale.
// Launched right after the split kernel, whose launch error finish_launch() here
// still sees.  Built in flashbob.hip.
template <typename T>
int32_t launch_parts_reduce(const Problem& p, int parts, const float* ws, float y_scale, void* x, void* y,
                            hipStream_t s) {
  const int64_t plane = p.B * p.Hkv * p.N * p.d;
  const int blocks = (int)std::min<int64_t>((plane / 2 + 255) / 256, 4096);
  hipLaunchKernelGGL((bob_column_parts_reduce_kernel<T>), dim3(blocks), dim3(256), 0, s, ws, parts, plane, p.scale,
                     y_scale, (T*)x, (T*)y);
  return finish_launch();
}
extern template int32_t launch_parts_reduce<bf16>(const Problem&, int, const float*, float, void*, void*, hipStream_t);
extern template int32_t launch_parts_reduce<float>(const Problem&, int, const float*, float, void*, void*, hipStream_t);

template <typename T, int D, bool kF>
int32_t launch_bwd_cols(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                        const float* L, const float* Dv, void* dK, void* dV, hipStream_t s, const ColumnPlan& cp,
                        float* parts_ws) {
  constexpr Shape cc = ColumnShape<T, D, false, kF>::kS;
  if constexpr (cc.mr == 0) {
    return BOB_EUNSUPPORTED;
  } else {
    const Grid& gc = cp.g;
    switch (cp.narrow) {
      case 4: return ColsSmall<T, D, 4>::launch(p, Q, K, V, dO, L, Dv, dK, dV, s);
      case 2: return ColsSmall<T, D, 2>::launch(p, Q, K, V, dO, L, Dv, dK, dV, s);
      case 1: return ColsSmall<T, D, 1>::launch(p, Q, K, V, dO, L, Dv, dK, dV, s);
    }
    (void)hipGetLastError();
    if (cp.parts > 1) {
      // each column block split over cp.parts workgroups, then one reduction
      hipLaunchKernelGGL((parts_kernel<T, D, false, kF>()), dim3(gc.total * cp.parts), dim3(64 * cc.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                         (const T*)dO, L, Dv, (T*)dK, (T*)dV, (int)p.N, gc.nRB, gc.total, p.scale, p.causal,
                         0, group(p), parts_ws, cp.parts, cp.flush_tiles);
      return launch_parts_reduce<T>(p, cp.parts, parts_ws, 1.0f, dK, dV, s);
    }
    auto cols = [&](auto gqa, auto ks) {
      constexpr auto kernel = &attn_bwd_cols_kernel<T, D, cc.mr, cc.nw, cc.occ, cc.st, decltype(gqa)::value,
                                                    decltype(ks)::value, false, kF, cc.kl != 0>;
      const int res = causal_resident<kernel>(p, gc, 64 * cc.nw * decltype(ks)::value);
      (void)hipGetLastError();
      hipLaunchKernelGGL(kernel, dim3(gc.total), dim3(64 * cc.nw * decltype(ks)::value), 0, s, (const T*)Q, (const T*)K,
                         (const T*)V, (const T*)dO, L, Dv, (T*)dK, (T*)dV, (int)p.N, gc.nRB, gc.total, p.scale,
                         p.causal, res, group(p), (float*)nullptr, 1, cp.flush_tiles);
    };
    const bool gqa = group(p) != 1;
    if constexpr (ColumnShape<T, D, false, kF>::kTwoFit) {
      if (cp.sets == 2) {
        gqa ? cols(std::true_type{}, std::integral_constant<int, 2>{})
            : cols(std::false_type{}, std::integral_constant<int, 2>{});
        return finish_launch();
      }
    }
    gqa ? cols(std::true_type{}, std::integral_constant<int, 1>{})
        : cols(std::false_type{}, std::integral_constant<int, 1>{});
    return finish_launch();
  }
}

template <typename T, int D>
int32_t launch_bwd_rows(const Problem& p, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* L, void* dQ, float* Dv, hipStream_t s) {
  constexpr Shape cr = Cfg<T, D>::kRows;
  constexpr auto rows = &attn_bwd_rows_kernel<T, D, cr.mr, cr.nw, cr.occ, cr.st>;
  switch (bwd_rows_form<T, D>(p)) {
    case 1: return RowsSmall<T, D, 4>::launch(p, Q, K, V, O, dO, L, dQ, Dv, s);
    case 2: return RowsSmall<T, D, 2>::launch(p, Q, K, V, O, dO, L, dQ, Dv, s);
    case 3: return RowsSmall<T, D, 1>::launch(p, Q, K, V, O, dO, L, dQ, Dv, s);
    case 4: return RowsWide<T, D>::launch(p, Q, K, V, O, dO, L, dQ, Dv, s);
  }
  const Grid gr = grid_for(p, 16 * cr.mr * cr.nw);
  const int res = causal_resident<rows>(p, gr, 64 * cr.nw);
  (void)hipGetLastError();
  hipLaunchKernelGGL(rows, dim3(gr.total), dim3(64 * cr.nw), 0, s,
                     (const T*)Q, (const T*)K, (const T*)V, (const T*)O, (const T*)dO, L, (T*)dQ, Dv,
                     (int)p.N, gr.nRB, gr.total, p.scale, p.causal, res, group(p));
  return finish_launch();
}

// The first backward: the row kernel (dQ, D), then the column kernel (dK, dV)
// laid out by `cp` (plan_columns<T, D, false>); parts_ws is the caller's
// workspace when cp.parts > 1.
template <typename T, int D>
int32_t launch_bwd(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                   const void* dO, const float* L, void* dQ, void* dK, void* dV, float* Dv,
                   hipStream_t s, const ColumnPlan& cp, float* parts_ws) {
  const int32_t rc = launch_bwd_rows<T, D>(p, Q, K, V, O, dO, L, dQ, Dv, s);
  if (rc != BOB_OK) return rc;
  if (cp.flush_tiles > 0)
    return launch_bwd_cols<T, D, true>(p, Q, K, V, dO, L, Dv, dK, dV, s, cp, parts_ws);
  return launch_bwd_cols<T, D, false>(p, Q, K, V, dO, L, Dv, dK, dV, s, cp, parts_ws);
}


template <typename T, int D>
int32_t launch_pass1(const Problem& p, const void* Q, const void* K, const void* V, const void* O,
                     const void* dO, const void* UQ, const void* UK, const void* UV, const float* L,
                     const float* Dv, const void* dQ, void* Qt, void* dOt, float* alpha, float* E,
                     hipStream_t s) {
  if (dQ != nullptr) {
    constexpr Shape c = Cfg<T, D>::kP1;
    constexpr auto kernel = &bob_pass1_kernel<T, D, c.mr, c.nw, c.occ, c.st, kWithDQ, c.ds, c.pf>;
    switch (pass1_form<T, D>(p, nullptr)) {
      case 1: return Pass1Small<T, D, 4>::launch(p, Q, K, V, O, dO, UQ, UK, UV, L, Dv, dQ, Qt, dOt, alpha, E, s);
      case 2: return Pass1Small<T, D, 2>::launch(p, Q, K, V, O, dO, UQ, UK, UV, L, Dv, dQ, Qt, dOt, alpha, E, s);
      case 3: return Pass1Small<T, D, 1>::launch(p, Q, K, V, O, dO, UQ, UK, UV, L, Dv, dQ, Qt, dOt, alpha, E, s);
    }
    const Grid g = grid_for(p, 16 * c.mr * c.nw);
    const int res = causal_resident<kernel>(p, g, 64 * c.nw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel, dim3(g.total, c.ds), dim3(64 * c.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (const T*)O,
                       (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, (const T*)dQ,
                       (const float*)nullptr, (T*)Qt, (T*)dOt, alpha, E, (int)p.N, g.nRB, g.total, p.scale,
                       p.causal, res, group(p));
  } else {
    constexpr Shape c = Cfg<T, D>::kP1Six;
    const Grid g = grid_for(p, 16 * c.mr * c.nw);
    constexpr auto kernel = &bob_pass1_kernel<T, D, c.mr, c.nw, c.occ, c.st, kSixAcc, c.ds, c.pf>;
    const int res = causal_resident<kernel>(p, g, 64 * c.nw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(kernel, dim3(g.total, c.ds), dim3(64 * c.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (const T*)O,
                       (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, (const T*)nullptr,
                       (const float*)nullptr, (T*)Qt, (T*)dOt, alpha, E, (int)p.N, g.nRB, g.total, p.scale,
                       p.causal, res, group(p));
  }
  return finish_launch();
}

// Three-pass control schedule: the alpha-only sweep and the second row sweep.
template <typename T, int D>
int32_t launch_alpha3(const Problem& p, const void* Q, const void* K, const void* UQ, const void* UK,
                      const float* L, float* alpha, hipStream_t s) {
  constexpr Shape c = Cfg<T, D>::kAlpha;
  const Grid g = grid_for(p, 16 * c.mr * c.nw);
  constexpr auto kernel = &bob3_alpha_kernel<T, D, c.mr, c.nw, c.occ, c.st>;
  const int res = causal_resident<kernel>(p, g, 64 * c.nw);
  (void)hipGetLastError();
  hipLaunchKernelGGL(kernel, dim3(g.total), dim3(64 * c.nw), 0, s,
                     (const T*)Q, (const T*)K, (const T*)UQ, (const T*)UK, L, alpha, (int)p.N, g.nRB, g.total,
                     p.scale, p.causal, res, group(p));
  return finish_launch();
}

template <typename T, int D>
int32_t launch_rows3(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                     const void* UQ, const void* UK, const void* UV, const float* L, const float* Dv,
                     const float* alpha, void* Qt, void* dOt, float* E, hipStream_t s) {
  constexpr Shape c = Cfg<T, D>::kP1;
  const Grid g = grid_for(p, 16 * c.mr * c.nw);
  constexpr auto kernel = &bob_pass1_kernel<T, D, c.mr, c.nw, c.occ, c.st, kAlphaGiven, c.ds, c.pf>;
  const int res = causal_resident<kernel>(p, g, 64 * c.nw);
  (void)hipGetLastError();
  hipLaunchKernelGGL(kernel, dim3(g.total, c.ds), dim3(64 * c.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (const T*)nullptr,
                     (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, (const T*)nullptr, alpha,
                     (T*)Qt, (T*)dOt, (float*)nullptr, E, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p));
  return finish_launch();
}

template <typename T, int D, bool kF>
int32_t launch_pass2_form(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                          const void* UQ, const void* UK, const void* UV, const float* L, const float* Dv,
                          const float* alpha, const float* E, void* Kt, void* Vt, hipStream_t s,
                          const ColumnPlan& cp, float* parts_ws) {
  constexpr Shape c = ColumnShape<T, D, true, kF>::kS;
  if constexpr (c.mr == 0) {
    return BOB_EUNSUPPORTED;
  } else {
    const Grid& g = cp.g;
    switch (cp.narrow) {
      case 4: return Pass2Small<T, D, 4>::launch(p, Q, K, V, dO, UQ, UK, UV, L, Dv, alpha, E, Kt, Vt, s);
      case 2: return Pass2Small<T, D, 2>::launch(p, Q, K, V, dO, UQ, UK, UV, L, Dv, alpha, E, Kt, Vt, s);
      case 1: return Pass2Small<T, D, 1>::launch(p, Q, K, V, dO, UQ, UK, UV, L, Dv, alpha, E, Kt, Vt, s);
    }
    (void)hipGetLastError();
    if (cp.parts > 1) {
      // each column block split over cp.parts workgroups, then one reduction
      hipLaunchKernelGGL((parts_kernel<T, D, true, kF>()), dim3(g.total * cp.parts), dim3(64 * c.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V,
                         (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, alpha, E, (T*)Kt, (T*)Vt,
                         (int)p.N, g.nRB, g.total, p.scale, p.causal, 0, group(p), parts_ws, cp.parts,
                         cp.flush_tiles);
      return launch_parts_reduce<T>(p, cp.parts, parts_ws, p.scale, Kt, Vt, s);
    }
    const bool gqa = group(p) != 1;
    if constexpr (!kF && Cfg<T, D>::kP2W.mr > 0) {
      constexpr Shape w = Cfg<T, D>::kP2W;
      auto wide = [&](auto kv) {
        hipLaunchKernelGGL((bob_pass2_kernel<T, D, w.mr, w.nw, w.occ, w.st, decltype(kv)::value, 1, w.pf != 0>),
                           dim3(g.total), dim3(64 * w.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (const T*)dO,
                           (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, alpha, E, (T*)Kt, (T*)Vt, (int)p.N,
                           g.nRB, g.total, p.scale, p.causal, 0, group(p), (float*)nullptr, 1, 0);
      };
      if (cp.wide) {
        gqa ? wide(std::true_type{}) : wide(std::false_type{});
        return finish_launch();
      }
    }
    if constexpr (!kF && Cfg<T, D>::kP2P.mr > 0) {
      constexpr Shape q = Cfg<T, D>::kP2P;
      auto pairs = [&](auto kv) {
        constexpr auto kernel = &bob_pass2_pair_kernel<T, D, q.nw / 2, decltype(kv)::value>;
        const int res = causal_resident<kernel>(p, g, 64 * q.nw);
        (void)hipGetLastError();
        hipLaunchKernelGGL(kernel, dim3(g.total), dim3(64 * q.nw), 0, s, (const T*)Q, (const T*)K, (const T*)V, (const T*)dO,
                           (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, alpha, E, (T*)Kt, (T*)Vt, (int)p.N,
                           g.nRB, g.total, p.scale, p.causal, res, group(p));
      };
      if (cp.pairs) {
        gqa ? pairs(std::true_type{}) : pairs(std::false_type{});
        return finish_launch();
      }
    }
    auto pass2 = [&](auto gqa, auto ks) {
      constexpr auto kernel = &bob_pass2_kernel<T, D, c.mr, c.nw, c.occ, c.st, decltype(gqa)::value,
                                                decltype(ks)::value, c.pf != 0, false, kF>;
      const int res = causal_resident<kernel>(p, g, 64 * c.nw * decltype(ks)::value);
      (void)hipGetLastError();
      hipLaunchKernelGGL(kernel, dim3(g.total), dim3(64 * c.nw * decltype(ks)::value), 0, s, (const T*)Q, (const T*)K,
                         (const T*)V, (const T*)dO, (const T*)UQ, (const T*)UK, (const T*)UV, L, Dv, alpha, E,
                         (T*)Kt, (T*)Vt, (int)p.N, g.nRB, g.total, p.scale, p.causal, res, group(p), (float*)nullptr, 1,
                         cp.flush_tiles);
    };
    if constexpr (ColumnShape<T, D, true, kF>::kTwoFit) {
      if (cp.sets == 2) {
        gqa ? pass2(std::true_type{}, std::integral_constant<int, 2>{})
            : pass2(std::false_type{}, std::integral_constant<int, 2>{});
        return finish_launch();
      }
    }
    gqa ? pass2(std::true_type{}, std::integral_constant<int, 1>{})
        : pass2(std::false_type{}, std::integral_constant<int, 1>{});
    return finish_launch();
  }
}

// Pass 2 laid out by `cp` (plan_columns<T, D, true>); parts_ws is the
// caller's workspace when cp.parts > 1.
template <typename T, int D>
int32_t launch_pass2(const Problem& p, const void* Q, const void* K, const void* V, const void* dO,
                     const void* UQ, const void* UK, const void* UV, const float* L, const float* Dv,
                     const float* alpha, const float* E, void* Kt, void* Vt, hipStream_t s, const ColumnPlan& cp,
                     float* parts_ws) {
  if (cp.flush_tiles > 0)
    return launch_pass2_form<T, D, true>(p, Q, K, V, dO, UQ, UK, UV, L, Dv, alpha, E, Kt, Vt, s, cp, parts_ws);
  return launch_pass2_form<T, D, false>(p, Q, K, V, dO, UQ, UK, UV, L, Dv, alpha, E, Kt, Vt, s, cp, parts_ws);
}

// Built in fb_passes_d128.hip.
extern template int32_t launch_pass1<bf16, 128>(const Problem&, const void*, const void*, const void*, const void*,
                                                const void*, const void*, const void*, const void*, const float*,
                                                const float*, const void*, void*, void*, float*, float*, hipStream_t);
extern template int32_t launch_pass2<bf16, 128>(const Problem&, const void*, const void*, const void*, const void*,
                                                const void*, const void*, const void*, const float*, const float*,
                                                const float*, const float*, void*, void*, hipStream_t,
                                                const ColumnPlan&, float*);

}  // namespace fb
