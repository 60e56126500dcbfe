// Which form of a kernel a launch runs, by estimated time.  Host code that depends
// on sizes alone (no HIP), so that a host compiler can build and test it.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <initializer_list>

namespace fb {

// The whole device, which the balanced causal order is laid out for: 8 XCDs, over
// which the dispatcher deals the workgroups in turn, of 32 compute units.
constexpr int kXCDs = 8;
constexpr int kCUsPerXCD = 32;

// A positive constant of the device that read() tells (0: it cannot be read now),
// kept in `known` once it has been read.  Threads that read it at once keep the same.
template <class F> int read_once(std::atomic<int>& known, F&& read) {
  int n = known.load(std::memory_order_relaxed);
  if (n <= 0 && (n = read()) > 0) known.store(n, std::memory_order_relaxed);
  return n;
}

// The `resident` argument of a causal grid's launch (`fit` workgroups of the kernel
// fit one of the device's `cus` compute units) if it is to run in the balanced order
// (map_block_causal), else 0 (heads one after another).  A grid of one round has a CU
// for every block, and on grids of many times the resident blocks the refills balance
// the load by themselves while blocks of one head in flight at a time share its
// streamed tiles in L2.  Measured on 270 kernels of causal problems, plain over
// balanced time: up to six multiples of the resident blocks 0.99 to 1.59, median 1.15;
// beyond eight, bf16 0.57 to 1.06, median 0.97 (fp32, whose tiles are reused longer,
// still gains there).  A part of a device (another CU count) keeps the plain order.
inline int balanced_order(int64_t total, int fit, int cus) {
  if (cus != kXCDs * kCUsPerXCD || total <= cus) return 0;
  return total <= (int64_t)6 * cus * fit ? fit : 0;
}

// One form of a kernel as pick_form() prices it: 16-row blocks per workgroup,
// wave sets, workgroups that fit one CU (0: not built), threads per workgroup,
// workgroups that split a block (column kernels) and what adding their parts takes,
// and what a block weighs in a step (more where it reads more LDS bytes per MFMA).
struct Form {
  int blocks = 0, sets = 1, resident = 0, threads = 256, parts = 1;
  double extra_us = 0, weight = 1;
};
// What the forms of one launch are chosen for: heads of N rows, each block
// streaming `tiles` tiles (all of them or, causal, up to the diagonal).
// One step (a streamed tile of every wave set on a CU) with n 16-row blocks takes
// base + per_block weight n times block_us (narrow: the weight of the narrow forms).
struct StepCost {
  double base, per_block, narrow;
};
struct FormQuery {
  int cus;  // compute units of the device
  int64_t heads, N, tiles;
  bool causal;
  double block_us;  // the tile contractions of one 16-row block at one CU's MFMA rate
  StepCost step;
  double merge_us;  // adding one more set's sums of one 16-row block at the end of a round
  double margin = 1.0;  // by which another unsplit form has to be faster than the whole blocks
};

// Estimated time of a kernel's forms.  Equal (dense) blocks cost the rounds of
// the fullest CU, causal ones the larger of the mean load and the heaviest
// block's steps; a step has at least the four 16-row blocks that occupy every
// SIMD, and kRound is a round's prologue and epilogue.  The constants (here, the
// steps' costs, the merge's and the margins) were fitted to 1380 shapes (N = 64 to
// 20000, 1 to 48 heads, both types, every head dim, dense and causal, grouped heads)
// timed in every form.  On 460 others the choice is 1% (Pass 1, dQ) to 2% (the rest)
// slower than the best form, and over 2% slower than the whole blocks at 1% of them,
// mostly calls of about 10 us.
// Measured, whole blocks -> chosen form (us), row kernels: bf16 B1 H1 N8192 d64
// causal forward 136 -> 34, Pass 1 206 -> 100; B1 H4 N4096 d128 dense 105 -> 48, 229
// -> 152; B2 H4 N777 d128 26 -> 13, 55 -> 33; fp32 B1 H1 N256 d64 14 -> 7, 46 -> 27.
// Column kernels, in sets: bf16 B1 H1 N256 d64 Pass 2 15 -> 7; B1 H12 N1024 d64
// causal 38 -> 21; split in parts: B1 H16 Hkv4 N4099 d128 causal Pass 2 606 -> 281,
// first backward 721 -> 277; B1 H8 Hkv1 N1024 d128 causal Pass 2 258 -> 51; fp32
// B1 H6 Hkv2 N700 d128 Pass 2 609 -> 101, first backward 347 -> 101.
// Returns the index of the form with the least time; 0 if the device is unknown.
// *chosen (may be null): that form.
inline int pick_form(const FormQuery& q, std::initializer_list<Form> forms, Form* chosen = nullptr) {
  constexpr double kRound = 4.0;
  if (chosen != nullptr) *chosen = *forms.begin();
  if (q.cus <= 0) return 0;
  int best = 0, i = -1;
  bool fills = false;
  double least = 0;
  for (const Form& f : forms) {
    ++i;
    if (f.resident == 0) continue;  // not built
    const int64_t total = q.heads * ((q.N + 16 * f.blocks - 1) / (16 * f.blocks)) * f.parts;
    // whole blocks that fill every slot of the device stay unless they are split
    // (bf16 B1 H20 N1800 d256 causal, 580 blocks in 512 slots: forward 64 us, 72 in
    // two sets)
    if (i == 0) fills = f.resident > 1 && total > q.cus * f.resident;
    // a launch takes fewer than 2^32 threads: 2^22 blocks of 1024, which 4 GB of bf16
    // d = 32 rows in 16-row blocks reach
    const bool launches = total <= INT32_MAX && total * f.threads <= (int64_t)UINT32_MAX;
    if (i > 0 && ((fills && f.parts == 1) || !launches)) continue;
    const int64_t shares = (int64_t)f.sets * f.parts;
    const double share = (double)((q.tiles + shares - 1) / shares);
    auto step = [&](int64_t workgroups) {
      const int64_t blocks = std::max<int64_t>(4, workgroups * f.blocks * f.sets);
      return q.block_us * (q.step.base + q.step.per_block * f.weight * (double)blocks);
    };
    const int64_t k = (total + q.cus - 1) / q.cus;  // workgroups of the fullest CU
    double t;
    if (q.causal) {
      const int64_t n = std::min<int64_t>(k, f.resident);
      const double mean = 0.5 * (share + 1) * total / (double)q.cus / n * step(n);
      t = std::max(mean, share * step(1));
    } else {
      t = share * ((double)(k / f.resident) * step(f.resident) + (k % f.resident != 0 ? step(k % f.resident) : 0));
    }
    t += (kRound + q.merge_us * f.blocks * (f.sets - 1)) * (double)((k + f.resident - 1) / f.resident);
    // splits cost what the estimate does not see (streams of several heads in flight,
    // the reduction's launch): they have to be clearly faster
    if (i > 0) t *= f.parts > 1 ? 1.08 : q.margin;
    t += f.extra_us;
    if (i == 0 || t < least) {
      best = i;
      least = t;
    }
  }
  if (chosen != nullptr) *chosen = forms.begin()[best];
  return best;
}

}  // namespace fb
