// C ABI of libflashbob.so: argument validation and kernel dispatch.
// The entry points are declared (and documented) in include/flashbob.h.
#include <atomic>
#include <type_traits>

#include "fb_launch.h"

namespace fb {

// Compute units of the current device, read from the runtime on every call
// (the library keeps no state of its own).
int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 0;
  return n;
}

// Dispatch on (dtype, d) to a templated function.
#define FB_DISPATCH(p, FN, ...)                                                  \
  do {                                                                           \
    if ((p).dtype == BOB_BF16 && (p).d == 32) return FN<fb::bf16, 32>(__VA_ARGS__);  \
    if ((p).dtype == BOB_BF16 && (p).d == 64) return FN<fb::bf16, 64>(__VA_ARGS__);  \
    if ((p).dtype == BOB_BF16 && (p).d == 128) return FN<fb::bf16, 128>(__VA_ARGS__); \
    if ((p).dtype == BOB_BF16 && (p).d == 256) return FN<fb::bf16, 256>(__VA_ARGS__); \
    if ((p).dtype == BOB_F32 && (p).d == 32) return FN<float, 32>(__VA_ARGS__);  \
    if ((p).dtype == BOB_F32 && (p).d == 64) return FN<float, 64>(__VA_ARGS__);  \
    if ((p).dtype == BOB_F32 && (p).d == 128) return FN<float, 128>(__VA_ARGS__); \
    return BOB_EUNSUPPORTED;                                                     \
  } while (0)

// Automatic choice for long blocks, from interleaved timing at B1 H16 N16384
// d128 bf16 with 1, 2, 4 and 16 key/value heads.  Causal: a column block's
// work grows with the query tiles at or below its diagonal, and splitting
// until there are about 8 jobs per CU made the heaviest block's share short
// enough to balance (Pass 2 and the first backward 1.3-2x faster with 1-4
// key/value heads; no gain with 16).  Dense Pass 2: blocks are equal, and the
// only gain was filling both workgroup slots of each CU on a grid smaller
// than the CU count (6% with one key/value head, against two wave sets in
// one workgroup).  The dense first backward gained from the same 8 jobs per
// CU as the causal one (9-18% with 1 and 4 key/value heads).
int resolve_parts(int workgroups, bool causal, bool pass2) {
  const int cus = device_cus();
  const bool fill_only = pass2 && !causal;
  if (workgroups <= 0 || cus <= 0 || (fill_only && workgroups > cus)) return 1;
  const int64_t target = (int64_t)(fill_only ? 2 : 8) * cus;
  const int64_t parts = (target + workgroups - 1) / workgroups;
  return parts < 2 ? 1 : (int)std::min<int64_t>(parts, kMaxParts);
}

// Automatic choice for blocks of kShortBlock up to kLongBlock iterations: the
// part count with the least estimated time.  Equal (dense) blocks cost the
// rounds of the fullest CU, where a partial round of n workgroups takes half of
// a full one and n / resident of the other half; causal blocks the larger of the mean load per CU and the
// heaviest block's share on a CU of its own; a split adds its parts' fp32 round
// trip through memory (at 4 TB/s) and a launch.  Two wave sets count as two
// workgroups of half the stream on one CU.  Measured, unsplit -> chosen (us): B1 H16 Hkv4
// N4099 d128 causal Pass 2 606 -> 281 (4 parts), first backward 721 -> 277 (8);
// dense 793 -> 610 (3), 877 -> 542 (3); B1 H8 Hkv1 N1024 d128 causal Pass 2
// 258 -> 51 (8); B1 H1 N8192 d64 causal Pass 2 230 -> 64 (8); B1 H4 N4096 d64
// Pass 2 121 -> 78 (4).  Below kShortBlock iterations a launch and the round
// trip cost about what the split gains (B2 H4 N777 d128, 25 iterations: 35 ->
// 31), and the causal B4 H12 grids at N = 2048 and 4096 (64 and 128) lost up to
// 14%.
int short_block_parts(const ColumnCost& c) {
  const int cus = device_cus();
  if (cus <= 0 || c.workgroups <= 0) return 1;
  // a round of n < resident workgroups on a CU, against a full round
  auto partial = [](int n, int resident) {
    return n == 0 ? 0.0 : 0.5 + 0.5 * n / resident;
  };
  auto cost = [&](int parts) {
    const int sets = parts == 1 && c.two_sets ? 2 : 1;
    const int resident = sets == 2 ? 2 : parts == 1 ? c.resident1 : c.resident;
    const double share = (double)((c.iters + parts * sets - 1) / (parts * sets));
    double t;
    if (c.causal) {
      const double mean = 0.5 * (1.0 + 1.0 / c.blocks) * c.iters * c.workgroups / ((double)cus * resident);
      t = std::max(mean, share * (sets < resident ? partial(sets, resident) : 1.0));
    } else {
      const int64_t k = ((int64_t)c.workgroups * parts + cus - 1) / cus * sets;
      t = share * ((double)(k / resident) + partial((int)(k % resident), resident));
    }
    t *= c.tile_us * resident;
    if (parts > 1) t += 4.0 + 16.0 * parts * (double)c.plane / 4e6;
    return t;
  };
  int best = 1;
  const double whole = cost(1);
  double least = 0.85 * whole;  // a split has to gain more than the estimate's error
  for (int parts = 2; parts <= kMaxParts; ++parts) {
    const double t = cost(parts);
    if (t < least) {
      best = parts;
      least = t;
    }
  }
  return best;
}

// Estimated time of a row kernel's forms.  A step (one streamed tile of every
// wave set on a CU) with n waves' worth of 16-row blocks takes 4.5 + 0.45 n times
// the MFMA time of one block, n at least the four that occupy every SIMD.  Equal
// (dense) blocks cost the rounds of the fullest CU, causal ones the larger of
// the mean load and the heaviest block's steps; kRound is a round's prologue,
// epilogue and merge of the sets.  The three constants were fitted to 37 shapes
// (N = 256 to 32768, 1 to 48 heads, both types, every head dim) timed in every
// form: the choice is on average 1.2% slower than the best form, and at most 23%.
// Measured, whole blocks -> chosen form (us): bf16 B1 H1 N8192 d64 causal forward
// 136 -> 34, Pass 1 206 -> 100; B1 H4 N4096 d128 dense 105 -> 48, 229 -> 152; B2
// H4 N777 d128 26 -> 13, 55 -> 33; fp32 B1 H1 N256 d64 14 -> 7, 46 -> 27.
int row_form(const Problem& p, int contractions, double rate, std::initializer_list<RowForm> forms) {
  constexpr int kCUs = kXCDs * kCUsPerXCD;
  constexpr double kRound = 4.0;
  const double block_us = 2.0 * contractions * 16 * kBS * (double)p.d / rate;  // one 16-row block, one tile
  const double tiles = (double)((p.N + kBS - 1) / kBS);
  int best = 0, i = -1;
  bool fills = false;
  double least = 0;
  for (const RowForm& f : forms) {
    ++i;
    if (f.resident == 0) continue;  // not built
    // whole blocks that fill every slot of the device stay (bf16 B1 H20 N1800
    // d256 causal, 580 blocks in 512 slots: forward 64 us, 72 in two sets)
    if (i > 0 && fills) break;
    const int64_t nRB = (p.N + 16 * f.blocks - 1) / (16 * f.blocks), total = p.B * p.H * nRB;
    if (i == 0) fills = f.resident > 1 && total > kCUs * f.resident;
    const double share = std::ceil(tiles / f.sets);
    auto step = [&](int64_t workgroups) {
      return block_us * (4.5 + 0.45 * std::max<int64_t>(4, workgroups * f.blocks * f.sets));
    };
    const int64_t k = (total + kCUs - 1) / kCUs;  // workgroups of the fullest CU
    double t;
    if (p.causal != 0) {
      const int64_t n = std::min<int64_t>(k, f.resident);
      const double mean = 0.5 * (share + 1) * total / (double)kCUs / n * step(n);
      t = std::max(mean, share * step(1));
    } else {
      t = share * ((double)(k / f.resident) * step(f.resident) + (k % f.resident != 0 ? step(k % f.resident) : 0));
    }
    t += kRound * (double)((k + f.resident - 1) / f.resident);
    if (i == 0 || t < least) {
      best = i;
      least = t;
    }
  }
  return best;
}

static ColumnOpts opts_of(const bob_column_opts* o) {
  ColumnOpts c;
  if (o != nullptr) {
    c.parts = o->parts;
    c.wave_sets = o->wave_sets;
    c.flush_tiles = o->flush_tiles;
  }
  return c;
}

// The plain (non-_ws) entry points never split a column block: they have no
// workspace.  Wave sets and sections are automatic.
constexpr ColumnOpts kUnsplit{1, 0, 0};

template <typename T, int D>
int32_t plan_bwd(const Problem& p, const ColumnOpts& o, ColumnPlan* c) {
  return plan_columns<T, D, false>(p, o, c);
}
template <typename T, int D>
int32_t plan_pass2(const Problem& p, const ColumnOpts& o, ColumnPlan* c) {
  return plan_columns<T, D, true>(p, o, c);
}

// Plan of a column kernel (pass2: Pass 2, else the first backward's) for a
// valid problem; an empty problem gets the trivial plan.
static int32_t column_plan(const Problem& p, bool pass2, const ColumnOpts& o, ColumnPlan* c) {
  bool empty;
  int32_t rc = check_problem(p, &empty);
  if (rc != BOB_OK) return rc;
  if (empty) {
    if (o.parts < 0 || o.parts > kMaxParts || o.wave_sets < 0 || o.wave_sets > 2 || o.flush_tiles < -1)
      return BOB_EINVAL;
    *c = ColumnPlan{};
    return BOB_OK;
  }
  if (pass2) FB_DISPATCH(p, plan_pass2, p, o, c);
  FB_DISPATCH(p, plan_bwd, p, o, c);
}

// The workspace checks of a *_ws entry point for a plan that splits.
static int32_t check_workspace(const Problem& p, const ColumnPlan& c, const void* ws, int64_t bytes) {
  if (c.parts <= 1) return BOB_OK;
  if (ws == nullptr || bytes < column_workspace_bytes(p, c.parts) || check_ptrs({ws}) != BOB_OK) return BOB_EINVAL;
  return BOB_OK;
}

static int32_t run_bwd(const Problem& p, const ColumnOpts& o, const void* Q, const void* K, const void* V,
                       const void* O, const void* dO, const float* L, void* dQ, void* dK, void* dV, float* D,
                       void* ws, int64_t ws_bytes, void* stream) {
  bool empty;
  int32_t rc = check_problem(p, &empty);
  if (rc != BOB_OK) return rc;
  ColumnPlan c;
  if ((rc = column_plan(p, false, o, &c)) != BOB_OK || empty) return rc;
  if ((rc = check_ptrs({Q, K, V, O, dO, L, dQ, dK, dV, D})) != BOB_OK) return rc;
  if ((rc = check_workspace(p, c, ws, ws_bytes)) != BOB_OK) return rc;
  FB_DISPATCH(p, launch_bwd, p, Q, K, V, O, dO, L, dQ, dK, dV, D, (hipStream_t)stream, c, (float*)ws);
}

static int32_t run_pass2(const Problem& p, const ColumnOpts& o, const void* Q, const void* K, const void* V,
                         const void* dO, const void* gdQ, const void* gdK, const void* gdV, const float* L,
                         const float* D, const float* alpha, const float* E, void* Kt, void* Vt, void* ws,
                         int64_t ws_bytes, void* stream) {
  bool empty;
  int32_t rc = check_problem(p, &empty);
  if (rc != BOB_OK) return rc;
  ColumnPlan c;
  if ((rc = column_plan(p, true, o, &c)) != BOB_OK || empty) return rc;
  if ((rc = check_ptrs({Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, E, Kt, Vt})) != BOB_OK) return rc;
  if ((rc = check_workspace(p, c, ws, ws_bytes)) != BOB_OK) return rc;
  FB_DISPATCH(p, launch_pass2, p, Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, E, Kt, Vt, (hipStream_t)stream, c,
              (float*)ws);
}

// Scratch of attn_bob_pass2_cols_gqa_noalloc, for callers that cannot
// allocate: the fp32 partial sums of a split Pass 2 (the *_ws workspace).
// Each device the library runs on holds its own copy until the process
// ends.  In host code `scratch` names a host-side stand-in, not device
// memory: kernels get the address hipGetSymbolAddress returns for the
// current device, read once per device and kept in scratch_dev.
constexpr int64_t kScratchBytes = int64_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
static std::atomic<void*> scratch_dev[kMaxDevices];

// Device address of `scratch` on the current device, or nullptr if it
// cannot be read.
static void* scratch_ptr() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* ptr = scratch_dev[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return nullptr;
    scratch_dev[dev].store(ptr, std::memory_order_release);   // the same address on every call
  }
  return ptr;
}

// The layout of Pass 2 with its workspace in `scratch`: as requested; when
// the part count is automatic and its workspace would not fit, the largest
// part count that fits (or none).  A forced part count that does not fit
// gives BOB_ESCRATCH.  Automatic splits here stay those of long blocks: calls
// that overlap race on the scratch buffer, so a call on short blocks, which
// callers may run on several streams at once, does not start to use it.
static int32_t noalloc_plan(const Problem& p, const ColumnOpts& o, ColumnPlan* c) {
  ColumnOpts long_only = o;
  long_only.min_iters = kLongBlock;
  int32_t rc = column_plan(p, true, long_only, c);
  if (rc != BOB_OK || column_workspace_bytes(p, c->parts) <= kScratchBytes) return rc;
  if (o.parts != 0) return BOB_ESCRATCH;
  const int64_t per_part = column_workspace_bytes(p, 2) / 2;
  const int fit = (int)std::min<int64_t>(kScratchBytes / per_part, kMaxParts);
  ColumnOpts capped = long_only;
  capped.parts = fit >= 2 ? std::min(fit, c->parts) : 1;
  return column_plan(p, true, capped, c);
}

}  // namespace fb

using fb::Problem;

extern "C" {

int32_t attn_fwd_lse(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale, int32_t causal,
                     const void* Q, const void* K, const void* V, void* O, float* L, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, H};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, V, O, L});
  if (rc != BOB_OK) return rc;
  FB_DISPATCH(p, fb::launch_fwd, p, Q, K, V, O, L, (hipStream_t)stream);
}

int32_t attn_bwd(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale, int32_t causal,
                 const void* Q, const void* K, const void* V, const void* O, const void* dO,
                 const float* L, void* dQ, void* dK, void* dV, float* D, void* stream) {
  return fb::run_bwd(Problem{dtype, B, H, N, d, scale, causal, H}, fb::kUnsplit, Q, K, V, O, dO, L, dQ, dK, dV, D,
                     nullptr, 0, stream);
}

int32_t attn_bob_pass1_rows(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale, int32_t causal,
                            const void* Q, const void* K, const void* V, const void* O,
                            const void* dO, const void* gdQ, const void* gdK, const void* gdV,
                            const float* L, const float* D, const void* dQ, void* Qt, void* dOt,
                            float* alpha, float* E, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, H};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, V, O, dO, gdQ, gdK, gdV, L, D, Qt, dOt, alpha, E});
  if (rc != BOB_OK) return rc;
  if (dQ != nullptr && !fb::aligned16(dQ)) return BOB_EINVAL;
  FB_DISPATCH(p, fb::launch_pass1, p, Q, K, V, O, dO, gdQ, gdK, gdV, L, D, dQ, Qt, dOt, alpha, E,
              (hipStream_t)stream);
}

int32_t attn_bob_pass2_cols(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale, int32_t causal,
                            const void* Q, const void* K, const void* V, const void* dO,
                            const void* gdQ, const void* gdK, const void* gdV, const float* L,
                            const float* D, const float* alpha, const float* E, void* Kt, void* Vt,
                            void* stream) {
  return fb::run_pass2(Problem{dtype, B, H, N, d, scale, causal, H}, fb::kUnsplit, Q, K, V, dO, gdQ, gdK, gdV, L,
                       D, alpha, E, Kt, Vt, nullptr, 0, stream);
}

// Grouped key/value heads: as above with Hkv key/value heads shared by the H
// query heads (H a multiple of Hkv).
int32_t attn_fwd_lse_gqa(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d, float scale,
                         int32_t causal, const void* Q, const void* K, const void* V, void* O, float* L,
                         void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, Hkv};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, V, O, L});
  if (rc != BOB_OK) return rc;
  FB_DISPATCH(p, fb::launch_fwd, p, Q, K, V, O, L, (hipStream_t)stream);
}

int32_t attn_bwd_gqa(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d, float scale,
                     int32_t causal, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                     const float* L, void* dQ, void* dK, void* dV, float* D, void* stream) {
  return fb::run_bwd(Problem{dtype, B, H, N, d, scale, causal, Hkv}, fb::kUnsplit, Q, K, V, O, dO, L, dQ, dK, dV,
                     D, nullptr, 0, stream);
}

int32_t attn_bob_pass1_rows_gqa(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                float scale, int32_t causal, const void* Q, const void* K, const void* V,
                                const void* O, const void* dO, const void* gdQ, const void* gdK,
                                const void* gdV, const float* L, const float* D, const void* dQ, void* Qt,
                                void* dOt, float* alpha, float* E, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, Hkv};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, V, O, dO, gdQ, gdK, gdV, L, D, Qt, dOt, alpha, E});
  if (rc != BOB_OK) return rc;
  if (dQ != nullptr && !fb::aligned16(dQ)) return BOB_EINVAL;
  FB_DISPATCH(p, fb::launch_pass1, p, Q, K, V, O, dO, gdQ, gdK, gdV, L, D, dQ, Qt, dOt, alpha, E,
              (hipStream_t)stream);
}

int32_t attn_bob_pass2_cols_gqa(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                float scale, int32_t causal, const void* Q, const void* K, const void* V,
                                const void* dO, const void* gdQ, const void* gdK, const void* gdV,
                                const float* L, const float* D, const float* alpha, const float* E, void* Kt,
                                void* Vt, void* stream) {
  return fb::run_pass2(Problem{dtype, B, H, N, d, scale, causal, Hkv}, fb::kUnsplit, Q, K, V, dO, gdQ, gdK, gdV,
                       L, D, alpha, E, Kt, Vt, nullptr, 0, stream);
}

int64_t bob_pass2_workspace_bytes(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                  int32_t causal, const bob_column_opts* opts) {
  const Problem p{dtype, B, H, N, d, 1.0f, causal, Hkv};
  fb::ColumnPlan c;
  return fb::column_plan(p, true, fb::opts_of(opts), &c) == BOB_OK ? fb::column_workspace_bytes(p, c.parts) : 0;
}

int64_t bob_bwd_workspace_bytes(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                int32_t causal, const bob_column_opts* opts) {
  const Problem p{dtype, B, H, N, d, 1.0f, causal, Hkv};
  fb::ColumnPlan c;
  return fb::column_plan(p, false, fb::opts_of(opts), &c) == BOB_OK ? fb::column_workspace_bytes(p, c.parts) : 0;
}

int32_t bob_column_layout(int32_t kernel, int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                          int32_t causal, const bob_column_opts* opts, bob_column_opts* resolved,
                          int64_t* workspace_bytes) {
  if (kernel != BOB_COLUMNS_BWD && kernel != BOB_COLUMNS_PASS2) return BOB_EINVAL;
  const Problem p{dtype, B, H, N, d, 1.0f, causal, Hkv};
  fb::ColumnPlan c;
  const int32_t rc = fb::column_plan(p, kernel == BOB_COLUMNS_PASS2, fb::opts_of(opts), &c);
  if (rc != BOB_OK) return rc;
  if (resolved != nullptr) {
    resolved->parts = c.parts;
    resolved->wave_sets = c.sets;
    resolved->flush_tiles = c.flush_tiles > 0 ? c.flush_tiles : -1;
  }
  if (workspace_bytes != nullptr) *workspace_bytes = fb::column_workspace_bytes(p, c.parts);
  return BOB_OK;
}

int32_t attn_bwd_gqa_ws(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d, float scale,
                        int32_t causal, const void* Q, const void* K, const void* V, const void* O, const void* dO,
                        const float* L, void* dQ, void* dK, void* dV, float* D, const bob_column_opts* opts,
                        void* workspace, int64_t workspace_bytes, void* stream) {
  return fb::run_bwd(Problem{dtype, B, H, N, d, scale, causal, Hkv}, fb::opts_of(opts), Q, K, V, O, dO, L, dQ, dK,
                     dV, D, workspace, workspace_bytes, stream);
}

int32_t attn_bob_pass2_cols_gqa_ws(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                   float scale, int32_t causal, const void* Q, const void* K, const void* V,
                                   const void* dO, const void* gdQ, const void* gdK, const void* gdV,
                                   const float* L, const float* D, const float* alpha, const float* E, void* Kt,
                                   void* Vt, const bob_column_opts* opts, void* workspace, int64_t workspace_bytes,
                                   void* stream) {
  return fb::run_pass2(Problem{dtype, B, H, N, d, scale, causal, Hkv}, fb::opts_of(opts), Q, K, V, dO, gdQ, gdK,
                       gdV, L, D, alpha, E, Kt, Vt, workspace, workspace_bytes, stream);
}

int32_t attn_bob_pass2_cols_gqa_noalloc(int32_t dtype, int64_t B, int64_t H, int64_t Hkv, int64_t N, int64_t d,
                                        float scale, int32_t causal, const void* Q, const void* K, const void* V,
                                        const void* dO, const void* gdQ, const void* gdK, const void* gdV,
                                        const float* L, const float* D, const float* alpha, const float* E,
                                        void* Kt, void* Vt, const bob_column_opts* opts, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, Hkv};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK) return rc;
  fb::ColumnPlan c;
  if ((rc = fb::noalloc_plan(p, fb::opts_of(opts), &c)) != BOB_OK || empty) return rc;
  if ((rc = fb::check_ptrs({Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, E, Kt, Vt})) != BOB_OK) return rc;
  float* ws = nullptr;
  if (c.parts > 1 && (ws = (float*)fb::scratch_ptr()) == nullptr) return BOB_ELAUNCH;
  FB_DISPATCH(p, fb::launch_pass2, p, Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, E, Kt, Vt, (hipStream_t)stream, c,
              ws);
}

int64_t bob_scratch_bytes(void) { return fb::kScratchBytes; }

int32_t attn_bob3_alpha_rows(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale,
                             int32_t causal, const void* Q, const void* K, const void* gdQ, const void* gdK,
                             const float* L, float* alpha, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, H};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, gdQ, gdK, L, alpha});
  if (rc != BOB_OK) return rc;
  FB_DISPATCH(p, fb::launch_alpha3, p, Q, K, gdQ, gdK, L, alpha, (hipStream_t)stream);
}

int32_t attn_bob3_rows(int32_t dtype, int64_t B, int64_t H, int64_t N, int64_t d, float scale, int32_t causal,
                       const void* Q, const void* K, const void* V, const void* dO, const void* gdQ,
                       const void* gdK, const void* gdV, const float* L, const float* D, const float* alpha,
                       void* Qt, void* dOt, float* E, void* stream) {
  const Problem p{dtype, B, H, N, d, scale, causal, H};
  bool empty;
  int32_t rc = fb::check_problem(p, &empty);
  if (rc != BOB_OK || empty) return rc;
  rc = fb::check_ptrs({Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, Qt, dOt, E});
  if (rc != BOB_OK) return rc;
  FB_DISPATCH(p, fb::launch_rows3, p, Q, K, V, dO, gdQ, gdK, gdV, L, D, alpha, Qt, dOt, E,
              (hipStream_t)stream);
}

int32_t bob_supported(int32_t dtype, int64_t d) {
  return fb::supported(dtype, d) ? 1 : 0;
}

const char* bob_status_string(int32_t status) {
  switch (status) {
    case BOB_OK: return "BOB_OK: success";
    case BOB_EINVAL: return "BOB_EINVAL: invalid argument (size, scale, dtype, or NULL/misaligned pointer)";
    case BOB_EUNSUPPORTED:
      return "BOB_EUNSUPPORTED: (dtype, head dim) not built; bf16 d = 32, 64, 128, 256; fp32 d = 32, 64, 128";
    case BOB_ELAUNCH: return "BOB_ELAUNCH: HIP kernel launch failed";
    case BOB_ESCRATCH:
      return "BOB_ESCRATCH: the requested layout needs more scratch than the library's static buffer "
             "(bob_scratch_bytes())";
    default: return "unknown bob_status";
  }
}

const char* bob_version(void) { return "flashbob-gfx950 0.2"; }


}  // extern "C"
