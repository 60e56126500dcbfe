// The bf16 d = 128 instances of the two BoB pass launchers (and so of their
// kernels), in a translation unit of their own so that the build can give it
// LLVM's iterative ILP machine scheduler (-amdgpu-sched-strategy=
// iterative-ilp).  Measured on gfx950 against the default scheduler, in
// interleaved runs on one device: Pass 1 3.7% and Pass 2 2.2% faster at
// d = 128, while the same scheduler made the forward 34% and the first
// backward 13% slower, and the d = 64 Pass 2 7-8% and the d = 256 passes far
// slower, so every other kernel stays in flashbob.hip with the default.  The
// small-grid forms of the two passes are built here too: against the default
// scheduler Pass 1 takes 30.0 us for 35.1 at B2 H4 N777, 150 for 163 at B1 H4 N4096
// and 211 for 266 at B1 H1 N8192 causal, Pass 2 26.7 for 27.9 at B2 H4 N777 and the
// same elsewhere.
#include "fb_launch.h"

namespace fb {

template int32_t launch_pass1<bf16, 128>(const Problem&, const void*, const void*, const void*, const void*,
                                         const void*, const void*, const void*, const void*, const float*,
                                         const float*, const void*, void*, void*, float*, float*, hipStream_t);
template int32_t launch_pass2<bf16, 128>(const Problem&, const void*, const void*, const void*, const void*,
                                         const void*, const void*, const void*, const float*, const float*,
                                         const float*, const float*, void*, void*, hipStream_t, const ColumnPlan&,
                                         float*);

template int pass1_form<bf16, 128>(const Problem&, Form*);
template int columns_resident<bf16, 128, true, false>(bool);
template int columns_resident<bf16, 128, true, true>(bool);
FB_PASS1_SMALL(, bf16, 128)
FB_PASS2_SMALL(, bf16, 128)

}  // namespace fb
