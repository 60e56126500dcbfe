// The column kernels' small-grid forms (16 to 64 key rows per workgroup in wave
// sets; Pass 2 at bf16 d = 128 is in fb_passes_d128.hip), in a translation unit of
// their own to build beside the others.
#include "fb_launch.h"

namespace fb {
FB_EACH_BUT_BF16_128(FB_COLS_SMALL, )
FB_COLS_SMALL(, bf16, 128)
FB_EACH_BUT_BF16_128(FB_PASS2_SMALL, )
}  // namespace fb
