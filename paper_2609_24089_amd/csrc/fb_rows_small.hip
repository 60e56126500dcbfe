// The row kernels' small-grid forms (wave sets, 16 to 64 query rows per
// workgroup) of the forward and the first backward, in a translation unit of
// their own to build beside the others.
#include "fb_launch.h"

namespace fb {
FB_EACH_BUT_BF16_128(FB_ROWS_SMALL, )
FB_ROWS_SMALL(, bf16, 128)
}  // namespace fb
