// The small-grid forms of Pass 1 (wave sets, 16 to 64 query rows per workgroup;
// bf16 d = 128 is in fb_passes_d128.hip), in a translation unit of their own to
// build beside the others.
#include "fb_launch.h"

namespace fb {
FB_EACH_BUT_BF16_128(FB_PASS1_SMALL, )
}  // namespace fb
