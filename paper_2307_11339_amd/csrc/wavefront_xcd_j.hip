// Variants of the XCD-resident kernel: bf16, groups on all XCDs, peephole and clipping terms (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 1
#define RNN_XR_WIDE 2
#include "wavefront_xcd.hip"
