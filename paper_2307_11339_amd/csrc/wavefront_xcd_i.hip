// Variants of the XCD-resident kernel: bf16, groups on all XCDs, plain cell (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 0
#define RNN_XR_WIDE 2
#include "wavefront_xcd.hip"
