// Variants of the XCD-resident kernel: bf16, groups on two XCDs, plain cell (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 0
#define RNN_XR_WIDE 1
#include "wavefront_xcd.hip"
