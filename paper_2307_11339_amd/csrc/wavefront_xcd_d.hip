// Variants of the XCD-resident kernel: fp32, plain cell (see wavefront_xcd.hip).
#define RNN_XR_DT 1
#define RNN_XR_KIND 0
#include "wavefront_xcd.hip"
