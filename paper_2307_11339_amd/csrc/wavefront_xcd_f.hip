// Variants of the XCD-resident kernel: fp32, GRU with the reset gate before the product (see wavefront_xcd.hip).
#define RNN_XR_DT 1
#define RNN_XR_KIND 2
#include "wavefront_xcd.hip"
