// Variants of the XCD-resident kernel: bf16, GRU with the reset gate before the product (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 2
#include "wavefront_xcd.hip"
