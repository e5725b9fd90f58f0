// Variants of the XCD-resident kernel: fp32, peephole and clipping terms (see wavefront_xcd.hip).
#define RNN_XR_DT 1
#define RNN_XR_KIND 1
#include "wavefront_xcd.hip"
