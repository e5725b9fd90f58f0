// Variants of the XCD-resident kernel: bf16, the sums of the two products apart, peephole and clipping terms (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 1
#define RNN_XR_APART 1
#include "wavefront_xcd.hip"
