// Variants of the XCD-resident kernel: bf16, the sums of the two products apart, plain cell (see wavefront_xcd.hip).
#define RNN_XR_DT 0
#define RNN_XR_KIND 0
#define RNN_XR_APART 1
#include "wavefront_xcd.hip"
