// One translation unit per nesting (-DNQ_INST_H=<h> -DNQ_INST_L=<l>) of the small-output GEMM / convolution.
#include "nq_gemm_slab.h"

namespace nq {
template void launch_nested_gemm_slab<NQ_INST_H, NQ_INST_L>(bool, const GemmParams &, int, hipStream_t, void *, void *);
}
