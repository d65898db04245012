// Instantiation of the fused kernel for 256 threads per QP and up to 256 rows of
// the bordered KKT system.
// phases inlined into the kernels: 1024 QPs of n = 100 (factor in global memory)
// solve in 5.18 instead of 6.57 ms and their backward takes 2.51 instead of 2.91
// (24 QPs, one per CU: 2.80 and 1.03 instead of 3.01 and 1.09); at 512 threads
// inlining is slower (64 QPs of n = 256 forward and backward 18.9 -> 22.8 ms, 24
// solves of n = 128 3.55 -> 4.0 ms), so those instantiations keep separate phases
#define QPK_INLINE_PHASES
#include "qp_kernel_impl.hpp"

namespace qpk {
template hipError_t launch_t<256, 4>(const Params &, bool, size_t, int, hipStream_t);
}  // namespace qpk
