// The GEMM kernels and their launch code (design notes: sdrop_gemm.hip).  Compiled once per operand type SDROP_T (F16,
// BF16) and group of kernels SDROP_PART, so that the groups build in parallel.
#include "gemm_launch.h"

namespace sdrop {
#if SDROP_PART == 0
template int dispatch_typed<FWD, SDROP_T>(bool, GemmParams &, hipStream_t);
#elif SDROP_PART == 1
template int dispatch_typed<DX, SDROP_T>(bool, GemmParams &, hipStream_t);
#elif SDROP_PART == 2
template int dispatch_typed<DW, SDROP_T>(bool, GemmParams &, hipStream_t);
template int fwd_seeded_typed<SDROP_T>(bool, const GemmParams &, hipStream_t);
#elif SDROP_PART == 4
template int fwd_dense_typed<SDROP_T>(const GemmParams &, hipStream_t);
#elif SDROP_PART == 5
template int bwd_gated_typed<SDROP_T>(bool, const GemmParams &, const GemmParams &, hipStream_t);
template int fwd_dw_typed<SDROP_T>(bool, const GemmParams &, const GemmParams &, hipStream_t);
#else
template int bwd_fused_typed<SDROP_T>(int, int, bool, bool, const GemmParams &, const GemmParams &, int, hipStream_t);
#endif
}  // namespace sdrop
