// The GEMM's kernels for 4-bit weights.
#include "qc_gemm_kernels.h"

namespace qc {
template hipError_t launch_gemm_kernel<4>(const GemmArgs &, qc_epilogue, qc_out, hipStream_t);
}
