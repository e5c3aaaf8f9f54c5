// Instantiations of the panel-fed matrix-core kernels (see qnn_gemm_panel_kernel.h, qnn_gemm_panel_wide_kernel.h).
#include "qnn_gemm_panel_kernel.h"
#include "qnn_gemm_panel_wide_kernel.h"

namespace qnn {
namespace panel {

KernelFn find_kernel(bool sign, bool narrow) {
    if (narrow) return sign ? gemm_panel_kernel<true, 2> : gemm_panel_kernel<false, 2>;
    return sign ? gemm_panel_kernel<true, 4> : gemm_panel_kernel<false, 4>;
}

KernelFn wide_kernel() { return panel_wide::gemm_panel_wide_kernel; }

}  // namespace panel
}  // namespace qnn
