// Instantiations of the panel-fed matrix-core kernels (see qnn_gemm_panel_kernel.h, qnn_gemm_panel_wide_kernel.h).
#include "qnn_gemm_panel_kernel.h"
#include "qnn_gemm_panel_wide_kernel.h"

namespace qnn {
namespace panel {

namespace {
template <bool kSign, int kRows>
KernelFn find(Shape t) {
    if (t == k128x256) return gemm_panel_kernel<kSign, 2, 4, kRows>;
    return t == k128x128 ? gemm_panel_kernel<kSign, 2, 2, kRows> : gemm_panel_kernel<kSign, 4, 4, kRows>;
}
}  // namespace
KernelFn find_kernel(bool sign, Shape t, bool whole) {
    if (whole) return sign ? find<true, kWholeRows>(t) : find<false, kWholeRows>(t);
    return sign ? find<true, kAnyRows>(t) : find<false, kAnyRows>(t);
}
MapFn map_kernel(Shape t) {
    if (t == k128x256) return gemm_map_kernel<2, 4>;
    return t == k128x128 ? gemm_map_kernel<2, 2> : gemm_map_kernel<4, 4>;
}
WideFn wide_kernel() { return panel_wide::gemm_panel_wide_kernel; }

}  // namespace panel
}  // namespace qnn
