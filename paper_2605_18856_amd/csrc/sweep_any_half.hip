// Instantiations of the any-shape matrix-core kernel: fp32 operands in two half-precision parts.
//
// Long rows are bound by the matrix pipe and the LDS reads of fragments beside the vector unit: three products of
// two parts (four for m <= 48) in place of six of three are half the matrix instructions and two thirds of the
// fragments (us, six and these: m = 60, n = 100, K = 20, 1000000 rows 1580 and 1070, 20000 rows 53 and 43; m = 128,
// n = 100, K = 10, 60000 rows 128 and 99; m = 128, n = 255, K = 4, 30000 rows 64 and 50; m = 45, n = 60, K = 20,
// 260000 rows 200 and 167; m = 64, n = 30, K = 12, 10000 rows 22 and 21).
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_half(int ks, int form, bool many)
{
    switch (ks) {
    case 3: return any_impl::any_kernel_half_form<3>(form, many);
    case 4: return any_impl::any_kernel_half_form<4>(form, many);
    case 6: return any_impl::any_kernel_half_form<6>(form, many);
    case 8: return any_impl::any_kernel_half_form<8>(form, many);
    }
    return nullptr;
}

}  // namespace bsse
