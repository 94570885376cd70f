// Instantiations of the any-shape matrix-core kernel: fp32 operands, payoffs and candidates in three bf16 parts.
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms6(int ks, int form, bool many)
{
    switch (ks) {
    case 1: return any_impl::any_kernel_form<6, 1>(form, many);
    case 2: return any_impl::any_kernel_form<6, 2>(form, many);
    case 3: return any_impl::any_kernel_form<6, 3>(form, many);
    case 4: return any_impl::any_kernel_form<6, 4>(form, many);
    case 6: return any_impl::any_kernel_form<6, 6>(form, many);
    case 8: return any_impl::any_kernel_form<6, 8>(form, many);
    }
    return nullptr;
}

}  // namespace bsse
