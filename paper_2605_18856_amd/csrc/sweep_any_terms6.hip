// Instantiations of the any-shape matrix-core kernel: fp32 operands, payoffs and candidates in three bf16 parts.
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms6(int ks, int form)
{
    switch (ks) {
    case 1: return any_impl::any_kernel_form<6, 1>(form);
    case 2: return any_impl::any_kernel_form<6, 2>(form);
    case 3: return any_impl::any_kernel_form<6, 3>(form);
    case 4: return any_impl::any_kernel_form<6, 4>(form);
    case 6: return any_impl::any_kernel_form<6, 6>(form);
    case 8: return any_impl::any_kernel_form<6, 8>(form);
    }
    return nullptr;
}

}  // namespace bsse
