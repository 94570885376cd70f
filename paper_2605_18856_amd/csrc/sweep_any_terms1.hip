// Instantiations of the any-shape matrix-core kernel: operands rounded to bf16 (bf16 storage).
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms1(int ks, int form, bool many)
{
    switch (ks) {
    case 1: return any_impl::any_kernel_form<1, 1>(form, many);
    case 2: return any_impl::any_kernel_form<1, 2>(form, many);
    case 3: return any_impl::any_kernel_form<1, 3>(form, many);
    case 4: return any_impl::any_kernel_form<1, 4>(form, many);
    case 6: return any_impl::any_kernel_form<1, 6>(form, many);
    case 8: return any_impl::any_kernel_form<1, 8>(form, many);
    }
    return nullptr;
}

}  // namespace bsse
