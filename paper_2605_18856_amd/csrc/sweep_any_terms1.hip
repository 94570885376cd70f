// Instantiations of the any-shape matrix-core kernel: operands rounded to bf16 (bf16 storage).
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms1(int ks, int form)
{
    switch (ks) {
    case 1: return any_impl::any_kernel_form<1, 1>(form);
    case 2: return any_impl::any_kernel_form<1, 2>(form);
    case 3: return any_impl::any_kernel_form<1, 3>(form);
    case 4: return any_impl::any_kernel_form<1, 4>(form);
    case 6: return any_impl::any_kernel_form<1, 6>(form);
    case 8: return any_impl::any_kernel_form<1, 8>(form);
    }
    return nullptr;
}

}  // namespace bsse
