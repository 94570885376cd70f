// Instantiations of the any-shape matrix-core kernel: fp32 candidates in three bf16 parts against
// payoffs that are bf16 numbers.
#include "sweep_any_impl.h"

namespace bsse {

any_impl::any_kernel_t any_kernel_terms3(int ks, int form, bool many)
{
    switch (ks) {
    case 2: return any_impl::any_kernel_form<3, 2>(form, many);
    case 4: return any_impl::any_kernel_form<3, 4>(form, many);
    case 8: return any_impl::any_kernel_form<3, 8>(form, many);
    }
    return nullptr;
}

}  // namespace bsse
