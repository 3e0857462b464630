// The one-piece (bf16) instantiations of the kernel in exact_x3_kernel.hpp.
#include "exact_x3_kernel.hpp"

namespace wgrad {

int x3_launch_bf16(int variant, const X3Multi &m, int blocks, size_t lds, hipStream_t st)
{
    switch (variant) {
#define X(ID, ...) case ID: return x3_launch(wgrad_exact_x3<X3Config<__VA_ARGS__>>, m, blocks, lds, st);
        WGRAD_X3_VARIANTS_BF16(X)
#undef X
        default: return WGRAD_UNSUPPORTED;
    }
}

}  // namespace wgrad
