// Layers of several kinds in one launch of the form of 16-bit pieces (exact_x3_kernel.hpp): the 16-wide tiles that a small network's
// layers take -- rows of whole pieces without a stride, with a column stride of two, and a first layer's few channels.  By
// themselves the strided and first layers of ResNet-20 were a launch of the fp32 matrix core's kernel, 24 us at N = 128 for a
// fourteenth of the work, which started when the other layers' launch had ended.  As workgroups of the one launch they run beside
// the others: ResNet-20 exact, N = 32 / 48 / 80 / 128: 44 / 53 / 76 / 100 us -> 30 / 38 / 57 / 80, every other layer, N = 80: 69 -> 56.
// The strided tiles take two fp16 pieces to a number: their staging registers leave no room for three pieces and their sums of
// their own beside two more workgroups on the CU (three bf16 pieces 230 registers; this kernel 160).  So do rows in sums too long
// for bf16 pieces (x3_flush).  Errors against 64 bits are 0.5 to 1.01 of the former launches' on every layer of ResNet-20, N = 40 to
// 128.
#include "exact_x3_kernel.hpp"

namespace wgrad {

namespace {
typedef X3Config<kX3Three, 16, 3, 3, 1, false, false, 16, 1, 2, 17, 33, 16> MixRows;
typedef X3Config<kX3Half, 16, 3, 3, 1, false, false, 16, 1, 2, 17, 33, 16> MixRowsLong;
typedef X3Config<kX3Half, 16, 3, 3, 2, false, false, 16, 1, 3, 17, 69, 16> MixStride;
typedef X3Config<kX3Three, 16, 1, 3, 1, false, false, 16, 1, 1, 17, 25, 7> MixFirst;

__global__ __launch_bounds__(kBlock, 3) void wgrad_exact_x3_mix(const X3Multi)
{
    extern __shared__ __align__(16) char x3_smem[];
    const X3Multi *mp = (const X3Multi *)__builtin_amdgcn_kernarg_segment_ptr();
    const int n = mp->n;
    int gi = 0;
    for (int i = 1; i < n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const int bid = (int)blockIdx.x - mp->begin[gi], nblk = mp->count[gi];
    if (bid >= nblk) return;
    const int first = mp->first[gi];
    const void *const *X = mp->X + first, *const *dY = mp->dY + first;
    float *const *out = mp->out + first;
    switch (mp->s[gi].body) {
        case 0: x3_body<MixRows>(mp->s[gi], X, dY, out, x3_smem, bid, nblk); break;
        case 1: x3_body<MixStride>(mp->s[gi], X, dY, out, x3_smem, bid, nblk); break;
        case 3: x3_body<MixRowsLong>(mp->s[gi], X, dY, out, x3_smem, bid, nblk); break;
        default: x3_body<MixFirst>(mp->s[gi], X, dY, out, x3_smem, bid, nblk); break;
    }
}
}  // namespace

int x3_mix_body(int variant) { return variant == 3 ? 0 : (variant == 5 ? 1 : (variant == 7 ? 2 : -1)); }
int x3_mix_lds()
{
    constexpr int a = MixRows::kLds, b = MixStride::kLds, c = MixFirst::kLds, d = MixRowsLong::kLds;
    static_assert(3 * (a > b ? a : b) <= 160 * 1024 && c <= a && d <= a, "three workgroups on a CU");
    return a > b ? a : b;
}
int x3_launch_mix(const X3Multi &m, int blocks, hipStream_t st) { return x3_launch(wgrad_exact_x3_mix, m, blocks, (size_t)x3_mix_lds(), st); }

}  // namespace wgrad
