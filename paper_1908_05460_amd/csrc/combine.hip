// Reduction of partial results: dW[o] = scale * sum_j partial[j][o], for a table of tensors in
// one launch.  The split reductions of the exact kernel and the batch chunks of the approximated
// one both end here.
#include <algorithm>

#include "common.hpp"

namespace wgrad {

struct CombineTable {
    int n;
    int begin[kTableMax + 1];        // first workgroup of each tensor; begin[n] = grid size
    CombineItem item[kTableMax];
    unsigned char pl_log[kTableMax]; // log2 of the lanes that share one output; kVec4: one lane, four outputs
};
constexpr int kVec4 = 8;

// PL = 2^pl_log lanes share one output: lane pl adds partials pl, pl+PL, ... in ascending order,
// then the PL sub-sums are added in ascending pl through LDS -- a fixed order, so the result is
// deterministic.  PL > 1 spreads a long list of partials of a small tensor over more lanes.  The sums are kept in 64 bits,
// which the loads hide: what is left of the error is the partials' own (16 -> 16 @ 32x32, N = 128, 512 partials, exact:
// 1.49e-7 of the result's 2-norm -> 0.67e-7, 15.5 us both ways).
__global__ __launch_bounds__(kBlock) void combine_table(const CombineTable t)
{
    __shared__ double red[kBlock];
    int it = 0;
    for (int i = 1; i < t.n; ++i) it += (int)blockIdx.x >= t.begin[i];
    const CombineItem c = t.item[it];
    if (t.pl_log[it] == kVec4) {
        // large tensors: four consecutive outputs per lane, 16-byte accesses (elems % 4 == 0, pointers 16-byte aligned)
        const long o = ((long)((int)blockIdx.x - t.begin[it]) * kBlock + threadIdx.x) * 4;
        if (o >= c.elems) return;
        const float *__restrict__ part = c.part;
        double acc[4] = {0., 0., 0., 0.};
        int i = 0;
        for (; i + 3 < c.nparts; i += 4) {
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = *(const float4 *)(part + (long)(i + u) * c.elems + o);
#pragma unroll
            for (int u = 0; u < 4; ++u) { acc[0] += v[u].x; acc[1] += v[u].y; acc[2] += v[u].z; acc[3] += v[u].w; }
        }
        for (; i < c.nparts; ++i) {
            const float4 v = *(const float4 *)(part + (long)i * c.elems + o);
            acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
        }
        *(float4 *)(c.dW + o) = make_float4((float)(acc[0] * c.scale), (float)(acc[1] * c.scale), (float)(acc[2] * c.scale), (float)(acc[3] * c.scale));
        return;
    }
    const int lg = t.pl_log[it];
    const int PL = 1 << lg, OB = kBlock >> lg;          // outputs per workgroup
    const int ol = threadIdx.x & (OB - 1), pl = threadIdx.x >> (8 - lg);
    const long o = (long)((int)blockIdx.x - t.begin[it]) * OB + ol;
    const float *__restrict__ part = c.part;
    const long elems = c.elems;
    double acc = 0.;
    if (o < elems) {
        int i = pl;
        for (; i + 7 * PL < c.nparts; i += 8 * PL) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(long)(i + u * PL) * elems + o];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        for (; i < c.nparts; i += PL) acc += part[(long)i * elems + o];
    }
    if (lg == 0) {
        if (o < elems) c.dW[o] = (float)(acc * c.scale);
        return;
    }
    red[pl * OB + ol] = acc;
    __syncthreads();
    if (pl == 0 && o < elems) {
        double s = 0.;
        for (int q = 0; q < PL; ++q) s += red[q * OB + ol];
        c.dW[o] = (float)(s * c.scale);
    }
}

// log2 of the lanes that share an output: few outputs and many partials are spread over lanes
static int combine_lanes_log(long elems, int nparts)
{
    return elems <= 16 * 1024 && nparts >= 64 ? 4 : (elems <= 256 * 1024 && nparts >= 16 ? 2 : 0);
}

// additions in a row that the reduction of a tensor's partials makes
int combine_chain(long elems, int nparts)
{
    const int lg = combine_lanes_log(elems, nparts);
    return lg ? ((nparts - 1) >> lg) + 1 + (1 << lg) : nparts;
}

int combine_flush(CombineQueue &q, hipStream_t st)
{
    for (size_t first = 0; first < q.item.size(); first += kTableMax) {
        const int n = (int)std::min<size_t>(kTableMax, q.item.size() - first);
        CombineTable t{};
        t.n = n;
        int blocks = 0;
        for (int i = 0; i < n; ++i) {
            const CombineItem &c = q.item[first + i];
            int lg = combine_lanes_log(c.elems, c.nparts);
            int ob = kBlock >> lg;
            if (lg == 0 && c.elems >= 64 * 1024 && c.elems % 4 == 0 && ((uintptr_t)c.part % 16) == 0 && ((uintptr_t)c.dW % 16) == 0) {
                lg = kVec4;
                ob = kBlock * 4;
            }
            t.item[i] = c;
            t.pl_log[i] = (unsigned char)lg;
            t.begin[i] = blocks;
            blocks += (c.elems + ob - 1) / ob;
        }
        t.begin[n] = blocks;
        WGRAD_LAUNCH(combine_table, dim3((unsigned)blocks), dim3(kBlock), 0, st, t);
        if (launch_status() != WGRAD_OK) { q.item.clear(); return WGRAD_LAUNCH_FAILED; }
    }
    q.item.clear();
    return WGRAD_OK;
}

int launch_combine(const float *partials, long prob_stride, int nparts, long elems, float scale,
                   float *const *dW, int nprob, hipStream_t st, CombineQueue *defer)
{
    CombineQueue local;
    CombineQueue &q = defer ? *defer : local;
    if (elems >= (1l << 31)) return WGRAD_UNSUPPORTED;        // a table entry counts its elements in an int
    for (int i = 0; i < nprob; ++i)
        q.item.push_back(CombineItem{partials + i * prob_stride, dW[i], nparts, (int)elems, scale});
    return defer ? WGRAD_OK : combine_flush(local, st);
}

}  // namespace wgrad
