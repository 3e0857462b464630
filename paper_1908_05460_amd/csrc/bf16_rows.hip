// Host side of the row-after-row bf16 kernel: which shapes it takes, how the batch is cut, launches.
#include <algorithm>
#include <type_traits>

#include "bf16_rows_kernel.hpp"

namespace wgrad {

constexpr int kRowsMultiMax = 10;    // groups per launch
struct RowsMulti {
    int n;
    int begin[kRowsMultiMax + 1];    // first workgroup of each group (multiples of 8: the XCD numbering of a group
                                     // then starts on XCD 0); begin[n] = grid size
    int per_prob[kRowsMultiMax];     // workgroups per problem
    int nprob[kRowsMultiMax];
    int W[kRowsMultiMax];
    RowsParams p[kRowsMultiMax];
};
static_assert(sizeof(RowsMulti) <= 4096, "kernel arguments");

// The groups of a run as one grid: a workgroup looks its group up in the kernel arguments, read in place.
template <bool SPARSE>
__device__ __forceinline__ void rows_group(char *rows_smem)
{
    const RowsMulti *mp = (const RowsMulti *)__builtin_amdgcn_kernarg_segment_ptr();
    const int n = mp->n;
    int gi = 0;
    for (int i = 1; i < n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const int bid = (int)blockIdx.x - mp->begin[gi], per = mp->per_prob[gi], prob = bid / per;
    if (prob >= mp->nprob[gi]) return;
    const RowsParams &p = mp->p[gi];
    switch (mp->W[gi]) {
        case 4: rows_body<4, SPARSE>(p, rows_smem, bid - prob * per, per, prob); break;
        case 8: rows_body<8, SPARSE>(p, rows_smem, bid - prob * per, per, prob); break;
        case 16: rows_body<16, SPARSE>(p, rows_smem, bid - prob * per, per, prob); break;
        default:
            if constexpr (!SPARSE) rows_body<32, SPARSE>(p, rows_smem, bid - prob * per, per, prob);
            break;
    }
}
__global__ __launch_bounds__(kRowsThreads, 2) void wgrad_bf16_rows(const RowsMulti)
{
    extern __shared__ char rows_smem[];
    rows_group<false>(rows_smem);
}
// the approximated gradient, from the selections
__global__ __launch_bounds__(kRowsThreads, 2) void approx_bf16_rows(const RowsMulti)
{
    extern __shared__ char rows_smem[];
    rows_group<true>(rows_smem);
}

struct RowsItem {
    Geometry g;
    Batch b;
    char *part;                      // partial results of the first problem; the next problem's lie `stride` bytes on
    size_t stride;
    int max_chunks;
};
struct RowsQueue {
    bool sparse = false;             // approximated layers: dY[] of the batches are the maps' words
    SelectQueue *sel = nullptr;      // selections that must be issued before these launches
    float scale = 1.0f;
    int n = 0;
    RowsItem item[kRowsMultiMax];
};
RowsQueue *rows_queue_new() { return new RowsQueue; }
RowsQueue *rows_queue_new_sparse(SelectQueue *selects)
{
    RowsQueue *q = new RowsQueue;
    q->sparse = true; q->sel = selects;
    return q;
}
void rows_queue_delete(RowsQueue *q) { delete q; }

bool rows_takes(const Geometry &g)
{
    if (!g.bf16 || g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || g.ph != 1 || g.pw != 1 || g.K % kRowsTile) return false;
    if (g.H != g.W || (g.W != 4 && g.W != 8 && g.W != 16 && g.W != 32)) return false;
    return tune_int("WGRAD_ROWS", 1) && (long)g.N * g.H * g.W * 2 * std::max(g.C, g.K) < (1l << 31);
}

int rows_tiles(const Geometry &g) { return (g.K / kRowsTile) * ((g.C + kRowsTile - 1) / kRowsTile); }
static int rows_groups(const Geometry &g) { return (g.N + rows_images(g.W) - 1) / rows_images(g.W); }
long rows_blocks(const Geometry &g) { return (long)rows_groups(g) * (g.H / 4); }

// How the batches of `n` groups of layers, launched together, are cut: chunks[i] workgroups share the images of every tile
// of group i.  A workgroup has a CU to itself and takes block_us for each block of four rows; finer cuts fill the CUs more
// evenly and cost partial results.  life[i]: of a workgroup of group i, as cut.
static void rows_cut(const RowsItem *const *it, int n, bool sparse, int *chunks, double *life)
{
    const double block_us = sparse ? tune_int("WGRAD_ROWS_SPARSE_NS", 900) * 1e-3 : tune_int("WGRAD_ROWS_BLOCK_NS", 1600) * 1e-3, fixed_us = 9.0;
    static const double kShare[] = {1.5, 1.25, 1.1, 1.0, 0.9, 0.8, 0.67, 0.57, 0.5, 0.4, 0.33, 0.25, 0.2};
    double total = 0;
    for (int i = 0; i < n; ++i) total += (double)rows_blocks(it[i]->g) * rows_tiles(it[i]->g) * it[i]->b.n;
    double best = 1e30;
    for (const double share : kShare) {
        const double target = total / kNumCU * share;
        int now[kRowsMultiMax];
        double sorted[kRowsMultiMax], lf[kRowsMultiMax], partial = 0;
        long count[kRowsMultiMax];
        for (int i = 0; i < n; ++i) {
            const Geometry &g = it[i]->g;
            const int groups = rows_groups(g), nb = g.H / 4;
            int ch = (int)(groups * nb / target + 0.95);
            ch = std::max(1, std::min(ch, std::min(groups, it[i]->max_chunks)));
            const int per = (groups + ch - 1) / ch;
            ch = (groups + per - 1) / per;
            now[i] = ch;
            if (ch > 1) partial += (double)ch * g.dw_elems() * 4 * it[i]->b.n;
            lf[i] = fixed_us + per * nb * block_us;
            int j = i;
            for (; j > 0 && sorted[j - 1] < lf[i]; --j) { sorted[j] = sorted[j - 1]; count[j] = count[j - 1]; }
            sorted[j] = lf[i];
            count[j] = (long)ch * rows_tiles(g) * it[i]->b.n;
        }
        const double cost = makespan_us(kNumCU, sorted, count, n) + partial / 5e6 + (partial > 0 ? 3.0 : 0.0);
        if (cost < best) {
            best = cost;
            std::copy(now, now + n, chunks);
            std::copy(lf, lf + n, life);
        }
    }
}

int rows_flush(RowsQueue &q, hipStream_t st, CombineQueue *combine)
{
    if (q.n == 0) return WGRAD_OK;
    if (q.sel) {
        const int rc = select_flush(*q.sel, st);
        if (rc != WGRAD_OK) return rc;
    }
    const RowsItem *it[kRowsMultiMax];
    int chunks[kRowsMultiMax];
    for (int i = 0; i < q.n; ++i) it[i] = &q.item[i];
    const int n = q.n;
    q.n = 0;
    double life[kRowsMultiMax];
    rows_cut(it, n, q.sparse, chunks, life);
    int order[kRowsMultiMax];                        // longest workgroups first
    for (int i = 0; i < n; ++i) {
        int j = i;
        for (; j > 0 && life[order[j - 1]] < life[i]; --j) order[j] = order[j - 1];
        order[j] = i;
    }
    RowsMulti m{};
    m.n = n;
    int blocks = 0;
    for (int o = 0; o < n; ++o) {
        const RowsItem &I = *it[order[o]];
        const Geometry &g = I.g;
        RowsParams &p = m.p[o];
        const int ch = chunks[order[o]], groups = rows_groups(g);
        p.N = g.N; p.C = g.C; p.K = g.K;
        p.ctiles = (g.C + kRowsTile - 1) / kRowsTile; p.ktiles = g.K / kRowsTile;
        p.chunks = ch; p.chunk_n = (groups + ch - 1) / ch * rows_images(g.W);
        p.scale = ch > 1 ? 1.0f : q.scale;
        for (int j = 0; j < kMaxBatch; ++j) {
            const int k = j < I.b.n ? j : 0;
            p.X[j] = I.b.X[k]; p.dY[j] = I.b.dY[k];
            p.out[j] = ch > 1 ? (float *)(I.part + k * I.stride) : I.b.dW[k];
        }
        m.W[o] = g.W;
        m.nprob[o] = I.b.n;
        m.per_prob[o] = p.ktiles * p.ctiles * ch;
        m.begin[o] = blocks;
        blocks += (m.per_prob[o] * I.b.n + 7) / 8 * 8;
    }
    m.begin[n] = blocks;
    if (hipFuncSetAttribute(q.sparse ? (const void *)approx_bf16_rows : (const void *)wgrad_bf16_rows, hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds) != hipSuccess)
        return WGRAD_LAUNCH_FAILED;
    if (q.sparse) WGRAD_LAUNCH(approx_bf16_rows, dim3((unsigned)blocks), dim3(kRowsThreads), kRowsLds, st, m);
    else WGRAD_LAUNCH(wgrad_bf16_rows, dim3((unsigned)blocks), dim3(kRowsThreads), kRowsLds, st, m);
    int rc = launch_status();
    for (int i = 0; i < n && rc == WGRAD_OK; ++i)
        if (chunks[i] > 1)
            rc = launch_combine((const float *)it[i]->part, (long)(it[i]->stride / 4), chunks[i], it[i]->g.dw_elems(), q.scale, it[i]->b.dW,
                                it[i]->b.n, st, combine);
    return rc;
}

// One group of identical layers: its own launch, or (with a queue) collected for rows_flush.
int launch_rows(const Geometry &g, const Batch &b, int max_chunks, void *ws, size_t stride, hipStream_t st, CombineQueue *defer,
                RowsQueue *queue)
{
    RowsQueue local;
    RowsQueue &q = queue ? *queue : local;
    if (q.n == kRowsMultiMax) {
        const int rc = rows_flush(q, st, defer);
        if (rc != WGRAD_OK) return rc;
    }
    q.item[q.n++] = RowsItem{g, b, (char *)ws, stride, max_chunks};
    return queue ? WGRAD_OK : rows_flush(local, st, defer);
}

// The same for the approximated gradient; b.dY: the maps' words, selected already (or recorded to be, in the queue's selections).
int launch_rows_sparse(const Geometry &g, const Batch &b, float scale, int max_chunks, void *part, size_t stride, hipStream_t st,
                       CombineQueue *defer, RowsQueue *queue)
{
    RowsQueue local;
    local.sparse = true;
    RowsQueue &q = queue ? *queue : local;
    q.scale = scale;                                 // (one for all layers of a run)
    const int rc = launch_rows(g, b, max_chunks, part, stride, st, defer, &q);
    return rc != WGRAD_OK || queue ? rc : rows_flush(local, st, defer);
}

}  // namespace wgrad
