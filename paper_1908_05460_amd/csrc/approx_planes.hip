// Approximated filter gradient of layers (3x3, padding up to 1) on planes of up to 256 positions: the planes in LDS, as fp32.  (bf16: what the
// matrix-core forms do not take.)
//
// dW[k][c][tap] = sum over n of sum[n][k] * X[n][c][position(n, k) + tap].  A lane is an output channel, so that a map's position is
// an address of its lane: the nine taps are LDS reads at offsets that all lanes share, and nothing moves to scalar registers.  Four input channels lie
// side by side, a position 16 bytes, so that a read serves four multiply-adds; the rows share a column of zeros.  A wavefront has
// images and LDS of its own -- it copies its four channels' planes two images ahead, through registers -- so that no barrier stands
// between its loads and its multiply-adds; the wavefronts' sums are added in 64 bits at the end.
// Bound by the LDS reads, which meet in banks as the positions fall, and, with the few images of a wavefront, by the first loads' latency
// and the exchange at the end.  128 -> 128 @ 16x16, N = 128: 9.9 us (channels in planes of their own, a read for each
// multiply-add: 11.5; two tiles of output channels to a lane spill), 1.7 TB/s; VGG-19's two such layers 15.4 where the fused
// form, whose patches come from L2, took 47 with their selections, 8 here.  Whole calls, before and now: that layer 27.0, 17.7;
// 200 -> 150 @ 9x9, N = 60: 42.3, 13.8 (bf16 41.7, 14.0); 200 -> 200 @ 7x7, N = 100: 66.6, 13.9; 128 -> 256 @ 16x16, stride 2, N = 128: 39.5, 18.5.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace wgrad {

constexpr int kPlanesWaves = 8;

struct PlanesParams {
    const void *X[kMaxBatch];
    const int32_t *at[kMaxBatch];                    // [N][K]: byte offset of a map's window in a plane with its border
    const float *sum[kMaxBatch];
    float *out[kMaxBatch];                           // dW, or the partials of the batch chunks
    int N, C, K, HW;
    int pitch, plane;                                // positions of a row and of a plane with its border; rows begin with a zero
    int first;                                       // positions before the window of position (0, 0)
    int ctiles, ktiles, chunk_n;
    FastDiv d_w;
    float scale;
};

typedef float pl_f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float planes_value(float x) { return x; }
__device__ __forceinline__ float planes_value(uint16_t x) { return bf16_bits_to_float(x); }

template <bool BF16, int NL>
__device__ __forceinline__ void planes_body(const PlanesParams &p, pl_f4 *smem, int bid, int prob)
{
    constexpr int CW = 4;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // (the tiles of output channels that read the same part of X are neighbours on one XCD)
    const int y = bid >> 3, kt = y % p.ktiles, tile = (y / p.ktiles) * 8 + (bid & 7), ct = tile % p.ctiles, chunk = tile / p.ctiles;
    const int c0 = ct * CW, k0 = kt * 64;
    const int n_begin = chunk * p.chunk_n, n_end = min(n_begin + p.chunk_n, p.N);
    if (n_begin >= n_end) return;
    typedef std::conditional_t<BF16, uint16_t, float> elem;
    const elem *X = (const elem *)p.X[prob] + (size_t)c0 * p.HW;
    const int32_t *at = p.at[prob];
    const float *sum = p.sum[prob];
    const int per_wave = p.plane + 1;                // (the last one takes what lanes without a position write)
    pl_f4 *const mine = smem + wave * per_wave;
    for (int e = lane; e < per_wave; e += 64) mine[e] = pl_f4{};

    int src[NL], dst[NL], chan[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) chan[c] = min(c, p.C - 1 - c0) * p.HW;     // (beyond the last channel: that one again, not stored)
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int e = lane + 64 * u;
        uint32_t row, col;
        p.d_w.divmod(e, row, col);
        src[u] = e < p.HW ? e : 0;
        dst[u] = e < p.HW ? ((int)row + 1) * p.pitch + 1 + (int)col : p.plane;
    }
    const bool live = k0 + lane < p.K;
    const int ko = min(k0 + lane, p.K - 1);
    float acc[CW][9];
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[c][t] = 0.f;

    elem x[2][NL][CW];
    float s[2];
    int a[2];
    const size_t image = (size_t)p.C * p.HW;
    auto load = [&](auto set, int n) {               // (behind the chunk's last image: that one again, so that as many loads are in flight)
        constexpr int i = decltype(set)::value;
        const int nn = min(n, n_end - 1);
        const elem *from = X + nn * image;
#pragma unroll
        for (int u = 0; u < NL; ++u)
#pragma unroll
            for (int c = 0; c < CW; ++c) x[i][u][c] = (from + chan[c])[src[u]];
        a[i] = at[(size_t)nn * p.K + ko];
        s[i] = sum[(size_t)nn * p.K + ko];
    };
    auto step = [&](auto set, int n) {
        constexpr int i = decltype(set)::value;
#pragma unroll
        for (int u = 0; u < NL; ++u) mine[dst[u]] = pl_f4{planes_value(x[i][u][0]), planes_value(x[i][u][1]), planes_value(x[i][u][2]), planes_value(x[i][u][3])};
        const pl_f4 *const w = (const pl_f4 *)((const char *)(mine + p.first) + a[i]);
        const float sv = live ? s[i] : 0.f;
        load(set, n + 2 * kPlanesWaves);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        // (the border's zeros are multiplied, too: a sum that is not finite makes NaNs there, as in the definition)
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const pl_f4 v = w[r * p.pitch + t];
#pragma unroll
                for (int c = 0; c < CW; ++c) acc[c][3 * r + t] = fmaf(sv, v[c], acc[c][3 * r + t]);
            }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    int n = n_begin + wave;
    load(set0, n);
    load(set1, n + kPlanesWaves);
    for (; n < n_end; n += 2 * kPlanesWaves) {
        step(set0, n);
        if (n + kPlanesWaves < n_end) step(set1, n + kPlanesWaves);
    }

    // the wavefronts' sums, two input channels at a time
    constexpr int J = 18, RP = J | 1;
    float *red = (float *)smem, *out = p.out[prob] + ((size_t)chunk * p.K + k0) * p.C * 9;
#pragma unroll
    for (int h = 0; h < CW / 2; ++h) {
        const int entries = min(2, p.C - c0 - 2 * h) * 9;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) red[(wave * 64 + lane) * RP + j] = acc[2 * h + j / 9][j % 9];
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * J; e += 64 * kPlanesWaves) {
            const int k = e / J, j = e - k * J;
            double v = 0;
#pragma unroll
            for (int w = 0; w < kPlanesWaves; ++w) v += red[(w * 64 + k) * RP + j];
            if (k0 + k < p.K && j < entries) out[((size_t)k * p.C + c0 + 2 * h) * 9 + j] = (float)(v * p.scale);
        }
    }
}

struct PlanesMulti {
    int n;
    int begin[kRegsMultiMax + 1];
    int per_prob[kRegsMultiMax];
    PlanesParams p[kRegsMultiMax];
};
static_assert(sizeof(PlanesMulti) <= 4096, "kernel arguments");

template <bool BF16>
__global__ __launch_bounds__(64 * kPlanesWaves, 4) void approx_gather_planes(const PlanesMulti)
{
    extern __shared__ __attribute__((aligned(16))) pl_f4 planes_smem[];
    const PlanesMulti *mp = (const PlanesMulti *)__builtin_amdgcn_kernarg_segment_ptr();
    const int n = mp->n;
    int gi = 0;
    for (int i = 1; i < n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const PlanesParams &p = mp->p[gi];
    const int bid = (int)blockIdx.x - mp->begin[gi], prob = bid / mp->per_prob[gi], at = bid - prob * mp->per_prob[gi];
    if (p.HW <= 64) planes_body<BF16, 1>(p, planes_smem, at, prob);
    else planes_body<BF16, 4>(p, planes_smem, at, prob);
}

// ---- host ----
// Against the direct form, which reads a patch an entry from L2, from 350 000 (image, channel of X, channel of dY) on (60 -> 150 @ 9x9, N = 35 /
// 45 / 60: 14.1 / 13.5 / 15.3 us there, 14.9 / 13.4 / 13.6 here; 30 -> 200 @ 13x13, N = 60 / 100: 16.9 / 21.8, 16.5 / 19.5); against the fused one, which selects in the same launch,
// from 750 000 (128 -> 128 @ 16x16, N = 32: 10.4, 13.0; N = 48: 15.5, 14.3; 16 -> 128, N = 200: 14.4, 17.6), in bf16, whose maps stream in half the time, from a million (128 -> 128 @ 16x16, stride 2, N = 48: 12.9, 14.0; N = 64: 15.5,
// 14.9), and where three
// lanes of four have an output channel.  The LDS gather keeps its layers, planes that the form in registers does not take, which would be
// faster here (66 -> 300 @ 8x8, stride 2, N = 40: 25.1 us there, 14.5 here; 100 -> 200, N = 60: 20.6, 14.9; 64 -> 300 @ 6x6, N = 128: 28.0, 16.1): the
// line is not drawn by these.
bool planes_takes(const Geometry &g, const ApproxPlan &alt)
{
    if (g.R != 3 || g.S != 3 || g.ph > 1 || g.pw > 1 || alt.sx || alt.mm || alt.use_lds) return false;
    if (g.H * g.W > 256 || kPlanesWaves * 16l * ((g.H + 2l) * (g.W + 1) + 2) > 64 * 1024) return false;
    const double work = (double)g.N * g.C * g.K;
    if (alt.fused) return work >= (g.bf16 ? 1e6 : 750e3) && 4 * g.K >= 3 * ((g.K + 63) / 64 * 64);
    return work >= 350e3;
}

RegsPosition planes_position(const Geometry &g) { return RegsPosition{(g.W + 1) * g.sh * 16, g.sw * 16}; }

// (of one element type)
int planes_launch(const RegsItem *const *it, int n, hipStream_t st, CombineQueue *combine)
{
    if (n == 0) return WGRAD_OK;
    PlanesMulti m{};
    m.n = n;
    int blocks = 0, chunks[kRegsMultiMax];
    size_t lds = 0;
    // workgroups for two to a CU, shared out by the layers' work, as the workspace has room for their partial results
    double work = 0;
    for (int i = 0; i < n; ++i) work += (double)it[i]->g.N * it[i]->g.C * it[i]->g.K * it[i]->b.n;
    for (int i = 0; i < n; ++i) {
        const RegsItem &I = *it[i];
        const Geometry &g = I.g;
        PlanesParams &p = m.p[i];
        p.N = g.N; p.C = g.C; p.K = g.K; p.HW = g.H * g.W;
        p.pitch = g.W + 1; p.plane = (g.H + 2) * p.pitch + 1;
        p.first = (1 - g.ph) * p.pitch + 1 - g.pw;
        p.d_w = FastDiv(g.W);
        p.ctiles = (g.C + 3) / 4; p.ktiles = (g.K + 63) / 64;
        const double share = 512 * (double)g.N * g.C * g.K * I.b.n / work;
        int ch = (int)(share / ((double)p.ctiles * p.ktiles * I.b.n) + 0.5);
        // ... in no longer sums than the fused or direct form's (24 layers of 64 -> 64 @ 8x16, N = 1000, which would be one chunk each:
        // 1.55e-7 off and 310 us, so 1.0e-7 and 308; the fused form 1.23e-7)
        ch = std::max(ch, (g.N + kPlanesWaves * I.in_a_row - 1) / (kPlanesWaves * I.in_a_row));
        ch = std::max(1, std::min(std::min(ch, I.max_chunks), (g.N + kPlanesWaves - 1) / kPlanesWaves));
        p.chunk_n = (g.N + ch - 1) / ch;
        ch = chunks[i] = (g.N + p.chunk_n - 1) / p.chunk_n;
        p.scale = ch > 1 ? 1.0f : I.scale;
        for (int j = 0; j < kMaxBatch; ++j) {
            const int k = j < I.b.n ? j : 0;
            p.X[j] = I.b.X[k]; p.at[j] = I.at[k]; p.sum[j] = I.sum[k];
            p.out[j] = ch > 1 ? (float *)(I.part + k * I.stride) : I.b.dW[k];
        }
        lds = std::max(lds, (size_t)kPlanesWaves * std::max(16 * (p.plane + 1), 64 * 19 * 4));
        m.per_prob[i] = (p.ctiles * ch + 7) / 8 * 8 * p.ktiles;
        m.begin[i] = blocks;
        blocks += m.per_prob[i] * I.b.n;
    }
    m.begin[n] = blocks;
    if (it[0]->g.bf16) WGRAD_LAUNCH(approx_gather_planes<true>, dim3((unsigned)blocks), dim3(64 * kPlanesWaves), lds, st, m);
    else WGRAD_LAUNCH(approx_gather_planes<false>, dim3((unsigned)blocks), dim3(64 * kPlanesWaves), lds, st, m);
    int rc = launch_status();
    for (int i = 0; i < n && rc == WGRAD_OK; ++i)
        if (chunks[i] > 1)
            rc = launch_combine((const float *)it[i]->part, (long)(it[i]->stride / 4), chunks[i], it[i]->g.dw_elems(), it[i]->scale,
                                it[i]->b.dW, it[i]->b.n, st, combine);
    return rc;
}

}  // namespace wgrad
