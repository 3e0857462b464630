// The exact filter gradient in 16-bit pieces (exact_x3_kernel.hpp) on 2x2 and 4x4 planes, position by position
// (fp32, 3x3 filters, stride 1, padding 1):
//
//     dW[k][c][r][s] = sum over positions p = (h, w) whose tap (r, s) lies inside X, q = (h + r - 1, w + s - 1), of
//                      G_pq[k][c],     G_pq[k][c] = sum_n dY[n][k][p] * X[n][c][q]
//
// The reduction of a G_pq runs over images, so an operand is "eight images of one position" and the (position, tap)
// pairs whose tap meets only padding are never multiplied: 100 of 144 are left on a 4x4 plane, 16 of 36 on a 2x2 plane.
// Matrix instructions and the staging's vector instructions (three to each with three pieces, five with two) take turns: the matrix
// core is busy 43 % of the cycles of VGG-19's launch with three pieces, 32 % with two, at 2.2 GHz, so a product left out is time saved.  512 -> 512 @ 4x4 takes 16.9 / 50 us at
// N = 16 / 128 with three bf16 pieces (the fp32 matrix core 28.8 / 72, the row form of exact_x3_kernel.hpp 63 at N = 128),
// 152 -> 101 us at N = 512 with two fp16 pieces, which long sums take (kX3HalfStages); 2x2 15.4 -> 45.7 us where the fp32 matrix
// core takes 49.7 (N = 512) and half of its time in a run of layers.
//
// A workgroup owns 64 output channels x 32 input channels; its four wavefronts share the taps out (13, 12, 12 and 15
// steps of a 4x4 plane's stage, 4 each of a 2x2 plane's; which wavefront has which changes with the workgroup), so that
// each holds the accumulators of its own two to four taps and nothing is added up across wavefronts.  A stage is 8
// images (4x4; the two lane groups of an operand take two positions of one tap) or 16 (2x2; they take two groups of
// images).  A thread loads four positions of one channel for eight images, 16 bytes each: a pair of images of one
// position is a word of each piece as it comes out of the split, so the transposition costs nothing.
#include <type_traits>

#include "exact_x3_kernel.hpp"

namespace wgrad {

namespace {

constexpr int kPK = 64, kPC = 32;                       // channels of the result tile

template <int HW, int KIND>
struct PlaneCfg {
    static constexpr int P = HW * HW, U = HW == 4 ? 16 : 8;            // positions; operand slots of a stage (2x2: position, image group)
    static constexpr int IMG = HW == 4 ? 8 : 16;                        // images of a stage
    static constexpr int kA = U * kPK * 16, kB = U * kPC * 16;          // bytes of one piece
    static constexpr bool HALF = KIND == kX3Half;
    static constexpr int NP = HALF ? 2 : 3;                             // pieces of a number
    static constexpr int kMark = HALF ? 4 * kBlock * 4 : 0;             // a bit for each of a thread's results
    static constexpr int kHead = 16 + (HALF ? (kPK + kPC) * 8 : 0) + kMark;     // flags; the channels' largest numbers and scales; those bits
    static constexpr int kLds = kHead + NP * (kA + kB);
};

// taps (r * 3 + s) of a role
template <int HW> constexpr int role_taps(int role, int i)
{
    constexpr int t4[4][4] = {{4, 0, -1, -1}, {1, 3, -1, -1}, {5, 7, -1, -1}, {2, 6, 8, -1}};
    constexpr int t2[4][4] = {{4, -1, -1, -1}, {1, 3, -1, -1}, {5, 7, -1, -1}, {0, 2, 6, 8}};
    return HW == 4 ? t4[role][i] : t2[role][i];
}
// i-th position whose tap lies inside X, or -1
template <int HW> constexpr int tap_position(int tap, int i)
{
    for (int p = 0; p < HW * HW; ++p) {
        const int h = p / HW + tap / 3 - 1, w = p % HW + tap % 3 - 1;
        if (h < 0 || h >= HW || w < 0 || w >= HW) continue;
        if (i-- == 0) return p;
    }
    return -1;
}
template <int HW> constexpr int tap_count(int tap)
{
    int n = 0;
    while (tap_position<HW>(tap, n) >= 0) ++n;
    return n;
}

template <int HW, int KIND, int ROLE>
struct PlaneRole {
    static constexpr int NT = (role_taps<HW>(ROLE, 0) >= 0) + (role_taps<HW>(ROLE, 1) >= 0) + (role_taps<HW>(ROLE, 2) >= 0) + (role_taps<HW>(ROLE, 3) >= 0);

    template <int T, int STEP>
    static __device__ __forceinline__ void step(x3_f16 (&acc)[NT][2], x3_f16 (&part)[2], const char *a0, const char *b0, int kk)
    {
        typedef PlaneCfg<HW, KIND> C;
        constexpr int tap = role_taps<HW>(ROLE, T), shift = (tap / 3 - 1) * HW + tap % 3 - 1;
        // operand slots of lane groups 0 and 1
        constexpr int p0 = tap_position<HW>(tap, HW == 4 ? 2 * STEP : STEP), p1 = HW == 4 ? tap_position<HW>(tap, 2 * STEP + 1) : p0;
        constexpr bool odd = p1 < 0;
        constexpr int q1 = odd ? p0 : p1;
        constexpr int ua0 = HW == 4 ? p0 : 2 * p0, ua1 = HW == 4 ? q1 : 2 * p0 + 1;
        constexpr int ub0 = HW == 4 ? p0 + shift : 2 * (p0 + shift), ub1 = HW == 4 ? q1 + shift : 2 * (p0 + shift) + 1;
        const char *const ap = a0 + (kk ? ua1 : ua0) * (kPK * 16), *const bp = b0 + (kk ? ub1 : ub0) * (kPC * 16);
        x3_u4 b[C::NP];
#pragma unroll
        for (int q = 0; q < C::NP; ++q) b[q] = *(const x3_u4 *)(bp + q * C::kB);
#pragma unroll
        for (int qa = C::NP - 1; qa >= 0; --qa) {
            x3_u4 a[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                a[m] = *(const x3_u4 *)(ap + qa * C::kA + m * 32 * 16);
                if (odd && kk) a[m] = x3_u4{0u, 0u, 0u, 0u};            // the last of an odd number of positions
            }
#pragma unroll
            for (int qb = C::NP - 1 - qa; qb >= 0; --qb)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    // Three pieces: the five smaller products of a stage's steps have a sum of their own, 2^-8 of the whole: it
                    // rounds that much finer, and the whole is rounded once a step instead of six times.  Two pieces: all
                    // products of a stage have, and the whole is rounded once a stage.
                    x3_mfma<KIND>(C::HALF || qa + qb ? part[m] : acc[T][m], a[m], b[qb]);
                }
        }
    }
    template <int T, int STEP>
    static __device__ __forceinline__ void steps(x3_f16 (&acc)[NT][2], x3_f16 (&part)[2], const char *a0, const char *b0, int kk, float sign)
    {
        constexpr int n = tap_count<HW>(role_taps<HW>(ROLE, T)), all = HW == 4 ? (n + 1) / 2 : n;
        if constexpr (STEP == 0) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int v = 0; v < 16; ++v) part[m][v] = 0.f;
        }
        step<T, STEP>(acc, part, a0, b0, kk);
        if constexpr (STEP + 1 < all) steps<T, STEP + 1>(acc, part, a0, b0, kk, sign);
        else {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[T][m][v] = KIND == kX3Half ? __builtin_fmaf(part[m][v], sign, acc[T][m][v]) : acc[T][m][v] + part[m][v];
            __builtin_amdgcn_sched_barrier(0);       // (across taps the scheduler's liking for early reads costs 67 spilled registers)
            if constexpr (T + 1 < NT) steps<T + 1, 0>(acc, part, a0, b0, kk, sign);
        }
    }

    // A stage's numbers themselves (eight images: four in the place of the first piece, four in the second's) on the fp32
    // matrix core, image by image.  Every position of dY takes part in every tap: one whose tap lies outside X meets a
    // zero there, which a NaN or infinity of dY makes a NaN of.
    template <int T>
    static __device__ __forceinline__ void plain_steps(x3_f16 (&acc)[NT][2], const char *a0, const char *b0, int kk)
    {
        typedef PlaneCfg<HW, KIND> C;
        constexpr int tap = role_taps<HW>(ROLE, T), dh = tap / 3 - 1, dw = tap % 3 - 1;
#pragma unroll 1
        for (int step = 0; step < (HW == 4 ? C::P / 2 : C::P); ++step) {
            const int p = HW == 4 ? 2 * step + kk : step, h = p / HW + dh, w = p % HW + dw;
            const bool here = h >= 0 && h < HW && w >= 0 && w < HW;
            const int q = here ? h * HW + w : p;
            const char *const ap = a0 + (HW == 4 ? p : 2 * p + kk) * (kPK * 16), *const bp = b0 + (HW == 4 ? q : 2 * q + kk) * (kPC * 16);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                float4_t b = *(const float4_t *)(bp + half * C::kB);
                if (!here) b = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const float4_t a = *(const float4_t *)(ap + half * C::kA + m * 32 * 16);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[T][m] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc[T][m], 0, 0, 0);
                }
            }
        }
        if constexpr (T + 1 < NT) plain_steps<T + 1>(acc, a0, b0, kk);
    }
};

template <int HW, int KIND, int ROLE>
__device__ __forceinline__ void planes_body(const X3Shape &p, const float *Xp, const float *dYp, float *out, char *smem, int k0, int c0,
                                            int st_begin, int st_end)
{
    typedef PlaneCfg<HW, KIND> C;
    typedef PlaneRole<HW, KIND, ROLE> R;
    const Geometry &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int i = lane & 31, kk = lane >> 5;
    uint32_t *const flag = (uint32_t *)smem;
    uint32_t *const over = flag + 1, *const asked = flag + 2, *const top = flag + 4;             // (see exact_x3_kernel.hpp; dY's channels, then X's)
    int *const expo = (int *)(top + kPK + kPC);
    char *const As = smem + C::kHead, *const Bs = As + C::NP * C::kA;

    // Staging items: (channel, four positions [4x4: a row of the plane], eight images).  4x4: every thread has one of dY and
    // half of one of X (four images); 2x2: 128 of dY, 64 of X, one for a thread.
    constexpr uint32_t kDead = 0x80000000u;
    constexpr int SETS = HW == 4 ? 2 : 1;
    uint32_t src[SETS], dst[SETS];                                      // byte offset of the first image's piece; LDS byte offset
    bool is_a[SETS];
    int first[SETS], chan[SETS];                                        // the item's first image in the stage; its row of `top`
    auto items = [&](int tid) {
#pragma unroll
        for (int u = 0; u < SETS; ++u) {
            int row, grp, half = 0;
            if (HW == 4) {
                is_a[u] = u == 0;
                row = u == 0 ? tid % kPK : tid % kPC;
                grp = u == 0 ? tid / kPK : tid / kPC & 3;                   // row of the plane
                half = u == 0 ? 0 : tid / (kPC * 4);
                first[u] = 4 * half;
            } else {
                is_a[u] = tid < 2 * kPK;
                const int f = is_a[u] ? tid : tid - 2 * kPK;
                row = is_a[u] ? f % kPK : f % kPC;
                grp = is_a[u] ? f / kPK : f / kPC;                          // group of eight images (2 and more: no item)
                first[u] = 8 * grp;
            }
            chan[u] = is_a[u] ? row : kPK + row;
            const bool live = HW == 4 || grp < 2;
            const int chans = is_a[u] ? g.K : g.C, rows = is_a[u] ? kPK : kPC;
            src[u] = live && (is_a[u] ? k0 : c0) + row < chans ? (uint32_t)((first[u] * chans + row) * C::P + (HW == 4 ? grp * 4 : 0)) * 4u : kDead;
            dst[u] = live ? (uint32_t)((is_a[u] ? 0 : C::NP * C::kA) + ((HW == 4 ? 4 * grp : grp) * rows + row) * 16 + 8 * half) : ~0u;
        }
    };
    items(tid);
    x3_u4 reg0[8], reg1[4];
    auto load = [&](int st) {
        const int n0 = st * C::IMG, left = g.N - n0;
        const auto ra = __builtin_amdgcn_make_buffer_rsrc((void *)(dYp + ((long)n0 * g.K + k0) * C::P), 0, kDead, 0x00020000);
        const auto rb = __builtin_amdgcn_make_buffer_rsrc((void *)(Xp + ((long)n0 * g.C + c0) * C::P), 0, kDead, 0x00020000);
        auto images = [&](auto &reg, int u, int count) {
            const uint32_t step = (uint32_t)((is_a[u] ? g.K : g.C) * C::P) * 4u;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (j >= count) break;
                const uint32_t off = src[u] != kDead && first[u] + j < left ? src[u] + j * step : kDead;
                if (is_a[u]) reg[j] = __builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0);
                else reg[j] = __builtin_amdgcn_raw_buffer_load_b128(rb, off, 0, 0);
            }
        };
        images(reg0, 0, 8);
        if constexpr (SETS > 1) images(reg1, 1, 4);
    };
    float scale[SETS];
#pragma unroll
    for (int u = 0; u < SETS; ++u) scale[u] = __builtin_inff();
    auto largest = [&](auto &reg, auto words) {
        float m = 0.f;
#pragma unroll
        for (int j = 0; j < 2 * decltype(words)::value; ++j)
#pragma unroll
            for (int q = 0; q < 4; q += 2)
                m = __builtin_fmaxf(__builtin_fmaxf(m, __builtin_fabsf(__uint_as_float(reg[j][q]))), __builtin_fabsf(__uint_as_float(reg[j][q + 1])));
        return m;
    };
    auto commit = [&](float sign, auto plain) {
        auto images = [&](auto &reg, int u, auto words) {
            constexpr int NW = decltype(words)::value;                  // words of a piece: pairs of images
            if (dst[u] == ~0u) return;
            const int rows = is_a[u] ? kPK : kPC, piece = is_a[u] ? C::kA : C::kB;
            const float by = (is_a[u] ? sign : 1.f) * x3_finite(scale[u]);
            if constexpr (decltype(plain)::value) {
                const int half = NW == 2 ? first[u] / 4 : 0;            // an item of four images is the first or the second four
#pragma unroll
                for (int h = 0; h < NW / 2; ++h)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(x3_u4 *)(As + dst[u] - 8 * half + (h + half) * piece + (HW == 4 ? q : 2 * q) * rows * 16) =
                            x3_u4{reg[4 * h][q], reg[4 * h + 1][q], reg[4 * h + 2][q], reg[4 * h + 3][q]};
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) {                          // position q of the item
                    typedef uint32_t words_t __attribute__((ext_vector_type(NW)));
                    words_t w[C::NP];
#pragma unroll
                    for (int e = 0; e < NW; ++e) {
                        const float x0 = __uint_as_float(reg[2 * e][q]), x1 = __uint_as_float(reg[2 * e + 1][q]);
                        uint32_t x, y, z;
                        if constexpr (C::HALF) x3_split2(x0, x1, by, x, y);
                        else x3_split3(x0, x1, kX3Scale, x, y, z);
                        w[0][e] = x; w[1][e] = y;
                        if constexpr (!C::HALF) w[2][e] = z;
                    }
#pragma unroll
                    for (int p = 0; p < C::NP; ++p) *(words_t *)(As + dst[u] + p * piece + (HW == 4 ? q : 2 * q) * rows * 16) = w[p];
                }
            }
        };
        images(reg0, 0, std::integral_constant<int, 4>{});
        if constexpr (SETS > 1) images(reg1, 1, std::integral_constant<int, 2>{});
    };

    load(st_begin);
    if (tid == 0) *flag = *over = *asked = 0;
    if constexpr (C::HALF) {
        if (tid < kPK + kPC) { top[tid] = 0; expo[tid] = kX3Unset; }
#pragma unroll
        for (int t = 0; t < R::NT; ++t) ((uint32_t *)(smem + C::kHead - C::kMark))[t * kBlock + tid] = 0;
        __syncthreads();
    }
    x3_f16 acc[R::NT][2];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < R::NT; ++t)
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[t][m][v] = 0.f;
    };
    clear();
    const char *const a0 = As + i * 16, *const b0 = Bs + i * 16;
    // Whether a result is known to be well held, a bit each (see exact_x3_kernel.hpp).  Here a wavefront has all of a result's products:
    // it looks at the sums after half of its stages, too.
    uint32_t *const mark = (uint32_t *)(smem + C::kHead - C::kMark);
    auto good = [&](int t) -> uint32_t & { return mark[t * kBlock + tid]; };
    auto weigh = [&](uint32_t (&good)[R::NT], const uint32_t *of, auto beyond) {
        const uint32_t nc = of[kPK + i];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            x3_u4 nk[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) nk[v] = *(const x3_u4 *)(of + m * 32 + 8 * v + 4 * kk);
#pragma unroll
            for (int v = 0; v < 16; ++v)
#pragma unroll
                for (int t = 0; t < R::NT; ++t)
                    good[t] = __builtin_amdgcn_alignbit(good[t], __float_as_uint(beyond(__builtin_fabsf(acc[t][m][v]), nk[v / 4][v % 4], nc)), 31);
        }
    };
    auto look = [&]() {
        uint32_t now[R::NT] = {};
        weigh(now, top, [](float sum, uint32_t row, uint32_t) { return (row == 0 ? -1.f : 2.f * kX3Need) - sum; });
        const uint32_t none = top[kPK + i] == 0 ? ~0u : 0u;
#pragma unroll
        for (int t = 0; t < R::NT; ++t) good(t) |= now[t] | none;
    };
    auto rescale = [&](float m0, float m1, bool sums) {                // (see exact_x3_kernel.hpp)
        auto note = [&](int u, float m) {
            if (m > 0.f) { const uint32_t b = __float_as_uint(m); atomicMax(top + chan[u], b < kX3Finite ? b : kX3Finite); }
        };
        note(0, m0);
        if constexpr (SETS > 1) note(1, m1);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SETS; ++u) scale[u] = x3_scale(top[chan[u]]);
        if (sums) {
            auto change = [&](int row) { return x3_exponent(top[row]) - expo[row]; };
            const int dc = change(kPK + i);
            uint32_t changed = 0;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int d = dc + change(m * 32 + 8 * (v / 4) + 4 * kk + v % 4);
#pragma unroll
                    for (int t = 0; t < R::NT; ++t) acc[t][m][v] = __builtin_ldexpf(acc[t][m][v], d);
                    changed = changed << 1 | (d != 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            // (what was large may be small in the new units)
#pragma unroll
            for (int t = 0; t < R::NT; ++t) good(t) &= ~changed;
            look();
        }
        __syncthreads();
        if (tid < kPK + kPC) expo[tid] = x3_exponent(top[tid]);
        if (tid == 0) *over = 0;
    };
    for (int st = st_begin; st < st_end; ++st) {
        if constexpr (C::HALF) {
            const float m0 = largest(reg0, std::integral_constant<int, 4>{}), m1 = SETS > 1 ? largest(reg1, std::integral_constant<int, 2>{}) : 0.f;
            X3Range r;
            r.item(m0, scale[0]);
            if constexpr (SETS > 1) r.item(m1, scale[1]);
            if (r.over()) *over = 1;
            __syncthreads();
            if (*(volatile uint32_t *)over) rescale(m0, m1, st != st_begin);
        } else if (st != st_begin) __syncthreads();
        __builtin_amdgcn_sched_barrier(0);                             // (see exact_x3_kernel.hpp)
        commit(C::HALF && st & 1 ? -1.f : 1.f, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        if (st + 1 < st_end) load(st + 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        x3_f16 part[2];
        R::template steps<0, 0>(acc, part, a0, b0, kk, C::HALF && st & 1 ? -1.f : 1.f);
        __builtin_amdgcn_sched_barrier(0);
        if (C::HALF && st + 1 == (st_begin + st_end) / 2) look();
    }
    float worst = 0.f;
#pragma unroll
    for (int t = 0; t < R::NT; ++t)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int v = 0; v < 16; ++v) worst = fmaf(acc[t][m][v], 0.f, worst);
    if (worst != worst) *flag = 1;
    if constexpr (C::HALF) {
        look();
        bool doubt = false;
#pragma unroll
        for (int t = 0; t < R::NT; ++t) doubt = doubt || ~good(t);
        if (doubt) *asked = 1;
    }
    __syncthreads();
    bool scaled = C::HALF;
    int few = 0;
    float unscale = C::HALF ? 1.f : kX3Unscale;
    if constexpr (C::HALF) {
        if (!*(volatile uint32_t *)flag && *(volatile uint32_t *)asked) {       // (see exact_x3_kernel.hpp)
            uint32_t *const count = (uint32_t *)As, *const tiny = count + kPK + kPC;
            for (int e = tid; e < 2 * (kPK + kPC); e += kBlock) count[e] = 0;
            int again = tid;
            asm volatile("" : "+v"(again));
            items(again);
            __syncthreads();
            auto note = [&](int u, uint32_t small) {
                if (small & 0x7fffffffu) atomicAdd(count + chan[u], small & 0x7fffffffu);
                if (small >> 31) tiny[chan[u]] = 1;
            };
#pragma unroll 1
            for (int st = st_begin; st < st_end; ++st) {
                load(st);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t v[4] = {reg0[j][0], reg0[j][1], reg0[j][2], reg0[j][3]};
                    note(0, x3_small<4>(v, scale[0]));
                }
                if constexpr (SETS > 1)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t v[4] = {reg1[j][0], reg1[j][1], reg1[j][2], reg1[j][3]};
                        note(1, x3_small<4>(v, scale[1]));
                    }
            }
            __syncthreads();
            uint32_t held[R::NT] = {}, now[R::NT] = {};
            const float one = kX3Need / (float)(C::IMG * C::P * (st_end - st_begin));
            weigh(now, count, [&](float sum, uint32_t row, uint32_t col) { return one * (float)(row + col) - sum; });
            weigh(held, tiny, [](float sum, uint32_t row, uint32_t col) { return 0.f - ((float)(row + col) + sum); });
#pragma unroll
            for (int t = 0; t < R::NT; ++t) held[t] &= ~(good(t) | now[t]);
            __syncthreads();
            if (tid == 0) mark[0] = 0;
            __syncthreads();
#pragma unroll
            for (int t = 0; t < R::NT; ++t)
                for (uint32_t rest = held[t]; rest; rest &= rest - 1) {
                    const uint32_t at = atomicAdd(mark, 1u), bit = 31 - __builtin_ctz(rest);        // m * 16 + v
                    if (at < (uint32_t)kX3Few) mark[1 + at] = (uint32_t)role_taps<HW>(ROLE, t) << 16 | (uint32_t)i << 8 | (bit / 4 * 8 + 4 * kk + bit % 4);
                }
            __syncthreads();
            few = mark[0] > (uint32_t)kX3Few ? 0 : (int)mark[0];
            if (mark[0] > (uint32_t)kX3Few) *flag = 1;
            for (int e = tid >> 6; e < few; e += kBlock / 64) {
                const uint32_t id = mark[1 + e];
                const int k = k0 + (int)(id & 255), c = c0 + (int)(id >> 8 & 255), tap = id >> 16;
                const double sum = k >= g.K || c >= g.C ? 0. : x3_dot(Xp, dYp, C::IMG * C::P * (st_end - st_begin), [&](int at, long &xi, long &yi) {
                    const int n = st_begin * C::IMG + at / C::P, pos = at % C::P, h = pos / HW + tap / 3 - 1, w = pos % HW + tap % 3 - 1;
                    xi = ((long)n * g.C + c) * C::P + h * HW + w;
                    yi = ((long)n * g.K + k) * C::P + pos;
                    return n < g.N && (unsigned)h < (unsigned)HW && (unsigned)w < (unsigned)HW;
                });
                if (lane == 0) mark[1 + kX3Few + e] = __float_as_uint((float)sum);
            }
            __syncthreads();
        }
    }
    if (*(volatile uint32_t *)flag) {                                  // (see exact_x3_kernel.hpp)
        scaled = false;
        unscale = 1.f;
        int again = tid;
        asm volatile("" : "+v"(again));             // (decoded again, not kept in registers over the loop above)
        items(again);
        clear();
        load(st_begin);
        for (int st = st_begin; st < st_end; ++st) {
            __syncthreads();
            commit(1.f, std::true_type{});
            if (st + 1 < st_end) load(st + 1);
            __syncthreads();
            R::template plain_steps<0>(acc, a0, b0, kk);
        }
    }
    // the result by half tiles of 32 output channels, gathered in LDS as rows of the tensor
    constexpr int Q = kPC * 9, PITCH = Q + 4;
    float *const rows = (float *)As;
    const int col_e = scaled ? expo[kPK + i] : 0;
    const int n = (g.C - c0 < kPC ? g.C - c0 : kPC) * 9, CRS = g.C * 9;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < R::NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 8 * (v / 4) + 4 * kk + v % 4;
                float z = acc[t][m][v];
                if constexpr (C::HALF) z = __builtin_ldexpf(z, scaled ? -(col_e + expo[m * 32 + row]) : 0);
                else z *= unscale;
                rows[row * PITCH + i * 9 + role_taps<HW>(ROLE, t)] = z;
            }
        __syncthreads();
        if (few > 0) {
            const uint32_t id = mark[1 + (tid < few ? tid : 0)];
            if (tid < few && (int)(id & 255) / 32 == m) rows[(id & 31) * PITCH + (id >> 8 & 255) * 9 + (id >> 16)] = __uint_as_float(mark[1 + kX3Few + tid]);
            __syncthreads();
        }
        const int kb = k0 + m * 32;
        if (n == Q && kb + 32 <= g.K && CRS % 4 == 0 && ((uintptr_t)out & 15) == 0) {
#pragma unroll
            for (int u = 0; u < 32 * Q / 4 / kBlock; ++u) {
                const int e = tid + u * kBlock, row = e / (Q / 4), x = e % (Q / 4) * 4;
                *(float4_t *)(out + (long)(kb + row) * CRS + c0 * 9 + x) = *(const float4_t *)(rows + row * PITCH + x);
            }
        } else {
            for (int row = tid >> 6; row < 32 && kb + row < g.K; row += 4)
                for (int x = lane; x < n; x += 64) out[(long)(kb + row) * CRS + c0 * 9 + x] = rows[row * PITCH + x];
        }
    }
}

template <int HW, int KIND>
__global__ __launch_bounds__(kBlock, 2) void wgrad_exact_x3_planes(const X3Multi)
{
    extern __shared__ __align__(16) char x3_smem[];
    const X3Multi *mp = (const X3Multi *)__builtin_amdgcn_kernarg_segment_ptr();
    int gi = 0;
    for (int i = 1; i < mp->n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const int bid = (int)blockIdx.x - mp->begin[gi], nblk = mp->count[gi];
    if (bid >= nblk) return;
    const X3Shape &p = mp->s[gi];
    uint32_t prob, logical, rest, coltile, ktile, split;
    p.d_prob.divmod((uint32_t)xcd_contiguous_id(bid, nblk), prob, logical);
    p.d_ctiles.divmod(logical, rest, coltile);
    p.d_ktiles.divmod(rest, split, ktile);
    const int st_begin = (int)split * p.tiles_each + min((int)split, p.tiles_more), st_end = st_begin + p.tiles_each + ((int)split < p.tiles_more);
    const int k0 = (int)ktile * kPK, c0 = (int)coltile * kPC;
    const float *const X = (const float *)mp->X[mp->first[gi] + prob], *const dY = (const float *)mp->dY[mp->first[gi] + prob];
    float *const out = mp->out[mp->first[gi] + prob] + (long)split * p.g.K * p.g.C * 9;
    // (the barriers inside are reached by all four wavefronts the same number of times, whatever their role)
    switch (__builtin_amdgcn_readfirstlane(((int)(threadIdx.x >> 6) + ((int)blockIdx.x >> 8)) & 3)) {
        case 0: planes_body<HW, KIND, 0>(p, X, dY, out, x3_smem, k0, c0, st_begin, st_end); break;
        case 1: planes_body<HW, KIND, 1>(p, X, dY, out, x3_smem, k0, c0, st_begin, st_end); break;
        case 2: planes_body<HW, KIND, 2>(p, X, dY, out, x3_smem, k0, c0, st_begin, st_end); break;
        default: planes_body<HW, KIND, 3>(p, X, dY, out, x3_smem, k0, c0, st_begin, st_end); break;
    }
}

}  // namespace

template <int HW, int KIND> constexpr int planes_lds()
{
    constexpr int tail = PlaneCfg<HW, KIND>::kHead + 32 * (kPC * 9 + 4) * 4, stage = PlaneCfg<HW, KIND>::kLds;
    return stage > tail ? stage : tail;
}
int x3_planes_lds(int hw) { return hw == 4 ? planes_lds<4, kX3Three>() : planes_lds<2, kX3Three>(); }
int x3_launch_planes(int hw, bool half, const X3Multi &m, int blocks, size_t lds, hipStream_t st)
{
    if (hw == 2) return x3_launch(wgrad_exact_x3_planes<2, kX3Three>, m, blocks, lds, st);
    return half ? x3_launch(wgrad_exact_x3_planes<4, kX3Half>, m, blocks, (size_t)planes_lds<4, kX3Half>(), st) : x3_launch(wgrad_exact_x3_planes<4, kX3Three>, m, blocks, lds, st);
}

}  // namespace wgrad
