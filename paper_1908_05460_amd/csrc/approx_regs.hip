// Approximated filter gradient of fp32 layers (3x3, padding 1) on 8x8, 4x4 and 2x2 planes: the planes in registers.
//
// dW[k][c][tap] = sum over n of sum[n][k] * X[n][c][position(n, k) + tap].  A lane is an input channel and a wavefront eight output
// channels (2x2: four).  Read from LDS patch by patch, each multiply-add costs an LDS read of its own, two clocks of a CU for each that
// four SIMDs do in one, and address arithmetic and waits besides.  Here a lane keeps its channel's whole plane in registers,
// read from LDS once for the wavefront's eight output channels, and the position -- the same for all lanes -- moves the register
// numbers that the multiply-adds name (s_set_gpr_idx): one scalar instruction a patch, no address arithmetic, no
// branch.  (Measured: the register numbers' moving costs nothing; a dependent chain of v_fma_f32 and this one both issue at one
// in four clocks.)
//   - 8x8, 4x4: the plane lies in a block of registers with a border of zeros; the position moves the source, nine taps.
//   - 2x2: each position has sums of its own, four elements of X go to four of them, which the position moves to; the five taps
//     in the padding are not computed, so that a map's sum that is not finite makes no NaN there, as in the plain product that takes
//     such a layer alone.  (Sums of a tap over all positions are chains four times as long: error against 64 bits
//     1.17e-7 against 0.91e-7, N = 128.)  Sixteen registers an output channel, so four of them to a wavefront.
// The block and the sums live in numbered registers, above those that the compiler is given (amdgpu_num_vgpr); they are
// touched by the asm blocks below only.  4x4 and 2x2: 127 registers, four wavefronts a SIMD, which hide each other's LDS and
// scalar latencies; 8x8: 233, two, bound by reading the planes (128 clocks of the CU's LDS a wavefront and image against 72 of
// multiply-adds).  X reaches LDS by loads that bypass the registers, a stage of 16 or 32 KB ahead.
// VGG-19 fp32 at N = 128: layers on 4x4 and 2x2 planes 87 us (54 of them the multiply-adds' own issue, 17 the results' way to
// memory), on 8x8 planes 28; the LDS gather took 197 for those on 8x8 and 4x4 planes, and the exact kernel on a sparsified dY
// 49 for those on 2x2 ones.
#include <algorithm>
#include <utility>

#include "exact_common.hpp"
#include "lds_copy.hpp"

namespace wgrad {

__host__ __device__ constexpr int regs_kw(int hw) { return hw == 2 ? 4 : 8; }
constexpr int kRegsWaves = 8;                        // most wavefronts of a workgroup
// KW: output channels of a wavefront; SUMS: registers of each; FREE: registers left to the compiler; X: first of the plane's, rows of PITCH (data rows begin at even numbers); ACC: first of
// the sums, [output channel][tap], 2x2: [output channel][position][element]; STAGE: bytes of X staged at a time; OCC: wavefronts a SIMD holds
template <int HW> struct RegsLayout;
template <> struct RegsLayout<2> { static constexpr int KW = 4, SUMS = 16, FREE = 19, X = 20, PITCH = 2, ACC = 55, STAGE = 16 * 1024, OCC = 4; };
template <> struct RegsLayout<4> { static constexpr int KW = 8, SUMS = 9, FREE = 19, X = 19, PITCH = 6, ACC = 55, STAGE = 16 * 1024, OCC = 4; };
template <> struct RegsLayout<8> { static constexpr int KW = 8, SUMS = 9, FREE = 61, X = 61, PITCH = 10, ACC = 161, STAGE = 32 * 1024, OCC = 2; };

struct RegsParams {
    const void *X[kMaxBatch];
    const int32_t *at[kMaxBatch];                    // [N][K]: by how much a map's position moves the register numbers
    const float *sum[kMaxBatch];
    float *out[kMaxBatch];                           // dW, or the partials of the batch chunks
    int N, C, K, hw;
    int ktiles, chunks, chunk_n;                     // tiles of (KW * wavefronts) output channels; 64 input channels
    float scale;
};

typedef int rg_i8 __attribute__((ext_vector_type(8)));
typedef float rg_f8 __attribute__((ext_vector_type(8)));
typedef int rg_i4 __attribute__((ext_vector_type(4)));
typedef float rg_f4 __attribute__((ext_vector_type(4)));
template <int KW> struct RegsScalars { typedef rg_i8 at; typedef rg_f8 sum; };
template <> struct RegsScalars<4> { typedef rg_i4 at; typedef rg_f4 sum; };

#define RG_CLOBBER "memory"
#define RG_CLOBBER_M0 "memory", "m0"     // (s_set_gpr_idx_* keep the offset there)

// nine taps of one patch into the sums of output channel J: v[...] += sum * X[tap]
#define RG_TAP(J, T, AT) "v_fmac_f32 v[%[A]+9*" #J "+" #T "], %[s" #J "], v[%[X]+" AT "]\n\t"
#define RG_PATCH(J)                                                                                              \
    "s_set_gpr_idx_idx %[i" #J "]\n\t"                                                                           \
    RG_TAP(J, 0, "0") RG_TAP(J, 1, "1") RG_TAP(J, 2, "2")                                                        \
    RG_TAP(J, 3, "%[P]") RG_TAP(J, 4, "%[P]+1") RG_TAP(J, 5, "%[P]+2")                                           \
    RG_TAP(J, 6, "2*%[P]") RG_TAP(J, 7, "2*%[P]+1") RG_TAP(J, 8, "2*%[P]+2")
// 2x2: the four elements into the sums of the position
#define RG_PATCH2(J)                                                                                             \
    "s_set_gpr_idx_idx %[i" #J "]\n\t"                                                                           \
    "v_fma_f32 v[%[A]+16*" #J "+0], v[%[X]+0], %[s" #J "], v[%[A]+16*" #J "+0]\n\t"                              \
    "v_fma_f32 v[%[A]+16*" #J "+1], v[%[X]+1], %[s" #J "], v[%[A]+16*" #J "+1]\n\t"                              \
    "v_fma_f32 v[%[A]+16*" #J "+2], v[%[X]+2], %[s" #J "], v[%[A]+16*" #J "+2]\n\t"                              \
    "v_fma_f32 v[%[A]+16*" #J "+3], v[%[X]+3], %[s" #J "], v[%[A]+16*" #J "+3]\n\t"
#define RG_SCALARS4(at, sum) [i0] "s"(at[0]), [i1] "s"(at[1]), [i2] "s"(at[2]), [i3] "s"(at[3]), [s0] "s"(sum[0]), [s1] "s"(sum[1]), \
    [s2] "s"(sum[2]), [s3] "s"(sum[3])
#define RG_SCALARS(at, sum) [i0] "s"(at[0]), [i1] "s"(at[1]), [i2] "s"(at[2]), [i3] "s"(at[3]), [i4] "s"(at[4]), [i5] "s"(at[5]), [i6] "s"(at[6]),    \
    [i7] "s"(at[7]), [s0] "s"(sum[0]), [s1] "s"(sum[1]), [s2] "s"(sum[2]), [s3] "s"(sum[3]), [s4] "s"(sum[4]), [s5] "s"(sum[5]),         \
    [s6] "s"(sum[6]), [s7] "s"(sum[7])

// Zeros in the border of the plane and in the sums.  (Naming the last numbered register makes it part of the kernel's allotment;
// the compiler remarks that it may not use it itself.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int HW>
__device__ __forceinline__ void regs_zero()
{
#define RG_ZERO ".set rg_i, %0\n\t.rept %1\n\tv_mov_b32 v[rg_i], 0\n\t.set rg_i, rg_i+1\n\t.endr"
    typedef RegsLayout<HW> L;
    if constexpr (HW == 8) asm volatile(RG_ZERO ::"n"(L::X), "n"(L::ACC + L::SUMS * L::KW - L::X) : "memory", "v232");
    else asm volatile(RG_ZERO ::"n"(L::X), "n"(L::ACC + L::SUMS * L::KW - L::X) : "memory", "v126");
    static_assert(L::ACC + L::SUMS * L::KW - 1 <= (HW == 8 ? 232 : 126) && L::X + (HW + 2) * L::PITCH <= L::ACC, "numbered registers");
#undef RG_ZERO
}
#pragma clang diagnostic pop
template <int R>
__device__ __forceinline__ float regs_get()
{
    float v;
    asm volatile("v_mov_b32 %0, v[%1]" : "=v"(v) : "n"(R) : "memory");
    return v;
}

// 4x4, 8x8: the lanes' planes of one image from LDS, waited for here.  The scalars pass through, so that the wait for
// them comes before and the next image's are loaded after: a wait for LDS is a wait for scalar loads too, and theirs take
// far longer.
template <int HW, int OFF, class AT, class SUM>
__device__ __forceinline__ void regs_load(const uint32_t *rd, const int32_t *&at_p, const float *&sum_p, AT &at, SUM &sum)
{
#define RG_ROW(R, V) "ds_read_b128 v[%[X]+" V ":%[X]+" V "+3], %[r" #R "] offset:%[o]\n\t"
#define RG_PASS "+s"(at_p), "+s"(sum_p), "+s"(at), "+s"(sum)
    typedef RegsLayout<HW> L;
    if constexpr (HW == 8)
        asm volatile(RG_ROW(0, "11") RG_ROW(1, "15") RG_ROW(2, "21") RG_ROW(3, "25") RG_ROW(4, "31") RG_ROW(5, "35") RG_ROW(6, "41") RG_ROW(7, "45")
                     RG_ROW(8, "51") RG_ROW(9, "55") RG_ROW(10, "61") RG_ROW(11, "65") RG_ROW(12, "71") RG_ROW(13, "75") RG_ROW(14, "81") RG_ROW(15, "85")
                     "s_waitcnt lgkmcnt(0)"
                     : RG_PASS
                     : [X] "n"(L::X), [o] "n"(OFF), [r0] "v"(rd[0]), [r1] "v"(rd[1]), [r2] "v"(rd[2]), [r3] "v"(rd[3]), [r4] "v"(rd[4]), [r5] "v"(rd[5]),
                       [r6] "v"(rd[6]), [r7] "v"(rd[7]), [r8] "v"(rd[8]), [r9] "v"(rd[9]), [r10] "v"(rd[10]), [r11] "v"(rd[11]), [r12] "v"(rd[12]),
                       [r13] "v"(rd[13]), [r14] "v"(rd[14]), [r15] "v"(rd[15]) : RG_CLOBBER);
    else
        asm volatile(RG_ROW(0, "7") RG_ROW(1, "13") RG_ROW(2, "19") RG_ROW(3, "25") "s_waitcnt lgkmcnt(0)"
                     : RG_PASS : [X] "n"(L::X), [o] "n"(OFF), [r0] "v"(rd[0]), [r1] "v"(rd[1]), [r2] "v"(rd[2]), [r3] "v"(rd[3]) : RG_CLOBBER);
#undef RG_ROW
#undef RG_PASS
}

// 2x2: the same for four images; four at a time, because the scalars of one are used before the next one's could arrive
template <int OFF>
__device__ __forceinline__ void regs_load4(uint32_t rd, rg_i4 (&at)[4], rg_f4 (&sum)[4])
{
    asm volatile("ds_read_b128 v[%[X]:%[X]+3], %[r0] offset:%[o]\n\tds_read_b128 v[%[X]+4:%[X]+7], %[r0] offset:%[o]+1024\n\t"
                 "ds_read_b128 v[%[X]+8:%[X]+11], %[r0] offset:%[o]+2048\n\tds_read_b128 v[%[X]+12:%[X]+15], %[r0] offset:%[o]+3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "+s"(at[0]), "+s"(at[1]), "+s"(at[2]), "+s"(at[3]), "+s"(sum[0]), "+s"(sum[1]), "+s"(sum[2]), "+s"(sum[3])
                 : [X] "n"(RegsLayout<2>::X), [o] "n"(OFF), [r0] "v"(rd) : RG_CLOBBER);
}

// the patches of one image; 2x2: of the one in the I-th four registers
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"     // (m0 named: see rows_copy)
template <int HW, int I, class AT, class SUM>
__device__ __forceinline__ void regs_patches(const AT &at, const SUM &sum)
{
    typedef RegsLayout<HW> L;
    if constexpr (HW >= 4)
        asm volatile("s_set_gpr_idx_on %[i0], gpr_idx(SRC1)\n\t"
                     RG_PATCH(0) RG_PATCH(1) RG_PATCH(2) RG_PATCH(3) RG_PATCH(4) RG_PATCH(5) RG_PATCH(6) RG_PATCH(7)
                     "s_set_gpr_idx_off" :: [X] "n"(L::X), [A] "n"(L::ACC), [P] "n"(L::PITCH), RG_SCALARS(at, sum) : RG_CLOBBER_M0);
    else
        asm volatile("s_set_gpr_idx_on %[i0], gpr_idx(SRC2,DST)\n\t"
                     RG_PATCH2(0) RG_PATCH2(1) RG_PATCH2(2) RG_PATCH2(3)
                     "s_set_gpr_idx_off" :: [X] "n"(L::X + 4 * I), [A] "n"(L::ACC), RG_SCALARS4(at, sum) : RG_CLOBBER_M0);
}
#pragma clang diagnostic pop

template <int... I, class F>
__device__ __forceinline__ void regs_each(std::integer_sequence<int, I...>, F &&f) { (f(std::integral_constant<int, I>()), ...); }

struct __attribute__((packed, aligned(4))) RegsRow { float v[4]; };

template <int HW>
__device__ __forceinline__ void regs_body(const RegsParams &p, char *smem, int bid, int nblk, int prob, int waves)
{
    typedef RegsLayout<HW> L;
    constexpr int PLANE = HW * HW * 4;               // bytes
    constexpr int IMG = 64 * PLANE;                  // of a tile's channels in one image
    constexpr int NI = L::STAGE / IMG;               // images of a stage
    constexpr int PIECES = HW * HW / 4;              // 16-byte pieces of a plane
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int logical = xcd_contiguous_id(bid, nblk);            // (the workgroups that read the same planes side by side)
    const int kt = logical % p.ktiles, rest = logical / p.ktiles, chunk = rest % p.chunks, ct = rest / p.chunks;
    const int C = p.C, K = p.K, c0 = ct * 64, k0 = (kt * waves + wave) * L::KW;
    const int n_begin = chunk * p.chunk_n, n_end = n_begin + p.chunk_n < p.N ? n_begin + p.chunk_n : p.N;
    const uint32_t ximg = (uint32_t)C * PLANE;

    // ---- copies, 1 KB each; loads past the last image bring zeros ----
    const br_u4 xbuf = rows_buffer((const char *)p.X[prob] + (size_t)n_begin * ximg, (uint32_t)(p.N - n_begin) * ximg);
    const uint32_t lds_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    // a channel's pieces are permuted by its number, so that the lanes of a read fall on all banks
    auto turn = [](int c) {
        if constexpr (HW == 8) return c & 15;
        else if constexpr (HW == 4) return ((c >> 2) & 1) | ((((c >> 1) ^ (c >> 3)) & 1) << 1);
        else return 0;
    };
    const int cl = lane / PIECES;
    const uint32_t from = (uint32_t)cl * PLANE + (((lane % PIECES) ^ turn(cl)) * 16);
    auto copy_stage = [&](int stage) {
        for (int q = wave; q < L::STAGE / 1024; q += waves) {
            const uint32_t img = (uint32_t)(stage * NI + q / (IMG / 1024));
            const uint32_t lanes_from = HW == 8 ? from ^ (uint32_t)((q & 3) * 64) : from;    // 8x8: four channels a copy
            rows_copy(xbuf, lanes_from + (img * ximg + (uint32_t)c0 * PLANE + (q % (IMG / 1024)) * 1024), lds_at + (stage & 1) * L::STAGE + q * 1024);
        }
    };
    uint32_t rd[PIECES];
#pragma unroll
    for (int r = 0; r < PIECES; ++r) rd[r] = lds_at + (uint32_t)lane * PLANE + ((r ^ turn(lane)) * 16);

    copy_stage(0);
    regs_zero<HW>();

    // (scalar loads: the selections were written by an earlier launch; volatile: where they stand is where they are issued)
    typedef const volatile __attribute__((address_space(4))) typename RegsScalars<L::KW>::at *at_ptr;
    typedef const volatile __attribute__((address_space(4))) typename RegsScalars<L::KW>::sum *sum_ptr;
    const size_t first = (size_t)n_begin * K + k0;
    const int32_t *at_p = p.at[prob] + first;
    const float *sum_p = p.sum[prob] + first;
    const int count = n_end - n_begin, full = count / NI, rest_n = count % NI, stages = full + (rest_n > 0);
    auto meet = [&](int stage) {                     // the stage is in LDS, the one before it read by all
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (stage + 1 < stages) copy_stage(stage + 1);
    };
    if constexpr (HW == 2) {
        rg_i4 at[2][4];
        rg_f4 sum[2][4];
        auto fetch = [&](int n, auto a_c) {          // of images n .. n + 3 of the chunk, the last one again past its end
            constexpr int A = decltype(a_c)::value;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t o = (uint32_t)std::min(n + j, count - 1) * (uint32_t)K;
                at[A][j] = *(at_ptr)(uintptr_t)(at_p + o);
                sum[A][j] = *(sum_ptr)(uintptr_t)(sum_p + o);
            }
        };
        typedef std::integral_constant<int, 0> i0;
        fetch(0, i0());
        for (int stage = 0; stage < full; ++stage) {
            meet(stage);
            regs_each(std::make_integer_sequence<int, NI / 4>(), [&](auto g_c) {
                constexpr int G = decltype(g_c)::value, A = G & 1;
                regs_load4<G * 4 * IMG>(rd[0], at[A], sum[A]);
                fetch(stage * NI + 4 * G + 4, std::integral_constant<int, A ^ 1>());
                __builtin_amdgcn_sched_barrier(0);
                regs_each(std::make_integer_sequence<int, 4>(), [&](auto j_c) { regs_patches<HW, decltype(j_c)::value>(at[A][decltype(j_c)::value], sum[A][decltype(j_c)::value]); });
            });
            rd[0] ^= L::STAGE;
        }
        if (rest_n > 0) {
            meet(full);
            for (int n = 0; n < rest_n; n += 4) {
                if (n > 0) fetch(full * NI + n, i0());
                regs_load4<0>(rd[0], at[0], sum[0]);
                regs_each(std::make_integer_sequence<int, 4>(), [&](auto j_c) {
                    constexpr int J = decltype(j_c)::value;
                    if (n + J < rest_n) regs_patches<HW, J>(at[0][J], sum[0][J]);
                });
                rd[0] += 4 * IMG;
            }
        }
    } else {
        typename RegsScalars<L::KW>::at at[2];
        typename RegsScalars<L::KW>::sum sum[2];
        at[0] = *(at_ptr)(uintptr_t)at_p;
        sum[0] = *(sum_ptr)(uintptr_t)sum_p;
        // image I of a stage or of its rest, with scalars I % 2; those of the next (step maps on) are loaded meanwhile
        auto image = [&](auto i_c, int step) {
            constexpr int I = decltype(i_c)::value, A = I & 1;
            at_p += step; sum_p += step;
            regs_load<HW, I * IMG>(rd, at_p, sum_p, at[A], sum[A]);
            at[A ^ 1] = *(at_ptr)(uintptr_t)at_p;
            sum[A ^ 1] = *(sum_ptr)(uintptr_t)sum_p;
            __builtin_amdgcn_sched_barrier(0);
            regs_patches<HW, 0>(at[A], sum[A]);
        };
        for (int stage = 0; stage < full; ++stage) {
            meet(stage);
            const int last_step = stage + 1 < stages ? K : 0;
            regs_each(std::make_integer_sequence<int, NI>(), [&](auto i_c) {
                constexpr int I = decltype(i_c)::value;
                image(i_c, I == NI - 1 ? last_step : K);
            });
#pragma unroll
            for (int r = 0; r < PIECES; ++r) rd[r] ^= L::STAGE;
        }
        if (rest_n > 0) {
            meet(full);
            for (int i = 0; i < rest_n; ++i) {
                image(std::integral_constant<int, 0>(), i + 1 < rest_n ? K : 0);
                at[0] = at[1]; sum[0] = sum[1];
#pragma unroll
                for (int r = 0; r < PIECES; ++r) rd[r] += IMG;
            }
        }
    }

    // the sums go out as rows of 576 values, through LDS
    __syncthreads();
    float *const row = (float *)smem + wave * 576;
    float *const out = p.out[prob] + ((size_t)chunk * K + k0) * C * 9 + (size_t)c0 * 9;
    auto put = [&](auto j_c) {
        constexpr int J = decltype(j_c)::value;
        float v[9] = {};
        regs_each(std::make_integer_sequence<int, L::SUMS>(), [&](auto i_c) {
            constexpr int I = decltype(i_c)::value;
            // 2x2: position p sees element e at tap e - p
            constexpr int T = HW == 2 ? 4 + 3 * ((I >> 1 & 1) - (I >> 3)) + (I & 1) - (I >> 2 & 1) : I;
            v[T] += regs_get<L::ACC + L::SUMS * J + I>();
        });
#pragma unroll
        for (int t = 0; t < 9; ++t) row[lane * 9 + t] = v[t] * p.scale;
        __builtin_amdgcn_wave_barrier();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        float *const o = out + (size_t)J * C * 9;
        for (int e = lane * 4; e < 576; e += 256) *(RegsRow *)(o + e) = *(const RegsRow *)(row + e);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    };
    regs_each(std::make_integer_sequence<int, L::KW>(), put);
}

struct RegsMulti {
    int n, waves;
    int begin[kRegsMultiMax + 1];    // first workgroup of each group (multiples of 8); begin[n] = grid size
    int per_prob[kRegsMultiMax], nprob[kRegsMultiMax];
    RegsParams p[kRegsMultiMax];
};
static_assert(sizeof(RegsMulti) <= 4096, "kernel arguments");

template <class F>
__device__ __forceinline__ void regs_group(F &&body)
{
    const RegsMulti *mp = (const RegsMulti *)__builtin_amdgcn_kernarg_segment_ptr();
    const int n = mp->n;
    int gi = 0;
    for (int i = 1; i < n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const int bid = (int)blockIdx.x - mp->begin[gi], per = mp->per_prob[gi], prob = bid / per;
    if (prob < mp->nprob[gi]) body(mp->p[gi], bid - prob * per, per, prob, mp->waves);
}

// layers on 4x4 and 2x2 planes
__global__ __launch_bounds__(64 * kRegsWaves, RegsLayout<4>::OCC) __attribute__((amdgpu_num_vgpr(RegsLayout<4>::FREE)))
void approx_gather_regs(const RegsMulti)
{
    extern __shared__ __attribute__((aligned(2 * RegsLayout<4>::STAGE))) char regs_smem[];    // (the two stages' addresses differ in one bit)
    regs_group([&](const RegsParams &p, int bid, int nblk, int prob, int waves) {
        if (p.hw == 4) regs_body<4>(p, regs_smem, bid, nblk, prob, waves);
        else regs_body<2>(p, regs_smem, bid, nblk, prob, waves);
    });
}

// layers on 8x8 planes
__global__ __launch_bounds__(64 * kRegsWaves, RegsLayout<8>::OCC) __attribute__((amdgpu_num_vgpr(RegsLayout<8>::FREE)))
void approx_gather_regs8(const RegsMulti)
{
    extern __shared__ __attribute__((aligned(2 * RegsLayout<8>::STAGE))) char regs8_smem[];
    regs_group([&](const RegsParams &p, int bid, int nblk, int prob, int waves) { regs_body<8>(p, regs8_smem, bid, nblk, prob, waves); });
}

// ---- host ----
bool regs_takes(const Geometry &g)
{
    if (g.bf16 || g.R != 3 || g.S != 3 || g.ph != 1 || g.pw != 1 || g.H != g.W || (g.H != 8 && g.H != 4 && g.H != 2)) return false;
    // Maps of up to four positions keep to the sparsified form, whose sums are the shorter chains (2x2, stride 2, 64 -> 128, N =
    // 256: error against 64 bits 0.99e-7 against 2.04e-7 here, 4x4, stride 2: 0.87e-7 against 1.40e-7); on 2x2 planes without a
    // stride the maps' four positions have sums of their own.
    if (g.Ho * g.Wo <= 4 && (g.H != 2 || g.sh != 1 || g.sw != 1)) return false;
    // (scalar loads of eight or four maps at a time, whole tiles; a byte offset in X is 32 bits)
    return g.C % 64 == 0 && g.K % 32 == 0 && g.K >= 128 && tune_int("WGRAD_REGS", 1) && (long)g.N * g.C * g.H * g.W * 4 < (1l << 31);
}

RegsPosition regs_position(const Geometry &g)
{
    if (g.H == 2) return RegsPosition{8 * g.sh, 4 * g.sw};
    return RegsPosition{(g.H == 8 ? RegsLayout<8>::PITCH : RegsLayout<4>::PITCH) * g.sh, g.sw};
}

struct RegsQueue {
    int n = 0;
    RegsItem item[kRegsMultiMax];
};
RegsQueue *regs_queue_new() { return new RegsQueue; }
void regs_queue_delete(RegsQueue *q) { delete q; }

// Which numbers of chunks lose no more to rounding than chunks of most_n images do, `least` of them.  What counts is how many
// additions in a row lie between a product and the result: a chunk's images and the reduction of the chunks, fewer and longer chunks
// where that is no more than with chunks of most_n (512 -> 512 @ 4x4, N = 128 in one / two / four chunks 1.45e-7 / 1.21e-7 / 1.09e-7;
// 64 -> 256 @ 4x4, N = 229 in 29 chunks, whose reduction is spread over lanes, 1.10e-7, in four 1.23e-7).  A partial result costs more than
// an image where X and the padding bring zeros, which round nothing, so that no chunk is cut into less than sixteen images without
// need (128 -> 160 @ 4x4, N = 128, two layers 1.11e-7 in sixteen chunks, 1.07e-7 in seven).
static int regs_additions(const RegsItem &I, int images)
{
    const int ch = (I.g.N + images - 1) / images;
    return images + (ch > 1 ? combine_chain(I.g.dw_elems(), ch) : 0);
}
static void regs_limits(RegsItem &I, int most_n)
{
    const int N = I.g.N, limit = regs_additions(I, most_n);
    I.additions = limit;
    I.least = (N + most_n - 1) / most_n;
    I.most = std::min(I.max_chunks, std::max(I.least, (N + 15) / 16));
    I.fewest = (N + limit - 1) / limit;
    while (I.fewest < I.least && regs_additions(I, (N + I.fewest - 1) / I.fewest) > limit) ++I.fewest;
}
static int regs_allowed(const RegsItem &I, int want)
{
    if (want <= I.fewest) return I.fewest;
    if (want >= I.least) return std::min(want, I.most);
    return regs_additions(I, (I.g.N + want - 1) / want) <= I.additions ? want : I.least;
}

// How the batches of n groups of layers, launched together, are cut, and how many wavefronts a workgroup has (eight share the
// copies of X among twice as many output channels as four do, four make twice as many workgroups).
// All of them on 8x8 planes, or none.
static int regs_cut(const RegsItem *const *it, int n, int *chunks, double *life)
{
    int best_waves = 8;
    double best = 1e30;
    for (int waves = 8; waves >= 4; waves -= 4) {
        bool fits = true;
        for (int i = 0; i < n; ++i) fits = fits && it[i]->g.K % (regs_kw(it[i]->g.H) * waves) == 0;
        if (!fits) continue;
        const bool big = it[0]->g.H == 8;
        const int most = big ? RegsLayout<8>::OCC : RegsLayout<4>::OCC, slots = kNumCU * 4 * most / waves;
        int now[kRegsMultiMax] = {};
        for (int want = 1; want <= 64; want += want < 8 ? 1 : want / 4) {     // chunks of a layer (2x2 planes: half as many, an image is half the work)
            double partial = 0, all_waves = 0;
            bool same = true;                        // (as with fewer wanted: the limits are reached)
            for (int i = 0; i < n; ++i) {
                const Geometry &g = it[i]->g;
                const int ch = regs_allowed(*it[i], g.H == 2 ? (want + 1) / 2 : want);
                const int per = (g.N + ch - 1) / ch, cut = (g.N + per - 1) / per;
                same = same && cut == now[i];
                now[i] = cut;
                if (now[i] > 1) partial += (double)now[i] * g.dw_elems() * 4 * it[i]->b.n;
                all_waves += (double)now[i] * (g.C / 64) * (g.K / regs_kw(g.H)) * it[i]->b.n;
            }
            if (same) continue;
            const double occ = std::min((double)most, std::max(waves / 4.0, all_waves / (kNumCU * 4)));
            double sorted[kRegsMultiMax], lf[kRegsMultiMax];
            long count[kRegsMultiMax];
            for (int i = 0; i < n; ++i) {
                const Geometry &g = it[i]->g;
                // a wavefront's time for an image, with occ of them on its SIMD (measured, 512 -> 512 @ 4x4 0.40 us at two and 0.71
                // at four, VGG-19's 8x8 layers 0.55 at two, 512 -> 512 @ 2x2 with eight output channels to a wavefront 0.24 and
                // 0.33, of which four take some 60 %); fewer wavefronts to a workgroup copy X more often
                const double image = g.H == 8 ? 0.11 + 0.22 * occ : (g.H == 4 ? std::max(0.177 * occ, 0.16 + 0.12 * occ) : 0.06 + 0.04 * occ);
                lf[i] = 9.0 + (g.N + now[i] - 1) / now[i] * image * (waves == 8 ? 1.0 : 1.1);
                int j = i;
                for (; j > 0 && sorted[j - 1] < lf[i]; --j) { sorted[j] = sorted[j - 1]; count[j] = count[j - 1]; }
                sorted[j] = lf[i];
                count[j] = (long)now[i] * (g.C / 64) * (g.K / (regs_kw(g.H) * waves)) * it[i]->b.n;
            }
            const double cost = makespan_us(slots, sorted, count, n) + partial / (partial < 40e6 ? 7e6 : 3.5e6) + (partial > 0 ? 2.0 : 0.0);
            if (cost < best) {
                best = cost;
                best_waves = waves;
                std::copy(now, now + n, chunks);
                std::copy(lf, lf + n, life);
            }
        }
    }
    return best_waves;
}

static int regs_launch(const RegsItem *const *it, int n, bool big, hipStream_t st, CombineQueue *combine)
{
    if (n == 0) return WGRAD_OK;
    int chunks[kRegsMultiMax];
    double life[kRegsMultiMax];
    const int waves = regs_cut(it, n, chunks, life);
    int order[kRegsMultiMax];                        // longest workgroups first
    for (int i = 0; i < n; ++i) {
        int j = i;
        for (; j > 0 && life[order[j - 1]] < life[i]; --j) order[j] = order[j - 1];
        order[j] = i;
    }
    RegsMulti m{};
    m.n = n; m.waves = waves;
    int blocks = 0;
    for (int o = 0; o < n; ++o) {
        const RegsItem &I = *it[order[o]];
        const Geometry &g = I.g;
        RegsParams &p = m.p[o];
        const int ch = chunks[order[o]];
        p.N = g.N; p.C = g.C; p.K = g.K; p.hw = g.H;
        p.ktiles = g.K / (regs_kw(g.H) * waves); p.chunks = ch; p.chunk_n = (g.N + ch - 1) / ch;
        p.scale = ch > 1 ? 1.0f : I.scale;
        for (int j = 0; j < kMaxBatch; ++j) {
            const int k = j < I.b.n ? j : 0;
            p.X[j] = I.b.X[k]; p.at[j] = I.at[k]; p.sum[j] = I.sum[k];
            p.out[j] = ch > 1 ? (float *)(I.part + k * I.stride) : I.b.dW[k];
        }
        m.nprob[o] = I.b.n;
        m.per_prob[o] = p.ktiles * (g.C / 64) * ch;
        m.begin[o] = blocks;
        blocks += (m.per_prob[o] * I.b.n + 7) / 8 * 8;
    }
    m.begin[n] = blocks;
    if (big) WGRAD_LAUNCH(approx_gather_regs8, dim3((unsigned)blocks), dim3(64 * waves), 2 * RegsLayout<8>::STAGE, st, m);
    else WGRAD_LAUNCH(approx_gather_regs, dim3((unsigned)blocks), dim3(64 * waves), 2 * RegsLayout<4>::STAGE, st, m);
    int rc = launch_status();
    for (int i = 0; i < n && rc == WGRAD_OK; ++i)
        if (chunks[i] > 1)
            rc = launch_combine((const float *)it[i]->part, (long)(it[i]->stride / 4), chunks[i], it[i]->g.dw_elems(), it[i]->scale,
                                it[i]->b.dW, it[i]->b.n, st, combine);
    return rc;
}

int regs_flush(RegsQueue &q, hipStream_t st, CombineQueue *combine)
{
    int rc = WGRAD_OK;
    for (int kind = 0; kind < 4 && rc == WGRAD_OK; ++kind) {       // 4x4 and 2x2 planes, 8x8 ones, those in LDS, fp32 and bf16
        const RegsItem *it[kRegsMultiMax];
        int n = 0;
        for (int i = 0; i < q.n; ++i)
            if ((q.item[i].planes ? 2 + (q.item[i].g.bf16 != 0) : q.item[i].g.H == 8) == kind) it[n++] = &q.item[i];
        rc = kind >= 2 ? planes_launch(it, n, st, combine) : regs_launch(it, n, kind == 1, st, combine);
    }
    q.n = 0;
    return rc;
}

// One group of identical layers, selected already (or recorded to be, where the launch is): its own launch, or (with a queue)
// collected for regs_flush.
int launch_regs(const Geometry &g, bool planes, const Batch &b, const int32_t *const *at, const float *const *sum, int max_chunks, int most_n, float scale,
                void *part, size_t stride, hipStream_t st, CombineQueue *defer, RegsQueue *queue)
{
    RegsQueue local;
    RegsQueue &q = queue ? *queue : local;
    RegsItem &I = q.item[q.n++];
    I.g = g; I.b = b; I.max_chunks = max_chunks; I.scale = scale; I.part = (char *)part; I.stride = stride; I.planes = planes;
    if (planes) I.in_a_row = most_n;
    else regs_limits(I, most_n);
    for (int i = 0; i < b.n; ++i) { I.at[i] = at[i]; I.sum[i] = sum[i]; }
    return queue ? WGRAD_OK : regs_flush(local, st, defer);
}
bool regs_full(const RegsQueue &q) { return q.n == kRegsMultiMax; }

}  // namespace wgrad
