// Exact filter gradient for fp32 inputs on the 16-bit matrix cores, with fp32 accumulation: a number is the sum of 16-bit
// pieces, a product of two numbers the sum of the larger products of their pieces, each exact in fp32.
//
// Three bf16 pieces (8 significant bits each, rounded to nearest: x = h + m + l exactly), six of nine products: what is left
// out is below 2^-24 |x y|, the rounding of one fp32 product.  bf16's smallest step is 2^-133, so both operands are scaled by
// 2^16 as they are split, and the sums scaled back: every fp32 number then has its 24 bits in the pieces (unscaled, a tensor
// of 1e-36 was 2.5e-5 off).
//
// Two fp16 pieces (11 bits and a sign: 23 bits of the 24 at least), three of four products: half the matrix instructions and
// 5 instead of 8 ns a number and SIMD of splitting.  fp16's range is met by a scale for every channel of a workgroup's tile, a
// power of two taken from the largest number of the channel so far: tile by tile the numbers, still in registers, are compared
// with fp16's range, and where one lies beyond it the channel's scale and the sums so far change to the new one (`rescale`;
// always in a workgroup's first tile, rarely later).  A number down to 2^-16 of its channel's largest has its 23 bits, a
// smaller one an error of 2^-39 of that.  That is less than fp32's roundings of a sum that the channel's larger numbers enter, but
// all there is of one whose larger numbers meet only zeros: such results are found at the end, by their own size (`weigh`), looked
// at more closely, and summed in full (64 -> 64 @ 32x32 / 512 -> 512 @ 4x4, N = 128 / 512, 48 / 101 us: 70 / 126 where the products are
// so sparse that many results are zero, 4 to 5 times as long where every other image is 2^26 larger and meets zeros).  The product
// left out is 2^-22 of the whole at most, where every number has the same bits behind its eleventh (all 1 + 2^-11, N = 128: 2.4e-7
// off, bf16 pieces 1.1 to 2.4e-7).  Of normally distributed numbers what the pieces leave out and what the core rounds inside of
// products of 22 bits is 1e-7 of a result, whatever the length of its sums, so this is the form of long sums: of the 32-wide tiles
// (VGG-19's run, N = 128: 4.5e-7 off with bf16 pieces, 2.8e-7; N = 16 to 40: 2.5 -> 2.1e-7) and of 4x4 planes
// (exact_x3_planes.hip), where it is no further from 64 bits; 16-wide tiles, whose sums are short or kept apart (64 -> 64 @ 8x8,
// N = 50: 0.86e-7, fp16 pieces 1.1e-7), keep bf16 pieces but for a run's strided and longest ones (exact_x3_mix.hip), with all four
// products.
// 64 -> 64 @ 32x32 / 256 -> 256 @ 8x8, N = 128: 62 / 59 us with bf16 pieces, 48 / 44; VGG-19's run 490 -> 342 us.
//
// What holds an infinity or a NaN, or numbers too large for the scale of bf16 pieces (beyond 2^111, sums beyond 2^96), or, in fp16
// pieces, more than a few results of numbers too small beside their channel's largest, is recomputed by its workgroup on the fp32
// matrix core, from the same tiles: the pieces would make NaNs of infinities.
//
// Implicit GEMM, rows = output channels k, columns = (input channel, filter row), reduction = "slots": the columns
// of X (stride 1) or of one phase of X (column mod stride), eight consecutive slots of one output row being one
// 16-byte chunk -- the operand of one lane.  The filter column s is applied by shifting the dY operand, in
// registers, by the distance between a slot and the output column that sees it through tap s (shift_of): a word
// read from each side of the chunk and four v_alignbit serve all filter rows and channels, and every X operand is
// one aligned 16-byte LDS read.
//
// A workgroup owns SH output channels x NTC * SH columns and a range of tiles (nti images x ht output rows x twc
// chunks, at most NCH chunks); its four wavefronts take a quarter of a tile's chunks each, with the whole output
// tile in their accumulators, and add them up through LDS at the end, so that a workgroup writes one partial
// result.  All irregularity -- odd widths, any padding, strides, ragged last tiles, any alignment -- is met while
// staging: dY and X rows are loaded in 16-byte pieces (4-byte aligned), split, and written to LDS as chunks of
// each piece, zero outside the tensors.  Two workgroups and more share a CU: one stages while another multiplies.  Timestamps
// (64 -> 64 @ 32x32, N = 128, 512 workgroups of 8 tiles, 36 us each): set-up and first loads 4.3, the first tile's scales 2.4,
// then a tile 0.7 of splitting, 0.5 of asking for the next, 1.4 of matrix instructions (0.9 alone), 0.4 at barriers; the
// exchange and write-out 4.3; loads are never waited for.
// bf16 inputs are their own only piece: the same kernel with one product per pair serves the bf16 shapes that
// exact_bf16_kernel.hpp does not take.
#pragma once
#include <type_traits>

#include "exact_common.hpp"

namespace wgrad {

typedef __bf16 x3_bf8 __attribute__((ext_vector_type(8)));
typedef _Float16 x3_h8 __attribute__((ext_vector_type(8)));
typedef _Float16 x3_h2 __attribute__((ext_vector_type(2)));
typedef float x3_f16 __attribute__((ext_vector_type(16)));
typedef uint32_t x3_u4 __attribute__((ext_vector_type(4)));

// Division of any 32-bit number by a run-time constant: the estimate is at most one low, and is put right.
struct X3Div {
    uint32_t d, m;
    __host__ __device__ X3Div() : d(1), m(0xffffffffu) {}
    __host__ explicit X3Div(uint32_t div) : d(div), m(div > 1 ? (uint32_t)((1ull << 32) / div) : 0xffffffffu) {}
    __device__ __forceinline__ void divmod(uint32_t n, uint32_t &q, uint32_t &r) const
    {
        q = __umulhi(n, m);
        r = n - q * d;
        if (r >= d) { ++q; r -= d; }
    }
};

struct X3Shape {
    Geometry g;
    int per_prob, ktiles, ctiles, splits;
    int nti, ht, iht, twc;       // tile: images, output rows, input rows, chunks per row
    int h_tiles, w_tiles, n_groups;
    int body;                    // of a launch that mixes variants (exact_x3_mix.hip)
    int nch;                     // live chunks of a tile (the table points the rest at a chunk of zeros)
    int ch;                      // channels staged per column tile
    int packed;                  // columns numbered c * R + r; otherwise column tile t is filter row t of SH channels
    int halo;                    // staged rows of dY carry their neighbours' words (tiles that are not whole rows)
    int vlo, xcol0;              // slot 0: its dY column, its X column in phase 0
    FastDiv d_nch, d_twc, d_ht, d_xrow, d_iht, d_htiles, d_wtiles, d_r, d_rows;      // (d_rows: output rows of a tile)
    X3Div d_prob, d_ctiles, d_ktiles;
    int tiles_each, tiles_more;  // tiles of a split; the first tiles_more splits have one more
};

constexpr int kX3MultiMax = 9;       // groups per launch
constexpr int kX3Tensors = 24;       // problems per launch
struct X3Multi {
    int n;
    int begin[kX3MultiMax + 1];      // first workgroup of each group (multiples of 8); begin[n] = grid size
    int count[kX3MultiMax];
    int first[kX3MultiMax];          // the group's first problem in the tensor tables
    X3Shape s[kX3MultiMax];
    const void *X[kX3Tensors], *dY[kX3Tensors];
    float *out[kX3Tensors];          // per problem: dW when splits == 1, else partials [splits][K][C*R*S]
};
static_assert(sizeof(X3Multi) <= 4096, "kernel arguments");

// filter column s of a filter of width S at stride SW: the phase of X it reads, and slot - output column
__host__ __device__ constexpr int x3_shift(int s, int S, int SW) { return (s - S / 2 + 8 * SW) / SW - 8; }
__host__ __device__ constexpr int x3_phase(int s, int S, int SW) { return (s - S / 2 + 8 * SW) % SW; }

// A = dY chunk as words w[0..3] with its neighbour words; element i of the result is element i - D of the row.
template <int D>
__device__ __forceinline__ x3_u4 x3_shifted(uint32_t L, x3_u4 w, uint32_t R)
{
    x3_u4 o;
    auto mid = [](uint32_t lo, uint32_t hi) { return __builtin_amdgcn_alignbit(hi, lo, 16); };
    if (D == 0) o = w;
    else if (D == -1) o = x3_u4{mid(w[0], w[1]), mid(w[1], w[2]), mid(w[2], w[3]), mid(w[3], R)};
    else if (D == 1) o = x3_u4{mid(L, w[0]), mid(w[0], w[1]), mid(w[1], w[2]), mid(w[2], w[3])};
    else if (D == -2) o = x3_u4{w[1], w[2], w[3], R};
    else o = x3_u4{L, w[0], w[1], w[2]};
    return o;
}

constexpr int kX3Bf16 = 0, kX3Three = 1, kX3Half = 2;       // bf16 inputs; fp32 as three bf16 pieces, as two fp16 pieces

constexpr float kX3Scale = 65536.f, kX3Unscale = 1.f / (kX3Scale * kX3Scale);      // bf16 pieces: of an operand; of a sum of products
// Two fp32 numbers, scaled -> one word (bf16 pair) of each of three pieces
__device__ __forceinline__ void x3_split3(float x0, float x1, float scale, uint32_t &h, uint32_t &m, uint32_t &l)
{
    x0 *= scale;
    x1 *= scale;
    // (written out: from a conversion in C the compiler makes a second instruction for the low half alone)
    auto pk = [](float a, float b) {
        uint32_t v;
        asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(v) : "v"(a), "v"(b));
        return v;
    };
    h = pk(x0, x1);
    const float r0 = x0 - __uint_as_float(h << 16), r1 = x1 - __uint_as_float(h & 0xffff0000u);
    m = pk(r0, r1);
    const float q0 = r0 - __uint_as_float(m << 16), q1 = r1 - __uint_as_float(m & 0xffff0000u);
    l = pk(q0, q1);
}

// fp16 pieces: the power of two that takes a channel's numbers to at most 2^15, given the bits of the largest so far (that to 2^14 at
// least; what is below 2^-111 is scaled by 2^126, where fp32's smallest step is one that fp16 has), and kX3Unset for a channel that
// has only zeros yet.
constexpr int kX3Unset = 127;
constexpr uint32_t kX3Finite = 0x7f7fffffu;             // an infinity's channel is scaled like that of the largest number
__device__ __forceinline__ int x3_exponent(uint32_t top) { const int e = 141 - (int)(top >> 23); return top == 0 ? kX3Unset : (e < kX3Unset ? e : kX3Unset - 1); }
__device__ __forceinline__ float x3_power(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }
constexpr float kX3Most = 65504.f;                      // fp16's largest number

// What fp16 pieces of scaled numbers leave out: 2^-23 of a number from kX3Whole on, 2^-25 of one below, which from kX3Coarse
// on is 2^-9 of it at most: no product of such numbers is lost altogether.  Of a sum of n products no more than m 2^-10 is left
// out that way, m of their 2 n numbers being below kX3Whole: within n roundings of fp32, 2^-24 each, of a sum of m kX3Need / n.
constexpr float kX3Whole = 0x1p-2f, kX3Coarse = 0x1p-16f, kX3Need = 0x1p14f;
constexpr int kX3Few = 32;                              // results of a workgroup that are summed by themselves (x3_dot)

// Two fp32 numbers, scaled -> one word (fp16 pair) of each piece.  (v_fma_mixlo_f16, which would scale, subtract and round at
// once, takes 3.6 ns a SIMD, these 1.2, 1.2, 1.8, 1.9, 1.9 and 1.8.)
__device__ __forceinline__ void x3_split2(float x0, float x1, float scale, uint32_t &h, uint32_t &l)
{
    auto pk = [](float a, float b) {
        uint32_t v;
        asm("v_cvt_pk_f16_f32 %0, %1, %2" : "=v"(v) : "v"(a), "v"(b));
        return v;
    };
    h = pk(x0 * scale, x1 * scale);
    float r0, r1;
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(r0) : "v"(x0), "v"(scale), "v"(h));
    asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r1) : "v"(x1), "v"(scale), "v"(h));
    l = pk(r0, r1);
}

// A channel's scale as its items keep it, given the largest number so far: an infinity for the channel that has only zeros yet, whose
// first other number is then beyond fp16's range (and 0 x infinity, a NaN, is not); and the scale that the split takes.
__device__ __forceinline__ float x3_scale(uint32_t top) { return top == 0 ? __builtin_inff() : x3_power(x3_exponent(top)); }
__device__ __forceinline__ float x3_finite(float scale) { return __builtin_amdgcn_fmed3f(scale, -x3_power(kX3Unset), x3_power(kX3Unset)); }

// Whether an item of a thread (a run of numbers of one channel, the largest given) lies beyond fp16's range at its channel's scale.
struct X3Range {
    float hi = 0.f;
    __device__ __forceinline__ void item(float largest, float scale) { hi = __builtin_fmaxf(hi, largest * __builtin_fabsf(scale)); }
    __device__ __forceinline__ bool over() const { return hi > kX3Most; }
};
// N numbers of a channel: how many are not zero and below kX3Whole at its scale, and whether one is below kX3Coarse (bit 31).
template <int N>
__device__ __forceinline__ uint32_t x3_small(const uint32_t *v, float scale)
{
    const float inverse = __uint_as_float(0x7f000000u - (__float_as_uint(scale) & 0x7fffffffu));     // (a channel of zeros: an infinity)
    auto twice = [](float x) { return (__float_as_uint(x) << 1) - 2u; };
    const uint32_t whole = twice(kX3Whole * inverse), coarse = twice(kX3Coarse * inverse);
    uint32_t n = 0, least = ~0u;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t m = (v[i] - 1u) << 1;            // twice a number's magnitude; most of a zero's
        n += m < whole;
        least = m < least ? m : least;
    }
    return n | (least < coarse ? 1u << 31 : 0u);
}
template <int N>
__device__ __forceinline__ float x3_largest(const uint32_t *v)
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < N; i += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, __builtin_fabsf(__uint_as_float(v[i]))), __builtin_fabsf(__uint_as_float(v[i + 1])));
    return m;
}

// A wavefront's sum of `count` products of fp32 numbers, in 64 bits; at(e, xi, yi): the places of the e-th, false if there is none
template <class F>
__device__ __forceinline__ double x3_dot(const float *X, const float *dY, int count, F at)
{
    double sum = 0;
#pragma unroll 1
    for (int e0 = threadIdx.x & 63; e0 < count; e0 += 64 * 8) {
        float x[8], y[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            long xi, yi;
            const bool live = e0 + 64 * u < count && at(e0 + 64 * u, xi, yi);
            x[u] = X[live ? xi : 0];
            y[u] = live ? dY[live ? yi : 0] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += y[u] == 0.f ? 0. : (double)x[u] * y[u];
    }
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    return sum;
}

// v = four columns loaded at a column clamped into the row, d = wanted column - loaded column: the wanted four,
// zero where they lie outside the row
__device__ __forceinline__ void x3_realign(float (&v)[4], int d)
{
    if (d >= 0) {
        if (d & 1) { v[0] = v[1]; v[1] = v[2]; v[2] = v[3]; v[3] = 0.f; }
        if (d & 2) { v[0] = v[2]; v[1] = v[3]; v[2] = v[3] = 0.f; }
        if (d >= 4) v[0] = v[1] = v[2] = v[3] = 0.f;
    } else {
        const int e = -d;
        if (e & 1) { v[3] = v[2]; v[2] = v[1]; v[1] = v[0]; v[0] = 0.f; }
        if (e & 2) { v[3] = v[1]; v[2] = v[0]; v[0] = v[1] = 0.f; }
        if (e >= 4) v[0] = v[1] = v[2] = v[3] = 0.f;
    }
}

template <int KIND>
__device__ __forceinline__ void x3_mfma(x3_f16 &z, x3_u4 a, x3_u4 b)
{
    if constexpr (KIND == kX3Half) z = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(x3_h8, a), __builtin_bit_cast(x3_h8, b), z, 0, 0, 0);
    else z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(x3_bf8, a), __builtin_bit_cast(x3_bf8, b), z, 0, 0, 0);
}
template <int KIND>
__device__ __forceinline__ void x3_mfma(float4_t &z, x3_u4 a, x3_u4 b)
{
    if constexpr (KIND == kX3Half) z = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(x3_h8, a), __builtin_bit_cast(x3_h8, b), z, 0, 0, 0);
    else z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(x3_bf8, a), __builtin_bit_cast(x3_bf8, b), z, 0, 0, 0);
}

// KIND: the pieces of a number (bf16 inputs are their own only piece).  SH: rows and columns of the matrix instruction (32: 32x32x16, 16: 16x16x32).  NTC: column tiles.  S: filter width.
// SW: column stride.  RAG: rows whose width is not a multiple of four, or that start before column 0 of a tensor.
// HALO: tiles may be parts of rows.  NCH: chunks of a tile; DI, XI:
// staging items per thread; KP, CP: LDS chunks per channel of dY and of X (odd: conflict-free 16-byte reads); CH: channels
// of X (compile-time, so that the operand reads have immediate offsets).
template <int KIND_, int SH_, int NTC_, int S_, int SW_, bool RAG_, bool HALO_, int NCH_, int DI_, int XI_, int KP_, int CP_, int CH_>
struct X3Config {
    static constexpr int SH = SH_, NTC = NTC_, S = S_, SW = SW_, NCH = NCH_, DI = DI_, XI = XI_, KP = KP_, CP = CP_, CH = CH_, NW = 4;
    static constexpr int KIND = KIND_;
    static constexpr bool BF = KIND == kX3Bf16, HALF = KIND == kX3Half, RAG = RAG_, HALO = HALO_;
    static constexpr int NP = BF ? 1 : (HALF ? 2 : 3);                  // pieces of a number
    static constexpr bool OWN = KIND == kX3Three && SH == 16 && S <= 3;   // the smaller products have sums of their own
    static constexpr bool STEP = HALF && SH == 16;                        // a step's products have
    static constexpr int DR = BF && !RAG ? 4 : 8;                       // registers of a chunk on its way to LDS
    static constexpr int kOcc = (SH == 32 && NTC > 1) || SW > 1 || S > 3 ? 2 : (RAG || SH == 32 || (OWN && NTC > 1) ? 3 : 4);      // workgroups that share a CU
    static constexpr int kDy = SH * KP * 16, kX = CH * CP * 16;         // bytes of one piece
    static constexpr int kBuf = 16 + NP * kDy + 16 + NP * kX;            // of a tile (16 spare bytes before each: a word left of a chunk 0)
    static constexpr int kTop = HALF ? ((SH + CH) * 8 + 15) / 16 * 16 : 0;      // the channels' largest numbers and scales
    static constexpr int kScales = HALF ? (DI + XI + (HALO ? 1 : 0)) * kBlock * 4 : 0;      // the scales of every thread's staging items
    static constexpr bool PARK = HALF && HALO && SH == 32 && NTC > 1;     // the items themselves are kept in LDS too
    static constexpr int kItems = PARK ? (DI + XI + 1) * kBlock * 8 : 0;
    static constexpr int NB = HALF ? NTC * S * (SH * SH / 64) : 0, WORDS = (NB + 31) / 32;      // a lane's sums, a bit each
    static constexpr int kFix = NCH * 4 + 16 + kTop + WORDS * 256;      // the chunk table, flags, the channels' scales, those bits
    static constexpr int kHead = kFix + kScales + kItems;               // ... and what the loop alone needs
    static constexpr int kTail = NW * NTC * S * SH * SH * 2;            // the final exchange: half of every wavefront's sums
    static constexpr int kCounts = HALF ? 2 * (SH + CH) * 4 + WORDS * 256 : 0;      // the second look at a workgroup's numbers (behind the tile, whose zeros stay)
    static constexpr int kLds = kHead + kBuf + kCounts > kFix + kTail ? kHead + kBuf + kCounts : kFix + kTail;
};

template <class T>
__device__ __forceinline__ void x3_body(const X3Shape &p, const void *const *Xt, const void *const *dYt, float *const *outt,
                                        char *smem, int bid, int nblk)
{
    constexpr int SH = T::SH, NTC = T::NTC, S = T::S, SW = T::SW, NCH = T::NCH, DI = T::DI, XI = T::XI, KP = T::KP, CP = T::CP,
                  NW = T::NW, NTHR = 64 * NW;
    constexpr int KIND = T::KIND;
    constexpr bool BF = T::BF, HALF = T::HALF, RAG = T::RAG, HALO = T::HALO;
    constexpr int NP = T::NP, DR = T::DR, ESZ = BF ? 2 : 4;
    constexpr int CPS = 64 / SH;                        // chunks per step (lane groups of an operand)
    constexpr int NST = NCH / (CPS * NW);                // steps per wavefront and tile
    constexpr int AV = SH * SH / 64;                    // accumulator registers per output tile
    static_assert(NCH % (CPS * NW) == 0 && DI * NTHR >= SH * NCH, "tile");
    typedef float acc_t __attribute__((ext_vector_type(AV)));

    const Geometry &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wq = tid >> 6;
    const int i = lane & (SH - 1), kk = lane / SH;
    const int R = g.R, CRS = g.C * R * S, L = g.Ho * g.Wo;

    uint32_t *const tab = (uint32_t *)smem;                       // [NCH] chunk -> A offset | B offset << 12 | mask left << 30 | mask right << 31
    uint32_t *const flag = tab + NCH;                        // set when the pieces cannot represent a tile
    uint32_t *const over = flag + 1;                         // set when a tile's numbers ask for smaller scales
    uint32_t *const top = flag + 4;                          // per channel of dY [SH] and X [CH]: bits of the largest number so far
    int *const expo = (int *)(top + SH + T::CH);             // ... and the exponent of its scale
    constexpr int NB = T::NB, WORDS = T::WORDS;
    uint32_t *const mark = (uint32_t *)(smem + T::kFix - WORDS * 256);      // [WORDS][64]: whether a sum is known to be well held (`weigh`)
    // Per staging item of a thread, the scale of its channel; PARK: what is known of the item.  (In registers these would be
    // what spills, and a reload among the loads of a tile waits for all of those: 64 -> 64 @ 224x224, N = 4, 82 us
    // against 79.)
    float *const scales = (float *)(smem + T::kFix);
    auto scale_at = [&](int item) -> float & { return scales[item * NTHR + (int)threadIdx.x]; };
    uint2 *const parked = (uint2 *)(smem + T::kFix + T::kScales);
    char *const buf = smem + T::kHead;                  // dY [NP][SH][KP] chunks, X [NP][CH][CP] chunks
    constexpr int dy_piece = T::kDy, x_piece = T::kX, kDyAt = 16, kXAt = 16 + NP * T::kDy + 16;

    const int logical_all = xcd_contiguous_id(bid, nblk);
    // (divisions by numbers that the host has prepared: the compiler's, of run-time numbers, are a hundred instructions each)
    uint32_t prob, logical, rest, coltile, ktile, split;
    p.d_prob.divmod((uint32_t)logical_all, prob, logical);
    p.d_ctiles.divmod(logical, rest, coltile);
    p.d_ktiles.divmod(rest, split, ktile);
    const char *const Xp = (const char *)Xt[prob], *const dYp = (const char *)dYt[prob];
    const int k0 = (int)ktile * SH;
    int c_first = (int)coltile * SH;
    if (p.packed) {
        uint32_t q, r;
        p.d_r.divmod(coltile * NTC * SH, q, r);
        c_first = (int)q;
    }

    const int wt_begin = (int)split * p.tiles_each + min((int)split, p.tiles_more);
    const int wt_end = wt_begin + p.tiles_each + ((int)split < p.tiles_more);

    // ---- staging items, decoded once: where in the tile (LDS chunk | row << 20 | chunk column << 28, all ones: none) and the
    //      byte offset of the row (of the chunk, where rows are whole) from the tile's first row ----
    constexpr uint32_t kDead = 0x80000000u;
    uint32_t d_at[DI], d_off[DI], x_at[XI], x_off[XI], h_at = ~0u, h_off = kDead;
    auto at_dst = [](uint32_t a) { return (a & 0xffffu) * 16u; };
    auto at_row = [](uint32_t a) { return (int)(a >> 20 & 255u); };
    auto at_wc = [](uint32_t a) { return (int)(a >> 28); };
#pragma unroll
    for (int u = 0; u < DI; ++u) {
        const int e = tid + u * NTHR;
        d_at[u] = ~0u; d_off[u] = kDead;
        if (e < SH * p.nch) {
            uint32_t k_l, chk, row, wc, n_l, h_l;
            p.d_nch.divmod(e, k_l, chk);
            p.d_twc.divmod(chk, row, wc);
            p.d_ht.divmod(row, n_l, h_l);
            const uint32_t idx = HALO && p.halo ? 1 + row * (p.twc + 1) + wc : chk;
            if (k0 + (int)k_l < g.K) d_at[u] = (k_l * KP + idx) | h_l << 20 | wc << 28;
            d_off[u] = (n_l * g.K + k_l) * L + h_l * g.Wo;
            d_off[u] = d_at[u] == ~0u ? kDead : (d_off[u] + (RAG ? 0 : wc * 8)) * ESZ;
        }
    }
    if (HALO && p.halo && tid < SH * p.nti * p.ht * 2) {           // one of a row's two neighbour words per thread
        uint32_t k_l, row, n_l, h_l;
        const uint32_t side = tid & 1;
        p.d_rows.divmod(tid >> 1, k_l, row);
        p.d_ht.divmod(row, n_l, h_l);
        if (k0 + (int)k_l < g.K) h_at = (k_l * KP + row * (p.twc + 1) + (side ? p.twc + 1 : 0)) | h_l << 20 | side << 28;
        if (h_at != ~0u) h_off = ((n_l * g.K + k_l) * L + h_l * g.Wo) * ESZ;
    }
#pragma unroll
    for (int u = 0; u < XI; ++u) {
        const int e = tid + u * NTHR;
        x_at[u] = ~0u; x_off[u] = kDead;
        if (e < p.ch * (int)p.d_xrow.d) {
            uint32_t c_l, rem, row, wc, n_l, ih_l;
            p.d_xrow.divmod(e, c_l, rem);
            p.d_twc.divmod(rem, row, wc);
            p.d_iht.divmod(row, n_l, ih_l);
            if (c_first + (int)c_l < g.C) x_at[u] = (c_l * CP + row * p.twc * SW + wc) | ih_l << 20 | wc << 28;
            x_off[u] = (n_l * g.C + c_l) * (g.H * g.W) + ih_l * g.W;
            x_off[u] = x_at[u] == ~0u ? kDead : (x_off[u] + (RAG ? 0 : wc * 8 * SW)) * ESZ;
        }
    }

    auto park = [&](int item, uint32_t at, uint32_t off) { parked[item * NTHR + tid] = uint2{at, off}; };
    if constexpr (T::PARK) {
#pragma unroll
        for (int u = 0; u < DI; ++u) park(u, d_at[u], d_off[u]);
#pragma unroll
        for (int u = 0; u < XI; ++u) park(DI + u, x_at[u], x_off[u]);
        park(DI + XI, h_at, h_off);
    }
    // (opaque: the fields are taken out of the word where they are used, not kept in registers of their own across the loop)
    auto fresh = [](uint32_t v) { asm volatile("" : "+v"(v)); return v; };
    auto item = [&](int item, uint32_t at, uint32_t off) {
        if constexpr (T::PARK) return parked[item * NTHR + (int)threadIdx.x];
        else return uint2{fresh(at), off};
    };
    uint32_t dr[DI][DR], xr[XI][DR * SW], hr[2];
    struct Tile { int n0, h0, wc0; };
    auto tile_of = [&](int wt) {
        uint32_t q, wti, ng, hti;
        p.d_wtiles.divmod(wt, q, wti);
        p.d_htiles.divmod(q, ng, hti);
        return Tile{(int)ng * p.nti, (int)hti * p.ht, (int)wti * p.twc};
    };
    // Loads go through a buffer descriptor from the tile's first row to the end of the tensor, 2^31 bytes at most; what is to be
    // zero is asked for beyond that, as the images past the last are anyway, and the hardware answers 0 without a memory
    // access: nothing is masked afterwards.
    // (The whole offset is the lanes': the check subtracts a scalar one from the size, which wraps where it is the larger.  Wide
    // padding puts a tile's first row behind the plane, and at the tensor's end nothing is left.)
    auto rsrc_of = [&](const char *base, long at, long elems) {
        const long left = elems > at ? (elems - at) * ESZ : 0;
        return __builtin_amdgcn_make_buffer_rsrc((void *)(base + at * ESZ), 0, left < (long)kDead ? (uint32_t)left : kDead, 0x00020000);
    };
    auto load4 = [&](__amdgpu_buffer_rsrc_t rs, uint32_t off, uint32_t *v) {      // whole pieces of a row
        if constexpr (BF) {
            const auto q = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
            v[0] = q[0]; v[1] = q[1];
        } else {
            const x3_u4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = q[e];
        }
    };
    // Four columns of a ragged row (byte offset `row`) from any column.  fp32 rows are read at a column clamped into the
    // row and realigned when they are staged; bf16 rows (2-byte aligned) element by element.
    auto load4_ragged = [&](__amdgpu_buffer_rsrc_t rs, bool live, uint32_t row, int col, int width, uint32_t *v) {
        if constexpr (BF) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = __builtin_amdgcn_raw_buffer_load_b16(rs, live && (unsigned)(col + e) < (unsigned)width ? row + (uint32_t)(col + e) * 2u : kDead, 0, 0);
        } else {
            const int c = col < 0 ? 0 : (col > width - 4 ? width - 4 : col);
            load4(rs, live && (unsigned)(col + 3) < (unsigned)(width + 3) ? row + (uint32_t)c * 4u : kDead, v);
        }
    };
    constexpr bool FIX = RAG && !BF, SHIFT = FIX && SW == 1;
    auto fix4 = [&](int col, int width, uint32_t *v) {   // the four that were clamped into the row, back to their columns
        float q[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) q[e] = __uint_as_float(v[e]);
        x3_realign(q, col - (col < 0 ? 0 : (col > width - 4 ? width - 4 : col)));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(q[e]);
    };
    auto load_tile = [&](int wt) {
        const Tile t = tile_of(wt);
        const int h_left = g.Ho - t.h0;
        const uint32_t wy = HALO ? t.wc0 * 8 * ESZ : 0, wx = wy * SW;   // the tile's first column
        const auto yb = rsrc_of(dYp, ((long)t.n0 * g.K + k0) * L + (long)t.h0 * g.Wo, (long)g.N * g.K * L);
#pragma unroll
        for (int u = 0; u < DI; ++u) {
            const auto [at, off0] = item(u, d_at[u], d_off[u]);
            if constexpr (RAG) {
                const bool live = at_row(at) < h_left;
                const int col = (at_wc(at) + t.wc0) * 8 + p.vlo;
                load4_ragged(yb, live, off0, col, g.Wo, dr[u]);
                load4_ragged(yb, live, off0, col + 4, g.Wo, dr[u] + DR / 2);
            } else {
                const uint32_t off = at_row(at) < h_left ? off0 + wy : kDead;
                const int left = g.Wo - t.wc0 * 8 - at_wc(at) * 8;
                load4(yb, !HALO || left > 0 ? off : kDead, dr[u]);
                load4(yb, left > 4 ? off + 4 * ESZ : kDead, dr[u] + DR / 2);
            }
        }
        if (HALO && p.halo) {
            const auto [at, off0] = item(DI + XI, h_at, h_off);
            const int col = (t.wc0 + (at_wc(at) ? p.twc : 0)) * 8 + p.vlo - (at_wc(at) ? 0 : 2);
            const bool live = at_row(at) < h_left;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t off = live && (unsigned)(col + e) < (unsigned)g.Wo ? off0 + (uint32_t)(col + e) * ESZ : kDead;
                if constexpr (BF) hr[e] = __builtin_amdgcn_raw_buffer_load_b16(yb, off, 0, 0);
                else hr[e] = __builtin_amdgcn_raw_buffer_load_b32(yb, off, 0, 0);
            }
        }
        // (the first input row of a tile may lie above the plane: offsets count from it, dead rows are never asked for)
        const int ih0 = t.h0 * g.sh - g.ph;
        const auto xb = rsrc_of(Xp, ((long)t.n0 * g.C + c_first) * g.H * g.W + (long)ih0 * g.W, (long)g.N * g.C * g.H * g.W);
#pragma unroll
        for (int u = 0; u < XI; ++u) {
            const auto [at, off0] = item(DI + u, x_at[u], x_off[u]);
            const bool in = (unsigned)(ih0 + at_row(at)) < (unsigned)g.H;
            if constexpr (RAG) {
                const int col = (at_wc(at) + t.wc0) * 8 * SW + p.xcol0;
#pragma unroll
                for (int q = 0; q < 2 * SW; ++q) load4_ragged(xb, in, off0, col + 4 * q, g.W, xr[u] + DR / 2 * q);
            } else {
                const uint32_t off = in ? off0 + wx : kDead;
                const int left = g.W - t.wc0 * 8 * SW - at_wc(at) * 8 * SW;
#pragma unroll
                for (int q = 0; q < 2 * SW; ++q) load4(xb, left > 4 * q ? off + 4 * q * ESZ : kDead, xr[u] + DR / 2 * q);
            }
        }
    };
    // The matrix core rounds downwards what it adds to a larger sum, and most of the products are small: the sums of the
    // products come out low, by as much as 4.5e-7 of the result's size (bf16 pieces, 64 -> 64 @ 224x224, N = 4).  Every other
    // workgroup of a reduction sums the negated products, so that what they lose cancels.
    const float sign = split & 1 ? -1.f : 1.f, dy_scale = sign * kX3Scale;
    auto range = [&]() {
        X3Range r;
#pragma unroll
        for (int u = 0; u < DI; ++u) r.item(x3_largest<8>(dr[u]), scale_at(u));
        if (HALO && p.halo) r.item(x3_largest<2>(hr), scale_at(DI + XI));
#pragma unroll
        for (int u = 0; u < XI; ++u) r.item(x3_largest<8 * SW>(xr[u]), scale_at(DI + u));
        return r;
    };
    // a chunk's pieces (plain: its fp32 numbers, in the place of the first two) to LDS; v(e): its element e (fp32 bits, or bf16
    // bits in the low half); lo, hi: bits by which its two groups of four columns, loaded clamped into the row, lie too high
    auto put = [&](auto v, char *dst, int piece, float scale, uint32_t lo, uint32_t hi, auto plain) {
        if constexpr (decltype(plain)::value && !BF) {
            *(x3_u4 *)dst = x3_u4{v(0), v(1), v(2), v(3)};
            *(x3_u4 *)(dst + piece) = x3_u4{v(4), v(5), v(6), v(7)};
            return;
        }
        x3_u4 w[NP];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (BF) w[0][e] = __builtin_amdgcn_perm(v(2 * e + 1), v(2 * e), 0x05040100u);
            else {
                uint32_t a, b, c;
                if constexpr (HALF) x3_split2(__uint_as_float(v(2 * e)), __uint_as_float(v(2 * e + 1)), scale, a, b);
                else x3_split3(__uint_as_float(v(2 * e)), __uint_as_float(v(2 * e + 1)), scale, a, b, c);
                w[0][e] = a; w[1][e] = b;
                if constexpr (!HALF) w[2][e] = c;
            }
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            if constexpr (SHIFT) {
                const uint64_t a = ((uint64_t)w[q][1] << 32 | w[q][0]) >> (lo & 63), b = ((uint64_t)w[q][3] << 32 | w[q][2]) >> (hi & 63);
                w[q] = x3_u4{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
            }
            *(x3_u4 *)(dst + q * piece) = w[q];
        }
    };
    // columns by which the four of `col` on, loaded at a column clamped into the row from the right, lie too far right (of four
    // that lie outside altogether nothing was loaded)
    auto behind = [](int col, int width) { return (uint32_t)(col > width - 4 ? col - (width - 4) : 0); };
    // element i of a run of columns in staging registers
    auto elem = [&](const uint32_t *v, int i) -> uint32_t {
        if constexpr (DR == 4) return i & 1 ? v[i / 2] >> 16 : v[i / 2];
        else return v[i];
    };
    auto commit_tile = [&](int wt, auto plain) {
        Tile t{0, 0, 0};
        if (FIX) t = tile_of(wt);
        // (rows that start left of the tensor's were also clamped from the left: rare, and put right in registers)
        const bool regs = SW > 1 || decltype(plain)::value;
#pragma unroll
        for (int u = 0; u < DI; ++u) {
            const auto [at, off0] = item(u, d_at[u], d_off[u]);
            uint32_t lo = 0, hi = 0;
            if constexpr (FIX) {
                const int col = (at_wc(at) + t.wc0) * 8 + p.vlo;
                if (regs || p.vlo < 0) {
                    fix4(col, g.Wo, dr[u]);
                    fix4(col + 4, g.Wo, dr[u] + 4);
                } else {
                    lo = behind(col, g.Wo) * 16u;
                    hi = behind(col + 4, g.Wo) * 16u;
                }
            }
            if (at != ~0u) {
                if constexpr (DR == 4) *(x3_u4 *)(buf + kDyAt + at_dst(at)) = x3_u4{dr[u][0], dr[u][1], dr[u][2], dr[u][3]};
                else put([&](int e) { return elem(dr[u], e); }, buf + kDyAt + at_dst(at), dy_piece, HALF ? x3_finite(scale_at(u)) : dy_scale, lo, hi, plain);
            }
        }
        if (HALO && p.halo) {
            const uint32_t at = item(DI + XI, h_at, h_off).x;
            char *const chunk = buf + kDyAt + at_dst(at);
            if (at == ~0u) {
            } else if constexpr (decltype(plain)::value && !BF) {
                *(uint2 *)(chunk + (at_wc(at) ? 0 : dy_piece + 8)) = uint2{hr[0], hr[1]};
            } else {
                uint32_t w[3];
                if constexpr (BF) w[0] = hr[0] | hr[1] << 16;
                else if constexpr (HALF) x3_split2(__uint_as_float(hr[0]), __uint_as_float(hr[1]), x3_finite(scale_at(DI + XI)), w[0], w[1]);
                else x3_split3(__uint_as_float(hr[0]), __uint_as_float(hr[1]), dy_scale, w[0], w[1], w[2]);
#pragma unroll
                for (int q = 0; q < NP; ++q) *(uint32_t *)(chunk + (at_wc(at) ? 0 : 12) + q * dy_piece) = w[q];
            }
        }
#pragma unroll
        for (int u = 0; u < XI; ++u) {
            const auto [at, off0] = item(DI + u, x_at[u], x_off[u]);
            uint32_t lo = 0, hi = 0;
            if constexpr (FIX) {
                const int col = (at_wc(at) + t.wc0) * 8 * SW + p.xcol0;
                if (regs || p.xcol0 < 0) {
#pragma unroll
                    for (int q = 0; q < 2 * SW; ++q) fix4(col + 4 * q, g.W, xr[u] + 4 * q);
                } else {
                    lo = behind(col, g.W) * 16u;
                    hi = behind(col + 4, g.W) * 16u;
                }
            }
            if (at != ~0u) {
                if constexpr (DR == 4 && SW == 1) *(x3_u4 *)(buf + kXAt + at_dst(at)) = x3_u4{xr[u][0], xr[u][1], xr[u][2], xr[u][3]};
                else {
#pragma unroll
                    for (int f = 0; f < SW; ++f)
                        put([&](int e) { return elem(xr[u], e * SW + f); }, buf + kXAt + at_dst(at) + f * p.twc * 16, x_piece, HALF ? x3_finite(scale_at(DI + u)) : kX3Scale, lo, hi, plain);
                }
            }
        }
    };

    load_tile(wt_begin);

    // ---- tables and the chunks of zeros, while the first loads are in flight ----
    for (int q = tid; q < NCH; q += NTHR) {
        uint32_t e = (KP - 1) * 16 | 3u << 30;   // (zeros times the first, finite or recomputed, chunk of X)
        if (q < p.nch) {
            uint32_t row, wc, n_l, h_l;
            p.d_twc.divmod(q, row, wc);
            p.d_ht.divmod(row, n_l, h_l);
            const int a = HALO && p.halo ? 1 + row * (p.twc + 1) + wc : q;
            const int b = ((n_l * p.iht + h_l * g.sh) * p.twc * SW + wc) * 16;
            e = a * 16 | b << 12;
            if (!HALO || !p.halo) e |= (wc == 0 ? 1u << 30 : 0u) | ((int)wc + 1 == p.twc ? 1u << 31 : 0u);
        }
        tab[q] = e;
    }
    if (tid == 0) *flag = *over = 0;
    if constexpr (HALF) {
        if (tid < SH + T::CH) { top[tid] = 0; expo[tid] = kX3Unset; }
        for (int e = tid; e < WORDS * 64; e += NTHR) mark[e] = 0;
#pragma unroll
        for (int u = 0; u < DI + XI + (HALO ? 1 : 0); ++u) scale_at(u) = __builtin_inff();
    }
    for (int e = tid; e < NP * SH; e += NTHR) *(x3_u4 *)(buf + kDyAt + (e * KP + KP - 1) * 16) = x3_u4{0u, 0u, 0u, 0u};
    if (k0 + SH > g.K || c_first + T::CH > g.C) {
        // rows and columns beyond the result are never staged: zeros, so that no left-over bits make infinities of them
        for (int e = tid; e < T::kBuf / 16; e += NTHR) *(x3_u4 *)(buf + e * 16) = x3_u4{0u, 0u, 0u, 0u};
        if (!HALF) __syncthreads();
    }
    if (HALF) __syncthreads();

    acc_t acc[NTC][S];
#pragma unroll
    for (int t = 0; t < NTC; ++t)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int v = 0; v < AV; ++v) acc[t][s][v] = 0.f;

    // 16-wide tiles: the five smaller products have a sum of their own, 2^-8 of the whole, which rounds that much finer; the
    // whole is then rounded once a step instead of six times
    acc_t small[T::OWN ? NTC : 1][T::OWN ? S : 1];
#pragma unroll
    for (int t = 0; t < (T::OWN ? NTC : 1); ++t)
#pragma unroll
        for (int s = 0; s < (T::OWN ? S : 1); ++s)
#pragma unroll
            for (int v = 0; v < AV; ++v) small[t][s][v] = 0.f;

    // column `col` of column tile t: its channel (of those staged) and filter row
    auto column = [&](int t, int col, int &c_l, int &r) {
        c_l = col; r = t;
        if (p.packed) {
            const int q = (int)coltile * NTC * SH + t * SH + col;
            uint32_t c, rr;
            p.d_r.divmod(q < g.C * R ? q : c_first * R, c, rr);
            c_l = (int)c - c_first; r = (int)rr;
        }
        if (c_l >= p.ch) c_l = p.ch - 1;                // a column beyond C: some staged channel, never written out
    };
    // this lane's columns: byte offset of (channel, filter row) in a piece of X
    int coloff[NTC];
    const int row_bytes = p.twc * SW * 16;
#pragma unroll
    for (int t = 0; t < NTC; ++t) {
        int c_l, r;
        column(t, i, c_l, r);
        coloff[t] = c_l * CP * 16 + r * row_bytes;
    }
    const char *const a_row = buf + kDyAt + i * KP * 16, *const Xs = buf + kXAt;
    // the rows of `top` that the thread's staging items belong to (items that there are not load zeros)
    auto item_rows = [&](uint32_t (&row)[DI + XI + 1]) {
        uint32_t rem;
#pragma unroll
        for (int u = 0; u < DI; ++u) {
            p.d_nch.divmod(tid + u * NTHR, row[u], rem);
            if (item(u, d_at[u], d_off[u]).x == ~0u) row[u] = 0;
        }
#pragma unroll
        for (int u = 0; u < XI; ++u) {
            p.d_xrow.divmod(tid + u * NTHR, row[DI + u], rem);
            row[DI + u] = item(DI + u, x_at[u], x_off[u]).x == ~0u ? SH : SH + row[DI + u];
        }
        row[DI + XI] = 0;
        if (HALO && p.halo && item(DI + XI, h_at, h_off).x != ~0u) p.d_rows.divmod(tid >> 1, row[DI + XI], rem);
    };
    // A tile has a number beyond fp16's range at the scale of its channel (in a workgroup's first tile they all do): scales
    // for the largest numbers so far, and the sums so far in units of them.
    auto rescale = [&](bool sums) {
        auto note = [&](int row, const float m) {
            if (m > 0.f) { const uint32_t b = __float_as_uint(m); atomicMax(top + row, b < kX3Finite ? b : kX3Finite); }
        };
        uint32_t row[DI + XI + 1];
        item_rows(row);
#pragma unroll
        for (int u = 0; u < DI; ++u) note((int)row[u], x3_largest<8>(dr[u]));
#pragma unroll
        for (int u = 0; u < XI; ++u) note((int)row[DI + u], x3_largest<8 * SW>(xr[u]));
        if (HALO && p.halo) note((int)row[DI + XI], x3_largest<2>(hr));
        __syncthreads();
#pragma unroll
        for (int u = 0; u < DI + XI + (HALO ? 1 : 0); ++u)
            scale_at(u) = (u < DI || u == DI + XI ? sign : 1.f) * x3_scale(top[row[u]]);
        if (sums) {
            auto change = [&](int row) { return x3_exponent(top[row]) - expo[row]; };
#pragma unroll
            for (int t = 0; t < NTC; ++t) {
                int c_l, r;
                column(t, i, c_l, r);
                const int dc = change(SH + c_l);
#pragma unroll
                for (int v = 0; v < AV; ++v) {
                    const int d = dc + change(SH == 32 ? 8 * (v / 4) + 4 * kk + v % 4 : 4 * kk + v);
#pragma unroll
                    for (int s = 0; s < S; ++s) acc[t][s][v] = __builtin_ldexpf(acc[t][s][v], d);
                    __builtin_amdgcn_sched_barrier(0);       // (one exponent at a time: there are no registers for all)
                }
            }
        }
        __syncthreads();
        if (tid < SH + T::CH) expo[tid] = x3_exponent(top[tid]);
        if (tid == 0) *over = 0;
    };
    for (int wt = wt_begin; wt < wt_end; ++wt) {
        if constexpr (HALF) {
            if (range().over()) *over = 1;
        }
        if (HALF || wt != wt_begin) __syncthreads();    // everyone has left the previous tile
        if constexpr (HALF)
            if (*(volatile uint32_t *)over) rescale(wt != wt_begin);
        // The scheduling fences keep the matrix instructions out of the staging: an instruction that waits for the matrix
        // core holds up what follows it, and then both workgroups of a CU stage while neither multiplies (N = 512,
        // 128 -> 128 @ 16x16: 190 us without them, 155 with).
        __builtin_amdgcn_sched_barrier(0);
        commit_tile(wt, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        if (wt + 1 < wt_end) load_tile(wt + 1);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
#pragma unroll
        for (int st = 0; st < NST; ++st) {
            const uint32_t e = tab[(wq * NST + st) * CPS + kk];
            const char *const ap = a_row + (e & 0xfff);
            const char *const bp = Xs + ((e >> 12) & 0x3fff);
            auto shifted = [&](int qa, x3_u4 (&a)[S]) {
                const x3_u4 w = *(const x3_u4 *)(ap + qa * dy_piece);
                uint32_t lw = *(const uint32_t *)(ap + qa * dy_piece - 4), rw = *(const uint32_t *)(ap + qa * dy_piece + 16);
                if (e & (1u << 30)) lw = 0;
                if (e & (1u << 31)) rw = 0;
                a[0] = x3_shifted<x3_shift(0, S, SW)>(lw, w, rw);
                a[1] = x3_shifted<x3_shift(1, S, SW)>(lw, w, rw);
                a[2] = x3_shifted<x3_shift(2, S, SW)>(lw, w, rw);
                if constexpr (S > 3) a[3] = x3_shifted<x3_shift(3, S, SW)>(lw, w, rw);
                if constexpr (S > 4) a[4] = x3_shifted<x3_shift(4, S, SW)>(lw, w, rw);
            };
            if constexpr (T::STEP) {
                // 16-wide fp16 pieces: a step's products are summed by themselves, and that is added to the whole, which is then
                // rounded once a step, to nearest, and not three times, downwards
                x3_u4 a[2][S];
                shifted(0, a[0]);
                shifted(1, a[1]);
#pragma unroll
                for (int t = 0; t < NTC; ++t)
#pragma unroll
                    for (int f = 0; f < SW; ++f) {
                        const char *const q0 = bp + coloff[t] + f * p.twc * 16;
                        const x3_u4 h = *(const x3_u4 *)q0, l = *(const x3_u4 *)(q0 + x_piece);
                        acc_t z[S];
#pragma unroll
                        for (int s = 0; s < S; ++s)
#pragma unroll
                            for (int v = 0; v < AV; ++v) z[s][v] = 0.f;
#pragma unroll
                        for (int q = 0; q < 4; ++q)     // (all four products: 32 -> 32 @ 16x16 in ResNet-20's run, N = 128, 1.36e-7 off, without the smallest 1.43e-7)
#pragma unroll
                            for (int s = 0; s < S; ++s)
                                if (x3_phase(s, S, SW) == f) x3_mfma<KIND>(z[s], a[q < 2][s], q % 2 == 0 ? l : h);
#pragma unroll
                        for (int s = 0; s < S; ++s)
                            if (x3_phase(s, S, SW) == f) acc[t][s] += z[s];
                    }
                continue;
            }
            // the products of dY's smallest piece first; a piece's shifted operands serve every column tile, X's pieces
            // are read again for each (reads that the LDS has to spare, against 24 registers that the loop has not)
#pragma unroll
            for (int qa = NP - 1; qa >= 0; --qa) {
                x3_u4 a[S];
                shifted(qa, a);
#pragma unroll
                for (int t = 0; t < NTC; ++t) {
#pragma unroll
                    for (int f = 0; f < SW; ++f) {
                        const char *const q0 = bp + coloff[t] + f * p.twc * 16;
#pragma unroll
                        for (int qb = NP - 1 - qa; qb >= 0; --qb) {
                            const x3_u4 b = *(const x3_u4 *)(q0 + qb * x_piece);
#pragma unroll
                            for (int s = 0; s < S; ++s) {
                                if (x3_phase(s, S, SW) != f) continue;
                                acc_t &z = T::OWN && qa + qb ? small[T::OWN ? t : 0][T::OWN ? s : 0] : acc[t][s];
                                x3_mfma<KIND>(z, a[s], b);
                            }
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }

    if constexpr (T::OWN) {
#pragma unroll
        for (int t = 0; t < NTC; ++t)
#pragma unroll
            for (int s = 0; s < S; ++s) acc[t][s] += small[t][s];
    }
    // An infinity, a NaN or a value whose largest piece rounds to infinity makes infinities or NaNs of every product it
    // enters, and an accumulator keeps them: one look at the sums finds what the pieces could not represent.
    float worst[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NTC; ++t)
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int v = 0; v < AV; ++v) worst[v & 3] = fmaf(acc[t][s][v], 0.f, worst[v & 3]);
    const float any = (worst[0] + worst[1]) + (worst[2] + worst[3]);
    if (any != any) *flag = 1;
    // fp16 pieces: numbers far below their channel's largest lose bits, which is nothing to a sum that larger ones enter, and
    // all to one whose larger ones meet only zeros.  Each wavefront's sum of a result's products is at most what the products'
    // magnitudes add up to: a result is well held if one of the four is so large (2 kX3Need) that what the pieces can have left out
    // of n products is within n roundings of fp32 of it; channels of zeros need nothing.  A bit a result: weigh shifts in the sign of
    // beyond(sum, its row's word of `of`, its column's).  Of normally distributed numbers, ReLU's zeros among them, no workgroup in
    // 10^4 has a result without one.
    [[maybe_unused]] auto weigh = [&](uint32_t (&good)[WORDS > 0 ? WORDS : 1], const uint32_t *of, auto beyond) {
        uint32_t nc[NTC];
        x3_u4 nk[AV / 4];
#pragma unroll
        for (int t = 0; t < NTC; ++t) {
            int c_l, r;
            column(t, i, c_l, r);
            nc[t] = of[SH + c_l];
        }
#pragma unroll
        for (int v = 0; v < AV / 4; ++v) nk[v] = *(const x3_u4 *)(of + (SH == 32 ? 8 * v : 0) + 4 * kk);
#pragma unroll
        for (int v = 0; v < AV; ++v)
#pragma unroll
            for (int t = 0; t < NTC; ++t)
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    uint32_t &w = good[((v * NTC + t) * S + s) / 32];
                    w = __builtin_amdgcn_alignbit(w, __float_as_uint(beyond(__builtin_fabsf(acc[t][s][v]), nk[v / 4][v % 4], nc[t])), 31);
                }
    };
    auto bits = [](int w) { return NB - 32 * w < 32 ? (1u << (NB - 32 * w)) - 1u : ~0u; };        // those of a word
    if constexpr (HALF) {
        uint32_t good[WORDS] = {};
        weigh(good, top, [](float sum, uint32_t row, uint32_t) { return (row == 0 ? -1.f : 2.f * kX3Need) - sum; });
#pragma unroll
        for (int t = 0; t < NTC; ++t) {
            int c_l, r;
            column(t, i, c_l, r);
            uint32_t of[WORDS] = {};                        // bits of this column
#pragma unroll
            for (int e = 0; e < NB; ++e)
                if (e / S % NTC == t) of[e / 32] |= 1u << ((NB - e / 32 * 32 < 32 ? NB - e / 32 * 32 : 32) - 1 - e % 32);
#pragma unroll
            for (int w = 0; w < WORDS; ++w) good[w] |= top[SH + c_l] == 0 ? of[w] : 0u;
        }
#pragma unroll
        for (int w = 0; w < WORDS; ++w) atomicOr(mark + w * 64 + lane, good[w]);
    }
    __syncthreads();
    bool scaled = HALF, again = *(volatile uint32_t *)flag;
    float unscale = KIND == kX3Three ? sign * kX3Unscale : 1.f;
    // a result by its bit's number and lane
    struct Result { int k, c, r, s, row, lc; };
    auto result = [&](uint32_t id) {
        const int v = (int)(id >> 8) / (NTC * S), t = (int)(id >> 8) / S % NTC, s = (int)(id >> 8) % S, i = id & (SH - 1), kk = (int)(id & 63) / SH;
        const int row = SH == 32 ? 8 * (v / 4) + 4 * kk + v % 4 : 4 * kk + v;
        int c_l, r;
        column(t, i, c_l, r);
        return Result{k0 + row, c_first + c_l, r, s, row, (p.packed ? t * SH + i : i * R + t) * S + s};
    };
    int few = 0;
    if constexpr (HALF) {
        bool doubt = false;
#pragma unroll
        for (int w = 0; w < WORDS; ++w) doubt = doubt || mark[w * 64 + lane] != bits(w);
        if (!again && __any(doubt)) {
            // The numbers once more, to count in each channel those that lose bits: a result is well held, too, if a sum is large beside
            // what so many can have lost, or if all are 0 and no number is so small that a product may have gone.
            uint32_t *const count = (uint32_t *)(buf + T::kBuf), *const tiny = count + SH + T::CH, *const some = tiny + SH + T::CH;     // some: [WORDS][64]
            for (int e = tid; e < T::kCounts / 4; e += NTHR) count[e] = 0;
            uint32_t row[DI + XI + 1];
            item_rows(row);
            __syncthreads();
            auto note = [&](uint32_t row, uint32_t small) {
                if (small & 0x7fffffffu) atomicAdd(count + row, small & 0x7fffffffu);
                if (small >> 31) tiny[row] = 1;
            };
#pragma unroll 1
            for (int wt = wt_begin; wt < wt_end; ++wt) {
                load_tile(wt);
#pragma unroll
                for (int u = 0; u < DI; ++u) note(row[u], x3_small<8>(dr[u], scale_at(u)));
#pragma unroll
                for (int u = 0; u < XI; ++u) note(row[DI + u], x3_small<8 * SW>(xr[u], scale_at(DI + u)));
                if (HALO && p.halo) note(row[DI + XI], x3_small<2>(hr, scale_at(DI + XI)));
            }
            __syncthreads();
            uint32_t good[WORDS] = {}, held[WORDS] = {};
            const float one = kX3Need / (float)(p.nch * 8 * (wt_end - wt_begin));
            weigh(good, count, [&](float sum, uint32_t row, uint32_t col) { return one * (float)(row + col) - sum; });
            weigh(held, tiny, [](float sum, uint32_t row, uint32_t col) { return 0.f - ((float)(row + col) + sum); });
#pragma unroll
            for (int w = 0; w < WORDS; ++w) {
                atomicOr(mark + w * 64 + lane, good[w]);
                atomicOr(some + w * 64 + lane, held[w]);
            }
            __syncthreads();
            // A few that are left (sums that happen to be small, as one in 2^10 of few products is) are summed by themselves, a
            // wavefront to each.  mark: their number, the results, the sums.
            uint32_t left[WORDS];
#pragma unroll
            for (int w = 0; w < WORDS; ++w) left[w] = some[w * 64 + lane] & ~mark[w * 64 + lane];
            __syncthreads();
            if (tid == 0) mark[0] = 0;
            __syncthreads();
            if (wq == 0)
#pragma unroll
                for (int w = 0; w < WORDS; ++w)
                    for (uint32_t rest = left[w]; rest; rest &= rest - 1) {
                        const uint32_t at = atomicAdd(mark, 1u), bit = (NB - 32 * w < 32 ? NB - 32 * w : 32) - 1 - __builtin_ctz(rest);
                        if (at < (uint32_t)kX3Few) mark[1 + at] = (32 * w + bit) << 8 | (uint32_t)lane;
                    }
            __syncthreads();
            again = mark[0] > (uint32_t)kX3Few;
            few = again ? 0 : (int)mark[0];
            for (int e = wq; e < few; e += NW) {
                const Result q = result(mark[1 + e]);
                const int shift = x3_shift(q.s, S, SW);
                const double sum = q.k >= g.K || q.c >= g.C ? 0. : x3_dot((const float *)Xp, (const float *)dYp, p.nch * 8 * (wt_end - wt_begin), [&](int at, long &xi, long &yi) {
                    uint32_t wt, chk, row, wc, n_l, h_l;
                    p.d_nch.divmod((uint32_t)at >> 3, wt, chk);
                    p.d_twc.divmod(chk, row, wc);
                    p.d_ht.divmod(row, n_l, h_l);
                    const Tile t = tile_of(wt_begin + (int)wt);
                    const int n = t.n0 + (int)n_l, h = t.h0 + (int)h_l, w = (t.wc0 + (int)wc) * 8 + (at & 7) + p.vlo - shift;
                    const int ih = h * g.sh + q.r - g.ph, iw = w * g.sw + q.s - g.pw;
                    xi = (((long)n * g.C + q.c) * g.H + ih) * g.W + iw;
                    yi = (((long)n * g.K + q.k) * g.Ho + h) * g.Wo + w;
                    return n < g.N && h < g.Ho && (unsigned)w < (unsigned)g.Wo && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
                });
                if (lane == 0) mark[1 + kX3Few + e] = __float_as_uint((float)sum);
            }
            __syncthreads();
        }
    }
    if (again) {
        // Once more on the fp32 matrix core, with the tiles' numbers as they are: a lane's chunk goes through it column by
        // column, dY's own eight and the two on each side, each with the X of its tap's slot.  X counts only where that
        // column of dY exists (an infinity of X is no product of a row's end), and a column whose slot lies before the
        // first chunk or behind the last meets the padding's zero.  (64 -> 64 @ 32x32, N = 128, 60 us: one infinity 128, an
        // infinity to every map or nothing but NaNs 190; with scalar multiply-adds from memory 4900 and 6500.)
        scaled = false;
        unscale = 1.f;
#pragma unroll
        for (int t = 0; t < NTC; ++t)
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int v = 0; v < AV; ++v) acc[t][s][v] = 0.f;
        load_tile(wt_begin);
        for (int wt = wt_begin; wt < wt_end; ++wt) {
            __syncthreads();
            commit_tile(wt, std::true_type{});
            if (wt + 1 < wt_end) load_tile(wt + 1);
            __syncthreads();
            const Tile tile = tile_of(wt);
#pragma unroll 1
            for (int st = 0; st < NST; ++st) {
                const int q = (wq * NST + st) * CPS + kk;
                const uint32_t e = tab[q];
                uint32_t row, wc, n_l, h_l;
                p.d_twc.divmod(q < p.nch ? q : 0, row, wc);
                p.d_ht.divmod(row, n_l, h_l);
                const bool live = q < p.nch && tile.n0 + (int)n_l < g.N && tile.h0 + (int)h_l < g.Ho;
                const int chunk = tile.wc0 + (int)wc, col0 = chunk * 8 + p.vlo;
                const bool first = chunk == 0, last = chunk + 1 == p.w_tiles * p.twc;
                const char *const ap = a_row + (e & 0xfff), *const bp = Xs + ((e >> 12) & 0x3fff);
                float y[12], x[8];                      // dY's columns col0 - 2 .. col0 + 9, X's slots
                auto words = [](const char *at, float *v, int n) {      // n bf16 numbers
#pragma unroll
                    for (int i = 0; i < n; i += 2) {
                        const uint32_t w = *(const uint32_t *)(at + 2 * i);
                        v[i] = __uint_as_float(w << 16); v[i + 1] = __uint_as_float(w & 0xffff0000u);
                    }
                };
                auto floats = [](const char *at, float *v, int n) {
#pragma unroll
                    for (int i = 0; i < n; ++i) v[i] = ((const float *)at)[i];
                };
                if constexpr (BF) words(ap - 4, y, 12);
                else {
                    floats(ap + dy_piece - 8, y, 2);
                    floats(ap, y + 2, 4);
                    floats(ap + dy_piece, y + 6, 4);
                    floats(ap + 16, y + 10, 2);
                }
                if (e & (1u << 30)) y[0] = y[1] = 0.f;
                if (e & (1u << 31)) y[10] = y[11] = 0.f;
#pragma unroll
                for (int t = 0; t < NTC; ++t)
#pragma unroll
                    for (int f = 0; f < SW; ++f) {
                        const char *const q0 = bp + coloff[t] + f * p.twc * 16;
                        if constexpr (BF) words(q0, x, 8);
                        else {
                            floats(q0, x, 4);
                            floats(q0 + x_piece, x + 4, 4);
                        }
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            if (x3_phase(s, S, SW) != f) continue;
#pragma unroll
                            for (int i = 0; i < 12; ++i) {
                                const int j = i - 2 + x3_shift(s, S, SW);
                                const bool slot = j >= 0 && j < 8;
                                const float a = slot || (j < 0 ? first : last) ? y[i] : 0.f;
                                const float b = slot && live && (unsigned)(col0 + i - 2) < (unsigned)g.Wo ? x[slot ? j : 0] : 0.f;
                                if constexpr (SH == 32) acc[t][s] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[t][s], 0, 0, 0);
                                else acc[t][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[t][s], 0, 0, 0);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
            }
        }
        __syncthreads();
    }
    float *const out = outt[prob] + (long)split * g.K * CRS;
    // ---- the wavefronts' sums: each pair of wavefronts two apart exchanges halves of its sums through LDS, then each
    //      neighbouring pair quarters, so that every wavefront has a quarter of the rows, which it lays out as rows of the
    //      result in LDS of its own and writes in whole lines: two barriers.  (With a round and a barrier for every filter tap a
    //      32-wide workgroup took 4.9 us of its life, 4.3 now, of which the partial results' way to memory, all workgroups at
    //      once, is most; 100 -> 100 @ 31x33, N = 20: 74.3 -> 72.2 us, bf16 64 -> 64 @ 56x56, N = 64: 41.4 -> 39.9.) ----
    constexpr int NTS = NTC * S, Q = AV / 4, COLS = NTC * SH * S, QROWS = SH / 4;
    typedef float quarter_t __attribute__((ext_vector_type(Q)));
    char *const tail = smem + T::kFix;
    constexpr int kQuarter = 64 * Q * 4, kSlot = NTS * 2 * kQuarter;                // bytes: of all lanes' quarter of a tile; of a wavefront's halves
    static_assert(QROWS * COLS * 4 == NTS * kQuarter, "rows of a quarter fill half a slot");
    const int hi = wq >> 1, lo = wq & 1;
    auto quarter = [&](int ts, int b) {
        quarter_t z;
#pragma unroll
        for (int e = 0; e < Q; ++e) z[e] = acc[ts / S][ts % S][b * Q + e];
        if (KIND == kX3Three) z *= unscale;             // (before they are added up, which could leave fp32's range)
        return z;
    };
    quarter_t mine[NTS][2];                             // quarters 2 hi and 2 hi + 1
    char *const own = tail + wq * kSlot + lane * Q * 4, *const theirs = tail + (wq ^ 2) * kSlot + lane * Q * 4;
#pragma unroll
    for (int ts = 0; ts < NTS; ++ts)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const quarter_t low = quarter(ts, h), high = quarter(ts, 2 + h);
            *(quarter_t *)(own + (ts * 2 + h) * kQuarter) = hi ? low : high;
            mine[ts][h] = hi ? high : low;
        }
    __syncthreads();
#pragma unroll
    for (int ts = 0; ts < NTS; ++ts)
#pragma unroll
        for (int h = 0; h < 2; ++h) mine[ts][h] += *(const quarter_t *)(theirs + (ts * 2 + h) * kQuarter);
    // (into the slot that nobody but this wavefront reads)
#pragma unroll
    for (int ts = 0; ts < NTS; ++ts) {
        *(quarter_t *)(theirs + ts * kQuarter) = lo ? mine[ts][0] : mine[ts][1];
        if (lo) mine[ts][0] = mine[ts][1];
    }
    __syncthreads();
    float *const rows = (float *)(tail + (wq ^ 2) * kSlot + kSlot / 2);             // [QROWS][COLS]
    const char *const last = tail + (wq ^ 3) * kSlot + lane * Q * 4;                // what the neighbour put into its slot
    const int part = 2 * hi + lo;
    auto row_of = [&](int r) { return SH == 32 ? 8 * part + r : 4 * r + part; };    // row of the quarter -> row of the tile
#pragma unroll
    for (int ts = 0; ts < NTS; ++ts) {
        const int t = ts / S, s = ts % S;
        quarter_t z = mine[ts][0] + *(const quarter_t *)(last + ts * kQuarter);
        if (HALF && scaled) {
            int c_l, r;
            column(t, i, c_l, r);
            const int e = expo[SH + c_l];
#pragma unroll
            for (int v = 0; v < Q; ++v) z[v] = sign * __builtin_ldexpf(z[v], -(e + expo[row_of(Q * kk + v)]));
        }
        // entry of an output channel's row: (c * R + r) * S + s
        const int lc = (p.packed ? t * SH + i : i * R + t) * S + s;
#pragma unroll
        for (int v = 0; v < Q; ++v) rows[(Q * kk + v) * COLS + lc] = z[v];
    }
    if (HALF && lane < few) {
        const Result q = result(mark[1 + lane]);
        const int r = SH == 32 ? q.row - 8 * part : q.row / 4;
        if (SH == 32 ? q.row / 8 == part : q.row % 4 == part) rows[r * COLS + q.lc] = __uint_as_float(mark[1 + kX3Few + lane]);
    }
    const int j0 = (p.packed ? (int)coltile * NTC * SH : c_first * R) * S;
    const int cols = p.packed ? COLS : SH * R * S, n = CRS - j0 < cols ? CRS - j0 : cols;
    if (n == COLS && k0 + SH <= g.K && CRS % 4 == 0 && j0 % 4 == 0 && ((uintptr_t)out & 15) == 0) {
        constexpr int P = COLS / 4, IT = (QROWS * P + 63) / 64;
#pragma unroll
        for (int u = 0; u < IT; ++u) {
            const int e = lane + u * 64, row = e / P, x = e % P * 4;
            if (QROWS * P % 64 == 0 || e < QROWS * P) *(float4_t *)(out + (long)(k0 + row_of(row)) * CRS + j0 + x) = *(const float4_t *)(rows + row * COLS + x);
        }
    } else {
#pragma unroll 1
        for (int row = 0; row < QROWS; ++row)
            if (k0 + row_of(row) < g.K)
                for (int x = lane; x < n; x += 64) out[(long)(k0 + row_of(row)) * CRS + j0 + x] = rows[row * COLS + x];
    }
}

// (id, KIND, SH, NTC, S, SW, RAG, HALO, NCH, DI, XI, KP, CP, CH)
#define WGRAD_X3_VARIANTS_FP32(X) \
    X(0, kX3Half, 32, 3, 3, 1, false, false, 16, 2, 3, 17, 25, 32) X(1, kX3Half, 32, 3, 3, 1, false, true, 16, 2, 3, 23, 25, 32) \
    X(2, kX3Half, 32, 3, 3, 1, true, true, 16, 2, 3, 23, 25, 32) X(3, kX3Three, 16, 3, 3, 1, false, false, 16, 1, 2, 17, 33, 16) \
    X(4, kX3Three, 16, 3, 3, 1, true, true, 16, 1, 2, 23, 33, 16) X(5, kX3Three, 16, 3, 3, 2, false, false, 16, 1, 3, 17, 69, 16) \
    X(6, kX3Three, 16, 3, 3, 2, true, true, 16, 1, 3, 23, 69, 16) X(7, kX3Three, 16, 1, 3, 1, false, false, 16, 1, 1, 17, 25, 7) \
    X(8, kX3Three, 16, 1, 3, 1, true, true, 16, 1, 1, 23, 25, 7) X(9, kX3Half, 32, 1, 3, 1, false, false, 16, 2, 2, 17, 25, 12) \
    X(10, kX3Half, 32, 1, 3, 1, true, true, 16, 2, 2, 23, 25, 12) X(11, kX3Three, 16, 5, 5, 1, true, true, 16, 1, 3, 23, 49, 16)
#define WGRAD_X3_VARIANTS_BF16(X) \
    X(12, kX3Bf16, 32, 3, 3, 1, false, false, 32, 4, 5, 33, 41, 32) X(13, kX3Bf16, 32, 3, 3, 1, false, true, 16, 2, 3, 23, 25, 32) \
    X(14, kX3Bf16, 32, 3, 3, 1, true, true, 16, 2, 3, 23, 25, 32) X(15, kX3Bf16, 16, 3, 3, 1, false, false, 32, 2, 3, 33, 41, 16) \
    X(16, kX3Bf16, 16, 3, 3, 1, true, true, 32, 2, 3, 43, 41, 16) X(17, kX3Bf16, 16, 3, 3, 2, false, false, 16, 1, 3, 17, 69, 16) \
    X(18, kX3Bf16, 16, 3, 3, 2, true, true, 16, 1, 3, 23, 69, 16) X(19, kX3Bf16, 16, 1, 3, 1, false, false, 32, 2, 2, 33, 41, 7) \
    X(20, kX3Bf16, 16, 1, 3, 1, true, true, 32, 2, 2, 43, 41, 7) X(21, kX3Bf16, 32, 1, 3, 1, false, false, 32, 4, 2, 33, 41, 12) \
    X(22, kX3Bf16, 32, 1, 3, 1, true, true, 16, 2, 2, 23, 25, 12) X(23, kX3Bf16, 16, 5, 5, 1, true, true, 16, 1, 3, 23, 49, 16)
constexpr int kX3FirstBf16 = 12, kX3Planes4 = 24, kX3Planes2 = 25, kX3Variants = 26;

// The parameters are read through the kernel-argument segment pointer: indexing the by-value argument with a run-time
// group number would make the compiler copy all of it into scratch memory first.
template <class T>
__global__ __launch_bounds__(kBlock, T::kOcc) void wgrad_exact_x3(const X3Multi)
{
    extern __shared__ __align__(16) char x3_smem[];
    const X3Multi *mp = (const X3Multi *)__builtin_amdgcn_kernarg_segment_ptr();
    const int n = mp->n;
    int gi = 0;
    for (int i = 1; i < n; ++i) gi += (int)blockIdx.x >= mp->begin[i];
    const int bid = (int)blockIdx.x - mp->begin[gi], nblk = mp->count[gi];
    if (bid >= nblk) return;
    const int first = mp->first[gi];
    x3_body<T>(mp->s[gi], mp->X + first, mp->dY + first, mp->out + first, x3_smem, bid, nblk);
}

inline int x3_launch(void (*kernel)(const X3Multi), const X3Multi &m, int blocks, size_t lds, hipStream_t st)
{
    // more than 64 KB of dynamic LDS has to be granted per kernel function (the CU has 160 KB)
    if (lds > 64 * 1024 && hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return WGRAD_LAUNCH_FAILED;
    WGRAD_LAUNCH(kernel, dim3((unsigned)blocks), dim3(kBlock), lds, st, m);
    return launch_status();
}
// 2x2 and 4x4 planes, position by position (exact_x3_planes.hip)
int x3_planes_lds(int hw);
int x3_launch_planes(int hw, bool half, const X3Multi &m, int blocks, size_t lds, hipStream_t st);
// 16-wide fp32 variants of several kinds in one launch (exact_x3_mix.hip): the body of a variant, or -1; a launch's LDS
int x3_mix_body(int variant);
int x3_mix_lds();
int x3_launch_mix(const X3Multi &m, int blocks, hipStream_t st);
int x3_launch_bf16(int variant, const X3Multi &m, int blocks, size_t lds, hipStream_t st);      // instantiated in a file of their own

}  // namespace wgrad
