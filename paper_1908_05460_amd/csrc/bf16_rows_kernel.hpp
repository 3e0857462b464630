// Filter gradient of bf16 layers (3x3, stride 1, padding 1) on planes of 4x4, 8x8, 16x16 or 32x32, row after row.
//
// Rows of the product = output channels, columns = input channels at one filter tap, reduction = positions.  A workgroup
// owns 64 x 64 channels and a range of images; each of its eight wavefronts 32 x 32 channels and four or five of the nine taps
// (v_mfma_f32_32x32x16_bf16, 16 accumulators a tap): filter column 0 and the centre, or filter column 2 and the other two of
// the middle column; a SIMD has one of either.  The wavefront walks down the rows.  A step is one row of
// sixteen positions per lane: a lane of an operand is (channel, half), its sixteen slots are half a row (W = 32), a row of
// one image (16), the same row of two images (8) or of four (4), so a group is 1, 2, 4 or 8 images.
//   - Filter row r of a step pairs the step's row of dY with the row of X one higher or lower, i.e. with registers of the
//     step before or after: every row of X is read from LDS once by a wavefront and kept for three steps.
//   - Filter columns 0 and 2 are X shifted by one element (v_alignbit), made once per row; a wavefront needs one of them.
//   - Rows above and below the plane are not multiplied; columns beside it are zeros that the shift brings in.  (Where dY
//     holds an infinity or a NaN in its first or last row, whose product with the padding is a NaN: see the end.)
// So a step's 8 or 10 matrix instructions come with about 13 others (over VGG-19's run, folds, copies and write-out included, 3.3 to each,
// matrix core busy 58 %).  That ratio is what bounds such a kernel here: measured on this core,
// a vector instruction between 32x32x16 instructions costs 1.3 clocks of their 36, between 16x16x32 ones 2 of 19 -- they
// do not run side by side -- and the row-window kernel (exact_bf16_kernel.hpp) has 3.6 of them to each.
//   - X and dY go to LDS by loads that bypass the registers, four rows (16 KB of each) at a time, into a ring: while four are
//     multiplied, the copies of the next three times four are under way; one barrier in four steps.  A channel's 16-byte pieces are permuted by its number (XOR), so that the
//     lanes of an operand read fall on all banks.  Loads past the end of a tensor bring zeros: ragged batches and
//     channel tiles need nothing else.
//   - A sum of many products in one register loses more to rounding than the older kernel's many short ones did, so every
//     kRowsFold blocks the sums are added to a second set of registers.  That is what the split of the taps buys: nine taps of
//     32 x 32 channels in one wavefront leave no room for it.  (Split into three filter columns and twelve wavefronts the
//     operands' reads were half again as many, and LDS bound the kernel: 128 -> 128 @ 16x16, N = 512: 44 us against 37.)
//   - A workgroup of few blocks (short batches) adds them to the second set after each or every other block: a chain of n additions
//     costs about n / 2 of the squared error, eight a block in the first set, one a fold in the second, so the two balance (8x8 planes, N =
//     9 / 16 / 33, error against 64 bits with four blocks to a sum 8.7e-8 / 9.2e-8 / 9.3e-8, so 6.5e-8 / 7.0e-8 / 7.5e-8, the row-window
//     kernel 5.7e-8 / 6.4e-8 / 7.6e-8).  It costs VGG-19 at N = 16 / 64 / 128 2 / 5 / 3 us (53 / 80 / 116).
// The kernel without the reduction behind it: 38.7 GFLOP in a launch (64 -> 64 @ 32x32 to 512 -> 512 @ 4x4, N = 512) 36 to 41 us, 9 of
// them set-up and write-out (the row-window kernel: 44 to 55); VGG-19's run, 395 GFLOP, 277 us of 350, where the card's power, not the
// kernel's instructions, sets the clock.
//
// SPARSE: the approximated gradient, which is the exact one of a dY with one value in each map (planes of up to 16x16).  That is a
// structured-sparse operand: of four consecutive positions at most one is not zero, and v_smfmac_f32_32x32x32_bf16
// contracts 32 such positions in the time of 16 (18.0 ns on a SIMD; two v_mfma_f32_32x32x16_bf16 34 to 38).  dY is not read
// again: a map is one word, its sum rounded to bf16 and its position, 256 bytes of them an image instead of 64 planes.
//   - A lane's four groups of four positions lie, by the instruction's layout, in both halves of the lanes' slots of X: groups 0 and
//     1 in the first half's, 2 and 3 in the second's, each in those 8 * half .. 8 * half + 7 (measured with one-hot operands).
//   - Each group has the sum in one of two kept places and the position's column as its index; which row and group of four
//     the position is in decides, by one comparison a group and step, whether it is there or a zero.
//   - One value a map and image: the sums need no second set of registers.
//   - A kept place is multiplied also where its value is zero, so that an infinity or a NaN of X that a map did not select makes NaNs
//     at that map's column and the next kept one's (column 3 of four): fewer than the row-window kernel's sparse operand, which
//     multiplies all of them.
#pragma once
#include <type_traits>

#include "exact_common.hpp"
#include "lds_copy.hpp"

namespace wgrad {

typedef __bf16 br_bf8 __attribute__((ext_vector_type(8)));
typedef float br_f16 __attribute__((ext_vector_type(16)));
typedef uint32_t br_u2 __attribute__((ext_vector_type(2)));
typedef uint32_t br_u8 __attribute__((ext_vector_type(8)));
typedef __bf16 br_bf16 __attribute__((ext_vector_type(16)));

constexpr int kRowsTile = 64;                        // channels of a workgroup's tile, each way
constexpr int kRowsThreads = 512;                    // eight wavefronts: two to a SIMD, one of either kind
constexpr int kRowsBlock = kRowsTile * 256;          // bytes of four rows of an operand: 256 a channel
constexpr int kRowsSlot = 2 * kRowsBlock;            // X and dY
constexpr int kRowsRing = 4;                         // slots: the copies of three blocks are under way while one is multiplied
constexpr int kRowsPitch = kRowsTile * 9 + 4;        // floats of a row of the result on its way out
constexpr int kRowsLds = kRowsRing * kRowsSlot > kRowsTile * kRowsPitch * 4 ? kRowsRing * kRowsSlot : kRowsTile * kRowsPitch * 4;
constexpr int kRowsShort = 12;                       // up to so many blocks a sum runs over one, up to twice as many over two
constexpr int kRowsFold = 4;                         // blocks that a sum runs over before it is added to the rest

constexpr int kRowsSparseSlot = kRowsBlock + 4096;   // SPARSE: X, and the maps of up to 16 images, 256 bytes an image
constexpr int kRowsSparseRing = 6;
static_assert(kRowsSparseRing * kRowsSparseSlot <= kRowsLds, "LDS");

struct RowsParams {
    const void *X[kMaxBatch], *dY[kMaxBatch];        // SPARSE: dY: the maps, [N][K] words: bf16 sum << 16 | position
    float *out[kMaxBatch];                           // dW, or the partials of the batch chunks
    int N, C, K;
    int ctiles, ktiles;                              // of 64 channels
    int chunks, chunk_n;                             // chunk_n: a multiple of the images of a group
    float scale;                                     // SPARSE: applied when the result is written
};

// images of a group
__host__ __device__ constexpr int rows_images(int W) { return 32 / W; }

// S: 0: the wavefront has the taps of filter column 0 and the centre, 2: those of filter column 2 and the rest of column 1
// SHORT: few blocks, after each or every other of which the sums are added to the rest
template <int W, int S, bool SPARSE, bool SHORT>
__device__ __forceinline__ void rows_wave(const RowsParams &p, char *smem, int bid, int nblk, int prob)
{
    constexpr int GI = rows_images(W), H = W;
    constexpr int NB = H / 4;                        // blocks of four rows in a plane
    constexpr int RING = SPARSE ? kRowsSparseRing : kRowsRing, SLOT = SPARSE ? kRowsSparseSlot : kRowsSlot;
    static_assert(!SPARSE || W <= 16, "a lane has at most four maps, a position's row and group of four 6 bits");
    int lane = threadIdx.x & 63, sub = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) & 3;
    asm volatile("" : "+v"(lane), "+s"(sub));        // (nothing of one variant is computed ahead for all of a kernel's)
    const int i32 = lane & 31, half = lane >> 5;
    const int kw = sub & 1, cw = sub >> 1;
    const int logical = xcd_contiguous_id(bid, nblk);
    const int kt = logical % p.ktiles, rest = logical / p.ktiles, ct = rest % p.ctiles, chunk = rest / p.ctiles;
    const int k0 = kt * kRowsTile, c0 = ct * kRowsTile;
    const int n_begin = chunk * p.chunk_n;
    const int n_end = n_begin + p.chunk_n < p.N ? n_begin + p.chunk_n : p.N;
    const int C = p.C, K = p.K;
    const int blocks = (n_end - n_begin + GI - 1) / GI * NB;
    constexpr uint32_t plane = H * W * 2;
    const uint32_t ximg = (uint32_t)C * plane, yimg = (uint32_t)K * (SPARSE ? 4u : plane);

    // ---- copies, by the wavefronts of four taps: one moves four channels (1 KB); wavefront `sub` moves channels
    //      16 sub .. 16 sub + 15 of X and of dY ----
    constexpr bool COPIES = S == 0;
    const br_u4 xbuf = rows_buffer((const char *)p.X[prob] + (size_t)n_begin * ximg, (uint32_t)(p.N - n_begin) * ximg);
    const br_u4 ybuf = rows_buffer((const char *)p.dY[prob] + (size_t)n_begin * yimg, (uint32_t)(p.N - n_begin) * yimg);
    const uint32_t lds_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    auto piece_off = [&](int piece, uint32_t img) {  // of a channel's piece (16 bytes) from the channel's first row
        if constexpr (W == 32) return (uint32_t)piece * 16;
        else if constexpr (W == 16) return (uint32_t)(piece >> 3) * img + (piece & 7) * 16;
        else if constexpr (W == 8) return (uint32_t)(piece >> 2) * img + (piece & 3) * 16;
        else return (uint32_t)(piece >> 1) * img + (piece & 1) * 16;
    };
    uint32_t xl[4], yl[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {                    // the copy's channels are 4q .. 4q + 3 of sixteen
        const int pc = (lane & 15) ^ (4 * q + (lane >> 4));
        xl[q] = piece_off(pc, ximg) + (lane >> 4) * plane;
        yl[q] = piece_off(pc, yimg) + (lane >> 4) * plane;
    }
    const uint32_t xg0 = (uint32_t)(c0 + 16 * sub) * plane, yg0 = (uint32_t)(SPARSE ? k0 * 4 : (k0 + 16 * sub) * plane);
    // SPARSE: the maps of four images; of none past the group: zeros
    const int mimg = 4 * sub + (lane >> 4);
    const uint32_t ml = mimg < GI ? (uint32_t)mimg * yimg + (lane & 15) * 16 : 0x80000000u;
    uint32_t xg = xg0, yg = yg0;                     // of the block to copy next
    int copied = 0;
    auto copy_block = [&](int slot) {
        if constexpr (COPIES) {
            const uint32_t at = lds_at + slot * SLOT + 16 * sub * 256;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                rows_copy(xbuf, xl[q] + (xg + 4 * q * plane), at + q * 1024);
                if constexpr (!SPARSE) rows_copy(ybuf, yl[q] + (yg + 4 * q * plane), at + kRowsBlock + q * 1024);
            }
            if constexpr (SPARSE) rows_copy(ybuf, ml + (mimg < GI ? yg : 0u), lds_at + slot * SLOT + kRowsBlock + sub * 1024);
            ++copied;
            const bool wrap = copied % NB == 0;
            xg += wrap ? GI * ximg - (uint32_t)(NB - 1) * (8 * W) : 8 * W;
            if constexpr (SPARSE) yg += wrap ? GI * yimg : 0u;
            else yg += wrap ? GI * yimg - (uint32_t)(NB - 1) * (8 * W) : 8 * W;
            if (copied >= blocks) { xg = xg0; yg = yg0; }        // past the last block: the first again, not read
        }
    };

    // ---- operand reads: sixteen slots of row s of the block at `base`, by channel ----
    const uint32_t piece0 = W == 32 ? 2 * half : 8 * half;
    const uint32_t rd = (uint32_t)i32 * 256 + ((piece0 ^ (i32 & 15)) * 16);
    auto read_row = [&](uint32_t base, int s) {
        if constexpr (W == 4) {
            br_u8 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const br_u2 u = *(const br_u2 *)(smem + ((rd ^ (uint32_t)(q * 32 + (s >> 1) * 16)) + base + (s & 1) * 8));
                v[2 * q] = u[0]; v[2 * q + 1] = u[1];
            }
            return v;
        } else {
            constexpr uint32_t SECOND = W == 8 ? 64 : 16;
            const uint32_t at = W == 32 ? s * 64 : (W == 16 ? s * 32 : s * 16);
            const br_u4 u = *(const br_u4 *)(smem + ((rd ^ at) + base)), v = *(const br_u4 *)(smem + ((rd ^ (at ^ SECOND)) + base));
            return br_u8{u[0], u[1], u[2], u[3], v[0], v[1], v[2], v[3]};
        }
    };
    // W = 32: the word beside the half row, from the other half: right of the first half (S = 2), left of the second (S = 0)
    const uint32_t rd_side = (uint32_t)i32 * 256 + (((S == 2 ? 2 : 1) ^ (i32 & 15)) * 16) + (S == 2 ? 0 : 12);
    auto read_side = [&](uint32_t base, int s) -> uint32_t {
        if constexpr (W == 32) return *(const uint32_t *)(smem + ((rd_side ^ (uint32_t)(s * 64)) + base));
        else return 0u;
    };
    auto mid = [](uint32_t lo, uint32_t hi) { return __builtin_amdgcn_alignbit(hi, lo, 16); };
    auto shifted = [&](const br_u8 &v, uint32_t side) {      // the row as filter column S sees it
        if constexpr (S == 0) {
            const uint32_t L = W == 32 && half ? side : 0u;
            if constexpr (W >= 16) return br_u8{mid(L, v[0]), mid(v[0], v[1]), mid(v[1], v[2]), mid(v[2], v[3]), mid(v[3], v[4]), mid(v[4], v[5]), mid(v[5], v[6]), mid(v[6], v[7])};
            else if constexpr (W == 8) return br_u8{v[0] << 16, mid(v[0], v[1]), mid(v[1], v[2]), mid(v[2], v[3]), v[4] << 16, mid(v[4], v[5]), mid(v[5], v[6]), mid(v[6], v[7])};
            else return br_u8{v[0] << 16, mid(v[0], v[1]), v[2] << 16, mid(v[2], v[3]), v[4] << 16, mid(v[4], v[5]), v[6] << 16, mid(v[6], v[7])};
        } else {
            const uint32_t R = W == 32 && !half ? side : 0u;
            if constexpr (W >= 16) return br_u8{mid(v[0], v[1]), mid(v[1], v[2]), mid(v[2], v[3]), mid(v[3], v[4]), mid(v[4], v[5]), mid(v[5], v[6]), mid(v[6], v[7]), mid(v[7], R)};
            else if constexpr (W == 8) return br_u8{mid(v[0], v[1]), mid(v[1], v[2]), mid(v[2], v[3]), v[3] >> 16, mid(v[4], v[5]), mid(v[5], v[6]), mid(v[6], v[7]), v[7] >> 16};
            else return br_u8{mid(v[0], v[1]), v[1] >> 16, mid(v[2], v[3]), v[3] >> 16, mid(v[4], v[5]), v[5] >> 16, mid(v[6], v[7]), v[7] >> 16};
        }
    };

    // sums of the last blocks, and of those before: filter rows 0, 1, 2 of column S, then the centre, or rows 0 and 2 of column 1
    constexpr int T = S == 0 ? 4 : 5;
    br_f16 acc[T], sum[SPARSE ? 1 : T];
#pragma unroll
    for (int r = 0; r < T; ++r)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[r][i] = sum[SPARSE ? 0 : r][i] = 0.f;
    auto lo = [](const br_u8 &v) { return __builtin_bit_cast(br_bf8, __builtin_shufflevector(v, v, 0, 1, 2, 3)); };
    auto hi = [](const br_u8 &v) { return __builtin_bit_cast(br_bf8, __builtin_shufflevector(v, v, 4, 5, 6, 7)); };
    auto first_half = [&](const br_u8 &a, const br_u8 &x, int r) { acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo(a), lo(x), acc[r], 0, 0, 0); };
    auto second_half = [&](const br_u8 &a, const br_u8 &x, int r) { acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi(a), hi(x), acc[r], 0, 0, 0); };

    // SPARSE: the lane's maps of a group of images, and its operand for row `row` of the planes
    constexpr int MAPS = W == 4 ? 4 : 2;
    constexpr int PLACES = W == 4 ? 1 : 2;           // groups of four positions of a row that a lane has of a map
    uint32_t word[MAPS], value[MAPS][PLACES], row_of[MAPS], index = 0;
    auto read_maps = [&](uint32_t base) {
#pragma unroll
        for (int m = 0; m < MAPS; ++m) {
            const int img = W == 4 ? 4 * (m >> 1) + 2 * half + (m & 1) : (W == 8 ? 2 * m + half : m);
            word[m] = *(const uint32_t *)(smem + base + kRowsBlock + img * 256 + (32 * kw + i32) * 4);
        }
    };
    auto take_maps = [&]() {
        index = 0;
#pragma unroll
        for (int m = 0; m < MAPS; ++m) {
            const uint32_t pos = word[m] & 0xffffu, col = pos & 3, v = word[m] & 0xffff0000u;
            const uint32_t placed = col == 3 ? v : v >> 16;      // in the first kept place, whose index is the column, or the second, whose is 3
            const uint32_t nibble = col == 3 ? 12u : col | 12u;
            row_of[m] = pos / W;
            if constexpr (W == 4) value[m][0] = placed;
            else
#pragma unroll
                for (int j = 0; j < 2; ++j) value[m][j] = ((pos >> 2) & (W / 4 - 1)) == (uint32_t)((W == 16 ? 2 * half : 0) + j) ? placed : 0u;
            index |= W == 4 ? nibble << (4 * m) : (nibble | nibble << 4) << (8 * m);
        }
    };
    auto operand = [&](int row) {
        br_u4 a;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = j / PLACES;
            a[j] = row_of[m] == (uint32_t)row ? value[m][j % PLACES] : 0u;
        }
        return a;
    };
    auto both_halves = [&](const br_u4 &a, const br_u8 &x, int r) {
        acc[r] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(br_bf8, a), __builtin_bit_cast(br_bf16, x), acc[r], (int)index, 0, 0);
    };

    // The copies of the next block have landed (those of two more may be under way) and own reads are over; then everyone's.
    auto meet = [&]() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((SPARSE ? 5 : 8) * (RING - 2)) : "memory"); };

    br_u8 x[3], m[3];                                // row q of the stream of rows is x[q % 3], shifted, and m[q % 3] as it is
    br_u8 a[2];                                      // and of dY a[q % 2]
    br_u8 ahead;                                     // SPARSE: the row of X after the next step's
    const uint32_t xbase = (uint32_t)cw * 8192, ybase = kRowsBlock + (uint32_t)kw * 8192;
    const int every = SHORT ? (blocks <= kRowsShort ? 1 : 2) : kRowsFold;
    int slot = 0, b = 0, fold = every;
    // One block of four steps.  PH: the number (mod 3) of its first row in the stream; FIRST, LAST: its place in the
    // plane.  At the start of a step its row of dY and the rows of X up to its own are in registers.
    auto block = [&](auto ph_c, auto first_c, auto last_c, auto at_c) {
        constexpr int PH = decltype(ph_c)::value, AT = decltype(at_c)::value;
        constexpr bool FIRST = decltype(first_c)::value, LAST = decltype(last_c)::value;
        const uint32_t cur = (uint32_t)slot * SLOT, nxt = (uint32_t)((slot + 1) % RING) * SLOT;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const br_u8 &xp = x[(PH + s + 2) % 3], &xc = x[(PH + s) % 3];
            const br_u8 &mp = m[(PH + s + 2) % 3], &mc = m[(PH + s) % 3];
            br_u8 &xn = x[(PH + s + 1) % 3], &mn = m[(PH + s + 1) % 3];
            const br_u8 &ac = a[s & 1];
            const bool above = !(FIRST && s == 0), below = !(LAST && s == 3);
            if constexpr (SPARSE) {
                const br_u4 sp = operand(4 * AT + s);
                if (s == 2) {
                    meet();
                    copy_block(slot);
                }
                const br_u8 after = read_row((s >= 2 ? nxt : cur) + xbase, (s + 2) & 3);       // (two rows ahead: there is room to wait longer)
                if (LAST && s == 3) read_maps(nxt);
                both_halves(sp, xc, 1);
                if (S == 0) both_halves(sp, mc, 3);
                if (above) {
                    both_halves(sp, xp, 0);
                    if (S == 2) both_halves(sp, mp, 3);
                }
                xn = shifted(ahead, 0);
                mn = ahead;
                if (below) {
                    both_halves(sp, xn, 2);
                    if (S == 2) both_halves(sp, mn, 4);
                }
                ahead = after;
                continue;
            }
            if (s == 3) {
                meet();                              // the next block is in LDS, this one's last rows are in registers
                copy_block(slot);
            }
            const uint32_t from = s == 3 ? nxt : cur;
            const br_u8 v = read_row(from + xbase, (s + 1) & 3);
            const uint32_t side = read_side(from + xbase, (s + 1) & 3);
            a[(s + 1) & 1] = read_row(from + ybase, (s + 1) & 3);
            first_half(ac, xc, 1);
            if (S == 0) first_half(ac, mc, 3);
            if (above) {
                first_half(ac, xp, 0);
                if (S == 2) first_half(ac, mp, 3);
            }
            second_half(ac, xc, 1);
            if (S == 0) second_half(ac, mc, 3);
            if (above) {
                second_half(ac, xp, 0);
                if (S == 2) second_half(ac, mp, 3);
            }
            xn = shifted(v, side);
            mn = v;
            if (below) {
                first_half(ac, xn, 2);
                if (S == 2) first_half(ac, mn, 4);
                second_half(ac, xn, 2);
                if (S == 2) second_half(ac, mn, 4);
            }
        }
        if constexpr (SPARSE && LAST) take_maps();
        slot = (slot + 1) % RING;
        ++b;
    };
    auto fold_sums = [&]() {
#pragma unroll
        for (int r = 0; r < (SPARSE ? 0 : T); ++r) {
            sum[r] += acc[r];
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][i] = 0.f;
        }
    };
    auto short_fold = [&]() {                        // (a branch that is always taken where `every` is 1: without it the registers do not suffice)
        if constexpr (SHORT)
            if (b >= fold) { fold = b + every; fold_sums(); }
    };
    typedef std::integral_constant<int, 0> i0;
    typedef std::integral_constant<int, 1> i1;
    typedef std::integral_constant<int, 2> i2;
    typedef std::integral_constant<int, 3> i3;
    typedef std::true_type yes;
    typedef std::false_type no;

#pragma unroll
    for (int i = 0; i < RING; ++i) {
        copy_block(i);
        if (i == RING - 2) meet();
    }
    const bool active = c0 + 32 * cw < C;
    if (!active)                                     // a wavefront without channels only copies
        for (; b < blocks; ++b, slot = (slot + 1) % RING) {
            meet();
            copy_block(slot);
        }
    if (active) {
    m[0] = read_row(xbase, 0);
    x[0] = shifted(m[0], read_side(xbase, 0));
    if constexpr (SPARSE) {
        read_maps(0);
        take_maps();
        ahead = read_row(xbase, 1);
    } else a[0] = read_row(ybase, 0);
    // a plane starts with its first row in x[0]; what follows its last row -- the next plane's first -- is moved there
    while (true) {
        if constexpr (NB == 1) {
            block(i0(), yes(), yes(), i0());
            x[0] = x[1]; m[0] = m[1];
        } else if constexpr (NB == 2) {
            block(i0(), yes(), no(), i0());
            short_fold();
            block(i1(), no(), yes(), i1());
            x[0] = x[2]; m[0] = m[2];
        } else if constexpr (NB == 4) {
            block(i0(), yes(), no(), i0());
            short_fold();
            block(i1(), no(), no(), i1());
            short_fold();
            block(i2(), no(), no(), i2());
            short_fold();
            block(i0(), no(), yes(), i3());
            x[0] = x[1]; m[0] = m[1];
        } else {
            block(i0(), yes(), no(), i0());
            short_fold();
#pragma unroll 1
            for (int q = 0; q < 2; ++q) {
                block(i1(), no(), no(), i0());       // (the last argument is for SPARSE alone, which has no such planes)
                short_fold();
                block(i2(), no(), no(), i0());
                short_fold();
                block(i0(), no(), no(), i0());
                if constexpr (SHORT) short_fold();
                else fold_sums();
            }
            block(i1(), no(), yes(), i0());
            x[0] = x[2]; m[0] = m[2];
        }
        // (before the loop is left: after the test the compiler moves all accumulators through memory)
        if constexpr (NB == 4 && !SHORT) fold_sums();
        if constexpr ((NB < 4 && !SPARSE) || SHORT)
            if (b >= fold) { fold = b + every; fold_sums(); }
        if (b == blocks) break;
    }
    }
    if constexpr (SPARSE) {
#pragma unroll
        for (int r = 0; r < T; ++r) acc[r] *= p.scale;
    } else {
#pragma unroll
        for (int r = 0; r < T; ++r) acc[r] += sum[r];
    }

    // An infinity or a NaN of dY reaches the sums of filter row 1.  In the first or last row it also meets the padding,
    // through filter row 0 or 2, whose sums are NaN then: products that were left out above.
    bool odd = false;
#pragma unroll
    for (int i = 0; i < 16; ++i) odd = odd || !(fabsf(acc[1][i]) < __builtin_inff());
    if (__any(odd)) {
        auto special = [](uint32_t w) { return (w & 0x7f80u) == 0x7f80u || (w & 0x7f800000u) == 0x7f800000u; };
        uint32_t seen = 0;                           // of output channel i32: bit 0: in a first row, bit 1: in a last row
        for (int n = n_begin + half; n < n_end; n += 2) {
            if constexpr (SPARSE) {
                const uint32_t w = *(const uint32_t *)((const char *)p.dY[prob] + (size_t)n * yimg + (size_t)(k0 + 32 * kw + i32) * 4);
                if ((w & 0x7f800000u) == 0x7f800000u) seen |= ((w & 0xffffu) < W ? 1u : 0u) | ((w & 0xffffu) >= (H - 1) * W ? 2u : 0u);
                continue;
            }
            const uint32_t *const map = (const uint32_t *)((const char *)p.dY[prob] + (size_t)n * yimg + (size_t)(k0 + 32 * kw + i32) * plane);
            for (int e = 0; e < W / 2; ++e) seen |= (special(map[e]) ? 1u : 0u) | (special(map[(H - 1) * (W / 2) + e]) ? 2u : 0u);
        }
        seen |= __shfl_xor(seen, 32, 64);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t f = __shfl(seen, 8 * (i >> 2) + 4 * half + (i & 3), 64);
            if (f & 1) acc[0][i] = __builtin_nanf("");
            if (f & 2) acc[2][i] = __builtin_nanf("");
            if (S == 2 && (f & 1)) acc[T - 2][i] = __builtin_nanf("");
            if (S == 2 && (f & 2)) acc[T - 1][i] = __builtin_nanf("");
        }
    }

    // The tile goes out through LDS, as whole rows of 576 values (lane: column i32, rows 8 * (i / 4) + 4 * half + i % 4); the
    // copies past the end have landed before.
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    float *const tile = (float *)smem;
    if (active) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float *const t = tile + (32 * kw + 8 * (i >> 2) + 4 * half + (i & 3)) * kRowsPitch + (32 * cw + i32) * 9;
#pragma unroll
            for (int r = 0; r < 3; ++r) t[3 * r + S] = acc[r][i];
            if (S == 0) t[4] = acc[3][i];
            else { t[1] = acc[T - 2][i]; t[7] = acc[T - 1][i]; }
        }
    }
    __syncthreads();
    float *const out = p.out[prob] + (size_t)chunk * K * C * 9 + ((size_t)k0 * C + c0) * 9;
    const int width = (C - c0 < kRowsTile ? C - c0 : kRowsTile) * 9;
    if (C % 4 == 0 && ((uintptr_t)p.out[prob] & 15) == 0) {
        for (int e = threadIdx.x; e < kRowsTile * (kRowsTile * 9 / 4); e += kRowsThreads) {
            const int k = e / (kRowsTile * 9 / 4), q = e % (kRowsTile * 9 / 4) * 4;
            if (q < width) *(float4_t *)(out + (size_t)k * C * 9 + q) = *(const float4_t *)(tile + k * kRowsPitch + q);
        }
    } else {
        for (int e = threadIdx.x; e < kRowsTile * kRowsTile * 9; e += kRowsThreads) {
            const int k = e / (kRowsTile * 9), q = e % (kRowsTile * 9);
            if (q < width) out[(size_t)k * C * 9 + q] = tile[k * kRowsPitch + q];
        }
    }
}

template <int W, bool SPARSE>
__device__ __forceinline__ void rows_body(const RowsParams &p, char *smem, int bid, int nblk, int prob)
{
    const bool first = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) == 0;
    if constexpr (!SPARSE)
        if (p.chunk_n / rows_images(W) * (W / 4) <= 2 * kRowsShort) {
            if (first) rows_wave<W, 0, SPARSE, true>(p, smem, bid, nblk, prob);
            else rows_wave<W, 2, SPARSE, true>(p, smem, bid, nblk, prob);
            return;
        }
    if (first) rows_wave<W, 0, SPARSE, false>(p, smem, bid, nblk, prob);
    else rows_wave<W, 2, SPARSE, false>(p, smem, bid, nblk, prob);
}

}  // namespace wgrad
