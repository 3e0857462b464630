// Host side of the exact filter gradient in 16-bit pieces (exact_x3_kernel.hpp): which shapes take it,
// their tiles, and launches that carry several shapes.
#include <algorithm>
#include <vector>

#include "exact_x3_kernel.hpp"

namespace wgrad {

struct X3Variant { int kind, sh, ntc, s, sw, rag, halo, nch, di, xi, kp, cp, ch, lds, occ, plane; };
static const X3Variant kVariant[kX3Variants] = {
#define X(ID, ...) {__VA_ARGS__, X3Config<__VA_ARGS__>::kLds, X3Config<__VA_ARGS__>::kOcc, 0},
    WGRAD_X3_VARIANTS_FP32(X)
    WGRAD_X3_VARIANTS_BF16(X)
#undef X
    {kX3Three, 32, 0, 3, 1, 0, 0, 0, 0, 0, 0, 0, 0, x3_planes_lds(4), 2, 4}, {kX3Three, 32, 0, 3, 1, 0, 0, 0, 0, 0, 0, 0, 0, x3_planes_lds(2), 2, 2},
};
// workgroups that the chip holds at once
static int x3_resident(const X3Variant &v) { return kNumCU * std::max(1, std::min(160 * 1024 / v.lds, v.occ)); }

static int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }
// Tile of a variant for a shape, or false.
static bool x3_tile(const Geometry &g, int id, X3Plan &pl)
{
    const X3Variant &v = kVariant[id];
    if (v.plane) {
        // position by position (exact_x3_planes.hip): a tile is 8 or 16 images
        if (g.H != v.plane || g.W != v.plane || g.R != 3 || g.S != 3 || g.sh != 1 || g.sw != 1 || g.ph != 1 || g.pw != 1) return false;
        if ((long)16 * std::max(g.K, g.C) * 16 * 4 >= (1l << 30)) return false;
        pl.variant = id;
        pl.ktiles = (g.K + 63) / 64; pl.ctiles = (g.C + 31) / 32;
        pl.nti = v.plane == 4 ? 8 : 16; pl.ht = g.Ho; pl.iht = g.H; pl.twc = 1;
        pl.h_tiles = pl.w_tiles = 1; pl.n_groups = (g.N + pl.nti - 1) / pl.nti;
        pl.lds = v.lds;
        return true;
    }
    const int half = v.s / 2;
    int dmin = 0, dmax = 0;
    for (int s = 0; s < v.s; ++s) { dmin = std::min(dmin, x3_shift(s, v.s, v.sw)); dmax = std::max(dmax, x3_shift(s, v.s, v.sw)); }
    int vlo = std::max(dmin, floor_div(g.pw - half, v.sw));
    int vhi = std::min(g.Wo - 1 + dmax, floor_div(g.W - 1 + g.pw - half, v.sw));
    if (vhi < vlo) return false;                         // (every product meets only padding)
    // Every column of dY meets a slot through some tap, also where the padding is as wide as the filter and the column's
    // taps all lie in it: an infinity or NaN there makes NaNs of the padding's zeros, and a column that no slot reaches
    // would never enter a sum.
    vlo = std::min(vlo, dmax);
    vhi = std::max(vhi, g.Wo - 1 + dmin);
    const int vw = vhi - vlo + 1;
    pl.vlo = vlo;
    pl.xcol0 = v.sw * vlo + half - g.pw;
    if (!v.rag && (g.Wo % 4 || g.W % 4 || vlo != 0 || pl.xcol0 != 0)) return false;
    pl.packed = v.ntc == 1;
    if (!pl.packed && v.ntc != g.R) return false;
    pl.ktiles = (g.K + v.sh - 1) / v.sh;
    if (pl.packed) {
        pl.ctiles = (g.C * g.R + v.sh * v.ntc - 1) / (v.sh * v.ntc);
        pl.ch = std::min(g.C, (v.sh * v.ntc - 1) / g.R + 2);
        if (pl.ch > v.ch) return false;
    } else {
        pl.ctiles = (g.C + v.sh - 1) / v.sh;
        pl.ch = std::min(v.sh, g.C);
    }
    const int vwc = (vw + 7) / 8;                            // (images of a tile, its rows and chunk columns are packed in 4, 8 and 4 bits)
    long best = -1;
    int best_x = 0;
    for (int twc = 1; twc <= std::min({vwc, v.nch, 16}); ++twc) {
        const int w_tiles = (vwc + twc - 1) / twc;
        if (twc > 1 && (vwc + twc - 2) / (twc - 1) == w_tiles) continue;      // the same number of narrower tiles does
        const int halo = w_tiles > 1 || vlo > 0 || vlo + 8 * twc < g.Wo;
        if (halo && !v.halo) continue;
        for (int ht = 1; ht <= g.Ho; ++ht) {
            if (ht * twc > v.nch) break;
            int nti = ht >= g.Ho ? std::min({g.N, v.nch / (ht * twc), 16}) : 1;
            const int iht = (ht - 1) * g.sh + g.R;
            if (iht > 255) break;
            for (; nti >= 1; --nti) {
                const int xr = nti * iht * twc;                        // staged chunks of a channel and phase
                if ((long)pl.ch * xr > (long)v.xi * kBlock) continue;
                if (halo && v.sh * nti * ht * 2 > kBlock) continue;
                const int nch = nti * ht * twc;
                // (the last chunk of a dY channel is the chunk of zeros)
                if ((halo ? 1 + nti * ht * (twc + 1) : nch) + 1 > v.kp || xr * v.sw > v.cp) continue;
                const long tiles = (long)w_tiles * ((g.Ho + ht - 1) / ht) * ((g.N + nti - 1) / nti);
                if (best >= 0 && (tiles > best || (tiles == best && xr >= best_x))) continue;
                best = tiles; best_x = xr;
                pl.nti = nti; pl.ht = ht; pl.iht = iht; pl.twc = twc; pl.nch = nch; pl.halo = halo;
                pl.w_tiles = w_tiles; pl.h_tiles = (g.Ho + ht - 1) / ht; pl.n_groups = (g.N + nti - 1) / nti;
            }
        }
    }
    if (best < 0) return false;
    pl.lds = v.lds;
    // index arithmetic: 32-bit element offsets within a tile, fast divisions of the tile number
    if ((long)pl.nti * g.K * g.Ho * g.Wo >= (1l << 28) || (long)(pl.nti + 1) * g.C * g.H * g.W >= (1l << 28)) return false;
    if (best * std::max(pl.w_tiles, pl.h_tiles) >= (1l << 31)) return false;
    pl.variant = id;
    return true;
}

// us that a workgroup spends on a tile when `share` of them are on its CU: bounded by the matrix instructions of all, or
// by its own staging and matrix instructions one after the other.  (Fitted to bf16 pieces and their six products; `half`, the longest
// rows of a launch of several variants, counts three.  The 32-wide tiles and 4x4 planes of fp16 pieces are cut by this figure as
// well, 4.2 us a tile where they take 3.0: their splits are those that were timed, not a minimum of the model.)
static double x3_tile_us(const X3Variant &v, int share, bool half = false)
{
    if (v.plane) return 1.1 * (v.plane == 4 ? std::max(share * 2.8, 4.2) : std::max(share * 0.85, 1.8));
    const double mfma = (double)v.nch / (64 / v.sh) / 4 * (v.kind == kX3Bf16 ? 1 : (half ? 3 : 6)) * v.ntc * v.s * (v.sh == 32 ? 32 : 16) / 1900.0;
    const double stage = 0.3 + (v.rag && v.sw > 1 ? 0.6 : (v.kind == kX3Bf16 ? 0.1 : 0.33)) * (v.di + v.xi * v.sw);
    return 1.1 * std::max(std::max(mfma * share, 0.3 * stage * share), mfma + stage);
}
static double x3_tile_us(const X3Variant &v) { return x3_tile_us(v, x3_resident(v) / kNumCU); }
// tiles a workgroup adds up in one accumulator: the error of the fp32 sums grows with their length (of the result's 2-norm,
// 64 -> 64 @ 32x32, N = 200, 13 tiles of 32-wide sums: 3.1e-7; 6 -> 196 @ 80x138, N = 34, 32 tiles: 4.4e-7; the fp32 matrix
// core's kernels 6.9e-7 in both; 16-wide tiles, whose smaller products have their own sums, 1.4e-7 at 32 tiles).  bf16's
// tiles of 32 chunks are two steps each: 182 -> 211 @ 22x8, N = 61, 1.9e-7 at 31 of them, 1.4e-7 at 16, the fp32 matrix
// core's kernel 1.3e-7.  The position form rounds its sums far less often (512 -> 512, N = 512, one sum of 64 / 32 tiles:
// 2.0e-7 at 4x4, 7.7e-8 at 2x2).
static long x3_most_tiles(const X3Variant &v) { return v.plane ? 64 : (v.kind == kX3Bf16 && v.sh == 16 && v.nch == 32 ? 16 : 32); }
// 4x4 planes: stages that a workgroup adds up from which on it takes two fp16 pieces to a number.  By themselves these are 1.3 to
// 1.5e-7 off whatever the sum's length, three bf16 pieces 0.65e-7 after 2 stages, 1.0e-7 after 8 and 1.9e-7 after 16 (VGG-19's run, N =
// 128); shorter sums would gain a fifth of their time (N = 128 alone, 4 stages: 50 us, 42).
constexpr long kX3HalfStages = 12;
// a launch of several variants, bf16 pieces: 24 tiles (ResNet-20, N = 90 to 128, sums of 18 / 24 / 28 tiles, error over that of the
// launches before: 64 -> 64 @ 8x8 0.86 / 0.97 / 1.17, the others less), and as many of the strided ones' fp16 pieces.  Layers that take
// bf16 pieces only in such a launch are in it where their workspace has room for that (x3_joins); the others' partial results are as
// many as in a launch of their own, x3_most_tiles to a sum.
constexpr long kX3MixMost = 24;
constexpr int kX3MixSlots = 3 * kNumCU;      // workgroups of such a launch that the chip holds at once
constexpr double kX3Fixed = 9.0;       // a workgroup's set-up, first loads and write-out

// How long a launch runs: its workgroups, longest first, each on the slot that is free earliest.  `n` kinds of
// workgroups, `count` of each, `life` us long, sorted by falling life.
double makespan_us(int slots, const double *life, const long *count, int n)
{
    struct { double at; long n; } free_at[64];
    int used = 1;
    free_at[0] = {0.0, slots};
    double end = 0;
    for (int i = 0; i < n; ++i) {
        long left = count[i];
        while (left > 0) {
            int e = 0;
            for (int j = 1; j < used; ++j)
                if (free_at[j].at < free_at[e].at) e = j;
            // whole rounds on the earliest slots while they stay the earliest
            const long take = std::min(left, free_at[e].n);
            const double done = free_at[e].at + life[i];
            left -= take;
            end = std::max(end, done);
            int same = -1;
            for (int j = 0; j < used; ++j)
                if (free_at[j].at > done - 0.05 && free_at[j].at < done + 0.05) same = j;
            if (take == free_at[e].n && same < 0) free_at[e].at = done;
            else {
                free_at[e].n -= take;
                if (same >= 0) free_at[same].n += take;
                else if (used < 64) free_at[used++] = {done, take};
                else free_at[e].n += take, free_at[e].at = done;              // (too many kinds: an estimate does)
                if (free_at[e].n == 0) free_at[e] = free_at[--used];
            }
        }
    }
    return end;
}

// us that writing and reading back `splits` partial results of a tensor take
static double x3_partial_us(const Geometry &g, long splits, int nprob)
{
    return splits > 1 ? (double)splits * nprob * g.dw_elems() * 8 / 4.5e6 : 0.0;
}

// How many workgroups share the reduction of one problem of `nprob`: the time of the launch, plus the traffic of the
// partial results.
static int x3_choose_splits(const Geometry &g, const X3Plan &pl, int nprob)
{
    const X3Variant &v = kVariant[pl.variant];
    const long tiles = (long)pl.w_tiles * pl.h_tiles * pl.n_groups, outs = (long)pl.ktiles * pl.ctiles * nprob;
    const int slots = x3_resident(v);
    const double t = x3_tile_us(v);
    double best_cost = 1e30;
    int best = 1;
    const long longest = x3_most_tiles(v), most = std::min(tiles, std::max({1l, 2 * slots / outs, (tiles + longest - 1) / longest}));
    for (long per = (tiles + most - 1) / most; per <= std::max(longest, (tiles + most - 1) / most) && per <= tiles; per += std::max(1l, per / 16)) {
        const long s = (tiles + per - 1) / per, n = outs * s;
        double life = kX3Fixed + per * t;
        if (n <= kNumCU) life = kX3Fixed + per * x3_tile_us(v, 1);      // a CU to itself
        const double cost = makespan_us(slots, &life, &n, 1) + (s > 1 ? 2.0 : 0.0) + x3_partial_us(g, s, nprob);
        if (cost < best_cost) { best_cost = cost; best = (int)s; }
    }
    return best;
}

// whether the variant reads bf16 rows in 8-byte pieces (4-byte aligned tensors), not element by element
bool x3_needs_alignment(const X3Plan &pl) { return kVariant[pl.variant].kind == kX3Bf16 && !kVariant[pl.variant].rag; }

// whether the variant stages rows of any width and cut rows; output channels of its tile
bool x3_ragged(const X3Plan &pl) { return kVariant[pl.variant].rag; }
int x3_tile_rows(const X3Plan &pl) { return kVariant[pl.variant].sh; }
bool x3_mixes(const X3Plan &pl) { return x3_mix_body(pl.variant) >= 0; }
bool x3_joins(const X3Plan &pl)
{
    return x3_mixes(pl) && (x3_mix_body(pl.variant) == 1 || (long)pl.w_tiles * pl.h_tiles * pl.n_groups <= kX3MixMost * pl.splits);
}

// at most `room` partial results; false if a workgroup would then add up more tiles than x3_most_tiles
bool x3_fit(X3Plan &pl, long room)
{
    const long tiles = (long)pl.w_tiles * pl.h_tiles * pl.n_groups;
    pl.splits = (int)std::max(1l, std::min((long)pl.splits, room));
    return (tiles + pl.splits - 1) / pl.splits <= x3_most_tiles(kVariant[pl.variant]);
}

bool plan_exact_x3(const Geometry &g, X3Plan &best)
{
    // Short layers of few channels, which the older forms took before, in the workspace of those
    auto small_room = [&](X3Plan &pl) {
        const double gflop = g.gflop();
        if (g.bf16 || gflop >= 0.5 || (gflop >= 0.03 && g.K > 16 && g.C > 16)) return true;
        return x3_fit(pl, exact_older_room(g));
    };
    if (!g.bf16 && g.H == g.W && (g.W == 2 || g.W == 4)) {
        // (every such layer: no slower than the row form or the fp32 matrix core anywhere, 64 -> 64 @ 4x4 at N = 128 14.5 us
        // against 16.7, 512 -> 512 at N = 2 11.5 against 11.4, at N = 512 153 against 227; figures in exact_x3_planes.hip)
        X3Plan pl{};
        if (x3_tile(g, g.W == 4 ? kX3Planes4 : kX3Planes2, pl)) {
            best = pl;
            best.splits = x3_choose_splits(g, best, 1);
            return small_room(best);
        }
    }
    if (g.W < 4 || g.Wo < 4 || g.pw >= 4096) return false;
    const double gflop = 2e-9 * g.N * g.K * g.Ho * g.Wo * (double)g.crs();
    double best_cost = 1e30;
    for (int id = 0; id < kX3Variants; ++id) {
        const X3Variant &v = kVariant[id];
        if (v.plane || (v.kind == kX3Bf16) != (g.bf16 != 0) || v.s != g.S || v.sw != g.sw) continue;
        X3Plan pl{};
        if (!x3_tile(g, id, pl)) continue;
        // Matrix instructions, in units of a 16x16 tile of the result, six products to either kind (32-wide tiles take fp16 pieces now,
        // and three: the line between the two, and its figures, are of bf16 pieces).  Long reductions do better with 32x32 tiles (a
        // staged element serves twice as many of them; 128 -> 128 @ 16x16, N = 128: 56 us against 65), short ones with
        // 16x16 tiles, whose workgroups are quicker to set up and share a CU by four (N = 16: 21 us against 22.5;
        // 48 -> 96 @ 27x27, N = 32, where 32x32 tiles would be a third padding besides: 35 against 49).
        double cost = (double)pl.ktiles * pl.ctiles * pl.w_tiles * pl.h_tiles * pl.n_groups * v.nch * v.ntc *
                      (v.sh == 32 ? 4.0 : (gflop < (g.bf16 ? 12.0 : 2.0) ? 0.9 : 1.15));
        // (ragged bf16 rows are loaded element by element: 64 -> 64 @ 56x56, stride 2, N = 128, 162 us that way, 53 with whole
        // rows and fewer of them to a tile)
        cost *= v.rag ? (g.bf16 ? (v.sw > 1 ? 2.5 : 1.5) : 1.1) : (v.halo ? 1.02 : 1.0);
        if (cost < best_cost) { best_cost = cost; best = pl; }
    }
    if (best_cost >= 1e30) return false;
    best.splits = x3_choose_splits(g, best, 1);
    return small_room(best);
}

// ---- launches ----
struct X3Group {
    Geometry g;
    X3Plan pl;
    Batch b;
    float *ws;                   // the group's slice of the workspace: slice_stride floats per problem
    long slice_stride;
    bool half;                   // two fp16 pieces where a launch of several variants could take three bf16 ones
};
struct X3Queue {
    std::vector<X3Group> item;
};
X3Queue *x3_queue_new() { return new X3Queue(); }
void x3_queue_delete(X3Queue *q) { delete q; }

static void x3_fill(const X3Group &it, X3Shape &s)
{
    const Geometry &g = it.g;
    const X3Plan &pl = it.pl;
    s.g = g;
    s.per_prob = pl.ktiles * pl.ctiles * pl.splits;
    s.ktiles = pl.ktiles; s.ctiles = pl.ctiles; s.splits = pl.splits;
    s.nti = pl.nti; s.ht = pl.ht; s.iht = pl.iht; s.twc = pl.twc;
    s.h_tiles = pl.h_tiles; s.w_tiles = pl.w_tiles; s.n_groups = pl.n_groups;
    s.nch = pl.nch; s.ch = pl.ch; s.packed = pl.packed;
    s.body = x3_mix_body(pl.variant);
    if (it.half) s.body = 3;
    s.halo = pl.halo; s.vlo = pl.vlo; s.xcol0 = pl.xcol0;
    const int tiles = pl.w_tiles * pl.h_tiles * pl.n_groups;
    s.tiles_each = tiles / pl.splits;
    s.tiles_more = tiles % pl.splits;
    s.d_prob = X3Div(s.per_prob);
    s.d_ctiles = X3Div(pl.ctiles);
    s.d_ktiles = X3Div(pl.ktiles);
    if (kVariant[pl.variant].plane) return;
    s.d_nch = FastDiv(pl.nch);
    s.d_twc = FastDiv(pl.twc);
    s.d_ht = FastDiv(pl.ht);
    s.d_xrow = FastDiv(pl.nti * pl.iht * pl.twc);
    s.d_iht = FastDiv(pl.iht);
    s.d_htiles = FastDiv(pl.h_tiles);
    s.d_wtiles = FastDiv(pl.w_tiles);
    s.d_r = FastDiv(g.R);
    s.d_rows = FastDiv(pl.nti * pl.ht);
}

static int x3_launch_groups(const X3Group *const *it, int n, hipStream_t st)
{
    X3Multi m{};
    m.n = n;
    size_t lds = 0;
    bool mixed = false;
    int blocks = 0, tensors = 0;
    for (int i = 0; i < n; ++i) {
        const X3Group &q = *it[i];
        x3_fill(q, m.s[i]);
        m.begin[i] = blocks;
        m.count[i] = m.s[i].per_prob * q.b.n;
        m.first[i] = tensors;
        for (int j = 0; j < q.b.n; ++j, ++tensors) {
            m.X[tensors] = q.b.X[j];
            m.dY[tensors] = q.b.dY[j];
            m.out[tensors] = q.pl.splits > 1 ? q.ws + (long)j * q.slice_stride : q.b.dW[j];
        }
        blocks += (m.count[i] + 7) / 8 * 8;
        lds = std::max(lds, (size_t)q.pl.lds);
        mixed = mixed || q.pl.variant != it[0]->pl.variant;
    }
    m.begin[n] = blocks;
    if (mixed) return x3_launch_mix(m, blocks, st);
    if (const int hw = kVariant[it[0]->pl.variant].plane) {
        bool half = hw == 4;
        for (int i = 0; i < n; ++i) half = half && it[i]->pl.n_groups >= kX3HalfStages * it[i]->pl.splits;
        return x3_launch_planes(hw, half, m, blocks, lds, st);
    }
    if (it[0]->pl.variant >= kX3FirstBf16) return x3_launch_bf16(it[0]->pl.variant, m, blocks, lds, st);
    switch (it[0]->pl.variant) {
#define X(ID, ...) case ID: return x3_launch(wgrad_exact_x3<X3Config<__VA_ARGS__>>, m, blocks, lds, st);
        WGRAD_X3_VARIANTS_FP32(X)
#undef X
        default: return WGRAD_UNSUPPORTED;
    }
}

// Issues what was collected, in launches of several groups (longest workgroups first), cut so that a launch's workgroups
// fill the chip about evenly; the partial results are recorded in `combine`.
// A launch of several variants: where one round of workgroups would add up more tiles than three bf16 pieces may (kX3MixMost), fp16
// pieces, which err no more at that length, on rows of more than one chunk (ResNet-20 exact, N = 128: 89 us in bf16 pieces, two
// rounds, 80 so; on 8x8 planes they err 1.15 times as much as bf16 pieces in the launches before)
void x3_choose_pieces(X3Kind *kind, int n)
{
    auto tile_us = [&](const X3Kind &k) { return x3_tile_us(kVariant[k.pl->variant], kX3MixSlots / kNumCU); };
    double rounds = 0;
    for (int i = 0; i < n; ++i) {
        const X3Plan &pl = *kind[i].pl;
        rounds += (double)((long)pl.w_tiles * pl.h_tiles * pl.n_groups) * pl.ktiles * pl.ctiles * kind[i].layers * tile_us(kind[i]) / tile_us(kind[0]);
    }
    for (int i = 0; i < n; ++i)
        kind[i].half = 1.08 * rounds > (double)kX3MixSlots * kX3MixMost && x3_mix_body(kind[i].pl->variant) == 0 && kind[i].g->Wo > 8;
}

int x3_flush(X3Queue &q, hipStream_t st, CombineQueue *combine)
{
    int rc = WGRAD_OK;
    auto tiles_of = [](const X3Group &it) { return (long)it.pl.w_tiles * it.pl.h_tiles * it.pl.n_groups; };
    auto key = [](const X3Group &g) { return x3_mixes(g.pl) ? -1 : g.pl.variant; };      // (those that share a launch side by side)
    std::stable_sort(q.item.begin(), q.item.end(), [&](const X3Group &a, const X3Group &b) { return key(a) < key(b) || (key(a) == key(b) && a.pl.variant < b.pl.variant); });
    for (size_t first = 0; first < q.item.size() && rc == WGRAD_OK;) {
        X3Group *sel[kX3MultiMax];
        int n = 0, tensors = 0;
        // (one variant, or the 16-wide ones that a launch can mix)
        const int variant = q.item[first].pl.variant;
        while (first < q.item.size() && n < kX3MultiMax && tensors + q.item[first].b.n <= kX3Tensors &&
               (q.item[first].pl.variant == variant || (x3_mix_body(variant) >= 0 && x3_mix_body(q.item[first].pl.variant) >= 0))) {
            tensors += q.item[first].b.n;
            sel[n++] = &q.item[first++];
        }
        const X3Variant &v = kVariant[variant];
        bool mixed = false;
        for (int i = 1; i < n; ++i) mixed = mixed || sel[i]->pl.variant != variant;
        const int slots = mixed ? kX3MixSlots : x3_resident(v);
        double t[kX3MultiMax];
        for (int i = 0; i < n; ++i) t[i] = x3_tile_us(kVariant[sel[i]->pl.variant], slots / kNumCU);
        if (mixed) {
            X3Kind kind[kX3MultiMax];
            for (int i = 0; i < n; ++i) kind[i] = X3Kind{&sel[i]->g, &sel[i]->pl, sel[i]->b.n, false};
            x3_choose_pieces(kind, n);
            for (int i = 0; i < n; ++i) {
                sel[i]->half = kind[i].half;
                if (sel[i]->half) t[i] = x3_tile_us(kVariant[sel[i]->pl.variant], slots / kNumCU, true);
            }
        }
        // Candidates: workgroups of `share` of the launch's even share of work, the first of a pair where the result is
        // large (its partial results are what splitting costs), the second elsewhere, to fill what those leave free.  (Shares
        // over 1 leave slots empty: 4x4 layers of 512 channels, whose partial sums weigh most, VGG-19 at N = 64 285 -> 269 us.)
        static const double kShare[][2] = {{1.4, 1.4}, {1.0, 1.0}, {1.0, 0.5}, {1.0, 0.33}, {0.67, 0.67}, {0.67, 0.33}, {0.5, 0.5}, {0.5, 0.25}, {0.33, 0.33}, {0.25, 0.25}, {1.07, 1.07}, {1.15, 1.15}, {1.25, 1.25}, {0.54, 0.54}, {0.58, 0.58}, {0.62, 0.62}, {0.36, 0.36}, {0.4, 0.4}};
        long largest = 0;
        double total = 0;                                // workgroup-tiles
        for (int i = 0; i < n; ++i) {
            total += (double)tiles_of(*sel[i]) * sel[i]->pl.ktiles * sel[i]->pl.ctiles * sel[i]->b.n * t[i] / t[0];
            largest = std::max(largest, sel[i]->g.dw_elems());
        }
        double best_cost = 1e30, life[kX3MultiMax], best_life[kX3MultiMax];
        int best[kX3MultiMax], now[kX3MultiMax];
        for (const auto &share : kShare) {
            double sorted[kX3MultiMax], partial = 0;
            long count[kX3MultiMax];
            for (int i = 0; i < n; ++i) {
                const long tiles = tiles_of(*sel[i]);
                const double target = std::max(1.0, total / slots * share[2 * sel[i]->g.dw_elems() < largest] * t[0] / t[i]);
                long s = (long)(tiles / target + 0.95);
                const long longest = mixed && !sel[i]->half ? kX3MixMost : x3_most_tiles(kVariant[sel[i]->pl.variant]);
                s = std::max(s, (tiles + longest - 1) / longest);
                s = std::max(1l, std::min(s, (long)std::min<long>(sel[i]->pl.splits, tiles)));
                now[i] = (int)s;
                partial += x3_partial_us(sel[i]->g, s, sel[i]->b.n);
                life[i] = kX3Fixed + (double)((tiles + s - 1) / s) * t[i];
                int j = i;
                for (; j > 0 && sorted[j - 1] < life[i]; --j) { sorted[j] = sorted[j - 1]; count[j] = count[j - 1]; }
                sorted[j] = life[i];
                count[j] = s * sel[i]->pl.ktiles * sel[i]->pl.ctiles * sel[i]->b.n;
            }
            const double cost = makespan_us(slots, sorted, count, n) + partial;
            if (cost < best_cost) {
                best_cost = cost;
                std::copy(now, now + n, best);
                std::copy(life, life + n, best_life);
            }
        }
        const X3Group *order[kX3MultiMax];
        for (int i = 0; i < n && rc == WGRAD_OK; ++i) {
            sel[i]->pl.splits = best[i];
            if (best[i] > 1)
                rc = launch_combine(sel[i]->ws, sel[i]->slice_stride, best[i], sel[i]->g.dw_elems(), 1.0f, sel[i]->b.dW, sel[i]->b.n, st, combine);
            int j = i;
            for (; j > 0 && life[j - 1] < best_life[i]; --j) { life[j] = life[j - 1]; order[j] = order[j - 1]; }
            life[j] = best_life[i];
            order[j] = sel[i];
        }
        if (rc == WGRAD_OK) rc = x3_launch_groups(order, n, st);
    }
    q.item.clear();
    return rc;
}

// One group of identical layers: its own launch, or (with a queue) collected for x3_flush.
int launch_exact_x3(const Geometry &g, const X3Plan &plan, const Batch &b, void *ws, size_t slice_bytes, hipStream_t st,
                    CombineQueue *defer, X3Queue *q)
{
    X3Group it{g, plan, b, (float *)ws, (long)(slice_bytes / 4), false};
    if (q) {
        q->item.push_back(it);
        return WGRAD_OK;
    }
    if (b.n > 1) it.pl.splits = std::min(plan.splits, x3_choose_splits(g, plan, b.n));
    const X3Group *one = &it;
    const int rc = x3_launch_groups(&one, 1, st);
    if (rc != WGRAD_OK || it.pl.splits == 1) return rc;
    return launch_combine(it.ws, it.slice_stride, it.pl.splits, g.dw_elems(), 1.0f, b.dW, b.n, st, defer);
}

}  // namespace wgrad
