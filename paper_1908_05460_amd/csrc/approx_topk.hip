// Top-k generalisation of the max-gradient approximation (arXiv 1908.05460, Section 2.3):
// every map of dY keeps its k entries of largest magnitude instead of one, and each kept
// position carries sum/k, so that the k = 1 case is Algorithm 1 and the retained mass is
// the map's sum whatever k is.  Two kernels: selection, then a gather over the kept
// positions; the batch-chunk partials go through the common reduction.
#include <type_traits>

#include "common.hpp"

namespace wgrad {

namespace {

// A position's rank key: magnitude bits above, inverted index below.  Keys of one map are
// all different, and "larger magnitude first, smaller index first among equals" is plain
// descending key order.  NaN ranks as zero magnitude.
__device__ __forceinline__ unsigned long long rank_key(uint32_t bits, uint32_t pos)
{
    uint32_t m = bits & 0x7fffffffu;
    m = m > 0x7f800000u ? 0u : m;
    return ((unsigned long long)m << 32) | (uint32_t)~pos;
}

template <bool BF16>
__device__ __forceinline__ uint32_t load_bits(const void *p, long i)
{
    return BF16 ? (uint32_t)((const uint16_t *)p)[i] << 16 : ((const uint32_t *)p)[i];
}

// maximum over aligned groups of G lanes (G a power of two up to 64)
__device__ __forceinline__ unsigned long long group_max(unsigned long long v, int G)
{
    for (int d = G >> 1; d > 0; d >>= 1) {
        const unsigned long long o = __shfl_xor(v, d, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Reduction over a wavefront by lane shifts within rows and broadcasts across them; the result is lane 63's, made uniform.
template <bool MAX>
__device__ __forceinline__ int wave_extreme(int v)
{
    auto step = [&](int o) { v = MAX ? (o > v ? o : v) : (o < v ? o : v); };
    step(__builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));        // row_shr:1, 2, 4, 8
    step(__builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    step(__builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));        // row_bcast:15, 31
    step(__builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// A group of G lanes per map (WG = 0; G a power of two, 64 / G maps per wavefront, so that maps of four
// positions take a lane each and not a wavefront each), or one workgroup per map for maps of more than 1024
// positions (WG = its threads: few, long maps would otherwise leave most of the chip idle).  Pass j finds the largest
// key below the one pass j-1 found; the map's sum rides along with pass 0.  Maps of up to T*REG entries (T = G or
// WG threads) stay in registers between the passes, longer ones are read again (from L2).
//
// What bounds it is vector instructions (a workgroup of 56x56 maps reads 12 KB, which takes a fraction of that), so
// the registers hold magnitudes alone, a thread keeps its own best as (magnitude, register) and goes over its
// registers again only when its best was the one taken, and `vec` (positions in quads: a multiple of four to a map,
// words of four bytes aligned) reads four positions at a time, past the end of a map without a branch.
// 56x56 maps, N = 32, K = 64, k = 4: 20.8 -> 14.0 us.  Up to 57344 positions stay in registers (to 4096 before: with the
// gather, 112x112, N = 4, K = 64, k = 4: 50 -> 18 us; 36x229, N = 7, K = 173, k = 8 in bf16: 66 -> 32).
// Beyond 16384 the workgroup has 1024 threads (146x154, N = 17, K = 13, k = 8: 140 -> 29 us; 224x224, N = 4, K = 64, k = 4:
// 272 -> 36); at 56 positions a thread some 50 registers spill, which costs less than reading the map k times.
template <bool BF16, int REG, int WG>
__global__ __launch_bounds__(WG ? WG : kBlock) void topk_select(const void *__restrict__ dY, long maps, int len, int Wo,
                                                      int k, int G, int32_t *__restrict__ hw_out,
                                                      int32_t *__restrict__ flat_out, float *__restrict__ sum_a,
                                                      float *__restrict__ sum_b, void *__restrict__ sparse, float w, bool vec)
{
    constexpr bool WIDE = WG > 0;
    constexpr int WAVES = (WIDE ? WG : kBlock) / 64;
    const int T = WIDE ? WG : G;
    __shared__ unsigned long long wg_best[2][WAVES];      // WIDE: the wavefronts' maxima, double-buffered over passes
    __shared__ float wg_sum[WAVES];
    const int lane = WIDE ? threadIdx.x : (threadIdx.x & 63) % G;
    const long map = WIDE ? (long)blockIdx.x
                          : ((long)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * (64 / G) + (threadIdx.x & 63) / G;
    if (map >= maps) return;                      // whole groups leave together (WIDE: the grid is exactly maps)
    const long base = map * len;

    constexpr int kTaken = -1, kAbsent = -2;                    // below every magnitude
    int mag[REG > 0 ? REG : 1];
    // (positions of a thread grow with the register, so the first of equal magnitudes is the smallest position)
    auto position = [&](int i) { return vec ? 4 * (lane + T * (i / 4)) + i % 4 : lane + T * i; };
    float sum = 0.f;
    if constexpr (REG > 0) {
        constexpr uint32_t kDead = 0x80000000u;                 // beyond the buffer: reads as zero
        constexpr int ES = BF16 ? 2 : 4;
        const long first = WIDE ? (long)blockIdx.x : (long)blockIdx.x * (kBlock / 64) * (64 / G);
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)dY + first * len * ES), 0, kDead, 0x00020000);
        const uint32_t off = (uint32_t)(map - first) * (uint32_t)(len * ES);
        // (in two halves where the bits of all of a thread's positions beside their magnitudes would spill)
        constexpr int PART = REG > 32 ? REG / 2 : (WG > 256 ? REG / 2 : REG);
#pragma unroll
        for (int i0 = 0; i0 < REG; i0 += PART) {
            uint32_t bits[PART];
            if (vec) {
#pragma unroll
                for (int i = 0; i < PART; i += 4) {
                    const int e = position(i0 + i);
                    const uint32_t at = e < len ? off + (uint32_t)(e * ES) : kDead;
                    if constexpr (BF16) {
                        const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, at, 0, 0);
                        bits[i] = v[0] << 16; bits[i + 1] = v[0] & 0xffff0000u; bits[i + 2] = v[1] << 16; bits[i + 3] = v[1] & 0xffff0000u;
                    } else {
                        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, 0, 0);
#pragma unroll
                        for (int q = 0; q < 4; ++q) bits[i + q] = v[q];
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < PART; ++i) {
                    const int e = position(i0 + i);
                    const uint32_t at = e < len ? off + (uint32_t)(e * ES) : kDead;
                    if constexpr (BF16) bits[i] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, at, 0, 0) << 16;
                    else bits[i] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < PART; ++i) {
                int m = (int)(bits[i] & 0x7fffffffu);
                m = m > 0x7f800000 ? 0 : m;
                mag[i0 + i] = position(i0 + i) < len ? m : kAbsent;
                sum += __uint_as_float(bits[i]);
            }
            if (PART < REG) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        for (int e = lane; e < len; e += T) sum += __uint_as_float(load_bits<BF16>(dY, base + e));
    }
    for (int d = (WIDE ? 64 : G) >> 1; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (WIDE) {
        if ((threadIdx.x & 63) == 0) wg_sum[threadIdx.x >> 6] = sum;
        __syncthreads();
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; w += 4) sum += (wg_sum[w] + wg_sum[w + 1]) + (wg_sum[w + 2] + wg_sum[w + 3]);
    }

    unsigned long long below = ~0ull;
    int own = kAbsent, own_reg = 0;                              // the thread's best
    auto scan = [&]() {
        own = mag[0], own_reg = 0;
#pragma unroll
        for (int i = 1; i < REG; ++i)
            if (mag[i] > own) own = mag[i], own_reg = i;
    };
    if (REG > 0) scan();
    for (int j = 0; j < k; ++j) {
        unsigned long long best = 0ull;
        const int own_pos = position(own_reg);
        if (REG > 0) {
            if (WIDE || G == 64) {
                const int m = wave_extreme<true>(own), pos = wave_extreme<false>(own == m ? own_pos : 0x7fffffff);
                if (m >= 0) best = (unsigned long long)(uint32_t)m << 32 | (uint32_t)~pos;
            } else {
                if (own >= 0) best = (unsigned long long)(uint32_t)own << 32 | (uint32_t)~own_pos;
                best = group_max(best, G);
            }
        } else {
            for (int e = lane; e < len; e += T) {
                unsigned long long c = rank_key(load_bits<BF16>(dY, base + e), (uint32_t)e);
                c = c < below ? c : 0ull;
                best = c > best ? c : best;
            }
            best = group_max(best, WIDE ? 64 : G);
        }
        if (WIDE) {
            // pass j writes buffer j & 1; the barrier of pass j+1 separates its readers from pass j+2's writers
            if ((threadIdx.x & 63) == 0) wg_best[j & 1][threadIdx.x >> 6] = best;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < WAVES; ++w) best = wg_best[j & 1][w] > best ? wg_best[j & 1][w] : best;
        }
        below = best;
        if (REG > 0 && own >= 0 && own_pos == (int)~(uint32_t)best) {
#pragma unroll
            for (int i = 0; i < REG; ++i) mag[i] = i == own_reg ? kTaken : mag[i];
            scan();
        }
        if (threadIdx.x == 0 || (!WIDE && lane == 0)) {
            const int32_t pos = (int32_t)~(uint32_t)best;
            if (flat_out) flat_out[map * k + j] = pos;
            hw_out[map * k + j] = ((pos / Wo) << 16) | (pos % Wo);
        }
    }
    if (threadIdx.x == 0 || (!WIDE && lane == 0)) {
        sum_a[map] = sum;
        if (sum_b) sum_b[map] = sum;
    }
    // optional: the sparsified map, sum * w at the kept positions (the k largest keys: those not below the
    // last one found) and zero elsewhere, in the element type of the inputs
    if (sparse) {
        const float kept = sum * w;
        auto put = [&](int e, bool is_kept) {
            const float v = is_kept ? kept : 0.f;
            if (BF16) {
                const uint32_t b = __float_as_uint(v);           // round to nearest even; v is finite
                ((uint16_t *)sparse)[base + e] = (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
            } else {
                ((float *)sparse)[base + e] = v;
            }
        };
        if (REG > 0) {
#pragma unroll
            for (int i = 0; i < REG; ++i) {
                const int e = position(i);
                if (e < len) put(e, mag[i] == kTaken);
            }
        } else {
            for (int e = lane; e < len; e += T)
                put(e, rank_key(load_bits<BF16>(dY, base + e), (uint32_t)e) >= below);
        }
    }
}

// One thread per filter-gradient entry (ko, c, r, s) and batch chunk: it walks the chunk's
// images and the k kept positions of map (n, ko), adding (sum/k) times the input element
// its tap sees there (zero outside the image).  The loads bound it: kDeep positions, then kDeep
// elements, are in flight at a time, and an XCD takes whole chunks, so that the input of a chunk
// is fetched into one L2 and not into all eight.  On small planes, whose loads hit, the addresses bound it instead: what a
// wavefront shares is added in scalar registers, a lane's part is 32 bits wide and its products 24 (FAR: sizes beyond
// that, with 64-bit parts).
// 64 -> 64 @ 56x56, N = 32, k = 4: 23.2 -> 12.4 us; 215 -> 62 @ 9x6, 5x5, stride 2, N = 84, k = 8: 282 -> 183 (216 without
// the loads ahead).
template <bool BF16, bool FAR>
__global__ __launch_bounds__(kBlock) void topk_gather(const void *__restrict__ X, const int32_t *__restrict__ hw,
                                                      const float *__restrict__ sum, float *__restrict__ out,
                                                      Geometry g, int k, float inv_k, int chunk_n, float scale, int eblocks)
{
    constexpr int kDeep = 8;
    const int logical = xcd_contiguous_id((int)blockIdx.x, (int)gridDim.x), chunk = __builtin_amdgcn_readfirstlane(logical / eblocks);
    const long o = (long)(logical - chunk * eblocks) * kBlock + threadIdx.x;
    const int RS = g.R * g.S, CRS = g.C * RS;
    if (o >= (long)g.K * CRS) return;
    const int ko = (int)(o / CRS), q = (int)(o % CRS);
    const int c = q / RS, r = (q % RS) / g.S - g.ph, s = (q % RS) % g.S - g.pw;
    constexpr int ES = BF16 ? 2 : 4;
    using part_t = std::conditional_t<FAR, uint64_t, uint32_t>;
    const part_t c_at = (part_t)c * (part_t)g.H * (part_t)g.W * ES, hw_at = (part_t)ko * (part_t)k * 4, sum_at = (part_t)ko * 4;
    auto times = [](int a, int b) { return FAR ? (part_t)a * (part_t)b : (part_t)(uint32_t)__mul24(a, b); };
    const int n_begin = chunk * chunk_n;
    const int n_end = n_begin + chunk_n < g.N ? n_begin + chunk_n : g.N;
    float acc = 0.f, part = 0.f;
    // the next kept position of the chunk: its image, its map's entries of filter 0, its place among the map's k
    const char *image = (const char *)X + (long)n_begin * g.C * g.H * g.W * ES;
    const int32_t *kept = hw + (long)n_begin * g.K * k;
    const float *sums = sum + (long)n_begin * g.K;
    const long next_image = (long)g.C * g.H * g.W * ES, next_map = (long)(g.K - 1) * k + 1;
    long left = (long)(n_end - n_begin) * k;
    int j = 0;
    auto batch = [&](auto whole) {                               // of kDeep positions; not whole: the last one is read again
        constexpr bool WHOLE = decltype(whole)::value;
        int at[kDeep];
        const char *img[kDeep];
        bool valid[kDeep], last[kDeep];                          // last of its map
        float share[kDeep];
        uint32_t x[kDeep];                                       // as loaded
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            valid[u] = WHOLE || u < left;
            img[u] = image;
            at[u] = *(const int32_t *)((const char *)kept + hw_at);
            last[u] = j == k - 1;
            share[u] = 0.f;
            if (last[u]) share[u] = *(const float *)((const char *)sums + sum_at);
            if (WHOLE || u + 1 < left) {
                ++j;
                if (j == k) { j = 0; image += next_image; sums += g.K; kept += next_map; }
                else ++kept;
            }
        }
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            const int ih = (int)times(at[u] >> 16, g.sh) + r, iw = (int)times(at[u] & 0xffff, g.sw) + s;
            const bool inside = (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W;
            const part_t xi = c_at + (inside ? times(ih, g.W) + (part_t)iw : 0) * ES;
            const uint32_t v = BF16 ? *(const uint16_t *)(img[u] + xi) : *(const uint32_t *)(img[u] + xi);
            x[u] = v & (inside && valid[u] ? ~0u : 0u);          // (a choice of v or 0 becomes a branch, which waits for its load)
        }
        // the same sums in the same order, whatever kDeep: a map's k elements, then their share
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            part += BF16 ? bf16_bits_to_float((uint16_t)x[u]) : __uint_as_float(x[u]);
            if (valid[u] && last[u]) {
                acc = fmaf(share[u] * inv_k, part, acc);
                part = 0.f;
            }
        }
        left -= kDeep;
    };
    // (the pointers stop at the chunk's last position: a whole batch may end there only if nothing is read after it)
    while (left >= kDeep) batch(std::true_type{});
    if (left > 0) batch(std::false_type{});
    out[(long)chunk * g.K * CRS + o] = acc * scale;
}

// When the kept positions are a sizeable share of a map, gathering their patches moves as much data as the
// dense kernel and loses to the matrix core: the gradient is then computed as the exact gradient of the
// sparsified dY (Section 2.4's identity).  Thresholds from measurements on the VGG-19 layers (N = 128): the
// LDS gather costs about k/2 of the dense kernel on 4x4 planes and k/5 on 8x8 planes; the general gather
// loses from three kept positions of 256 on; with bf16 inputs the dense kernel is twice as fast again.
bool topk_sparse_exact(const Geometry &g, int k, ExactPlan &ex)
{
    if (!tune_int("WGRAD_TOPK_SX", 1)) return false;
    const int L = g.Ho * g.Wo;
    ex = plan_exact_plain(g);
    if (!ex.ok) return false;
    // the bf16 matrix-core kernel runs a dense layer in the time the gather needs for one kept position
    const bool fast_bf16 = ex.mm16 && k >= 2;
    // large maps, few channels: the fused kernel, unless the bf16 matrix core beats it (maps of up to 256 positions)
    bool take;
    if (topk_takes_fused(g, k)) take = fast_bf16 && L <= 256;
    else {
        const ApproxPlan ap = plan_approx(g, /*allow_lds=*/true, /*allow_fused=*/false, /*allow_mm=*/false);
        const bool lds = ap.use_lds && ap.m * k <= 64;
        const bool dense_enough = L <= 4 || (lds ? k >= 2 && k * 14 >= L : k * 80 >= L);
        take = fast_bf16 || ((ex.stream || ex.mm16) && dense_enough);
    }
    if (take) ex = plan_exact(g);
    return take;
}

int topk_chunks(const Geometry &g)
{
    // enough (entry, chunk) threads to fill the chip, at least 4 images per chunk
    const long entries = g.dw_elems();
    long chunks = (256l * 1024 + entries - 1) / entries;
    const long most = (g.N + 3) / 4;
    chunks = chunks > most ? most : chunks;
    return (int)(chunks < 1 ? 1 : chunks);
}

}  // namespace

bool topk_supported(const Geometry &g, int k)
{
    return k >= 1 && k <= kTopKMax && (long)k <= (long)g.Ho * g.Wo && g.Ho < 32768 && g.Wo < 65536;
}

// batch-chunk partials of whichever form runs: the general gather here, the fused kernel or the LDS gather
static size_t topk_partial_bytes(const Geometry &g)
{
    const int chunks = topk_chunks(g);
    size_t general = chunks > 1 ? (size_t)chunks * g.dw_elems() * sizeof(float) : 0;
    const size_t borrowed = topk_borrowed_partial_bytes(g);
    return align_up(general > borrowed ? general : borrowed);
}

size_t topk_ws_bytes(const Geometry &g, int k)
{
    const size_t maps = (size_t)g.N * g.K;
    size_t tail = topk_partial_bytes(g);
    ExactPlan ex;
    if (topk_sparse_exact(g, k, ex)) {
        const size_t sx = align_up(maps * g.Ho * g.Wo * (g.bf16 ? 2 : 4)) + align_up(ex.ws_bytes);
        if (sx > tail) tail = sx;
    }
    return align_up(maps * k * sizeof(int32_t)) + align_up(maps * sizeof(float)) + tail;
}

bool launch_topk_group(const Geometry &g, const Batch &b, int k, float scale, void *ws, size_t slice_bytes,
                       hipStream_t st, int *rc, FusedQueue *fq, CombineQueue *defer)
{
    ExactPlan ex;
    if (topk_sparse_exact(g, k, ex)) return false;         // that form runs layer by layer
    // a slice holds the kept positions, the sums, then the partials (as in launch_approx_topk)
    const long maps = (long)g.N * g.K;
    const size_t off = align_up((size_t)maps * k * sizeof(int32_t)) + align_up((size_t)maps * sizeof(float));
    return topk_fused(g, b, k, scale, nullptr, nullptr, (float *)((char *)ws + off), (long)(slice_bytes / 4), st, rc, fq, defer);
}

// fq, defer: a schedule run's queue of fused launches and of reductions (the fused form then only records its work)
int launch_approx_topk(const Geometry &g, const void *X, const void *dY, float *dW, int k, float scale,
                       int32_t *idx_out, float *sum_out, void *ws, hipStream_t st, FusedQueue *fq, CombineQueue *defer)
{
    const long maps = (long)g.N * g.K;
    const int len = g.Ho * g.Wo;
    char *w = (char *)ws;
    int32_t *hw = (int32_t *)w;  w += align_up((size_t)maps * k * sizeof(int32_t));
    float *sum = (float *)w;     w += align_up((size_t)maps * sizeof(float));
    float *partials = (float *)w;

    int rc;
    // kept positions a sizeable share of a map: the selection also writes the sparsified dY, and the exact
    // kernel contracts it
    ExactPlan ex;
    const bool sx = topk_sparse_exact(g, k, ex);
    void *sparse = sx ? (void *)partials : nullptr;
    // maps of up to 1024 positions and C*R*S <= 2304: selection and gather in one launch
    Batch one{};
    one.n = 1; one.X[0] = X; one.dY[0] = dY; one.dW[0] = dW;
    if (!sx && topk_fused(g, one, k, scale, idx_out, sum_out, partials, 0, st, &rc, fq, defer)) return rc;

    const bool wide = len > 1024;
    // lanes per map: four positions each up to 256 positions, sixteen up to 1024
    int G = 1;
    while (G < 64 && G * 4 < len) G <<= 1;
    const long waves = (maps + 64 / G - 1) / (64 / G);
    const long grid = wide ? maps : (waves + kBlock / 64 - 1) / (kBlock / 64);
    if (grid >= (1l << 31)) return WGRAD_UNSUPPORTED;
    const bool vec = len % 4 == 0 && ((uintptr_t)dY & 3) == 0;
#define SEL(BF, REG, WG) WGRAD_LAUNCH((topk_select<BF, REG, WG>), dim3((unsigned)grid), dim3(WG ? WG : kBlock), 0, st, dY, maps, len, g.Wo, k, G, hw, idx_out, sum, sum_out, sparse, scale / k, vec)
#define SEL_PICK(BF)                                     \
    if (len <= 256)        SEL(BF, 4, 0);                \
    else if (len <= 1024)  SEL(BF, 16, 0);               \
    else if (len <= 4096)  SEL(BF, 16, 256);             \
    else if (len <= 8192)  SEL(BF, 32, 256);             \
    else if (len <= 16384) SEL(BF, 64, 256);             \
    else if (len <= 32768) SEL(BF, 32, 1024);            \
    else if (len <= 57344) SEL(BF, 56, 1024);            \
    else                   SEL(BF, 0, 256)
    if (g.bf16) { SEL_PICK(true); } else { SEL_PICK(false); }
#undef SEL_PICK
#undef SEL
    rc = launch_status();
    if (rc != WGRAD_OK) return rc;

    if (sx) {
        Batch eb{};
        eb.n = 1; eb.X[0] = X; eb.dY[0] = sparse; eb.dW[0] = dW;
        return launch_exact(g, ex, eb, (char *)partials + align_up((size_t)maps * len * (g.bf16 ? 2 : 4)), st);
    }

    // small planes and many output channels: the LDS-staged gather of the k = 1 path, over k positions per map
    if (topk_gather_lds(g, X, hw, sum, k, scale, dW, partials, topk_partial_bytes(g), st, &rc)) return rc;

    const int chunks = topk_chunks(g);
    const int chunk_n = (g.N + chunks - 1) / chunks;
    const int nchunk = (g.N + chunk_n - 1) / chunk_n;
    const long entries = g.dw_elems();
    float *out = nchunk > 1 ? partials : dW;
    const int eblocks = (int)((entries + kBlock - 1) / kBlock);
    const dim3 gg((unsigned)eblocks * (unsigned)nchunk);
    const float gscale = nchunk > 1 ? 1.0f : scale;
    // (kept rows and columns beyond the first bound their stride by the padded plane's side; without any the product is zero)
    const bool far = (long)g.C * g.H * g.W * (g.bf16 ? 2 : 4) >= (1l << 32) || (long)g.K * k * 4 >= (1l << 32) ||
                     (long)g.H + 2l * g.ph >= (1l << 23) || (long)g.W + 2l * g.pw >= (1l << 23);
#define GATHER(BF, FAR) WGRAD_LAUNCH((topk_gather<BF, FAR>), gg, dim3(kBlock), 0, st, X, hw, sum, out, g, k, 1.0f / k, chunk_n, gscale, eblocks)
    if (g.bf16) { if (far) GATHER(true, true); else GATHER(true, false); }
    else        { if (far) GATHER(false, true); else GATHER(false, false); }
#undef GATHER
    rc = launch_status();
    if (rc != WGRAD_OK || nchunk == 1) return rc;
    float *dst[1] = {dW};
    return launch_combine(partials, 0, nchunk, entries, scale, dst, 1, st, nullptr);
}

}  // namespace wgrad
