// Bounded matching cost over all views, Sec. 3.5: Eq. (12) (l2 of the
// bilinearly shifted views) and Eq. (15) (Census Hamming at the nearest shift).
//
// Work is flattened over the cells of the CSR volume so that pixels whose range
// is the full hypothesis set and pixels with a 2*lambda+1 window share the
// machine evenly; a cell, or a hypothesis of a few adjacent pixels, is found by binary
// search over offsets staged in LDS.  Consecutive threads handle consecutive
// hypotheses and then the next pixels of the row, so the taps of a view are read from
// a narrow band of rows (L1/L2 resident) and the cost writes are close together.
//
// The view loop runs t outer, s inner, float32, with the shift of each view and
// hypothesis rounded once: this is the precision the quantised integer cost is
// decided in.  The reference view contributes exactly +0 and is skipped.
#include "lf_internal.h"

#include <algorithm>
#include <type_traits>

namespace lf {
namespace {

constexpr int kThreads = 256;
// Workgroups of a launch at most.  A launch has fewer than 2^32 work items, 2^24 of these
// workgroups, which volumes of 2^33 cells (worst case) would exceed; those walk their
// slices instead.
constexpr int64_t kMostBlocks = 1 << 23;

// The pixel that owns cell c0, off[p0] <= c0 < off[p0 + 1], of HW pixels: every wave
// searches by itself, 64 pixels at a time (four rounds for 2^24 of them; a binary search
// is 24 loads one after the other, which took most of a slice's time with few views).
__device__ __forceinline__ int first_pixel(const int64_t* __restrict__ off, int HW, int64_t c0) {
    int p0 = 0, n = HW;                       // p0 <= the pixel < p0 + n
    while (n > 1) {
        const int step = (n + 63) / 64;
        const int at = p0 + (int)(threadIdx.x & 63) * step;
        const bool below = at < p0 + n && off[at] <= c0;          // the first lane is
        const int hit = max(__popcll(__builtin_amdgcn_ballot_w64(below)) - 1, 0);
        const int end = p0 + n;
        p0 += hit * step;
        n = min(step, end - p0);
    }
    return p0;
}

// The same by one thread, among the pixels from p on.
__device__ __forceinline__ int pixel_of(const int64_t* __restrict__ off, int p, int end,
                                        int64_t c) {
    while (end - p > 1) {
        const int mid = p + (end - p) / 2;
        if (off[mid] <= c) p = mid; else end = mid;
    }
    return p;
}

// ---------------------------------------------------------------------------
// l2 cost, Eq. (12).  Work is dealt in equal slices of cells: slice i is the
// cells [i*chunk, (i+1)*chunk) of the CSR volume, whatever pixels they belong
// to, so pixels with the full hypothesis range and pixels with a 2*lambda+1
// window cost the same per cell and no workgroup is a straggler.  The number of
// slices is only known on the device (the last offset), so a light field gets
// nblk workgroups sized for its worst case, and workgroup b walks the slices
// b, b + nblk, ... that exist.  The first pixel of a slice is searched for over
// the offsets; the offsets and lower bounds of the slice's pixels are staged in LDS.
//
// What bounds this kernel is the issue of its scattered gathers (about four lanes a
// cycle per CU, whatever their width up to 16 bytes), then its VALU.  So a slice's
// pixels form groups of G horizontally adjacent ones: at one hypothesis a view shifts
// them alike, and one load of G + 1 elements per tap row (and channel) serves them all.
// The copy of 8-bit colour views interleaves the channels of a pixel in a word.

// Pixels per group.  A larger group has fewer loads per cell, a wider hull of its pixels'
// ranges (on the benchmark bounds 1, 3, 5 pixels: 1.0, 2.0, 2.6 cells per hypothesis of
// the hull) and so more arithmetic per cell.  Float views are bound by the loads: 3,
// what 16 bytes hold.  8-bit grayscale ones by both: 3 (338 us; 4 or 5 with 8-byte
// loads 418 us, one cell per thread with four 2-byte loads 512 us; 9x9x512^2, N = 100).
// 8-bit colour ones by the arithmetic of three channels: 1 (625 us; 2 and 3 pixels
// 916 and 1232 us, the planes apart 1870 us; the same size).
template <typename T, int C>
constexpr int kGroupOf = sizeof(T) == 4 ? 3 : C == 1 ? 3 : 1;

// Items per 100 cells above which a slice takes one cell at a time instead.  An item takes
// as long as 1.5 cells alone (8-bit), 1.6 (colour), also one of a hull's gap, and where
// neighbours' windows have little in common a hull is mostly gaps.  9x9x512^2: windows of 7
// anywhere in 64 hypotheses 379 us in groups, 268 so (8-bit), 429 / 304 (float), 2385 / 1288
// (colour float); a third of them anywhere in 100, a tenth of the pixels full, 462 / 376,
// 479 / 365, 2298 / 1995; a twentieth 317 / 309, 328 / 313, 1481 / 1360; on the benchmark
// bounds the same.  With 50 for 75 windows anywhere gain more (a third 1745 us), but colour
// float views of real bounds lose (7x3x61x1867, N = 137, 607 us for 512).  Colour 8-bit
// views have no groups.
template <typename T, int C>
constexpr int kSparse = C == 3 ? 75 : 100;

// Views with a replicated edge: padded (y', x') holds the view at (clamp(y' - 1),
// clamp(x' - L)), y' < H + 2, x' < W + P (one row above and below, L >= G columns left,
// P - L right).  With it, the two clamped taps of a bilinear row, (clamp(X),
// clamp(X+1)), are always the two consecutive elements starting at clamp(X, -1, W-1) +
// L -- one load, no edge cases, and the same values (so the same float32 sums) as
// clamping each tap; and the taps of the pixels g = 1 .. G-1 to the right, (clamp(X+g),
// clamp(X+g+1)), are always elements g, g+1 of the G+1 starting at clamp(X, -L, W-1) + L
// (X outside that range reads replicas).
constexpr int kPadT = 1;
constexpr int kPadL = 3;
static_assert(kPadW == 2 * kPadL && kPadH == 2, "the view copy's margins");
// Columns of the copy.  Single-byte rows a multiple of 128 bytes apart, and up to 9 bytes
// less or more, get up to 23 more: the bottom taps conflict with the top ones in the cache
// (9x9x256xW, N = 100, in us per pixel column: rows of 498 and 502 bytes 0.38, 506 0.41, 510
// and 514 0.54, 518 0.40, 522 0.354, 526 0.349, up to 600 0.35; the same around 256, 384,
// 640, 768, 1024 and 1920).  Fits the workspace, which is of floats, and a row of views of
// 2^31 bytes stays below 2^32.
__host__ __device__ __forceinline__ int copy_width(int H, int W, size_t elem) {
    const int w = W + kPadW, m = w & 127;
    if (elem != 1 || H < 8 || W < 64 || (m > 9 && m < 119)) return w;
    return (w + 9) / 128 * 128 + 14;
}

struct PadArgs {
    gptr<const void> src;          // [planes][H][pitch] (a view is C planes)
    gptr<void> dst;                // [planes][H + 2][W + P]
    int H, W, pitch;
};

// Element of the copy at x from the three planes' rows of an 8-bit colour view.
__device__ __forceinline__ uint32_t rgb_word(const uint8_t* r, size_t plane, int x) {
    return (uint32_t)r[x] | (uint32_t)r[plane + x] << 8 | (uint32_t)r[2 * plane + x] << 16;
}

// A workgroup copies kPadRows padded rows of one plane: block b is rows
// kPadRows * (b % g) .. of plane b / g (g row groups per plane).  Each thread
// loads its elements of all the rows (3 x kPadRows per 768 columns) before it
// stores them, so that many loads are in flight.
constexpr int kPadRows = 4;

// kRGB: 8-bit colour views, copied [views][H + 2][W + P] with a pixel's channels
// in bytes 0..2 of a word.
template <class Src, typename T, bool kRGB>
__global__ __launch_bounds__(kThreads) void pad_views_kernel(Src src) {
    using E = typename std::conditional<kRGB, uint32_t, T>::type;
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const PadArgs& a = member(src, vb, b);
        const int Hp = a.H + kPadH, Wp = copy_width(a.H, a.W, sizeof(E));
        const int g = (Hp + kPadRows - 1) / kPadRows;
        const int z = (int)(b / (uint32_t)g);
        const int y0 = ((int)b - z * g) * kPadRows;
        for (int xb = 0; xb < Wp; xb += 3 * kThreads) {
            E v[kPadRows][3];
#pragma unroll
            for (int r = 0; r < kPadRows; ++r) {
                const T* __restrict__ row =
                    (const T*)a.src + ((size_t)z * (kRGB ? 3 : 1) * a.H +
                                       clampi(y0 + r - kPadT, 0, a.H - 1)) * a.pitch;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int x = clampi(xb + e * kThreads + (int)threadIdx.x - kPadL, 0, a.W - 1);
                    if constexpr (kRGB) v[r][e] = rgb_word(row, (size_t)a.H * a.pitch, x);
                    else v[r][e] = row[x];
                }
            }
#pragma unroll
            for (int r = 0; r < kPadRows; ++r) {
                if (y0 + r >= Hp) break;
                E* __restrict__ out = (E*)a.dst + ((size_t)z * Hp + y0 + r) * Wp;
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const int x = xb + e * kThreads + (int)threadIdx.x;
                    if (x < Wp) out[x] = v[r][e];
                }
            }
        }
    }
}

struct L2Args {
    gptr<const void> views;        // padded: [T][S][C][H + 2][W + P], 8-bit colour ones
                                   // [T][S][H + 2][W + P] words
    gptr<const float> hyp;
    gptr<const int16_t> lo;
    gptr<const int64_t> off;       // [H*W + 1]
    gptr<uint16_t> cost;
    gptr<float> cost_f32;          // nullable
    int64_t cap_cells;
    int S, T, H, W, N;
    float alpha, cap;
    uint32_t nblk;            // workgroups of this light field
};

// The taps of a group of G pixels in one tap row at p: n = G + 1 consecutive elements
// per channel, or the first G of them, one load per plane (planes `plane` bytes apart).
template <int C, int n>
struct Taps {
    float e[C][n];
};
template <typename T, int C, int n>
__device__ __forceinline__ Taps<C, n> ld_taps(const char* __restrict__ p, uint32_t plane) {
    Taps<C, n> r;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int c = 0; c < C; ++c) __builtin_memcpy(r.e[c], p + (size_t)c * plane, 4 * n);
    } else if constexpr (C == 1) {
        static_assert(n <= 4, "one word");
        uint32_t w;
        __builtin_memcpy(&w, p, 4);
#pragma unroll
        for (int g = 0; g < n; ++g) r.e[0][g] = (float)(w >> (8 * g) & 0xFF);
    } else {
        uint32_t w[n];
        __builtin_memcpy(w, p, 4 * n);
#pragma unroll
        for (int g = 0; g < n; ++g)
#pragma unroll
            for (int c = 0; c < 3; ++c) r.e[c][g] = (float)(w[g] >> (8 * c) & 0xFF);
    }
    return r;
}

// The correctly rounded square root of 0 and of every x in [2^-100, 2^100] (one
// Newton step in fused arithmetic from the reciprocal square root; compared with
// sqrtf on all 1.7e9 floats of the range): 6 instructions for the library's 17.
constexpr float kRootMin = 0x1p-100f, kRootMax = 0x1p100f;
__device__ __forceinline__ float root(float x) {
    const float y = __builtin_amdgcn_rsqf(fmaxf(x, kRootMin));
    const float s = x * y, h = 0.5f * y;
    return fmaf(fmaf(-s, s, x), h, s);
}

// Exclusive prefix sum of one value per thread over the workgroup; *total its sum.
__device__ __forceinline__ uint32_t block_prefix(uint32_t own, uint32_t* s_wave, uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t n = __shfl_up(inc, o);
        if (lane >= o) inc += n;
    }
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        const uint32_t x = s_wave[w];
        if (w < wave) before += x;
        all += x;
    }
    *total = all;
    return before + inc - own;
}

// LDS of one slice's pixels and groups.
template <int CPT>
struct SliceLds {
    int rel[kThreads * CPT + 1];       // a pixel's first cell, from the slice's first
    int16_t lo[kThreads * CPT];
    uint32_t pre[kThreads * CPT];      // per group: items of the groups before it,
    uint32_t uv[kThreads * CPT];       // its first pixel's u | v << 16,
    uint32_t rec[kThreads * CPT];      // that pixel's index | pixels << 12 | first k << 16
    uint32_t wave[kThreads / 64];
    int np;
};

template <typename T, int CPT, bool Walk, int C>
__device__ __forceinline__ void l2_slices(const L2Args& a, uint32_t b, SliceLds<CPT>& sl) {
    constexpr int kChunk = kThreads * CPT, G = kGroupOf<T, C>;
    // planes of a view in the copy, bytes of an element
    constexpr int CP = sizeof(T) == 1 && C == 3 ? 1 : C;
    constexpr int kElem = sizeof(T) == 1 && C == 3 ? 4 : (int)sizeof(T);
    static_assert(G <= kPadL, "the group's taps lie inside the margins");
    const int S = a.S, T_ = a.T, H = a.H, W = a.W, N = a.N;
    const int Wp = copy_width(H, W, kElem);
    const int16_t* __restrict__ lo = a.lo;
    const int64_t* __restrict__ off = a.off;
    const int HW = H * W;
    const int64_t total = min(off[HW], a.cap_cells);
    const int sh = (S - 1) / 2, th = (T_ - 1) / 2;
    const uint32_t row = (uint32_t)Wp * kElem, plane = (uint32_t)(H + kPadH) * row;
    const uint32_t vw_stride = (uint32_t)(H + kPadH) * Wp * CP;
    const uint32_t vbytes = plane * CP;            // of a view: below 2^32
    const char* __restrict__ views = (const char*)(const void*)a.views;
    auto view_at = [&](int t, int s) { return views + ((size_t)t * S + s) * vbytes; };

    auto store = [&](int64_t c, float acc) {
        const float q = rintf(a.alpha * acc);
        a.cost[c] = (uint16_t)(q > a.cap ? a.cap : q);
        if (a.cost_f32) a.cost_f32[c] = acc;
    };

    // Eq. (12) for the G pixels (u + g, v) at one hypothesis d, over the views t
    // outer, s inner; one view of row t takes taps at horizontal fraction fx from two
    // rows Wp apart.  Pixel g's taps are pixel 0's moved by g elements.  Two cases
    // skip taps that are weighted by an exact 0, since fma(0, b - a, a) is a exactly:
    // the reference row of views (t = t_hat, flat: fy = 0, no bottom taps) and the
    // reference column (s = s_hat, col: fx = 0, only the left tap of each row).  Each
    // case is its own branch-free copy of the loop body.
    // kRoot: the colour norm by root(), whose range the caller looks after: lim[] takes
    // the smallest and largest squared norm other than 0 (as bits, the smallest less 1).
    auto group = [&](int u, int v, float d, auto& acc, uint32_t (&lim)[2], auto kRoot) {
        constexpr int G = std::extent_v<std::remove_reference_t<decltype(acc)>>;
        const Taps<C, G> ref = ld_taps<T, C, G>(
            view_at(th, sh) + ((uint32_t)(v + kPadT) * Wp + u + kPadL) * kElem, plane);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[g] = 0.0f;
        constexpr std::true_type yes;
        constexpr std::false_type no;
        auto view = [&](const char* __restrict__ rt, float fy, int s, auto kFlat, auto kCol) {
            const float shx = (float)(sh - s) * d;
            const float x0 = floorf(shx);
            const float fx = shx - x0;
            const char* __restrict__ vw = rt + (size_t)((uint32_t)s * vw_stride) * kElem +
                                          (uint32_t)(clampi(u + (int)x0, -kPadL, W - 1) + kPadL) * kElem;
            constexpr int n = decltype(kCol)::value ? G : G + 1;
            const Taps<C, n> top = ld_taps<T, C, n>(vw, plane);
            Taps<C, n> bot;
            if constexpr (!decltype(kFlat)::value) bot = ld_taps<T, C, n>(vw + row, plane);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float sq = 0.0f, dist = 0.0f;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    float val = top.e[c][g];
                    if constexpr (!decltype(kCol)::value)
                        val = fmaf(fx, top.e[c][g + 1] - top.e[c][g], top.e[c][g]);
                    if constexpr (!decltype(kFlat)::value) {
                        float bv = bot.e[c][g];
                        if constexpr (!decltype(kCol)::value)
                            bv = fmaf(fx, bot.e[c][g + 1] - bot.e[c][g], bot.e[c][g]);
                        val = fmaf(fy, bv - val, val);
                    }
                    const float dl = ref.e[c][g] - val;
                    dist = fabsf(dl);
                    sq = c == 0 ? dl * dl : fmaf(dl, dl, sq);   // colour: l2 norm
                }
                if constexpr (C == 1) {
                    acc[g] = acc[g] + dist;
                } else if constexpr (!decltype(kRoot)::value) {
                    acc[g] = acc[g] + sqrtf(sq);
                } else {
                    acc[g] = acc[g] + root(sq);
                    if constexpr (sizeof(T) == 4) {
                        lim[0] = min(lim[0], __float_as_uint(sq) - 1u);
                        lim[1] = max(lim[1], __float_as_uint(sq));
                    }
                }
            }
        };
        // s ascending; the reference view itself adds exactly +0 and is skipped
        auto view_row = [&](const char* __restrict__ rt, float fy, auto flat) {
            for (int s = 0; s < sh; ++s) view(rt, fy, s, flat, no);
            if constexpr (!decltype(flat)::value) view(rt, fy, sh, no, yes);
            for (int s = sh + 1; s < S; ++s) view(rt, fy, s, flat, no);
        };
        for (int t = 0; t < T_; ++t) {
            const float shy = (float)(th - t) * d;
            const float y0 = floorf(shy);
            const float fy = shy - y0;
            // the top tap row, from its element at x = 0; the bottom one follows it
            const char* __restrict__ rt =
                view_at(t, 0) + (uint32_t)(clampi(v + (int)y0, -1, H - 1) + kPadT) * row;
            if (t == th) view_row(rt, fy, yes);
            else view_row(rt, fy, no);
        }
    };

    // the same with the root where it holds
    auto sums = [&](int u, int v, float d, auto& acc) {
        uint32_t lim[2] = {~0u, 0u};
        if constexpr (C == 1) {
            group(u, v, d, acc, lim, std::false_type());
        } else if constexpr (sizeof(T) == 1) {
            // 8-bit samples: a bilinear sum that is not its reference differs from
            // it by at least 2^-24, or where that is 0 by a product of two
            // fractions, each 0 or at least 2^-24 for such shifts
            if (d == 0.0f || fabsf(d) >= 0x1p-24f)
                group(u, v, d, acc, lim, std::true_type());
            else
                group(u, v, d, acc, lim, std::false_type());
        } else {
            group(u, v, d, acc, lim, std::true_type());
            if (lim[0] < __float_as_uint(kRootMin) - 1u || lim[1] > __float_as_uint(kRootMax))
                group(u, v, d, acc, lim, std::false_type());
        }
    };

    for (int64_t slice = b; slice * kChunk < total; slice += a.nblk) {   // uniform
        const int64_t c0 = slice * kChunk;
        const int64_t c1 = min(c0 + kChunk, total);
        if constexpr (Walk) __syncthreads();      // LDS of the previous slice is read
        const int p0 = first_pixel(off, HW, c0);
        const int npx = min(kChunk, HW - p0), len = (int)(c1 - c0);
        const int v0 = p0 / W, u0 = p0 - v0 * W;  // wave-uniform
        for (int i = threadIdx.x; i <= npx; i += kThreads) {
            sl.rel[i] = (int)(off[p0 + i] - c0);
            if (i < npx) sl.lo[i] = lo[p0 + i];
        }
        if (threadIdx.x == 0) sl.np = 0;
        __syncthreads();
        // pixels that own cells of the slice: up to the last one that starts in it
        for (int i = threadIdx.x; i < npx; i += kThreads)
            if (sl.rel[i] < len && (i + 1 == npx || sl.rel[i + 1] >= len)) atomicMax(&sl.np, i + 1);
        __syncthreads();
        const int np = sl.np, stop = min(sl.rel[npx], len);     // of the staged pixels' cells

        // Groups: a pixel at u = 0 mod G (or the slice's first pixel) with the following
        // pixels of its row up to the next such u that are in the slice.  A group's
        // items are the hypotheses k of the hull of its pixels' slice cells; an item
        // computes the cells (p + g, k) of the group that exist.  The slice cells of pixel
        // i are [max(rel[i], 0), min(rel[i + 1], len)), cell c is hypothesis
        // lo[i] + c - rel[i]; a pixel whose range is empty adds nothing.
        uint32_t cnt[CPT], rec[CPT], uv[CPT], own = 0;
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            const int i = (int)threadIdx.x * CPT + e;     // consecutive pixels per thread
            cnt[e] = 0;
            if (i >= np) continue;
            int u = u0 + i, v = v0;
            if (u >= W) {
                v += u / W;
                u = u % W;
            }
            if (i != 0 && u % G != 0) continue;
            const int n = min(min(G - u % G, np - i), W - u);
            int kl = INT_MAX, kh = INT_MIN;
            for (int g = 0; g < n; ++g) {
                const int r = sl.rel[i + g], f = max(r, 0), t = min(sl.rel[i + g + 1], len);
                if (f >= t) continue;
                const int l = sl.lo[i + g] - r;
                kl = min(kl, l + f);
                kh = max(kh, l + t - 1);
            }
            kl = max(kl, 0);                      // ranges outside [0, N) add nothing there
            kh = min(kh, N - 1);
            if (kl > kh) continue;
            cnt[e] = (uint32_t)(kh - kl + 1);
            rec[e] = (uint32_t)i | (uint32_t)n << 12 | (uint32_t)kl << 16;
            uv[e] = (uint32_t)u | (uint32_t)v << 16;
            own += 1u << 20 | cnt[e];             // at most 2,048 groups of 256 items
        }
        uint32_t total_groups;
        uint32_t at = block_prefix(own, sl.wave, &total_groups);
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            if (cnt[e] == 0) continue;
            sl.pre[at >> 20] = at & 0xFFFFFu;
            sl.rec[at >> 20] = rec[e];
            sl.uv[at >> 20] = uv[e];
            at += 1u << 20 | cnt[e];
        }
        __syncthreads();
        const int ngroups = (int)(total_groups >> 20), nitems = (int)(total_groups & 0xFFFFFu);
        // One cell at a time: where the hulls are mostly gaps, and where some cells are of
        // pixels past the staged ones (only if some of those own no cell).
        auto singles = [&](int from) {
            for (int c = from + threadIdx.x; c < len; c += kThreads) {
                int i = 0, k;
                if (G > 1 && c < stop) {
                    int end = np;                 // largest i with rel[i] <= c
                    while (end - i > 1) {
                        const int mid = (i + end) >> 1;
                        if (sl.rel[mid] <= c) i = mid; else end = mid;
                    }
                    k = sl.lo[i] + c - sl.rel[i];
                } else {
                    const int p = pixel_of(off, p0 + npx, HW, c0 + c);
                    i = p - p0;
                    k = lo[p] + (int)(c0 + c - off[p]);
                }
                if ((unsigned)k >= (unsigned)N) continue;
                int u = u0 + i, v = v0;
                if (u >= W) {
                    v += u / W;
                    u %= W;
                }
                float acc[1];
                sums(u, v, a.hyp[k], acc);
                store(c0 + c, acc[0]);
            }
        };
        const bool gaps = G > 1 && 100 * nitems > kSparse<T, C> * len;
        // before the items, or after them, as the registers come out better: after them the
        // gray kernels took 4 % longer, before them the colour float one 6 %
        constexpr bool kAfter = C == 3 && sizeof(T) == 4;
        if (!kAfter && __builtin_expect(gaps || stop < len, 0)) {    // uniform
            singles(G > 1 ? 0 : stop);
            if constexpr (G > 1) {
                if constexpr (Walk) continue; else break;
            }
        }
        for (int j = threadIdx.x; j < (kAfter && gaps ? 0 : nitems); j += kThreads) {
            int x = 0, y = ngroups;               // largest x with pre[x] <= j
            while (y - x > 1) {
                const int mid = (x + y) >> 1;
                if ((int)sl.pre[mid] <= j) x = mid; else y = mid;
            }
            const uint32_t gr = sl.rec[x], at = sl.uv[x];
            const int i = (int)(gr & 0xFFFu), n = (int)(gr >> 12 & 15u);
            const int k = (int)(gr >> 16) + (j - (int)sl.pre[x]);
            const int u = (int)(at & 0xFFFFu), v = (int)(at >> 16);
            int cell[G];                          // of the slice, or -1
            bool any = false;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                cell[g] = -1;
                if (g < n) {
                    const int r = sl.rel[i + g], c = r + k - sl.lo[i + g];
                    if (c >= max(r, 0) && c < min(sl.rel[i + g + 1], len)) cell[g] = c;
                }
                any |= cell[g] >= 0;
            }
            if (!any) continue;                   // a gap of the hull
            float acc[G];
            sums(u, v, a.hyp[k], acc);
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (cell[g] >= 0) store(c0 + cell[g], acc[g]);
        }
        if constexpr (kAfter) singles(gaps ? 0 : stop);
        if constexpr (!Walk) break;               // one slice per workgroup
    }
}

template <class Src, typename T, int CPT, bool Walk, int C>
__global__ __launch_bounds__(kThreads) void cost_l2_kernel(Src src) {
    __shared__ SliceLds<CPT> sl;
    uint32_t b;
    const L2Args& a = member(src, blockIdx.x, b);
    l2_slices<T, CPT, Walk, C>(a, b, sl);
}

// ---------------------------------------------------------------------------
// l2 cost where every pixel has the full range (a search without bounds, whose volume is
// dense).  A lane has a block of R rows x G columns of pixels at one hypothesis: the
// R + 1 tap rows of a view serve them all and are interpolated along the row once, and
// neighbouring lanes load neighbouring taps.  The waves of a workgroup have the same
// pixels at consecutive hypotheses, whose taps are in the same lines; they pass their
// costs through LDS, to be written together (2-byte stores 2 N bytes apart took longer
// than the sums where the views are few: 1x11x540x960 u8, N = 96, 257 us with them, 175
// us with 4 hypotheses a store, 144 us with 8).  Bound by its arithmetic, about 8
// instructions per cell and view, and nearly as much by the 16 bytes a lane loads per
// row, which the cache delivers at 64 bytes a cycle; 2 or 4 hypotheses per lane leave
// fewer waves to hide the loads' latency (667, 824 us against 568, 9x9x512^2 f32, N =
// 100), as do more rows (4: 580 us; 2 rows load more, 613 us).  Faster than the slices
// at every size tried (there 1141 us; 5x5x96^2 u8, N = 32: 17 us for 25; 3x3x64^2: 10 for
// 16; colour 5x5x331x449, N = 77, f32 269 us for 424, u8 260 for 656).
constexpr int kFullHyps = 8;
template <typename T, int C>
constexpr int kFullRows = C == 1 ? 3 : sizeof(T) == 1 ? 4 : 2;

// Costs of the pixels u .. u + G-1 of the rows v0 .. v0 + R-1 at hypothesis d.
template <typename T, int C, bool kRoot>
__device__ __forceinline__ void full_item(const L2Args& a, int u, int v0, float d,
                                          uint16_t (&cost)[kFullRows<T, C>][kGroupOf<T, C>]) {
    constexpr int G = kGroupOf<T, C>, R = kFullRows<T, C>;
    constexpr int CP = sizeof(T) == 1 && C == 3 ? 1 : C;
    constexpr int kElem = sizeof(T) == 1 && C == 3 ? 4 : (int)sizeof(T);
    const int S = a.S, T_ = a.T, H = a.H, W = a.W;
    const int sh = (S - 1) / 2, th = (T_ - 1) / 2;
    const int Wp = copy_width(H, W, kElem);
    const uint32_t row = (uint32_t)Wp * kElem, plane = (uint32_t)(H + kPadH) * row;
    const size_t vbytes = (size_t)plane * CP;
    const char* __restrict__ views = (const char*)(const void*)a.views;

    Taps<C, G> ref[R];
    float acc[R][G];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        ref[r] = ld_taps<T, C, G>(views + ((size_t)th * S + sh) * vbytes +
                                      (uint32_t)(min(v0 + r, H - 1) + kPadT) * row +
                                      (uint32_t)(u + kPadL) * kElem, plane);
#pragma unroll
        for (int g = 0; g < G; ++g) acc[r][g] = 0.0f;
    }
    uint32_t lim_lo = ~0u, lim_hi = 0;            // as group()'s lim
    for (int t = 0; t < T_; ++t) {
        // the image rows v0 + y0 + 0..R, clamped: row i is pixel row i's top tap row and
        // pixel row i-1's bottom one (the replicas are equal)
        const float shy = (float)(th - t) * d;
        const float y0 = floorf(shy);
        const float fy = shy - y0;
        uint32_t ro[R + 1];
#pragma unroll
        for (int r = 0; r <= R; ++r)
            ro[r] = (uint32_t)(clampi(v0 + (int)y0 + r, 0, H - 1) + kPadT) * row;
        const char* __restrict__ rt = views + (size_t)t * S * vbytes;
        auto view = [&](int s, auto kFlat, auto kCol) {     // the cases of group()
            const char* __restrict__ vw = rt + (size_t)(uint32_t)s * vbytes;
            constexpr bool flat = decltype(kFlat)::value, col = decltype(kCol)::value;
            const float shx = (float)(sh - s) * d;
            const float x0 = floorf(shx);
            const float fx = shx - x0;
            const uint32_t xo = (uint32_t)(clampi(u + (int)x0, -kPadL, W - 1) + kPadL) * kElem;
            float h[R + 1][C][G];
#pragma unroll
            for (int r = 0; r < (flat ? R : R + 1); ++r) {
                constexpr int n = col ? G : G + 1;
                const Taps<C, n> e = ld_taps<T, C, n>(vw + (ro[r] + xo), plane);
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        if constexpr (col) h[r][c][g] = e.e[c][g];
                        else h[r][c][g] = fmaf(fx, e.e[c][g + 1] - e.e[c][g], e.e[c][g]);
                    }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    float sq = 0.0f, dist = 0.0f;
#pragma unroll
                    for (int c = 0; c < C; ++c) {
                        float val = h[r][c][g];
                        if constexpr (!flat) val = fmaf(fy, h[r + 1][c][g] - val, val);
                        const float dl = ref[r].e[c][g] - val;
                        dist = fabsf(dl);
                        sq = c == 0 ? dl * dl : fmaf(dl, dl, sq);
                    }
                    if constexpr (C == 1) {
                        acc[r][g] += dist;
                    } else if constexpr (!kRoot) {
                        acc[r][g] += sqrtf(sq);
                    } else {
                        acc[r][g] += root(sq);
                        if constexpr (sizeof(T) == 4) {
                            lim_lo = min(lim_lo, __float_as_uint(sq) - 1u);
                            lim_hi = max(lim_hi, __float_as_uint(sq));
                        }
                    }
                }
        };
        constexpr std::true_type yes;
        constexpr std::false_type no;
        if (t == th) {
            for (int s = 0; s < S; ++s)
                if (s != sh) view(s, yes, no);    // the reference view adds +0
        } else {
            for (int s = 0; s < sh; ++s) view(s, no, no);
            view(sh, no, yes);
            for (int s = sh + 1; s < S; ++s) view(s, no, no);
        }
    }
    if constexpr (C == 3 && sizeof(T) == 4 && kRoot) {
        if (lim_lo < __float_as_uint(kRootMin) - 1u || lim_hi > __float_as_uint(kRootMax)) {
            full_item<T, C, false>(a, u, v0, d, cost);
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const float q = rintf(a.alpha * acc[r][g]);
            cost[r][g] = (uint16_t)(q > a.cap ? a.cap : q);
        }
}

template <typename T, int C>
__host__ __device__ __forceinline__ uint32_t full_items(int H, int W) {
    constexpr int G = kGroupOf<T, C>, R = kFullRows<T, C>;
    return (uint32_t)((W + G - 1) / G) * (uint32_t)((H + R - 1) / R);
}

// Workgroup b: 64 items at kFullHyps hypotheses, one per wave; those of the same items
// follow each other.
template <class Src, typename T, int C>
__global__ __launch_bounds__(64 * kFullHyps) void cost_l2_full_kernel(Src src) {
    constexpr int G = kGroupOf<T, C>, R = kFullRows<T, C>;
    __shared__ uint16_t s_cost[R][64 * G][kFullHyps];
    uint32_t b;
    const L2Args& a = member(src, blockIdx.x, b);
    const uint32_t nk = (uint32_t)(a.N + kFullHyps - 1) / kFullHyps;
    const uint32_t set = b / nk, wg = (uint32_t)((a.W + G - 1) / G);
    const uint32_t items = full_items<T, C>(a.H, a.W);
    const int k0 = (int)(b - set * nk) * kFullHyps;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k0 + wave < a.N) {
        const uint32_t item = min(set * 64 + lane, items - 1);
        const int v = (int)(item / wg), u = (int)(item - (uint32_t)v * wg);
        const float d = a.hyp[k0 + wave];
        uint16_t cost[R][G];
        // the root of 8-bit colour norms: as in l2_slices
        if (C == 3 && sizeof(T) == 1 && d != 0.0f && !(fabsf(d) >= 0x1p-24f))
            full_item<T, C, false>(a, u * G, v * R, d, cost);
        else
            full_item<T, C, C == 3>(a, u * G, v * R, d, cost);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int g = 0; g < G; ++g) s_cost[r][lane * G + g][wave] = cost[r][g];
    }
    __syncthreads();
    const int n = min(kFullHyps, a.N - k0);
    for (int j = threadIdx.x; j < R * 64 * G; j += 64 * kFullHyps) {
        const int r = j / (64 * G), q = j - r * (64 * G);
        const uint32_t item = set * 64 + (uint32_t)(q / G);
        const int vi = (int)(item / wg);
        const int v = vi * R + r, u = (int)(item - (uint32_t)vi * wg) * G + q % G;
        if (item >= items || v >= a.H || u >= a.W) continue;
        uint16_t* out = a.cost + ((int64_t)v * a.W + u) * a.N + k0;
        if (n == kFullHyps) {
            __builtin_memcpy(out, s_cost[r][q], 2 * kFullHyps);
        } else {
            for (int i = 0; i < n; ++i) out[i] = s_cost[r][q][i];
        }
    }
}

// ---------------------------------------------------------------------------
// Census kind, Eq. (15), in slices of cells like the l2 cost, a cell per thread and
// round.  The gathers of the views' strings bound it, about 25 cycles of a CU for the 64
// lanes of one.  A workgroup for 64 pixels, whatever their ranges, had stragglers (7x7x384^2,
// N = 64: 261 us; 97 us in slices, 88 us with two views in flight, 93 us with four).
struct CensusAllArgs {
    gptr<const uint64_t> census;   // [S*T][C][H*W]
    gptr<const float> hyp;
    gptr<const int16_t> lo;
    gptr<const int64_t> off;
    gptr<uint16_t> cost;
    gptr<float> cost_f32;
    int64_t cap_cells;
    int S, T, H, W, N;
    uint32_t cap;
    uint32_t nblk;                 // workgroups of this light field
};

constexpr int kCensusChunk = 2 * kThreads;

struct CensusLds {
    int rel[kCensusChunk + 1];     // a pixel's first cell, from the slice's first
    int16_t lo[kCensusChunk];
    int np;
};

template <int C>
__device__ __forceinline__ void census_slice(const CensusAllArgs& a, int64_t b, CensusLds& sl) {
    const int S = a.S, T = a.T, H = a.H, W = a.W, N = a.N;
    const int HW = H * W;
    const int64_t* __restrict__ off = a.off;
    const int64_t total = min(off[HW], a.cap_cells), c0 = b * kCensusChunk;
    if (c0 >= total) return;                                // uniform
    const int len = (int)min((int64_t)kCensusChunk, total - c0);
    const int p0 = first_pixel(off, HW, c0);
    const int npx = min(kCensusChunk, HW - p0);
    const int v0 = p0 / W, u0 = p0 - v0 * W;
    for (int i = threadIdx.x; i <= npx; i += kThreads) {
        sl.rel[i] = (int)(off[p0 + i] - c0);
        if (i < npx) sl.lo[i] = a.lo[p0 + i];
    }
    if (threadIdx.x == 0) sl.np = 0;
    __syncthreads();
    // pixels that start before the slice's end
    for (int i = threadIdx.x; i < npx; i += kThreads)
        if (sl.rel[i] < len && (i + 1 == npx || sl.rel[i + 1] >= len)) atomicMax(&sl.np, i + 1);
    __syncthreads();
    const int np = sl.np, stop = min(sl.rel[npx], len);     // of the staged pixels' cells
    const int sh = (S - 1) / 2, th = (T - 1) / 2;
    const uint64_t* __restrict__ census = a.census;
    const uint64_t* __restrict__ cref = census + ((size_t)th * S + sh) * C * HW;
    for (int c = threadIdx.x; c < len; c += kThreads) {
        int i = 0, k, u = u0, v = v0;
        if (__builtin_expect(c < stop, 1)) {
            int end = np;                                   // largest i with rel[i] <= c
            while (end - i > 1) {
                const int mid = (i + end) >> 1;
                if (sl.rel[mid] <= c) i = mid; else end = mid;
            }
            k = sl.lo[i] + c - sl.rel[i];
        } else {                                            // past the staged pixels, of
            const int p = pixel_of(off, p0 + npx, HW, c0 + c);    // which some own no cell
            i = p - p0;
            k = a.lo[p] + (int)(c0 + c - off[p]);
        }
        if ((unsigned)k >= (unsigned)N) continue;
        u += i;
        if (u >= W) {
            v += u / W;
            u %= W;
        }
        const float d = a.hyp[k];
        uint64_t ref[C];
#pragma unroll
        for (int ch = 0; ch < C; ++ch) ref[ch] = cref[(size_t)ch * HW + (p0 + i)];
        uint32_t acc = 0;
        for (int t = 0; t < T; ++t) {
            const int y = clampi(v + (int)rintf((float)(th - t) * d), 0, H - 1);
            const uint64_t* __restrict__ row = census + (size_t)t * S * C * HW + (size_t)y * W;
#pragma unroll 2
            for (int s = 0; s < S; ++s) {
                const int x = clampi(u + (int)rintf((float)(sh - s) * d), 0, W - 1);
#pragma unroll
                for (int ch = 0; ch < C; ++ch)              // colour: summed per channel
                    acc += (uint32_t)__popcll(ref[ch] ^ row[((size_t)s * C + ch) * HW + x]);
            }
        }
        a.cost[c0 + c] = (uint16_t)min(acc, a.cap);
        if (a.cost_f32) a.cost_f32[c0 + c] = (float)acc;
    }
}

template <class Src, bool Walk, int C>
__global__ __launch_bounds__(kThreads) void cost_census_kernel(Src src) {
    __shared__ CensusLds sl;
    uint32_t b;
    const CensusAllArgs& a = member(src, blockIdx.x, b);
    if constexpr (Walk) {
        const int64_t total = min(a.off[a.H * a.W], a.cap_cells);
        for (int64_t slice = b; slice * kCensusChunk < total; slice += a.nblk) {   // uniform
            census_slice<C>(a, slice, sl);
            __syncthreads();                      // LDS of the slice is read
        }
    } else {
        census_slice<C>(a, b, sl);
    }
}

// The workgroups of a launch over slices, args[i].nblk each; true if they were too many
// and are fewer now, which then walk.
template <class A>
bool limit_blocks(std::vector<A>& args, std::vector<uint32_t>& blocks) {
    int64_t all = 0;
    for (const A& a : args) all += a.nblk;
    const int64_t most = std::max<int64_t>(1, kMostBlocks / (int64_t)args.size());
    for (A& a : args) {
        if (all > kMostBlocks) a.nblk = (uint32_t)std::min<int64_t>(a.nblk, most);
        blocks.push_back(a.nblk);
    }
    return all > kMostBlocks;
}

template <int C>
hipError_t census_walk(Runner& r, std::vector<CensusAllArgs>& args) {
    std::vector<uint32_t> blocks;
    const bool walk = limit_blocks(args, blocks);
    return walk ? launch(r, kStCost, cost_census_kernel<Single<CensusAllArgs>, true, C>,
                         cost_census_kernel<Group<CensusAllArgs>, true, C>, args, blocks, kThreads)
                : launch(r, kStCost, cost_census_kernel<Single<CensusAllArgs>, false, C>,
                         cost_census_kernel<Group<CensusAllArgs>, false, C>, args, blocks,
                         kThreads);
}

template <typename T, bool Walk, int C>
hipError_t l2_variant(Runner& r, const std::vector<L2Args>& args,
                      const std::vector<uint32_t>& blocks) {
    switch (r.tune.cost_cpt) {
        case 2:
            return launch(r, kStCost, cost_l2_kernel<Single<L2Args>, T, 2, Walk, C>,
                          cost_l2_kernel<Group<L2Args>, T, 2, Walk, C>, args, blocks, kThreads);
        case 8:
            return launch(r, kStCost, cost_l2_kernel<Single<L2Args>, T, 8, Walk, C>,
                          cost_l2_kernel<Group<L2Args>, T, 8, Walk, C>, args, blocks, kThreads);
        default:
            return launch(r, kStCost, cost_l2_kernel<Single<L2Args>, T, 4, Walk, C>,
                          cost_l2_kernel<Group<L2Args>, T, 4, Walk, C>, args, blocks, kThreads);
    }
}

template <typename T, int C>
hipError_t l2_walk(Runner& r, std::vector<L2Args>& args) {
    std::vector<uint32_t> blocks;
    const bool walk = limit_blocks(args, blocks);
    return walk || r.tune.cost_stride > 1 ? l2_variant<T, true, C>(r, args, blocks)
                                  : l2_variant<T, false, C>(r, args, blocks);
}

template <typename T, int C>
hipError_t l2_full(Runner& r, const std::vector<L2Args>& args) {
    std::vector<uint32_t> blocks;
    for (const L2Args& a : args) {
        blocks.push_back((full_items<T, C>(a.H, a.W) + 63) / 64 *
                         ((uint32_t)(a.N + kFullHyps - 1) / kFullHyps));
    }
    return launch(r, kStCost, cost_l2_full_kernel<Single<L2Args>, T, C>,
                  cost_l2_full_kernel<Group<L2Args>, T, C>, args, blocks,
                  64 * kFullHyps);
}

// The bounded l2 cost goes by slices, but where every pixel has the full range.
bool takes_slices(const Job* j) {
    return j->prm.cost_kind == LF_COST_L2 && !(j->full_range && !j->cost_f32);
}

}  // namespace

hipError_t stage_cost_inputs(Runner& r, const Jobs& jobs) {
    // l2 cost: the edge-replicated copy of every view plane; Eq. (15) cost: the
    // Census strings of every view
    std::vector<PadArgs> pads[3];                  // u8, f32, u8 colour
    std::vector<uint32_t> pad_blocks[3];
    Jobs census_jobs;
    for (const Job* j : jobs) {
        if (j->prm.cost_kind != LF_COST_L2) {
            census_jobs.push_back(j);
            continue;
        }
        PadArgs pa{};
        pa.src = j->views;
        pa.dst = j->padded;
        pa.H = j->H;
        pa.W = j->W;
        pa.pitch = j->pitch;
        const int k = j->dtype != LF_U8 ? 1 : j->C == 3 ? 2 : 0;
        pads[k].push_back(pa);
        pad_blocks[k].push_back((uint32_t)((j->H + kPadH + kPadRows - 1) / kPadRows) * j->S *
                                j->T * (k == 2 ? 1 : j->C));
    }
    hipError_t e = hipSuccess;
    if (!pads[0].empty() &&
        (e = launch(r, kStCostInputs, pad_views_kernel<Single<PadArgs>, uint8_t, false>,
                    pad_views_kernel<Group<PadArgs>, uint8_t, false>, pads[0], pad_blocks[0],
                    kThreads)) != hipSuccess)
        return e;
    if (!pads[2].empty() &&
        (e = launch(r, kStCostInputs, pad_views_kernel<Single<PadArgs>, uint8_t, true>,
                    pad_views_kernel<Group<PadArgs>, uint8_t, true>, pads[2], pad_blocks[2],
                    kThreads)) != hipSuccess)
        return e;
    if (!pads[1].empty() &&
        (e = launch(r, kStCostInputs, pad_views_kernel<Single<PadArgs>, float, false>,
                    pad_views_kernel<Group<PadArgs>, float, false>, pads[1], pad_blocks[1],
                    kThreads)) != hipSuccess)
        return e;
    if (!census_jobs.empty()) e = stage_census(r, census_jobs, true);
    return e;
}

// Longer slices spread a slice's setup over more cells but leave fewer workgroups: 4 cells
// per thread where an image is large (377 against 500 us, 1x11x1080x1920 u8, N = 96, 199 M
// cells at most), 2 otherwise (325 against 357 us, 9x9x512^2 f32 with N = 100, 26 M; 21
// against 28 us, 5x5x96^2).
int default_cost_cpt(const Jobs& jobs) {
    for (const Job* j : jobs)
        if (takes_slices(j) && (int64_t)j->H * j->W * j->N > (int64_t)1 << 26) return 4;
    return 2;
}

bool uses_cost_slices(const Jobs& jobs) {
    return std::any_of(jobs.begin(), jobs.end(), takes_slices);
}

hipError_t stage_cost(Runner& r, const Jobs& jobs) {
    std::vector<L2Args> l2[2][2];                  // [u8/f32][gray/colour]
    std::vector<L2Args> full[2][2];
    std::vector<CensusAllArgs> ca[2];              // [gray/colour]
    const int cpt = r.tune.cost_cpt == 2 || r.tune.cost_cpt == 8 ? r.tune.cost_cpt : 4;
    const int stride = std::max(1, r.tune.cost_stride);
    for (const Job* j : jobs) {
        const int64_t HW = (int64_t)j->H * j->W;
        if (j->prm.cost_kind == LF_COST_L2) {
            L2Args a{};
            a.views = j->padded;
            a.hyp = j->hyp;
            a.lo = j->lo;
            a.off = j->offsets;
            a.cost = j->cost;
            a.cost_f32 = j->cost_f32;
            a.cap_cells = j->cap_cells;
            a.S = j->S;
            a.T = j->T;
            a.H = j->H;
            a.W = j->W;
            a.N = j->N;
            a.alpha = j->alpha;
            a.cap = (float)j->cap;
            // worst-case slices; those past the device-side cell count are skipped
            const int64_t slices = (HW * j->N + kThreads * cpt - 1) / (kThreads * cpt);
            a.nblk = (uint32_t)std::max<int64_t>(1, (slices + stride - 1) / stride);
            const int t = j->dtype == LF_U8 ? 0 : 1, col = j->C == 3 ? 1 : 0;
            (takes_slices(j) ? l2 : full)[t][col].push_back(a);
        } else {
            CensusAllArgs a{};
            a.census = j->census_all;
            a.hyp = j->hyp;
            a.lo = j->lo;
            a.off = j->offsets;
            a.cost = j->cost;
            a.cost_f32 = j->cost_f32;
            a.cap_cells = j->cap_cells;
            a.S = j->S;
            a.T = j->T;
            a.H = j->H;
            a.W = j->W;
            a.N = j->N;
            a.cap = (uint32_t)j->cap;
            a.nblk = (uint32_t)((HW * j->N + kCensusChunk - 1) / kCensusChunk);
            ca[j->C == 3 ? 1 : 0].push_back(a);
        }
    }
    hipError_t e = hipSuccess;
    if (!l2[0][0].empty() && (e = l2_walk<uint8_t, 1>(r, l2[0][0])) != hipSuccess)
        return e;
    if (!l2[1][0].empty() && (e = l2_walk<float, 1>(r, l2[1][0])) != hipSuccess)
        return e;
    if (!l2[0][1].empty() && (e = l2_walk<uint8_t, 3>(r, l2[0][1])) != hipSuccess)
        return e;
    if (!l2[1][1].empty() && (e = l2_walk<float, 3>(r, l2[1][1])) != hipSuccess)
        return e;
    if (!full[0][0].empty() && (e = l2_full<uint8_t, 1>(r, full[0][0])) != hipSuccess) return e;
    if (!full[1][0].empty() && (e = l2_full<float, 1>(r, full[1][0])) != hipSuccess) return e;
    if (!full[0][1].empty() && (e = l2_full<uint8_t, 3>(r, full[0][1])) != hipSuccess) return e;
    if (!full[1][1].empty() && (e = l2_full<float, 3>(r, full[1][1])) != hipSuccess) return e;
    if (!ca[0].empty() && (e = census_walk<1>(r, ca[0])) != hipSuccess) return e;
    if (!ca[1].empty()) e = census_walk<3>(r, ca[1]);
    return e;
}

}  // namespace lf
