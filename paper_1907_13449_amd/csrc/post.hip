// Per-pixel stages around the two SGM passes (Sec. 3.4-3.6): fusion of the
// intermediate maps, median hole filling, Sobel edge exclusion and the borders
// of Eq. (11), the prefix sum that indexes the bounded volume, WTA with the
// parabola sub-pixel refinement, and the 3x3 median.  All HBM-light: mostly one thread
// per pixel, coalesced along rows.
#include "lf_internal.h"

#include <type_traits>

namespace lf {
namespace {

constexpr int kThreads = 256;

uint32_t blocks_for(int64_t n) { return (uint32_t)((n + kThreads - 1) / kThreads); }

// --- fusion with confidence threshold phi (Sec. 3.4) -----------------------
struct FuseArgs {
    gptr<const int16_t> maps;      // [nv][HW]
    gptr<int16_t> dinit;
    int nv, HW, phi;
};

template <class Src>
__global__ __launch_bounds__(kThreads) void fuse_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const FuseArgs& a = member(src, vb, b);
        const int p = (int)b * kThreads + threadIdx.x;
        if (p >= a.HW) continue;
        int d[4];                                 // |V| <= 4: all loads in flight at once
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = i < a.nv ? a.maps[(size_t)i * a.HW + p] : 0;
        int acc = d[0];
        bool valid = true;
#pragma unroll
        for (int i = 1; i < 4; ++i) {
            if (i >= a.nv) break;
            if (valid && abs(acc - d[i]) < a.phi)
                acc = (acc + d[i]) >> 1;
            else
                valid = false;
        }
        a.dinit[p] = (int16_t)(valid ? acc : -1);
    }
}

// --- one median hole-filling pass: lower median of the valid 8-neighbours ---
struct FillArgs {
    gptr<const int16_t> in;
    gptr<int16_t> out;
    int H, W;
};

__device__ __forceinline__ void fill_pixel(const FillArgs& a, int p) {
    const int H = a.H, W = a.W;
    const int v = p / W, u = p - v * W;
    const int d0 = a.in[p];
    if (d0 >= 0) {
        a.out[p] = (int16_t)d0;
        return;
    }
    // the 8 neighbours in fixed slots, invalid or outside ones as a sentinel above
    // every index; a sorting network (Batcher's odd-even merge, 19 comparators)
    // moves the n valid values to the front in order, and the lower median is
    // the one at (n-1)/2
    constexpr int kNone = 0x7FFF;
    int s[8], n = 0;
#pragma unroll
    for (int i = 0, q = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (i == 1 && j == 1) continue;
            const int y = v + i - 1, x = u + j - 1;
            const int d = y < 0 || y >= H || x < 0 || x >= W ? -1 : a.in[(size_t)y * W + x];
            s[q++] = d >= 0 ? d : kNone;
            n += d >= 0;
        }
    constexpr int kNet[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6},
                                 {5, 7}, {1, 2}, {5, 6}, {0, 4}, {1, 5}, {2, 6}, {3, 7},
                                 {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
    for (int c = 0; c < 19; ++c) {
        const int x = s[kNet[c][0]], y = s[kNet[c][1]];
        s[kNet[c][0]] = min(x, y);
        s[kNet[c][1]] = max(x, y);
    }
    const int want = (n - 1) / 2;
    int res = -1;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (n > 0 && i == want) res = s[i];
    a.out[p] = (int16_t)res;
}

template <class Src>
__global__ __launch_bounds__(kThreads) void fill_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const FillArgs& a = member(src, vb, b);
        const int p = (int)b * kThreads + threadIdx.x;
        if (p < a.H * a.W) fill_pixel(a, p);
    }
}

// --- Sobel edge exclusion and borders, Eq. (11) -----------------------------
struct BordersArgs {
    gptr<const int16_t> dinit;
    gptr<const void> ref;          // C planes of H x pitch
    gptr<int16_t> lo;
    gptr<int16_t> hi;
    int pitch, H, W, N, lambda, lambda_far, C;
    float alpha, tau;
};

// Half-width at initial index d (Sec. 4.6): lambda_far at index 0 (the smallest
// disparity, the farthest point) falling linearly to lambda at N-1, rounded
// half up; lambda_far <= lambda keeps lambda.
__device__ __forceinline__ int border_width(int lambda, int lambda_far, int d, int N) {
    if (lambda_far <= lambda || N < 2) return lambda;
    return lambda + ((lambda_far - lambda) * (N - 1 - d) + (N - 1) / 2) / (N - 1);
}

// d: the filled initial index of pixel p (dinit[p])
template <typename T>
__device__ __forceinline__ void borders_pixel(const BordersArgs& a, int p, int d) {
    const int H = a.H, W = a.W;
    const T* __restrict__ ref = (const T*)a.ref;
    const int v = p / W, u = p - v * W;
    const int ym = max(v - 1, 0), yp = min(v + 1, H - 1);
    const int xm = max(u - 1, 0), xp = min(u + 1, W - 1);
    float g = 0.0f;                               // colour: the strongest channel
    for (int c = 0; c < a.C; ++c) {
        const T* __restrict__ img = ref + (size_t)c * H * a.pitch;
        auto I = [&](int y, int x) { return ld(img + (size_t)y * a.pitch + x); };
        const float gx = ((I(ym, xp) + 2.0f * I(v, xp)) + I(yp, xp)) -
                         ((I(ym, xm) + 2.0f * I(v, xm)) + I(yp, xm));
        const float gy = ((I(yp, xm) + 2.0f * I(yp, u)) + I(yp, xp)) -
                         ((I(ym, xm) + 2.0f * I(ym, u)) + I(ym, xp));
        const float gc = fabsf(gx) + fabsf(gy);
        g = gc > g ? gc : g;
    }
    const bool edge = a.alpha * g > a.tau;
    if (a.lambda < 0 || d < 0 || edge) {          // lambda < 0: boundary-less search
        a.lo[p] = 0;
        a.hi[p] = (int16_t)(a.N - 1);
    } else {
        const int lam = border_width(a.lambda, a.lambda_far, d, a.N);
        a.lo[p] = (int16_t)max(d - lam, 0);
        a.hi[p] = (int16_t)min(d + lam, a.N - 1);
    }
}

template <class Src, typename T>
__global__ __launch_bounds__(kThreads) void borders_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const BordersArgs& a = member(src, vb, b);
        const int p = (int)b * kThreads + threadIdx.x;
        if (p < a.H * a.W) borders_pixel<T>(a, p, a.dinit[p]);
    }
}

// --- fusion, hole filling and borders in one launch -------------------------
// A workgroup owns a 32 x 8 tile of pixels.  It fuses the cross views' maps over
// the tile plus a halo of F = fill_passes pixels into LDS, runs the F Jacobi
// fill passes there (pass f is exact on the tile grown by F - f, since a pass
// reads only the 8 neighbours), and then applies the Sobel test and Eq. (11) to
// its own pixels: the same values as the fuse / fill / borders kernels, with no
// round trips of the intermediate maps and one launch instead of 2 + F.
// Halo positions outside the image read as invalid (-1), which the fill treats
// as it treats a missing neighbour.
constexpr int kPrepTX = 32, kPrepTY = 8, kMaxPrepFill = 3;
constexpr int kPrepMax = (kPrepTX + 2 * kMaxPrepFill) * (kPrepTY + 2 * kMaxPrepFill);

struct PrepArgs {
    FuseArgs fuse;            // fuse.dinit: the filled map (dinit)
    BordersArgs brd;
    int fill;                 // passes, <= kMaxPrepFill
    int tx;                   // tiles along x
};

template <class Src, typename T>
__global__ __launch_bounds__(kThreads) void prep_kernel(Src src) {
    __shared__ int16_t buf[2][kPrepMax];
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const PrepArgs& a = member(src, vb, b);
        const int H = a.brd.H, W = a.brd.W, F = a.fill;
        const int by = (int)b / a.tx, bx = (int)b - by * a.tx;
        const int EW = kPrepTX + 2 * F, EH = kPrepTY + 2 * F;
        const int x0 = bx * kPrepTX - F, y0 = by * kPrepTY - F;
        __syncthreads();                          // LDS of the previous tile is read
        for (int i = threadIdx.x; i < EW * EH; i += kThreads) {
            const int ey = i / EW, ex = i - ey * EW;
            const int y = y0 + ey, x = x0 + ex;
            int out = -1;
            if (y >= 0 && y < H && x >= 0 && x < W) {
                const int p = y * W + x;
                const FuseArgs& f = a.fuse;
                int d[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) d[v] = v < f.nv ? f.maps[(size_t)v * f.HW + p] : 0;
                int acc = d[0];
                bool valid = true;
#pragma unroll
                for (int v = 1; v < 4; ++v) {
                    if (v >= f.nv) break;
                    if (valid && abs(acc - d[v]) < f.phi)
                        acc = (acc + d[v]) >> 1;
                    else
                        valid = false;
                }
                out = valid ? acc : -1;
            }
            buf[0][i] = (int16_t)out;
        }
        __syncthreads();
        int cur = 0;
        for (int pass = 1; pass <= F; ++pass) {
            const int16_t* in = buf[cur];
            int16_t* o = buf[cur ^ 1];
            for (int i = threadIdx.x; i < EW * EH; i += kThreads) {
                const int ey = i / EW, ex = i - ey * EW;
                if (ey < pass || ey >= EH - pass || ex < pass || ex >= EW - pass) continue;
                const int d0 = in[i];
                const int y = y0 + ey, x = x0 + ex;
                if (d0 >= 0 || y < 0 || y >= H || x < 0 || x >= W) {
                    o[i] = (int16_t)d0;               // outside the image: stays absent (-1)
                    continue;
                }
                // lower median of the valid neighbours (as fill_pixel)
                constexpr int kNone = 0x7FFF;
                int sv[8], n = 0;
#pragma unroll
                for (int dy = 0, q = 0; dy < 3; ++dy)
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
                        if (dy == 1 && dx == 1) continue;
                        const int d = in[i + (dy - 1) * EW + dx - 1];
                        sv[q++] = d >= 0 ? d : kNone;
                        n += d >= 0;
                    }
                constexpr int kNet[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6},
                                             {5, 7}, {1, 2}, {5, 6}, {0, 4}, {1, 5}, {2, 6}, {3, 7},
                                             {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
                for (int c = 0; c < 19; ++c) {
                    const int x = sv[kNet[c][0]], y = sv[kNet[c][1]];
                    sv[kNet[c][0]] = min(x, y);
                    sv[kNet[c][1]] = max(x, y);
                }
                const int want = (n - 1) / 2;
                int res = -1;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (n > 0 && k == want) res = sv[k];
                o[i] = (int16_t)res;
            }
            __syncthreads();
            cur ^= 1;
        }
        // this thread's pixel of the tile
        const int lx = threadIdx.x % kPrepTX, ly = threadIdx.x / kPrepTX;
        const int x = bx * kPrepTX + lx, y = by * kPrepTY + ly;
        if (x < W && y < H) {
            const int p = y * W + x;
            const int d = buf[cur][(ly + F) * EW + lx + F];
            a.fuse.dinit[p] = (int16_t)d;
            borders_pixel<T>(a.brd, p, d);
        }
    }
}

// --- boundary-less search (Sec. 4.5): every pixel keeps the full range -------
struct FullArgs {
    gptr<int16_t> lo;
    gptr<int16_t> hi;
    int HW, N;
};

template <class Src>
__global__ __launch_bounds__(kThreads) void full_range_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const FullArgs& a = member(src, vb, b);
        const int p = (int)b * kThreads + threadIdx.x;
        if (p >= a.HW) continue;
        a.lo[p] = 0;
        a.hi[p] = (int16_t)(a.N - 1);
    }
}

// --- exclusive prefix sum of the range widths -> CSR offsets ----------------
// Two launches: per-tile totals, then per tile the sum of the totals before it
// (its base) and the scan of its own widths.
constexpr int kScanPerThread = 8;
constexpr int kScanTile = kThreads * kScanPerThread;

struct ScanArgs {
    gptr<const int16_t> lo;
    gptr<const int16_t> hi;
    gptr<int64_t> bsum;            // [nb]: tile totals
    gptr<int64_t> offsets;         // [HW + 1]
    int64_t HW;
    int nb;
};

__device__ __forceinline__ int64_t block_exclusive_scan(int64_t x, int64_t* sh, int64_t& total) {
    // Hillis-Steele over the 256 per-thread partial sums in LDS
    const int t = threadIdx.x;
    sh[t] = x;
    __syncthreads();
    for (int o = 1; o < kThreads; o <<= 1) {
        const int64_t y = t >= o ? sh[t - o] : 0;
        __syncthreads();
        sh[t] += y;
        __syncthreads();
    }
    total = sh[kThreads - 1];
    const int64_t excl = sh[t] - x;
    __syncthreads();
    return excl;
}

template <class Src>
__global__ __launch_bounds__(kThreads) void scan_reduce_kernel(Src src) {
    __shared__ int64_t sh[kThreads];
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const ScanArgs& a = member(src, vb, b);
        const int64_t base = (int64_t)b * kScanTile;
        int64_t s = 0;
        for (int i = 0; i < kScanPerThread; ++i) {
            const int64_t p = base + (int64_t)i * kThreads + threadIdx.x;
            if (p < a.HW) s += (int64_t)(a.hi[p] - a.lo[p] + 1);
        }
        int64_t total;
        block_exclusive_scan(s, sh, total);
        if (threadIdx.x == 0) a.bsum[b] = total;
    }
}

template <class Src>
__global__ __launch_bounds__(kThreads) void scan_apply_kernel(Src src) {
    __shared__ int64_t sh[kThreads];
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const ScanArgs& a = member(src, vb, b);
        // the tile's base: the sum of the totals of the tiles before it (a tile
        // count of HW / 2048, so each thread adds a few)
        int64_t pre = 0;
        for (int i = threadIdx.x; i < (int)b; i += kThreads) pre += a.bsum[i];
        int64_t tile_base;
        block_exclusive_scan(pre, sh, tile_base);
        // each thread owns kScanPerThread consecutive pixels of the tile
        const int64_t base = (int64_t)b * kScanTile + (int64_t)threadIdx.x * kScanPerThread;
        int w[kScanPerThread];
        int64_t s = 0;
        for (int i = 0; i < kScanPerThread; ++i) {
            const int64_t p = base + i;
            w[i] = p < a.HW ? a.hi[p] - a.lo[p] + 1 : 0;
            s += w[i];
        }
        int64_t total;
        int64_t run = tile_base + block_exclusive_scan(s, sh, total);
        for (int i = 0; i < kScanPerThread; ++i) {
            const int64_t p = base + i;
            if (p < a.HW) a.offsets[p] = run;
            run += w[i];
        }
        if ((int)b == a.nb - 1 && threadIdx.x == 0) a.offsets[a.HW] = tile_base + total;
    }
}

// --- WTA (Eq. 10) and the parabola sub-pixel step (Sec. 3.6) ----------------
struct WtaArgs {
    gptr<const void> csum;
    gptr<const int64_t> off;
    gptr<const int16_t> lo;
    gptr<const int16_t> hi;
    gptr<const float> hyp;
    gptr<int16_t> d_index;
    gptr<float> disp;
    int HW, N;
};

// What bounds the search is the loads of the costs.  A thread per pixel has one load
// instruction per hypothesis, each touching a line or more per lane, and a wave waits for
// its widest pixel (79 us of 37 M 32-bit costs, 1080 x 1920 pixels, an eighth of which
// have 96 hypotheses; 90 us of 512^2 x 100).  So a lane loads a narrow pixel's costs 8 at
// a time, and wide pixels are left to 16 lanes each, which load neighbouring costs.
// Now 38 and 22 us; the bytes take 38 and 21 us at the rate of a large copy.
// Four rounds are still quicker than leaving the pixel to others where the image is too
// small to hide their latency: 175 x 294, N = 30, 4.8 us, with 16 here 6.8 us (10.3 us if
// the 16 lanes also took one pixel at a time).
constexpr int kNarrow = 32;        // hypotheses of the widest narrow pixel

// 8 consecutive costs.
__device__ __forceinline__ void ld8(const uint32_t* c, uint32_t (&x)[8]) {
    __builtin_memcpy(x, c, 16);
    __builtin_memcpy(x + 4, c + 4, 16);
}
__device__ __forceinline__ void ld8(const uint16_t* c, uint32_t (&x)[8]) {
    uint32_t w[4];
    __builtin_memcpy(w, c, 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = w[i] & 0xFFFF;
        x[2 * i + 1] = w[i] >> 16;
    }
}

// Smallest value of 16 lanes, in each of them.
__device__ __forceinline__ uint32_t row_least(uint32_t x) {
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, true));
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xF, 0xF, true));
    x = min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xF, 0xF, true));
    return min(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xF, 0xF, true));
}

// A wave's wide pixels: where their costs start, how many there are and the lane that
// has the pixel; and the winners by that lane.
struct WideLds {
    int64_t off[64];
    int n[64];                     // hypotheses | lane << 16
    int best[64];
};

template <typename SumT>
__device__ __forceinline__ void wta_pixels(const WtaArgs& a, int p, WideLds& wl) {
    const int lane = threadIdx.x & 63;
    const int pc = min(p, a.HW - 1);
    const SumT* __restrict__ csum = (const SumT*)a.csum;
    const int64_t o = a.off[pc];
    // bounds outside the documented 0 <= lo <= hi < N are clamped into it, so no
    // hypothesis outside [0, N) is read (the result is then unspecified)
    const int l = clampi(a.lo[pc], 0, a.N - 1), h = clampi(a.hi[pc], l, a.N - 1);
    const int n = h - l + 1;
    const SumT* __restrict__ c = csum + o;                  // c[i] is hypothesis l + i
    // in increasing order, strict <, so the lowest index wins ties
    int best = 0;
    uint32_t bv = 0;
    const bool wide = p < a.HW && n > kNarrow;
    if (!wide) {
        const int64_t left = a.off[a.HW] - o;               // costs from here to the end
        for (int i0 = 0; i0 < n; i0 += 8) {
            uint32_t x[8];
            if (__builtin_expect(i0 + 8 <= left, 1)) {
                ld8(c + i0, x);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = c[min(i0 + i, n - 1)];
            }
            if (i0 == 0) bv = x[0];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i0 + i < n && x[i] < bv) {
                    bv = x[i];
                    best = i0 + i;
                }
        }
    }
    const uint64_t wides = __builtin_amdgcn_ballot_w64(wide);
    if (wides != 0) {                                       // uniform
        if (wide) {
            const int at = __popcll(wides & ((1ull << lane) - 1));
            wl.off[at] = o;
            wl.n[at] = n | lane << 16;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int count = __popcll(wides), sub = lane & 15;
        // Q pixels at a time per 16 lanes, 8 loads in flight for them together
        auto search = [&](int r, auto kQ) {
            constexpr int Q = decltype(kQ)::value, L = 8 / Q;
            const SumT* __restrict__ w[Q];
            int m[Q], owner[Q], at[Q], longest = 0;
            uint32_t least[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                // past the last one: that again
                const int i = min(r + 4 * q + (lane >> 4), count - 1);
                w[q] = csum + wl.off[i];
                m[q] = wl.n[i] & 0xFFFF;
                owner[q] = wl.n[i] >> 16;
                longest = max(longest, m[q]);
                least[q] = ~0u;
                at[q] = INT_MAX;                  // any real one is before it
            }
            for (int k0 = sub; k0 < longest; k0 += 16 * L) {
                uint32_t x[Q][L];
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int j = 0; j < L; ++j) x[q][j] = w[q][min(k0 + 16 * j, m[q] - 1)];
#pragma unroll
                for (int q = 0; q < Q; ++q)
#pragma unroll
                    for (int j = 0; j < L; ++j) {
                        const int k = k0 + 16 * j;
                        if (k < m[q] && (x[q][j] < least[q] || at[q] == INT_MAX)) {
                            least[q] = x[q][j];
                            at[q] = k;
                        }
                    }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const uint32_t all = row_least(least[q]);
                const uint32_t first = row_least(least[q] == all ? (uint32_t)at[q] : ~0u);
                if (sub == 0) wl.best[owner[q]] = (int)first;
            }
        };
        for (int r = 0; r < count;) {                       // uniform
            const int left = count - r;
            if (left > 8) search(r, std::integral_constant<int, 4>()), r += 16;
            else if (left > 4) search(r, std::integral_constant<int, 2>()), r += 8;
            else search(r, std::integral_constant<int, 1>()), r += 4;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (wide) {
            best = wl.best[lane];
            bv = c[best];
        }
    }
    if (p >= a.HW) return;
    a.d_index[p] = (int16_t)(l + best);
    const float* __restrict__ hyp = (const float*)a.hyp + l;
    float d = hyp[best];
    if (best >= 1 && best + 1 < n && n >= 5) {
        const int64_t cm = c[best - 1], c0 = bv, cp = c[best + 1];
        const float o = (float)(cm - cp) / (2.0f * (float)(cm + cp - 2 * c0));
        d = o >= 0.0f ? fmaf(o, hyp[best + 1] - hyp[best], hyp[best])
                      : fmaf(o, hyp[best] - hyp[best - 1], hyp[best]);
    }
    a.disp[p] = d;
}

template <class Src, typename SumT>
__global__ __launch_bounds__(kThreads) void wta_subpixel_kernel(Src src) {
    __shared__ WideLds wl[kThreads / 64];
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const WtaArgs& a = member(src, vb, b);
        wta_pixels<SumT>(a, (int)b * kThreads + threadIdx.x, wl[threadIdx.x >> 6]);
    }
}

// --- 3x3 median, clamp-to-edge ----------------------------------------------
struct MedianArgs {
    gptr<const float> in;
    gptr<float> out;
    int H, W;
};

// A thread takes kMedianRows pixels of a column, whose windows share rows: a row's three
// values are ordered once, and the median of nine is the median of the largest of the
// rows' least, the median of their medians and the least of their largest.  Bound by
// its loads, 18 for four pixels (1080 x 1920: 6 us; by ranks, a pixel per thread, 46 us).
constexpr int kMedianRows = 4;

// Order-preserving integers of the floats other than NaN (-0 before +0), and back.
__device__ __forceinline__ int ordered(float x) {
    const int i = __float_as_int(x);
    return i ^ (i >> 31 & 0x7FFFFFFF);
}
__device__ __forceinline__ float unordered(int i) {
    return __int_as_float(i ^ (i >> 31 & 0x7FFFFFFF));
}
__device__ __forceinline__ int mid3(int x, int y, int z) {
    return max(min(x, y), min(max(x, y), z));
}

// The median of a window with NaN: by ranks, a NaN having none (the centre if no value
// has at most 4 values below it and at least 5 at or below).
__device__ __forceinline__ float median_by_rank(const MedianArgs& a, int v, int u) {
    float w[9];
#pragma unroll
    for (int i = 0; i < 9; ++i)
        w[i] = a.in[(size_t)clampi(v + i / 3 - 1, 0, a.H - 1) * a.W +
                    clampi(u + i % 3 - 1, 0, a.W - 1)];
    float med = w[4];
#pragma unroll
    for (int x = 0; x < 9; ++x) {
        int below = 0, atmost = 0;
#pragma unroll
        for (int y = 0; y < 9; ++y) {
            below += w[y] < w[x];
            atmost += w[y] <= w[x];
        }
        if (below <= 4 && 4 < atmost) med = w[x];
    }
    return med;
}

__device__ __forceinline__ void median_pixels(const MedianArgs& a, int i) {
    const int H = a.H, W = a.W;
    const int q = i / W, u = i - q * W, v0 = q * kMedianRows;
    if (v0 >= H) return;
    const float* __restrict__ in = a.in;
    const int um = max(u - 1, 0), up = min(u + 1, W - 1);
    float x[kMedianRows + 2][3];
#pragma unroll
    for (int r = 0; r < kMedianRows + 2; ++r) {
        const float* __restrict__ row = in + (size_t)clampi(v0 + r - 1, 0, H - 1) * W;
        x[r][0] = row[um];
        x[r][1] = row[u];
        x[r][2] = row[up];
    }
    float any = 0.0f;                             // NaN if one of the values is
    int lo[kMedianRows + 2], mid[kMedianRows + 2], hi[kMedianRows + 2];
#pragma unroll
    for (int r = 0; r < kMedianRows + 2; ++r) {
        any += x[r][0] + x[r][1] + x[r][2];
        const int p = ordered(x[r][0]), c = ordered(x[r][1]), n = ordered(x[r][2]);
        lo[r] = min(min(p, c), n);
        mid[r] = mid3(p, c, n);
        hi[r] = max(max(p, c), n);
    }
    float* __restrict__ out = a.out + (size_t)v0 * W + u;
    if (__builtin_expect(any != any, 0)) {
#pragma unroll 1
        for (int r = 0; r < min(kMedianRows, H - v0); ++r)
            out[(size_t)r * W] = median_by_rank(a, v0 + r, u);
        return;
    }
#pragma unroll
    for (int r = 0; r < kMedianRows; ++r)
        if (v0 + r < H)
            out[(size_t)r * W] = unordered(mid3(max(max(lo[r], lo[r + 1]), lo[r + 2]),
                                                mid3(mid[r], mid[r + 1], mid[r + 2]),
                                                min(min(hi[r], hi[r + 1]), hi[r + 2])));
}

template <class Src>
__global__ __launch_bounds__(kThreads) void median3_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const MedianArgs& a = member(src, vb, b);
        median_pixels(a, (int)b * kThreads + threadIdx.x);
    }
}

}  // namespace

size_t scan_scratch_bytes(int64_t HW) {
    const int64_t nb = (HW + kScanTile - 1) / kScanTile;
    return (size_t)(nb + 1) * sizeof(int64_t);
}

hipError_t stage_borders(Runner& r, const Jobs& jobs) {
    // light fields with at most kMaxPrepFill fill passes: one tile kernel; others:
    // fusion, the fill passes and the borders as separate launches
    std::vector<PrepArgs> prep[2];
    std::vector<uint32_t> prep_blocks[2];
    std::vector<FuseArgs> fuse;
    std::vector<uint32_t> fuse_blocks;
    std::vector<BordersArgs> brd[2];
    std::vector<uint32_t> brd_blocks[2];
    Jobs sep;
    int max_passes = 0;
    for (const Job* j : jobs) {
        const int HW = j->H * j->W;
        const int t = j->dtype == LF_U8 ? 0 : 1;
        const int sh = (j->S - 1) / 2, th = (j->T - 1) / 2;
        const size_t elem = j->dtype == LF_U8 ? 1 : 4;
        BordersArgs b{};
        b.dinit = j->dinit;
        b.ref = (const char*)j->views + ((size_t)th * j->S + sh) * j->C * j->H * j->pitch * elem;
        b.lo = j->lo;
        b.hi = j->hi;
        b.pitch = j->pitch;
        b.H = j->H;
        b.W = j->W;
        b.N = j->N;
        b.lambda = j->prm.lambda;
        b.lambda_far = j->prm.lambda_far;
        b.C = j->C;
        b.alpha = j->alpha;
        b.tau = j->prm.edge_tau;
        if (j->prm.fill_passes <= kMaxPrepFill) {
            PrepArgs pa{};
            pa.fuse = FuseArgs{j->maps, j->dinit, j->nv, HW, j->prm.phi};
            pa.brd = b;
            pa.fill = j->prm.fill_passes;
            pa.tx = (j->W + kPrepTX - 1) / kPrepTX;
            prep[t].push_back(pa);
            prep_blocks[t].push_back((uint32_t)pa.tx * ((j->H + kPrepTY - 1) / kPrepTY));
            continue;
        }
        sep.push_back(j);
        int16_t* buf[2] = {j->dinit, j->fill_tmp};
        // the passes ping-pong between the two buffers and end in dinit
        fuse.push_back(FuseArgs{j->maps, buf[j->prm.fill_passes % 2], j->nv, HW, j->prm.phi});
        fuse_blocks.push_back(blocks_for(HW));
        max_passes = std::max(max_passes, j->prm.fill_passes);
        brd[t].push_back(b);
        brd_blocks[t].push_back(blocks_for(HW));
    }
    hipError_t e = hipSuccess;
    if (!prep[0].empty() &&
        (e = launch(r, kStBorders, prep_kernel<Single<PrepArgs>, uint8_t>,
                    prep_kernel<Group<PrepArgs>, uint8_t>, prep[0], prep_blocks[0],
                    kThreads)) != hipSuccess)
        return e;
    if (!prep[1].empty() &&
        (e = launch(r, kStBorders, prep_kernel<Single<PrepArgs>, float>,
                    prep_kernel<Group<PrepArgs>, float>, prep[1], prep_blocks[1],
                    kThreads)) != hipSuccess)
        return e;
    if (sep.empty()) return hipSuccess;
    e = launch(r, kStBorders, fuse_kernel<Single<FuseArgs>>, fuse_kernel<Group<FuseArgs>>, fuse,
               fuse_blocks, kThreads);
    if (e != hipSuccess) return e;
    for (int f = 0; f < max_passes; ++f) {
        std::vector<FillArgs> fill;
        std::vector<uint32_t> fill_blocks;
        for (const Job* j : sep) {
            if (f >= j->prm.fill_passes) continue;
            int16_t* buf[2] = {j->dinit, j->fill_tmp};
            const int cur = (j->prm.fill_passes + f) % 2;
            fill.push_back(FillArgs{buf[cur], buf[cur ^ 1], j->H, j->W});
            fill_blocks.push_back(blocks_for((int64_t)j->H * j->W));
        }
        e = launch(r, kStBorders, fill_kernel<Single<FillArgs>>, fill_kernel<Group<FillArgs>>,
                   fill, fill_blocks, kThreads);
        if (e != hipSuccess) return e;
    }
    if (!brd[0].empty()) {
        e = launch(r, kStBorders, borders_kernel<Single<BordersArgs>, uint8_t>,
                   borders_kernel<Group<BordersArgs>, uint8_t>, brd[0], brd_blocks[0], kThreads);
        if (e != hipSuccess) return e;
    }
    if (!brd[1].empty())
        e = launch(r, kStBorders, borders_kernel<Single<BordersArgs>, float>,
                   borders_kernel<Group<BordersArgs>, float>, brd[1], brd_blocks[1], kThreads);
    return e;
}

hipError_t stage_full_range(Runner& r, const Jobs& jobs) {
    std::vector<FullArgs> args;
    std::vector<uint32_t> blocks;
    for (const Job* j : jobs) {
        args.push_back(FullArgs{j->lo, j->hi, j->H * j->W, j->N});
        blocks.push_back(blocks_for((int64_t)j->H * j->W));
    }
    return launch(r, kStBorders, full_range_kernel<Single<FullArgs>>,
                  full_range_kernel<Group<FullArgs>>, args, blocks, kThreads);
}

hipError_t stage_offsets(Runner& r, const Jobs& jobs) {
    std::vector<ScanArgs> args;
    std::vector<uint32_t> tiles;
    for (const Job* j : jobs) {
        const int64_t HW = (int64_t)j->H * j->W;
        ScanArgs a{};
        a.lo = j->lo;
        a.hi = j->hi;
        a.bsum = (int64_t*)j->scan;
        a.offsets = j->offsets;
        a.HW = HW;
        a.nb = (int)((HW + kScanTile - 1) / kScanTile);
        args.push_back(a);
        tiles.push_back((uint32_t)a.nb);
    }
    hipError_t e = launch(r, kStOffsets, scan_reduce_kernel<Single<ScanArgs>>,
                          scan_reduce_kernel<Group<ScanArgs>>, args, tiles, kThreads);
    if (e != hipSuccess) return e;
    return launch(r, kStOffsets, scan_apply_kernel<Single<ScanArgs>>,
                  scan_apply_kernel<Group<ScanArgs>>, args, tiles, kThreads);
}

hipError_t stage_wta(Runner& r, const Jobs& jobs) {
    std::vector<WtaArgs> wta[2];
    std::vector<uint32_t> wta_blocks[2];
    std::vector<MedianArgs> med;
    std::vector<uint32_t> med_blocks;
    for (const Job* j : jobs) {
        const int HW = j->H * j->W;
        const bool median = j->prm.median == 3;
        WtaArgs a{};
        a.csum = j->csum;
        a.off = j->offsets;
        a.lo = j->lo;
        a.hi = j->hi;
        a.hyp = j->hyp;
        a.d_index = j->d_index;
        a.disp = median ? j->pre_median : j->disparity;
        a.HW = HW;
        a.N = j->N;
        const int sb = j->prm.sum_bits == 16 ? 0 : 1;
        wta[sb].push_back(a);
        wta_blocks[sb].push_back(blocks_for(HW));
        if (median) {
            med.push_back(MedianArgs{j->pre_median, j->disparity, j->H, j->W});
            med_blocks.push_back(
                blocks_for((int64_t)((j->H + kMedianRows - 1) / kMedianRows) * j->W));
        }
    }
    hipError_t e = hipSuccess;
    if (!wta[0].empty()) {
        e = launch(r, kStWta, wta_subpixel_kernel<Single<WtaArgs>, uint16_t>,
                   wta_subpixel_kernel<Group<WtaArgs>, uint16_t>, wta[0], wta_blocks[0], kThreads);
        if (e != hipSuccess) return e;
    }
    if (!wta[1].empty()) {
        e = launch(r, kStWta, wta_subpixel_kernel<Single<WtaArgs>, uint32_t>,
                   wta_subpixel_kernel<Group<WtaArgs>, uint32_t>, wta[1], wta_blocks[1], kThreads);
        if (e != hipSuccess) return e;
    }
    if (!med.empty())
        e = launch(r, kStWta, median3_kernel<Single<MedianArgs>>, median3_kernel<Group<MedianArgs>>,
                   med, med_blocks, kThreads);
    return e;
}

}  // namespace lf
