// Semi-global matching, Eq. (8)-(10), on gfx950.
//
// Schedule.  All path directions of all views run in ONE launch: a wavefront
// owns one path line (or four, see the kernels with 16 lanes per line) of one
// direction of one view, and writes that direction's
// path costs L_r to a buffer of its own (no read-modify-write, no atomics); a
// second kernel sums the directions, Eq. (9), and for the initial stage takes
// the WTA of Eq. (10) in the same pass.  With 8 directions x |V| views the launch
// has enough independent waves to keep every SIMD busy while each wave walks its
// line step by step.
//
// Inside a wave, lane l holds hypotheses k = K*l .. K*l+K-1 (K = ceil(N/64)), so
// the state of one pixel lives in the registers of one wave.  Per step:
//   - the matching cost of the K hypotheses, read from a cost volume whose row of
//     the pixel is contiguous (initial stage: the 8-bit Census cost volume, built
//     once by a popcount kernel; final stage: the CSR volume), with the loads of
//     the next D steps in flight (D is a tuning parameter);
//   - the neighbours k-1 / k+1 of the previous pixel come from the lane's own
//     registers or, at the lane boundary, from lane l-1 / l+1 by a DPP wave
//     shift (wave_shr:1 / wave_shl:1);
//   - m = min_k L_r(p-r, k) is a DPP reduction (quad perms, half/row mirror, row
//     broadcasts) and a readlane, so it is wave-uniform in an SGPR.
// The initial stage stages each step's path-cost row in LDS and copies D rows
// at a time out with 16-byte stores.
// Path costs use the normalised recurrence (subtract m), which keeps them in
// [0, C + P2]: 8 bits suffice for the Census stage when bits + P2 <= 255.
// Hypotheses outside a pixel's range hold +inf (kInf) so they never win a min.
#include "lf_internal.h"

#include <algorithm>
#include <climits>
#include <type_traits>
#include <utility>

namespace lf {
namespace {

template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROW_MASK, 0xF, false);
}

// Minimum over the 64 lanes, returned wave-uniform.
// The DPP source operand "old" is UINT_MAX, the identity of umin, so that each
// move fuses into the v_min_u32 that consumes it (one v_min_u32_dpp per stage).
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
    v = min(v, dpp<0xB1>(UINT_MAX, v));        // quad_perm [1,0,3,2]
    v = min(v, dpp<0x4E>(UINT_MAX, v));        // quad_perm [2,3,0,1]
    v = min(v, dpp<0x141>(UINT_MAX, v));       // row_half_mirror
    v = min(v, dpp<0x140>(UINT_MAX, v));       // row_mirror: every lane holds its row's min
    v = min(v, dpp<0x142, 0xA>(UINT_MAX, v));  // row_bcast:15 into rows 1, 3
    v = min(v, dpp<0x143, 0xC>(UINT_MAX, v));  // row_bcast:31 into rows 2, 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Path directions (du, dv): the 8 axis and diagonal neighbours, then the 8
// knight moves of the 16-path setting (Sec. 4.3).
constexpr int kDirs[16][2] = {{1, 0},  {-1, 0},  {0, 1},  {0, -1}, {1, 1},  {-1, -1},
                              {1, -1}, {-1, 1},  {1, 2},  {-1, -2}, {2, 1},  {-2, -1},
                              {2, -1}, {-2, 1},  {1, -2}, {-1, 2}};

// kDirs[r][c] + 2 of every direction, four bits each: a wave-uniform r reads its
// direction by a scalar shift.
constexpr uint64_t packed_dirs(int c) {
    uint64_t x = 0;
    for (int r = 0; r < 16; ++r) x |= (uint64_t)(kDirs[r][c] + 2) << (4 * r);
    return x;
}
__host__ __device__ inline int dir_u(int r) {
    constexpr uint64_t x = packed_dirs(0);
    return (int)(x >> (4 * r) & 15) - 2;
}
__host__ __device__ inline int dir_v(int r) {
    constexpr uint64_t x = packed_dirs(1);
    return (int)(x >> (4 * r) & 15) - 2;
}

// f(integral_constant 0), ..., f(integral_constant n - 1)
template <int n, class F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int n, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_<n>(f, std::make_integer_sequence<int, n>());
}
constexpr int kMaxPaths = 16;

// A path starts at every pixel whose predecessor p - r lies outside the image:
// the |dv| rows and |du| columns on the entry sides.
__host__ __device__ inline int num_lines(int H, int W, int du, int dv) {
    const int su = min(abs(du), W), sv = min(abs(dv), H);
    return sv * W + su * (H - sv);
}

// Lines of every direction, numbered consecutively: direction r owns global
// lines [base[r], base[r+1]); nlines = base[npaths].
struct Lines {
    int base[kMaxPaths + 1];
    int8_t du[kMaxPaths], dv[kMaxPaths];
    int npaths, nlines;
};

Lines make_lines(int H, int W, int npaths) {
    Lines L{};
    L.npaths = npaths;
    L.base[0] = 0;
    for (int r = 0; r < npaths; ++r) {
        L.du[r] = (int8_t)kDirs[r][0];
        L.dv[r] = (int8_t)kDirs[r][1];
        L.base[r + 1] = L.base[r] + num_lines(H, W, L.du[r], L.dv[r]);
    }
    L.nlines = L.base[npaths];
    return L;
}

struct LineInfo {
    int r, u0, v0, du, dv, len;
};

// Start pixel and length of global line g (wave-uniform; scalar arithmetic).
// Lines of a direction are the entry rows first (row-major), then the entry
// columns below / above them.
__device__ __forceinline__ LineInfo locate(const Lines& L, int H, int W, int g) {
    LineInfo li;
    // the direction of line g and its fields, read with constant indices only (the
    // argument record stays in registers)
    int r = 0, lbase = 0, du = L.du[0], dv = L.dv[0];
#pragma unroll
    for (int i = 1; i < kMaxPaths; ++i)
        if (i < L.npaths && g >= L.base[i]) {
            r = i;
            lbase = L.base[i];
            du = L.du[i];
            dv = L.dv[i];
        }
    const int line = g - lbase;
    const int su = min(abs(du), W), sv = min(abs(dv), H);
    li.r = r;
    li.du = du;
    li.dv = dv;
    if (line < sv * W) {                 // an entry row
        const int j = line / W;
        li.u0 = line - j * W;
        li.v0 = dv >= 0 ? j : H - 1 - j;
    } else {                             // an entry column, below/above the entry rows
        const int l2 = line - sv * W;
        const int i = l2 / su, j = l2 - i * su;
        li.u0 = du >= 0 ? j : W - 1 - j;
        li.v0 = dv >= 0 ? sv + i : H - 1 - sv - i;
    }
    const int lu = du > 0 ? (W - 1 - li.u0) / du + 1 : du < 0 ? li.u0 / -du + 1 : INT_MAX;
    const int lv = dv > 0 ? (H - 1 - li.v0) / dv + 1 : dv < 0 ? li.v0 / -dv + 1 : INT_MAX;
    li.len = min(lu, lv);
    return li;
}

// Work units of the path kernels with one line per wave.  Besides |W - H| + 1
// lines of length M = min(H, W), a diagonal direction (|du| = |dv| = 1) has one
// line of each length 1 .. M - 1 among its entry-row lines and one among its
// entry-column lines.  Its units are the full lines alone and the pairs of
// lengths m and M - m, run one after the other: every unit is M steps long, so
// all the waves of the launch have the same work and none is left running
// alone at the end.  Any other direction has one unit per line.
__host__ __device__ inline bool paired_dir(int du, int dv) {
    return (du == 1 || du == -1) && (dv == 1 || dv == -1);
}

__host__ __device__ inline int num_units(int H, int W, int du, int dv) {
    return paired_dir(du, dv) ? max(H, W) : num_lines(H, W, du, dv);
}

struct Units {
    int base[kMaxPaths + 1];       // direction r owns units [base[r], base[r+1])
    int nunits;
};

Units make_units(const Lines& L, int H, int W) {
    Units U{};
    for (int r = 0; r < L.npaths; ++r)
        U.base[r + 1] = U.base[r] + num_units(H, W, L.du[r], L.dv[r]);
    U.nunits = U.base[L.npaths];
    return U;
}

// The global lines of unit u (wave-uniform): line[0], and line[1] or -1.  In a
// diagonal direction, entry-row line j is min(W - j', H) long, j' = j for du > 0
// and W - 1 - j for du < 0, and entry-column line i (index W + i within the
// direction) min(W, H - 1 - i).
__device__ __forceinline__ void unit_lines(const Lines& L, const Units& U, int H, int W, int u,
                                           int (&line)[2]) {
    int r = 0, ub = 0, lb = 0, du = L.du[0], dv = L.dv[0];
#pragma unroll
    for (int i = 1; i < kMaxPaths; ++i)    // constant indices: the record stays in registers
        if (i < L.npaths && u >= U.base[i]) {
            r = i;
            ub = U.base[i];
            lb = L.base[i];
            du = L.du[i];
            dv = L.dv[i];
        }
    const int x = u - ub;
    int first = x, second = -1;
    if (paired_dir(du, dv)) {
        if (x < W && du < 0) first = W - 1 - x;        // the row line of length min(W - x, H)
        if (W >= H) {
            if (x > W - H) second = 2 * W - 1 - x;      // lengths W - x and H - (W - x)
        } else if (x >= 1 && x < W) {
            second = W + H - 1 - x;                    // lengths W - x and x
        }                                              // x >= W: a full column line
    }
    line[0] = lb + first;
    line[1] = second < 0 ? -1 : lb + second;
}

constexpr int kWavesPerBlock = 4;

size_t round256(size_t x) { return (x + 255) / 256 * 256; }

uint32_t div_up(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

// Copies a wave-uniform value into a VGPR that the compiler treats as divergent.
// Loads addressed through it stay vector-memory loads, which complete in order,
// so a wave can keep several steps of them in flight and wait for the oldest
// only (scalar loads can only be awaited all at once).
__device__ __forceinline__ uint32_t in_vgpr(uint32_t x) {
    asm volatile("" : "=v"(x) : "0"(x));
    return x;
}

// One step of the normalised recurrence for K consecutive hypotheses.  Lanes
// whose hypotheses do not exist carry costs >= kInf and so path costs >= kInf,
// which never win a min; the neighbour shift brings UINT_MAX (the identity of
// umin) in at the wave edges.
template <int K>
__device__ __forceinline__ void sgm_step(const uint32_t (&Lp)[K], uint32_t m, uint32_t P1,
                                         uint32_t P2, const uint32_t (&C)[K], uint32_t (&L)[K]) {
    // X = Lp + P1 first: each DPP neighbour move then fuses into the min that
    // consumes it, and (for K = 2) none of the sources needs a copy
    uint32_t X[K];
#pragma unroll
    for (int j = 0; j < K; ++j) X[j] = Lp[j] + P1;
    const uint32_t left = dpp<0x138>(UINT_MAX, X[K - 1]);    // wave_shr:1 -> from lane l-1
    const uint32_t right = dpp<0x130>(UINT_MAX, X[0]);       // wave_shl:1 -> from lane l+1
    const uint32_t mP2 = m + P2;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const uint32_t lm = j == 0 ? left : X[j - 1];
        const uint32_t lp = j == K - 1 ? right : X[j + 1];
        const uint32_t t = min(min(Lp[j], mP2), min(lm, lp));
        L[j] = t + (C[j] - m);               // the cost byte less m: one SDWA subtract
    }
}

template <int K>
__device__ __forceinline__ uint32_t lane_min(const uint32_t (&L)[K]) {
    uint32_t mn = L[0];
#pragma unroll
    for (int j = 1; j < K; ++j) mn = min(mn, L[j]);
    return mn;
}

// ---------------------------------------------------------------------------
// Initial stage, Eq. (7): the Census cost volume C[z][p][NPc] (8-bit; NPc = N + 2
// rounded up to 4, at most 256) of every cross view, computed once and read by
// all path directions.  Bytes k >= N of a row hold 255.  A workgroup builds the tile of 64 consecutive pixels x NP
// hypotheses in LDS with lanes over pixels -- for a fixed hypothesis the 64
// gathered Census strings are consecutive in memory for both shift axes -- and
// then writes the tile, which is contiguous in C, with 32-bit stores.
constexpr int kTilePix = 64;

struct CcvArgs {
    gptr<const uint64_t> cref;     // [C][H*W]
    gptr<const uint64_t> cview;    // [nv][C][H*W]
    gptr<const float> hyp;
    uint64_t cs4, ct4;        // s_hat - s, t_hat - t of cross view z in bits 16z..16z+15
                              // (int16; packed so that the record is never indexed)
    int nv, H, W, N, NP;      // NP: the row stride NPc
    uint32_t tiles;           // pixel tiles per view
    gptr<uint8_t> cvol;            // [nv][H*W][NPc]
};

template <int C>
__device__ __forceinline__ void ccv_block(const CcvArgs& a, uint32_t b, uint32_t* tile,
                                          int* s_sh) {
    const int z = (int)(b / a.tiles);
    const uint32_t t = b - (uint32_t)z * a.tiles;
    const int H = a.H, W = a.W, N = a.N, NP = a.NP;
    const uint32_t HW = (uint32_t)H * W;
    const uint32_t p0 = t * kTilePix;
    const int npix = (int)min((uint32_t)kTilePix, HW - p0);
    const int csz = (int16_t)(a.cs4 >> (16 * z)), ctz = (int16_t)(a.ct4 >> (16 * z));
    const bool along_u = ctz == 0;
    const int cs = along_u ? csz : ctz;
    for (int k = threadIdx.x; k < NP; k += 256)
        s_sh[k] = (int)rintf((float)cs * a.hyp[min(k, N - 1)]);
    __syncthreads();

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t p = p0 + (uint32_t)min(lane, npix - 1);
    const int v = (int)(p / W), u = (int)(p - (uint32_t)v * W);
    // colour: one Census string per channel, Hamming distances summed (<= 3*64)
    uint64_t r[C];
#pragma unroll
    for (int c = 0; c < C; ++c) r[c] = a.cref[(size_t)c * HW + p];
    const uint64_t* __restrict__ cv = a.cview + (size_t)z * C * HW;
    // The rounded shift is monotone in k, so consecutive hypotheses mostly share
    // it (at |s_hat - s| * (d_k+1 - d_k) < 1 a shift spans several k): wave w
    // walks its quarter of the row's 4-hypothesis words in order, gathers and
    // counts a Census string only when the shift changes, and writes each word
    // of four costs (255 past N) with one LDS store.
    const int NW = NP / 4;
    const int wb = NW * wave / 4, we = NW * (wave + 1) / 4;
    // Where most hypotheses have a shift of their own, the strings of kWords words are
    // gathered before the first is counted, without looking for equal shifts: one at a
    // time their latency was most of the kernel (2 views of 1080x1920, N = 96, 1.3 pixels
    // per hypothesis: 353 us, now 273; gathering only the changed ones ahead 257, but
    // then 0.3 pixels per hypothesis, 4 views of 512x512, N = 100, take 56 us for 54).
    // With fewer pixels per hypothesis the walk gathers less; 4 views of 512x512, N = 100,
    // at 0.5, 0.65, 0.8, 1 and 1.2: 62, 70, 79, 89, 89 us against 71, in colour 98, 124,
    // 151, 180, 177 against 152.
    auto gather = [&](int sh, int c) {
        const uint32_t qq = along_u ? (uint32_t)(v * W + clampi(u + sh, 0, W - 1))
                                    : (uint32_t)(clampi(v + sh, 0, H - 1) * W + u);
        return cv[(size_t)c * HW + qq];
    };
    const int span = __builtin_amdgcn_readfirstlane(s_sh[N - 1] - s_sh[0]);
    if (20 * llabs(span) > (C == 1 ? 13 : 16) * N) {
        constexpr int kWords = C == 1 ? 2 : 1;
        for (int w4 = wb; w4 < we; w4 += kWords) {
            uint64_t x[4 * kWords][C];
#pragma unroll
            for (int j = 0; j < kWords; ++j) {
                const int4 sh4 = *(const int4*)(s_sh + 4 * min(w4 + j, we - 1));
                const int shq[4] = {sh4.x, sh4.y, sh4.z, sh4.w};
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int c = 0; c < C; ++c) x[4 * j + q][c] = gather(shq[q], c);
            }
#pragma unroll
            for (int j = 0; j < kWords; ++j) {
                uint32_t word = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t hd = 0;
#pragma unroll
                    for (int c = 0; c < C; ++c) hd += (uint32_t)__popcll(r[c] ^ x[4 * j + q][c]);
                    word |= (4 * (w4 + j) + q < N ? hd : 255u) << (8 * q);
                }
                if (w4 + j < we) tile[lane * NW + w4 + j] = word;
            }
        }
    } else {
        int prev = INT_MIN;
        uint32_t hd = 0;
        for (int w4 = wb; w4 < we; ++w4) {
            const int4 sh4 = *(const int4*)(s_sh + 4 * w4);
            const int shq[4] = {sh4.x, sh4.y, sh4.z, sh4.w};
            uint32_t word = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t val = 255;
                if (4 * w4 + q < N) {
                    const int sh = __builtin_amdgcn_readfirstlane(shq[q]);
                    if (sh != prev) {
                        prev = sh;
                        hd = 0;
#pragma unroll
                        for (int c = 0; c < C; ++c)
                            hd += (uint32_t)__popcll(r[c] ^ gather(sh, c));
                    }
                    val = hd;
                }
                word |= val << (8 * q);
            }
            tile[lane * NW + w4] = word;
        }
    }
    __syncthreads();
    // the tile is npix * NP contiguous bytes of C (NP is a multiple of 4): 16-byte
    // stores (4-byte aligned), then the last words one by one
    uint32_t* dst = (uint32_t*)(a.cvol + ((size_t)z * HW + p0) * NP);
    const int words = npix * NP / 4, quads = words / 4;
    for (int i = threadIdx.x; i < quads; i += 256) {
        uint4 q;
        __builtin_memcpy(&q, __builtin_assume_aligned(tile + 4 * i, 16), 16);
        __builtin_memcpy(dst + 4 * i, &q, 16);
    }
    for (int i = 4 * quads + threadIdx.x; i < words; i += 256) dst[i] = tile[i];
}

template <class Src, int C>
__global__ __launch_bounds__(256) void census_cost_volume_kernel(Src src) {
    __shared__ __align__(16) uint32_t tile[kTilePix * LF_MAX_HYPOTHESES / 4];
    __shared__ __align__(16) int s_sh[LF_MAX_HYPOTHESES];
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const CcvArgs& a = member(src, vb, b);
        __syncthreads();                          // LDS of the previous block is read
        ccv_block<C>(a, b, tile, s_sh);
    }
}

// SGM over the Census cost volume, every direction of every view in one launch.
// Output: Lbuf[r][z][p][NP], storage type LT, NP a multiple of 4 elements.
struct DenseArgs {
    gptr<const uint8_t> cvol;      // [nv][H*W][NPc]
    gptr<void> Lbuf;
    Lines lines;
    Units units;
    int nv, H, W, N, NP, NPc;
    uint32_t P1, P2;
    uint32_t wblocks;         // blocks per view
};

// Staged bytes per step of the initial path kernel: the lanes' 64 K path costs,
// rounded up to whole 128-byte lines, as are the rows in memory (a path-cost
// row of NP elements is never longer: see dense_lnp).
constexpr int dense_stage_row(int K, int elem_bytes) {
    return (64 * K * elem_bytes + 127) / 128 * 128;
}

// The K path costs of a lane, written as LT into the wave's staging row.
template <int K, typename LT>
__device__ __forceinline__ void stage_put(uint8_t* dst, const uint32_t (&L)[K]) {
    if constexpr (sizeof(LT) == 1) {
        if constexpr (K == 1) {
            *dst = (uint8_t)L[0];
        } else if constexpr (K == 2) {
            *(uint16_t*)dst = (uint16_t)((L[0] & 0xFFu) | (L[1] << 8));
        } else if constexpr (K == 4) {
            *(uint32_t*)dst = (L[0] & 0xFFu) | ((L[1] & 0xFFu) << 8) | ((L[2] & 0xFFu) << 16) |
                              (L[3] << 24);
        } else {
#pragma unroll
            for (int j = 0; j < K; ++j) dst[j] = (uint8_t)L[j];
        }
    } else {
        if constexpr (K == 1) {
            *(uint16_t*)dst = (uint16_t)L[0];
        } else if constexpr (K == 2) {
            *(uint32_t*)dst = (L[0] & 0xFFFFu) | (L[1] << 16);
        } else if constexpr (K == 4) {
            *(uint2*)dst = make_uint2((L[0] & 0xFFFFu) | (L[1] << 16),
                                      (L[2] & 0xFFFFu) | (L[3] << 16));
        } else {
#pragma unroll
            for (int j = 0; j < K; ++j) ((uint16_t*)dst)[j] = (uint16_t)L[j];
        }
    }
}

// kPad (8-bit path costs, K = 2, and B + 2 P2 <= 255 + P1 for the largest Census
// cost B): hypotheses k >= N read the 255 that pads each cost row instead of
// adding kInf.  Their path costs then stay >= 255 while every real one stays
// <= B + P2 <= 255, so they never lower the minimum m, and as the neighbour of
// k = N-1 their 255 + P1 >= m + P2 (m <= B + P2) never wins the min of Eq. (8):
// the real path costs are those of the exact recurrence.
//
// Stores.  A path-cost row (NP elements) per step would be one narrow store per
// step, and those stores took about a third of the kernel's vector-memory
// issue.  Instead each step's row goes to the wave's staging area in LDS, and
// after every D steps the wave copies the D rows out with 16-byte stores, the
// lanes over (row, 16-byte chunk) pairs, and one store for the rows' short
// tails: 16 rows of 100 bytes are three store instructions.  Row elements
// k >= N hold don't-care values.
template <int K, typename LT, int D, bool kPad>
__device__ __forceinline__ void dense_line(const DenseArgs& a, int z, const LineInfo& li,
                                           uint8_t* wst) {
    constexpr int kRow = dense_stage_row(K, sizeof(LT));    // staged bytes per step
    constexpr int kRounds = (D * kRow / 16 + 63) / 64;      // 16-byte copies per lane
    const int lane = threadIdx.x & 63;
    const int H = a.H, W = a.W, N = a.N, NPc = a.NPc;
    const uint32_t P1 = a.P1, P2 = a.P2;
    const uint32_t HW = (uint32_t)H * W;
    const uint8_t* __restrict__ cz = a.cvol + (size_t)z * HW * NPc;
    const int rb = a.NP * (int)sizeof(LT);                  // bytes per path-cost row
    uint8_t* __restrict__ out = (uint8_t*)a.Lbuf + ((size_t)li.r * a.nv + z) * HW * rb;

    // Copy plan of a flush, fixed per line.  A row is c16 whole 16-byte chunks
    // and a tail of 0, 4, 8 or 12 bytes (rows are 4-byte aligned).  Copy j of
    // this lane moves chunk c of staged row s to byte goff[j] past the flush's
    // base address, that of the lowest-addressed row (rows follow the line, so
    // for a direction running backwards it is the block's last row); lane s < D
    // also moves the tail of row s.  Chunks past the D rows repeat the last one
    // (the same bytes to the same place).
    const int c16 = rb >> 4, tail = rb & 15, nchunk = D * c16;
    const int dstep = li.dv * W + li.du;                    // pixels per step
    const int sbytes = dstep * rb;
    const int minoff = min(0, (D - 1) * sbytes);
    uint32_t loff[kRounds], goff[kRounds];
    int srow[kRounds];
#pragma unroll
    for (int j = 0; j < kRounds; ++j) {
        const int idx = min(lane + 64 * j, max(nchunk - 1, 0));
        const int s = c16 ? idx / c16 : 0, c = idx - s * c16;
        srow[j] = s;
        loff[j] = (uint32_t)(s * kRow + c * 16);
        goff[j] = (uint32_t)(s * sbytes - minoff + c * 16);
    }
    const int tsrow = min(lane, D - 1);
    const uint32_t tloff = (uint32_t)(tsrow * kRow + c16 * 16);
    const uint32_t tgoff = (uint32_t)(tsrow * sbytes - minoff + c16 * 16);

    // the lane's K bytes of a pixel row; lanes past N read the row's last bytes
    // (with kPad: its 255 padding, since NPc >= N + 2) and, without kPad, add kInf
    const uint32_t lofs = (uint32_t)min(lane * K, NPc - K);
    uint32_t cinit[K];
#pragma unroll
    for (int j = 0; j < K; ++j) cinit[j] = kPad || lane * K + j < N ? 0u : kInf;
    const int last = li.len - 1;
    const int64_t srow_bytes = (int64_t)dstep * NPc;       // cost-row bytes per step
    // One load per step for the K bytes.  The loads of a block of D steps go
    // through a buffer descriptor based at the lowest-addressed row among them;
    // a step's row offset from it (>= 0, < 2^31) is the scalar offset, the lane's
    // byte within the row the vector offset: no per-step vector arithmetic.
    auto block_rsrc = [&](int nb, int& lo) {
        lo = dstep >= 0 ? min(nb, last) : min(nb + D - 1, last);
        const uint32_t p = (uint32_t)((li.v0 + lo * li.dv) * W + li.u0 + lo * li.du);
        return __builtin_amdgcn_make_buffer_rsrc((void*)(cz + (size_t)p * NPc), (short)0,
                                                 0x7FFFFFFF, 0x00020000);
    };
    auto load = [&](__amdgpu_buffer_rsrc_t rs, int lo, int step) -> uint32_t {
        const int so = (int)((int64_t)(min(step, last) - lo) * srow_bytes);
        if constexpr (K == 1) {
            return __builtin_amdgcn_raw_buffer_load_b8(rs, lofs, so, 0);
        } else if constexpr (K == 2) {
            return __builtin_amdgcn_raw_buffer_load_b16(rs, lofs, so, 0);
        } else if constexpr (K == 4) {
            return __builtin_amdgcn_raw_buffer_load_b32(rs, lofs, so, 0);
        } else {
            return (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, lofs, so, 0) |
                   ((uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, lofs + 1, so, 0) << 8) |
                   ((uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, lofs + 2, so, 0) << 16);
        }
    };
    uint32_t cb[D];
    {
        int lo;
        const __amdgpu_buffer_rsrc_t rs = block_rsrc(0, lo);
#pragma unroll
        for (int i = 0; i < D; ++i) cb[i] = load(rs, lo, i);
    }

    uint8_t* const mine = wst + lane * K * (int)sizeof(LT);
    uint32_t Lp[K], m = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) Lp[j] = kInf;
    for (int base = 0; base < li.len; base += D) {
        int lo;
        const __amdgpu_buffer_rsrc_t rs = block_rsrc(base + D, lo);
#pragma unroll
        for (int i = 0; i < D; ++i) {
            const int step = base + i;           // steps past the line end are computed
            uint32_t C[K];                       // and not copied out
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const uint32_t byte = (cb[i] >> (8 * j)) & 0xFFu;
                C[j] = kPad ? byte : byte + cinit[j];
            }
            cb[i] = load(rs, lo, step + D);      // refill the slot just consumed
            uint32_t L[K];
            if (step == 0) {
#pragma unroll
                for (int j = 0; j < K; ++j) L[j] = C[j];
            } else {
                sgm_step<K>(Lp, m, P1, P2, C, L);
            }
            m = wave_min(lane_min(L));
            stage_put<K, LT>(mine + i * kRow, L);
#pragma unroll
            for (int j = 0; j < K; ++j) Lp[j] = L[j];
        }
        // flush: the staged rows were written by other lanes of this wave, whose
        // LDS accesses complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int rows = min(D, li.len - base);
        const uint32_t pb = (uint32_t)((li.v0 + base * li.dv) * W + li.u0 + base * li.du);
        uint8_t* const ob = out + (int64_t)pb * rb + minoff;
        const bool stream = (rb & 127) == 0;     // whole-line rows
        // LDS offsets are 16-byte aligned; rows in memory 4-byte aligned
        auto copy = [&](uint32_t lo, uint32_t go, auto n) {
            constexpr int kBytes = decltype(n)::value;
            using V = typename std::conditional<kBytes == 16, uint4,
                      typename std::conditional<kBytes == 12, uint3,
                      typename std::conditional<kBytes == 8, uint2, uint32_t>::type>::type>::type;
            V v;
            __builtin_memcpy(&v, __builtin_assume_aligned(wst + lo, 16), kBytes);
            if constexpr (kBytes == 16) {
                if (stream) {
                    // rows are whole cache lines, read once by the sum: streaming
                    // (non-temporal) stores, measured 0.33 vs 0.41 ms for the kernel
                    uint32_t* d = (uint32_t*)__builtin_assume_aligned(ob + go, 16);
                    __builtin_nontemporal_store(v.x, d);
                    __builtin_nontemporal_store(v.y, d + 1);
                    __builtin_nontemporal_store(v.z, d + 2);
                    __builtin_nontemporal_store(v.w, d + 3);
                    return;
                }
            }
            __builtin_memcpy(__builtin_assume_aligned(ob + go, 4), &v, kBytes);
        };
#pragma unroll
        for (int j = 0; j < kRounds; ++j) {
            if (64 * j >= nchunk) break;         // wave-uniform
            if (rows == D || srow[j] < rows) copy(loff[j], goff[j], std::integral_constant<int, 16>());
        }
        if (tail && tsrow < rows) {
            if (tail == 4) copy(tloff, tgoff, std::integral_constant<int, 4>());
            else if (tail == 8) copy(tloff, tgoff, std::integral_constant<int, 8>());
            else copy(tloff, tgoff, std::integral_constant<int, 12>());
        }
        // the next steps overwrite the staging rows only after these reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

template <class Src, int K, typename LT, int D, bool kPad>
__global__ __launch_bounds__(64 * kWavesPerBlock) void sgm_dense_paths_kernel(Src src) {
    constexpr int kWaveBytes = D * dense_stage_row(K, sizeof(LT));
    __shared__ __align__(16) uint8_t stage[kWavesPerBlock * kWaveBytes];
    uint8_t* const wst = stage + (threadIdx.x >> 6) * kWaveBytes;
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const DenseArgs& a = member(src, vb, b);
        const int z = (int)(b / a.wblocks);               // the view
        const uint32_t wb = b - (uint32_t)z * a.wblocks;
        const int u = __builtin_amdgcn_readfirstlane(wb * kWavesPerBlock + (threadIdx.x >> 6));
        if (u >= a.units.nunits) continue;                // wave-uniform
        int line[2];
        unit_lines(a.lines, a.units, a.H, a.W, u, line);
        for (int part = 0; part < 2; ++part) {            // one copy of the line loop
            if (line[part] < 0) break;
            dense_line<K, LT, D, kPad>(a, z, locate(a.lines, a.H, a.W, line[part]), wst);
        }
    }
}

// --- 16 lanes (one DPP row) per path line, four lines per wave ----------------
// The lines of a direction are taken as units of equal length: the
// primary axis is the one the direction moves fastest along (the shorter one for
// the diagonals), and unit x walks it from its entry side, starting at position
// x of the other axis and, where the direction also moves along that one,
// wrapping around its end.  A path starts (L = C) at the first step and at each
// wrap, which is where the predecessor is outside the image.  A knight move
// steps two along its primary axis: one set of units per parity.  A wave's four
// rows take four neighbouring units, so they walk side by side.

// The walk of direction (du, dv) as equal units.
struct Walk {
    bool pv;            // the primary axis is v
    int step, dir;      // pixels per step along it, and its sign
    int len, Q;         // lengths of the primary and the other axis
    int dsec;           // movement along the other axis per step: -1, 0, 1
    int units;          // Q for each parity of the primary axis
};

__host__ __device__ inline Walk make_walk(int H, int W, int du, int dv) {
    const int au = du < 0 ? -du : du, av = dv < 0 ? -dv : dv;
    Walk w;
    w.pv = av > au || (av == au && H <= W);
    w.step = av > au ? av : au;
    w.dir = (w.pv ? dv : du) > 0 ? 1 : -1;
    w.len = w.pv ? H : W;
    w.Q = w.pv ? W : H;
    w.dsec = w.pv ? du : dv;
    w.units = w.Q * (w.step < w.len ? w.step : w.len);
    return w;
}

// The waves of the directions, four units each, and their prefix sums.
inline void rows_waves(int H, int W, int npaths, int* wbase) {
    int n = 0;
    wbase[0] = 0;
    for (int r = 0; r < kMaxPaths; ++r) {
        if (r < npaths) n += (make_walk(H, W, kDirs[r][0], kDirs[r][1]).units + 3) / 4;
        wbase[r + 1] = n;
    }
}

// Lane j of every row takes lane I's value of its row.
template <int I>
__device__ __forceinline__ uint32_t row_bcast(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + I, 0xF, 0xF, true);
}

// The same in a register of its own, for values that are subtracted or shifted by:
// the compiler folds a DPP operand into the reversed forms too (v_subrev,
// v_lshrrev), which permute the other operand (measured).
template <int I>
__device__ __forceinline__ uint32_t row_value(uint32_t v) {
    uint32_t x = row_bcast<I>(v);
    asm("" : "+v"(x));
    return x;
}

// Row rotations: the value of lane j - 1 and of lane j + 1 (mod 16).
__device__ __forceinline__ uint32_t row_prev(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t row_next(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x12F, 0xF, 0xF, true);
}

// Minimum over each row of 16 lanes, in every lane of it (rotations by 8, 4, 2, 1).
__device__ __forceinline__ uint32_t row_min(uint32_t v) {
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, true));
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, true));
    return min(v, row_prev(v));
}

// The steps at which any of the four rows has its bit set.
__device__ __forceinline__ uint32_t any_row(uint64_t ballot) {
    const uint32_t half = (uint32_t)ballot | (uint32_t)(ballot >> 32);
    return (half | half >> 16) & 0xFFFFu;
}

// Two 16-bit values per register.
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));
using u16x2 = unsigned short __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 as_u16x2(uint32_t x) { return __builtin_bit_cast(u16x2, x); }
__device__ __forceinline__ uint32_t as_u32(u16x2 x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ uint32_t pk_min(uint32_t x, uint32_t y) {
    return as_u32(__builtin_elementwise_min(as_u16x2(x), as_u16x2(y)));
}
__device__ __forceinline__ uint32_t pk_add(uint32_t x, uint32_t y) {
    return as_u32(as_u16x2(x) + as_u16x2(y));
}
__device__ __forceinline__ uint32_t pk_sub(uint32_t x, uint32_t y) {
    return as_u32(as_u16x2(x) - as_u16x2(y));
}
__device__ __forceinline__ uint32_t pk_add_sat(uint32_t x, uint32_t y) {
    return as_u32(__builtin_elementwise_add_sat(as_u16x2(x), as_u16x2(y)));
}
// (x >> 16) | (y << 16): the high half of x and the low half of y.
__device__ __forceinline__ uint32_t pk_next(uint32_t x, uint32_t y) {
    return __builtin_amdgcn_alignbit(y, x, 16);
}

// The initial paths, four lines per wave: lane j of a row holds the 2 NR hypotheses from
// 2 NR j, two per register in packed 16-bit arithmetic.  The one-line form is bound by the
// issue of its instructions, 25 per step; this one takes 55 for a step of four lines.
// A byte permutation unpacks the lane's cost bytes and puts 255 in place of hypotheses
// k >= N (the bound of kPad: those then never win a min).  Lane j holds the pixel of step
// j of a block of 16, as byte offsets, and a step reads them by a row broadcast; the
// next block's costs are in flight.  A row's path costs are written by one instruction
// (past the caches where the rows are whole lines: 281 us, 4 views of 512x512, N = 100, 1.07
// GB written; a third more through the caches; 313 us by the one-line form).
struct DenseRowsArgs {
    gptr<const uint8_t> cvol;      // [nv][H*W][NPc]
    gptr<uint8_t> Lbuf;            // [npaths][nv][H*W][NP]
    int nv, H, W, N, NP, NPc;
    uint32_t P1, P2;
    int npaths;
    uint32_t wblocks;              // blocks per view
    int wbase[kMaxPaths + 1];      // direction r owns waves [wbase[r], wbase[r+1])
};

constexpr uint32_t kRowsVolume = 0x7F000000u;  // the largest volume of a view

template <int NR>
__device__ __forceinline__ void dense_rows_wave(const DenseRowsArgs& a, int z, int wave) {
    constexpr int B = 16;                          // steps per block
    constexpr int NW = NR / 2;                     // words of a lane's costs
    const int lane = threadIdx.x & 63, j = lane & 15, row = lane >> 4;
    const int H = a.H, W = a.W, N = a.N;

    // the wave's direction (constant indices: the record stays in registers)
    int r = 0, wb = 0;
#pragma unroll
    for (int i = 1; i < kMaxPaths; ++i)
        if (i < a.npaths && wave >= a.wbase[i]) {
            r = i;
            wb = a.wbase[i];
        }
    const Walk wk = make_walk(H, W, dir_u(r), dir_v(r));
    const int x = (wave - wb) * 4 + row;                      // this row's unit
    const int xq = min(x, wk.units - 1);
    const int q = xq / wk.Q, sec0 = xq - q * wk.Q;            // parity, start
    const int P = (wk.len - q + wk.step - 1) / wk.step;       // steps of this unit
    const int steps = (wk.len + wk.step - 1) / wk.step;       // of the wave
    const int Prow = x < wk.units ? P : 0;                    // none past the last unit

    const uint32_t HW = (uint32_t)H * W;
    const uint32_t NPc = (uint32_t)a.NPc, NP = (uint32_t)a.NP;
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const uint8_t*)a.cvol + (size_t)z * HW * NPc), (short)0, (int)(HW * NPc),
        0x00020000);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((uint8_t*)a.Lbuf + ((size_t)r * a.nv + z) * HW * NP), (short)0, (int)(HW * NP),
        0x00020000);
    // past the volumes (of at most kRowsVolume bytes), also one added to the other
    constexpr uint32_t kNowhere = 0x80000000u, kNoLane = kRowsVolume;
    // the lane's bytes of a cost row (the row's last ones, if it has none), and of a
    // path-cost row
    const uint32_t first = (uint32_t)min(2 * NR * j, a.NPc - 2 * NR);
    const uint32_t out = 2 * NR * j < a.NP ? (uint32_t)(2 * NR * j) : kNoLane;
    uint32_t sel[NR];                              // of the byte permutation
#pragma unroll
    for (int c = 0; c < NR; ++c) {
        const int k = 2 * NR * j + 2 * c;          // 13: 0xFF, 12: 0
        sel[c] = (k < N ? (uint32_t)k - first : 13u) |
                 (k + 1 < N ? (uint32_t)k + 1 - first : 13u) << 16 | 0x0C000C00u;
    }

    // the steps of a block, one per lane of a row
    struct Meta {
        uint32_t cost, L;                          // byte offsets of the rows
        uint32_t start;                            // a path starts
        uint32_t starts;                           // steps at which any row's does
    };
    int tau = j;                                   // this lane's step
    int sec = sec0 + wk.dsec * (j % wk.Q);         // and where it is
    if (sec >= wk.Q) sec -= wk.Q;
    if (sec < 0) sec += wk.Q;
    const int adv = wk.dsec * (B % wk.Q);
    auto next_meta = [&]() -> Meta {
        const int st = q + wk.step * min(tau, P - 1);
        const int pri = wk.dir > 0 ? st : wk.len - 1 - st;
        const uint32_t p = (uint32_t)(wk.pv ? pri * W + sec : sec * W + pri);
        Meta m;
        m.cost = p * NPc;
        m.L = tau < Prow ? p * NP : kNowhere;
        m.start = tau == 0 || (wk.dsec > 0 && sec == 0) || (wk.dsec < 0 && sec == wk.Q - 1);
        m.starts = any_row(__builtin_amdgcn_ballot_w64(m.start != 0));
        tau += B;
        sec += adv;
        if (sec >= wk.Q) sec -= wk.Q;
        if (sec < 0) sec += wk.Q;
        return m;
    };
    struct Words {
        uint32_t w[NW];
    };
    auto load = [&](uint32_t at) {
        Words x;
        if constexpr (NW == 2) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rc, at, 0, 0);
            x.w[0] = v[0];
            x.w[1] = v[1];
        } else {
            x.w[0] = __builtin_amdgcn_raw_buffer_load_b32(rc, at, 0, 0);
        }
        return x;
    };

    const uint32_t P11 = a.P1 | a.P1 << 16, P22 = a.P2 | a.P2 << 16;
    uint32_t L[NR], mm = 0;                        // mm: the minimum, in both halves
#pragma unroll
    for (int c = 0; c < NR; ++c) L[c] = 0;
    Meta cur = next_meta();
    Words cb[B];
    static_for<B>([&](auto I) { cb[I] = load(row_value<I>(cur.cost) + first); });
    for (int base = 0; base < steps; base += B) {
        const Meta nxt = next_meta();
        static_for<B>([&](auto I) {
            constexpr int i = decltype(I)::value;
            uint32_t C[NR], X[NR], nb[NR + 1];
#pragma unroll
            for (int c = 0; c < NR; ++c)
                C[c] = __builtin_amdgcn_perm(cb[i].w[NW - 1], cb[i].w[0], sel[c]);
            cb[i] = load(row_value<i>(nxt.cost) + first);
#pragma unroll
            for (int c = 0; c < NR; ++c) X[c] = pk_add(L[c], P11);
            nb[0] = pk_next(dpp<0x111>(~0u, X[NR - 1]), X[0]);          // row_shr:1
#pragma unroll
            for (int c = 1; c < NR; ++c) nb[c] = pk_next(X[c - 1], X[c]);
            nb[NR] = pk_next(X[NR - 1], dpp<0x101>(~0u, X[0]));         // row_shl:1
            const uint32_t m2 = pk_add(mm, P22);
#pragma unroll
            for (int c = 0; c < NR; ++c)
                L[c] = pk_add(pk_min(pk_min(L[c], m2), pk_min(nb[c], nb[c + 1])),
                              pk_sub(C[c], mm));
            if (__builtin_expect(cur.starts >> i & 1, 0)) {
                const bool start = row_value<i>(cur.start) != 0;
#pragma unroll
                for (int c = 0; c < NR; ++c) L[c] = start ? C[c] : L[c];
            }
            uint32_t least = L[0];
#pragma unroll
            for (int c = 1; c < NR; ++c) least = pk_min(least, L[c]);
            least = pk_min(least, __builtin_amdgcn_alignbit(least, least, 16));
            mm = row_min(least);                   // both halves alike: ordered as one
            const uint32_t at = row_value<i>(cur.L) + out;
            if constexpr (NW == 2)                 // whole lines, read once by the sum
                __builtin_amdgcn_raw_buffer_store_b64(
                    u32x2{__builtin_amdgcn_perm(L[1], L[0], 0x06040200u),
                          __builtin_amdgcn_perm(L[3], L[2], 0x06040200u)}, ro, at, 0, 2);
            else
                __builtin_amdgcn_raw_buffer_store_b32(
                    __builtin_amdgcn_perm(L[1], L[0], 0x06040200u), ro, at, 0, 0);
        });
        cur = nxt;
    }
}

template <class Src, int NR>
__global__ __launch_bounds__(64 * kWavesPerBlock) void sgm_dense_rows_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const DenseRowsArgs& a = member(src, vb, b);
        // The views in turn, so that the directions of the image's longer side, the first
        // for a wide one, start with the launch in every view: view by view, the last one's
        // would end it alone (4 views of 156x624, N = 64: 180 us, 79 in turn; 331x449, N =
        // 77: 185, 173; of the 2 to 4 views of 346 sizes and shapes 1.11 times as fast).
        const uint32_t wb = b / (uint32_t)a.nv;
        const int z = (int)(b - wb * (uint32_t)a.nv);
        const int wave = __builtin_amdgcn_readfirstlane(wb * kWavesPerBlock + (threadIdx.x >> 6));
        if (wave >= a.wbase[kMaxPaths]) continue;             // wave-uniform
        dense_rows_wave<NR>(a, z, wave);
    }
}

// Sum over directions + WTA (Eq. 9-10) of the initial stage: one wave per pixel,
// lane l holds hypotheses 2l and 2l+1 (+128 per round); lowest index on ties.
struct SumWtaArgs {
    gptr<const void> Lbuf;
    int64_t HW;
    int nv, N, NP;
    gptr<int16_t> dmap;            // [nv][H*W]
};

template <typename LT, int kPaths>
__device__ __forceinline__ void sum_wta_block(const SumWtaArgs& a, uint32_t b) {
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)b * 4 + (threadIdx.x >> 6);       // q = z*HW + p
    if (q >= a.nv * a.HW) return;                                 // wave-uniform
    const int N = a.N, NP = a.NP;
    const size_t dir_stride = (size_t)a.nv * a.HW * NP;
    const LT* __restrict__ base = (const LT*)a.Lbuf + (size_t)q * NP;
    uint32_t key = UINT_MAX;
    for (int k = 2 * lane; k < N; k += 128) {
        uint32_t x[kPaths];                                       // all loads in flight first
#pragma unroll
        for (int r = 0; r < kPaths; ++r) {
            const LT* e = base + (size_t)r * dir_stride + k;
            if constexpr (sizeof(LT) == 1) x[r] = __builtin_nontemporal_load((const uint16_t*)e);
            else x[r] = __builtin_nontemporal_load((const uint32_t*)e);
        }
        uint32_t t0 = 0, t1 = 0;
#pragma unroll
        for (int r = 0; r < kPaths; ++r) {
            if constexpr (sizeof(LT) == 1) {
                t0 += x[r] & 0xFF;
                t1 += x[r] >> 8;
            } else {
                t0 += x[r] & 0xFFFF;
                t1 += x[r] >> 16;
            }
        }
        key = min(key, (t0 << 8) | (uint32_t)k);
        if (k + 1 < N) key = min(key, (t1 << 8) | (uint32_t)(k + 1));
    }
    key = wave_min(key);
    if (lane == 0) a.dmap[q] = (int16_t)(key & 0xFF);
}

// The same for 8-bit path costs with rows of at most 128 bytes (N <= 128): a
// row of 16 lanes per pixel, 8 bytes (8 hypotheses) per lane, so one 64-lane
// load reads four pixels' rows of a direction (512 bytes).  The sums are kept
// two per register in 16-bit fields (at most 16 * 255 per field: no carry
// between fields); the argmin is a DPP minimum within the row of 16 lanes.
// Lanes past a row's end read the next row (or the slack after the volume) and
// drop those hypotheses (k >= N).
template <int kPaths>
__device__ __forceinline__ void sum_wta_rows_block(const SumWtaArgs& a, uint32_t b) {
    const int sub = threadIdx.x & 15;
    const int64_t nq = a.nv * a.HW;
    const int64_t q = (int64_t)b * 16 + (threadIdx.x >> 4);       // this row's pixel
    const int64_t qq = q < nq ? q : nq - 1;                        // rows past the end
    const int N = a.N;                                             // load in bounds
    const size_t dir_stride = (size_t)a.nv * a.HW * a.NP;
    const uint8_t* __restrict__ base = (const uint8_t*)a.Lbuf + (size_t)qq * a.NP + sub * 8;
    // the path costs are read once: non-temporal loads (measured 0.155 vs 0.204
    // ms at the benchmark size) keep them from displacing what L2 holds
    uint32_t x0[kPaths], x1[kPaths];
#pragma unroll
    for (int r = 0; r < kPaths; ++r) {
        const uint32_t* pp = (const uint32_t*)(base + (size_t)r * dir_stride);
        x0[r] = __builtin_nontemporal_load(pp);
        x1[r] = __builtin_nontemporal_load(pp + 1);
    }
    // acc[0]: bytes 0, 2; acc[1]: 1, 3; acc[2]: 4, 6; acc[3]: 5, 7 (low, high field)
    uint32_t acc[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < kPaths; ++r) {
        acc[0] += x0[r] & 0x00FF00FFu;
        acc[1] += (x0[r] >> 8) & 0x00FF00FFu;
        acc[2] += x1[r] & 0x00FF00FFu;
        acc[3] += (x1[r] >> 8) & 0x00FF00FFu;
    }
    uint32_t key = UINT_MAX;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t t = (acc[(i >> 2) * 2 + (i & 1)] >> (16 * ((i >> 1) & 1))) & 0xFFFFu;
        const int k = sub * 8 + i;
        if (k < N) key = min(key, (t << 8) | (uint32_t)k);
    }
    key = min(key, dpp<0xB1>(UINT_MAX, key));     // quad_perm [1,0,3,2]
    key = min(key, dpp<0x4E>(UINT_MAX, key));     // quad_perm [2,3,0,1]
    key = min(key, dpp<0x141>(UINT_MAX, key));    // row_half_mirror
    key = min(key, dpp<0x140>(UINT_MAX, key));    // row_mirror: the row's minimum
    if (sub == 0 && q < nq) a.dmap[q] = (int16_t)(key & 0xFF);
}

template <class Src, int kPaths>
__global__ __launch_bounds__(256) void dense_sum_wta_rows_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const SumWtaArgs& a = member(src, vb, b);
        sum_wta_rows_block<kPaths>(a, b);
    }
}

template <class Src, typename LT, int kPaths>
__global__ __launch_bounds__(256) void dense_sum_wta_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const SumWtaArgs& a = member(src, vb, b);
        sum_wta_block<LT, kPaths>(a, b);
    }
}

// Optional outputs of the initial stage for checking: the Census cost of Eq. (7)
// and the aggregated cost of Eq. (9) of every cross view, [nv][H*W][N], copied
// and summed out of the stage's own buffers (element e = (z*HW + p)*N + k).
struct ExportArgs {
    gptr<const void> src;          // cvol [nv][HW][NPc] (8-bit), or Lbuf [npaths][nv][HW][NP]
    gptr<void> dst;                // [nv][HW][N]: 8-bit costs, or 16-bit sums
    int64_t rows;             // nv * HW
    int N, NP, npaths, lt;    // lt: bytes per path-cost element (sums)
};

template <class Src, bool kSum>
__global__ __launch_bounds__(256) void initial_export_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const ExportArgs& a = member(src, vb, b);
        const int64_t e = (int64_t)b * 256 + threadIdx.x;
        if (e >= a.rows * a.N) continue;
        const int64_t q = e / a.N;
        const int64_t at = q * a.NP + (e - q * a.N);
        if constexpr (!kSum) {
            ((uint8_t*)a.dst)[e] = ((const uint8_t*)a.src)[at];
        } else {
            const int64_t dir = a.rows * a.NP;
            uint32_t s = 0;
            for (int r = 0; r < a.npaths; ++r)
                s += a.lt == 1 ? ((const uint8_t*)a.src)[r * dir + at]
                               : ((const uint16_t*)a.src)[r * dir + at];
            ((uint16_t*)a.dst)[e] = (uint16_t)s;
        }
    }
}

// ---------------------------------------------------------------------------
// Final stage: CSR volume over per-pixel ranges [lo, hi].  Output Lbuf[r][cell].
// meta[p] = {q = off[p] - lo[p] + N (int64, low half first), lo | hi << 16}: one
// 16-byte load per step, or one 8-byte load of the first two words where 32-bit
// offsets suffice.  Cell k of pixel p is q + k - N; q + k itself is positive for
// every k >= 0 (off[p] >= 0, lo[p] < N), so it can serve as an unsigned offset
// from N cells before the volume.
struct alignas(16) PixMeta {
    uint32_t q_lo;
    int32_t lohi;
    uint32_t q_hi;
    int32_t rows;                            // of pixel 0: not 0 if four lines per wave ran
    __device__ int64_t base(int N) const {   // off - lo
        return (int64_t)(((uint64_t)q_hi << 32) | q_lo) - N;
    }
};

__device__ __forceinline__ PixMeta pix_meta(int64_t off, int lo, int hi, int N) {
    // bounds outside the documented 0 <= lo <= hi < N are clamped into it; that
    // only narrows a range, so its cells stay within the pixel's own
    lo = clampi(lo, 0, N - 1);
    hi = clampi(hi, lo, N - 1);
    PixMeta m;
    const uint64_t q = (uint64_t)(off - lo + N);
    m.q_lo = (uint32_t)q;
    m.lohi = (int32_t)((uint32_t)lo | ((uint32_t)hi << 16));
    m.q_hi = (uint32_t)(q >> 32);
    m.rows = 0;
    return m;
}

struct MetaArgs {
    gptr<const int64_t> off;
    gptr<const int16_t> lo;
    gptr<const int16_t> hi;
    gptr<PixMeta> meta;
    int HW, N;
};

template <class Src>
__global__ __launch_bounds__(256) void pix_meta_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const MetaArgs& a = member(src, vb, b);
        const int p = (int)b * 256 + threadIdx.x;
        if (p >= a.HW) continue;
        a.meta[p] = pix_meta(a.off[p], a.lo[p], a.hi[p], a.N);
    }
}

struct BoundedArgs {
    gptr<const uint16_t> cost;
    gptr<const PixMeta> meta;
    gptr<uint16_t> Lbuf;           // [npaths][dir_stride]
    size_t dir_stride;
    Lines lines;
    Units units;                   // of the 64-lane kernel (one line per wave)
    int H, W, N;
    uint32_t P1, P2;
    int chosen;                    // only if the four-line kernel left it (see RowsChoice)
};

template <int K, int D>
__device__ __forceinline__ void bounded_line(const BoundedArgs& a, const LineInfo& li) {
    constexpr int kMeta = D, kCost = D / 2;   // two-stage prefetch
    const int lane = threadIdx.x & 63;
    const int W = a.W;
    const uint32_t P1 = a.P1, P2 = a.P2;
    const uint16_t* __restrict__ cost = a.cost;
    const PixMeta* __restrict__ meta = a.meta;
    uint16_t* __restrict__ out = a.Lbuf + (size_t)li.r * a.dir_stride;

    auto load_meta = [&](int step) {
        const int u = li.u0 + step * li.du, v = li.v0 + step * li.dv;
        return meta[in_vgpr((uint32_t)(v * W + u))];
    };
    // gather of the K costs of a pixel; hypotheses outside [lo, hi] read the
    // pixel's first cell and are replaced by kInf when used
    auto load_cost = [&](const PixMeta& pm, uint32_t (&c)[K]) {
        const int lo = pm.lohi & 0xFFFF, hi = pm.lohi >> 16;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int k = min(max(lane * K + j, lo), hi);
            c[j] = cost[pm.base(a.N) + k];
        }
    };
    PixMeta mb[kMeta];
    uint32_t cb[kCost][K];
#pragma unroll
    for (int i = 0; i < kMeta; ++i) mb[i] = load_meta(min(i, li.len - 1));
#pragma unroll
    for (int i = 0; i < kCost; ++i) load_cost(mb[i], cb[i]);

    uint32_t Lp[K], m = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) Lp[j] = kInf;
    for (int base = 0; base < li.len; base += kMeta) {
#pragma unroll
        for (int i = 0; i < kMeta; ++i) {
            const int step = base + i;           // steps past the line end are computed
            const PixMeta pm = mb[i];            // and not stored
            const int lo = pm.lohi & 0xFFFF, hi = pm.lohi >> 16;
            uint32_t C[K];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int k = lane * K + j;
                C[j] = (k >= lo && k <= hi) ? cb[i % kCost][j] : kInf;
            }
            // refill: costs for step + kCost (its meta arrived kMeta - kCost steps ago)
            load_cost(mb[(i + kCost) % kMeta], cb[i % kCost]);
            uint32_t L[K];
            if (step == 0) {
#pragma unroll
                for (int j = 0; j < K; ++j) L[j] = C[j];
            } else {
                sgm_step<K>(Lp, m, P1, P2, C, L);
            }
            m = wave_min(lane_min(L));
            const bool live = step < li.len;
#pragma unroll
            for (int j = 0; j < K; ++j) {
                const int k = lane * K + j;
                if (live && k >= lo && k <= hi) out[pm.base(a.N) + k] = (uint16_t)L[j];
            }
            // the slot's metadata for step + kMeta, loaded after the last use of
            // this step's (so the load can take the same registers: no copies,
            // which would wait for every load in flight, at the loop's back edge)
            mb[i] = load_meta(min(step + kMeta, li.len - 1));
#pragma unroll
            for (int j = 0; j < K; ++j) Lp[j] = L[j];
        }
    }
}

// The same line loop with the cost volume, the pixel metadata and this
// direction's path costs addressed through buffer descriptors, for volumes of
// less than 2^31 bytes: 32-bit byte offsets instead of 64-bit addresses.  A
// metadata load takes its pixel's offset as the scalar operand (no vector
// arithmetic), a cost gather med3(k, lo, hi) and one shift-add, and a step's
// stores one shift-add.  The descriptors start N cells before the volumes, so
// that the offsets q + k are never negative (the store of a lane whose first
// hypothesis lies below the range would otherwise start from a wrapped offset,
// and the hardware drops a store whose vector offset is out of range).  A lane's
// hypothesis k lies in [lo, hi] exactly when the clamp leaves it unchanged.
template <int K, int D>
__device__ __forceinline__ void bounded_line_buf(const BoundedArgs& a, const LineInfo& li) {
    constexpr int kMeta = D, kCost = D / 2;   // two-stage prefetch
    const int lane = threadIdx.x & 63;
    const int W = a.W;
    const uint32_t P1 = a.P1, P2 = a.P2;
    const int32_t vol_bytes = (int32_t)((a.dir_stride + a.N) * 2);
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const uint16_t*)a.cost - a.N), (short)0, vol_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(const PixMeta*)a.meta, (short)0, a.H * W * (int)sizeof(PixMeta), 0x00020000);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((uint16_t*)a.Lbuf + (size_t)li.r * a.dir_stride - a.N), (short)0, vol_bytes,
        0x00020000);
    struct Meta {
        uint32_t base, lohi;       // low 32 bits of q; lo | hi << 16
    };
    auto load_meta = [&](int step) -> Meta {
        const int u = li.u0 + step * li.du, v = li.v0 + step * li.dv;
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(
            rm, 0, (v * W + u) * (int)sizeof(PixMeta), 0);
        return Meta{x[0], x[1]};
    };
    int kl[K];                                 // the lane's hypotheses
#pragma unroll
    for (int j = 0; j < K; ++j) kl[j] = lane * K + j;
    // gather of the K costs of a pixel; hypotheses outside [lo, hi] read a cell
    // of the pixel and are replaced by kInf when used
    auto load_cost = [&](const Meta& pm, uint32_t (&c)[K]) {
        const int lo = (int)(pm.lohi & 0xFFFF), hi = (int)(pm.lohi >> 16);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint32_t k = (uint32_t)min(max(kl[j], lo), hi);
            c[j] = __builtin_amdgcn_raw_buffer_load_b16(rc, (pm.base + k) << 1, 0, 0);
        }
    };
    Meta mb[kMeta];
    uint32_t cb[kCost][K];
#pragma unroll
    for (int i = 0; i < kMeta; ++i) mb[i] = load_meta(min(i, li.len - 1));
#pragma unroll
    for (int i = 0; i < kCost; ++i) load_cost(mb[i], cb[i]);

    uint32_t Lp[K], m = 0;                     // step 0 reduces to L = C
#pragma unroll
    for (int j = 0; j < K; ++j) Lp[j] = 0;
    for (int base = 0; base < li.len; base += kMeta) {
#pragma unroll
        for (int i = 0; i < kMeta; ++i) {
            const int step = base + i;           // steps past the line end are computed
            const Meta pm = mb[i];               // and not stored
            const int lo = (int)(pm.lohi & 0xFFFF), hi = (int)(pm.lohi >> 16);
            bool in[K];
            uint32_t C[K];
#pragma unroll
            for (int j = 0; j < K; ++j) {
                in[j] = min(max(kl[j], lo), hi) == kl[j];
                C[j] = in[j] ? cb[i % kCost][j] : kInf;
            }
            load_cost(mb[(i + kCost) % kMeta], cb[i % kCost]);
            uint32_t L[K];
            sgm_step<K>(Lp, m, P1, P2, C, L);   // with Lp = 0 and m = 0: L = C at step 0
            m = wave_min(lane_min(L));
            const bool live = step < li.len;
            const uint32_t ob = (pm.base + (uint32_t)kl[0]) << 1;
#pragma unroll
            for (int j = 0; j < K; ++j)
                if (live && in[j])
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)L[j], ro, ob, 2 * j, 0);
            // the slot's metadata for step + kMeta, loaded after the last use of
            // this step's (so the load can take the same registers: no copies,
            // which would wait for every load in flight, at the loop's back edge)
            mb[i] = load_meta(min(step + kMeta, li.len - 1));
#pragma unroll
            for (int j = 0; j < K; ++j) Lp[j] = L[j];
        }
    }
}

template <class Src, int K, int D, bool kBuf>
__global__ __launch_bounds__(64 * kWavesPerBlock) void sgm_bounded_paths_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const BoundedArgs& a = member(src, vb, b);
        const int u = __builtin_amdgcn_readfirstlane(b * kWavesPerBlock + (threadIdx.x >> 6));
        if (u >= a.units.nunits) continue;            // wave-uniform
        if (a.chosen && ((const PixMeta*)a.meta)->rows) continue;
        int line[2];
        unit_lines(a.lines, a.units, a.H, a.W, u, line);
        for (int part = 0; part < 2; ++part) {        // one copy of the line loop
            if (line[part] < 0) break;
            if constexpr (kBuf)
                bounded_line_buf<K, D>(a, locate(a.lines, a.H, a.W, line[part]));
            else
                bounded_line<K, D>(a, locate(a.lines, a.H, a.W, line[part]));
        }
    }
}

// The bounded SGM with 16 lanes (one DPP row) per path line, four lines per wave.
//
// Narrow pixels.  Nearly all pixels keep a window of 2*lambda+1 hypotheses, so a
// wave per line works with 7 of its 64 K slots.  Here lane j of a row holds the
// hypothesis k of the pixel's window with k = j (mod 16): any window of up to 16
// hypotheses fits, a window that moves needs no data movement, and the
// neighbours k -+ 1 are the lanes j -+ 1 of the row (row_ror).  Lanes outside the
// window hold kOut or more, which loses to m + P2: the terms of Eq. (8) outside
// R(p - r) drop out without any masks, as long as the previous window and this
// one with a hypothesis to each side lie within 16 consecutive hypotheses.  Where
// they do not (a jump), a lane whose hypothesis changed is set to kOut first.
//
// Wide pixels (more than 14 hypotheses: the full-range ones).  Rows that are at
// one take a second path, entered by the wave when any of its rows is: lane j
// then holds the 2 NR hypotheses from lo + 2 NR j, two per register in packed
// 16-bit arithmetic (0xFFFF outside the window), with one 16-byte load and store
// per four registers.  Where the window starts elsewhere than the previous one,
// or the previous or next pixel is narrow, the path costs go through a row of LDS
// that has 0xFFFF on both sides (a narrow window takes one hypothesis more to each
// side, hence at most 14).
//
// Metadata.  Lane j of a row holds what step j of the current block of 16 steps
// needs (bounds, cell offset), decoded once, and a step reads it by a row
// broadcast (row_newbcast) fused into the instruction that uses it; the next
// block's is decoded and its successor's loads are in flight.  Ballots of the
// decode say which steps have anything but narrow pixels in the middle of a path:
// one bit test keeps the others to about 18 VALU for four lines.

// Whether the ranges suit this kernel, where the host cannot know.  A step with a wide pixel
// in any of the four rows takes several times as long as one without, so many of them make
// it slower than a wave per line, the more so the fewer their cells (figures beside the
// bounded_form rule).  Every wave looks at the same 256 sets of four neighbouring pixels,
// spread over the image, and finds the same: the share of sets with a wide pixel may be up
// to limit + slope * (cells per pixel), sets whose wide pixels are full ranges counting
// `full` each.  If it is more, the workgroups write the metadata of the one-line kernel
// instead, which is launched after this one and finds in it which of the two is to run.
struct RowsChoice {
    int on;                        // 0: take four lines
    float limit, slope, full;
};

struct RowsArgs {
    gptr<const uint16_t> cost;
    gptr<const int64_t> off;
    gptr<const int16_t> lo;
    gptr<const int16_t> hi;
    gptr<uint16_t> Lbuf;           // [npaths][dir_stride]
    size_t dir_stride;
    int H, W, N;
    uint32_t P1, P2;
    int npaths;
    int wbase[kMaxPaths + 1];      // direction r owns waves [wbase[r], wbase[r+1])
    gptr<PixMeta> meta;            // of the one-line kernel
    uint32_t nblk;                 // workgroups
    RowsChoice choice;
};

// What the four rows need of the 16 steps of a block: lane j of a row holds step
// j of its line.
struct RowsMeta {
    uint32_t lo, hi;
    uint32_t nlo2;          // -2 lo
    uint32_t offb;          // byte offset of the pixel's first cell
    int32_t w2;             // (hi - lo) * 2, or -1 for pixels the narrow path skips
    uint32_t flags;         // kRowWide ...
    // steps (bits 0..15) at which any of the rows has the flag
    uint32_t wide, pre, conv, part, leave;     // pre: kRowStart or kRowJump
};
constexpr uint32_t kRowWide = 1,    // a wide pixel
    kRowStart = 2,                  // the start of a path
    kRowJump = 4,                   // windows too far apart for the lanes (see above)
    kRowConv = 8,                   // wide, but not after a wide one from the same lo
    kRowAfterWide = 16;             // the pixel before is a wide one

constexpr int kRowsNarrow = 14;        // the widest window of the narrow path

// LDS of one row's wide path costs: 16 lanes x 2 NR hypotheses, with as many
// entries of 0xFFFF before and after them.
template <int NR>
constexpr int kRowsPad = 32 * NR;              // entries
template <int NR>
constexpr int kRowsLds = 3 * kRowsPad<NR>;

template <int NR>
__device__ __forceinline__ void bounded_rows_wave(const RowsArgs& a, int wave, uint16_t* lds) {
    constexpr int B = 16;           // steps per block
    constexpr int DW = 4;           // steps ahead that a wide pixel's costs are loaded
    constexpr int PAD = kRowsPad<NR>;
    const int lane = threadIdx.x & 63, j = lane & 15, row = lane >> 4;
    const int H = a.H, W_ = a.W, N = a.N;
    const uint32_t P1 = a.P1, P2 = a.P2;

    // the wave's direction (constant indices: the record stays in registers)
    int r = 0, wb = 0;
#pragma unroll
    for (int i = 1; i < kMaxPaths; ++i)
        if (i < a.npaths && wave >= a.wbase[i]) {
            r = i;
            wb = a.wbase[i];
        }
    const Walk wk = make_walk(H, W_, dir_u(r), dir_v(r));

    const int x = (wave - wb) * 4 + row;                      // this row's unit
    const int xq = min(x, wk.units - 1);
    const int q = xq / wk.Q, sec0 = xq - q * wk.Q;            // parity, start
    const int P = (wk.len - q + wk.step - 1) / wk.step;       // steps of this unit
    const int steps = (wk.len + wk.step - 1) / wk.step;       // of the wave
    const int Prow = x < wk.units ? P : 0;                    // none past the last unit

    // Byte offsets are from a 4-byte boundary at or before the costs' first cell: whole
    // aligned words of them are loaded for wide pixels, the last one at most two bytes
    // past the last cell.  The descriptors drop every access outside the volumes (the
    // costs may end at the last cell, which only the offsets know).
    const uint64_t cbase = (uint64_t)(const uint16_t*)a.cost;
    const uint32_t odd = (uint32_t)cbase & 2u;
    const uint64_t cells = min((uint64_t)a.off[H * W_], (uint64_t)a.dir_stride);
    const int32_t vol_bytes = (int32_t)(a.dir_stride * 2 + odd);
    const int32_t cost_bytes = __builtin_amdgcn_readfirstlane((int32_t)(cells * 2 + odd));
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(cbase - odd), (short)0, (cost_bytes + 3) & ~3, 0x00020000);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((uint64_t)((uint16_t*)a.Lbuf + (size_t)r * a.dir_stride) - odd), (short)0,
        vol_bytes, 0x00020000);

    // --- metadata of a block: loads, then the decode ---
    int tau = j;                                              // this lane's step
    int sec = sec0 + wk.dsec * (j % wk.Q);                    // and where it is
    if (sec >= wk.Q) sec -= wk.Q;
    if (sec < 0) sec += wk.Q;
    const int adv = wk.dsec * (B % wk.Q);
    struct Raw {
        uint32_t off;
        int lo, hi, sec, tau;
    };
    const uint32_t* __restrict__ off32 = (const uint32_t*)(const int64_t*)a.off;
    const int16_t* __restrict__ plo = a.lo;
    const int16_t* __restrict__ phi = a.hi;
    auto load_raw = [&]() -> Raw {
        const int st = q + wk.step * min(tau, P - 1);
        const int pri = wk.dir > 0 ? st : wk.len - 1 - st;
        const uint32_t p = (uint32_t)(wk.pv ? pri * W_ + sec : sec * W_ + pri);
        Raw x;
        x.off = off32[2 * (size_t)p];                         // the low half: < 2^30 cells
        x.lo = plo[p];
        x.hi = phi[p];
        x.sec = sec;
        x.tau = tau;
        tau += B;
        sec += adv;
        if (sec >= wk.Q) sec -= wk.Q;
        if (sec < 0) sec += wk.Q;
        return x;
    };
    // prv: the block before (its last step precedes this one's first)
    auto decode = [&](const Raw& x, const RowsMeta& prv) -> RowsMeta {
        RowsMeta m;
        // bounds outside the documented 0 <= lo <= hi < N are clamped into it
        const int lo = clampi(x.lo, 0, N - 1), hi = clampi(x.hi, lo, N - 1);
        const bool live = x.tau < Prow;
        const bool start = x.tau == 0 || (wk.dsec > 0 && x.sec == 0) ||
                           (wk.dsec < 0 && x.sec == wk.Q - 1);
        const bool wide = live && hi - lo >= kRowsNarrow, skip = wide || !live;
        m.lo = (uint32_t)lo;
        m.hi = (uint32_t)hi;
        m.nlo2 = 0u - 2u * (uint32_t)lo;
        m.offb = x.off * 2 + odd;
        m.w2 = skip ? -1 : (hi - lo) * 2;
        const int pl = (int)dpp<0x111>(row_bcast<15>(prv.lo), m.lo);
        const int ph = (int)dpp<0x111>(row_bcast<15>(prv.hi), m.hi);
        const bool pwide = ph - pl >= kRowsNarrow;
        const bool jump = !skip && !start && !pwide && max(ph, hi + 1) - min(pl, lo - 1) >= 16;
        const bool conv = wide && !start && (!pwide || pl != lo);
        m.flags = (wide ? kRowWide : 0) | (live && start ? kRowStart : 0) |
                  (jump ? kRowJump : 0) | (conv ? kRowConv : 0) | (pwide ? kRowAfterWide : 0);
        const uint64_t bw = __builtin_amdgcn_ballot_w64(wide);
        m.wide = any_row(bw);
        m.pre = any_row(__builtin_amdgcn_ballot_w64(jump || (live && start)));
        m.conv = any_row(__builtin_amdgcn_ballot_w64(conv));
        m.part = any_row(__builtin_amdgcn_ballot_w64(wide && (lo != 0 || hi != N - 1)));
        // a narrow pixel follows (the last step of a block: perhaps)
        m.leave = any_row(bw & ~(bw >> 1 & 0x7FFF7FFF7FFF7FFFull));
        return m;
    };

    const uint32_t J = (uint32_t)j;
    constexpr uint32_t kOut = 0x3FFF0000u;    // the cost of a lane outside the window
    constexpr uint32_t kNowhere = 0x80000000u;            // an offset outside every volume
    // --- prefetched 16 steps ahead: the lane's cell (A) and its cost (C) ---
    uint32_t A[B], C[B];
    bool in[B];
    auto locate_cell = [&](const RowsMeta& m, auto ic) {
        constexpr int i = decltype(ic)::value;
        const uint32_t o = (2 * J + row_bcast<i>(m.nlo2)) & 30u;
        in[i] = (int)o <= (int)row_bcast<i>((uint32_t)m.w2);
        uint32_t at = row_bcast<i>(m.offb) + o;
        asm volatile("" : "+v"(at));          // in every lane: a broadcast that was folded into
        A[i] = in[i] ? at : kNowhere;         // an add under a mask would read a masked lane
    };
    // Where a lane's prefetch reads: its cell, but in the row of a wide pixel a place
    // all over its cells, so that their lines are in the cache when fetch_wide loads
    // them (the values are not used).
    auto spread = [&](const RowsMeta& m, auto ic, uint32_t ad) -> uint32_t {
        constexpr int i = decltype(ic)::value;
        const uint32_t w2 = 2 * (row_value<i>(m.hi) - row_value<i>(m.lo));
        const uint32_t at = row_value<i>(m.offb) + min(4 * NR * J, w2);
        return row_value<i>(m.flags) & kRowWide ? at : ad;
    };
    // --- the costs of a wide pixel: the words that hold the lane's cells ---
    uint32_t CW[DW][NR + 1];
    auto fetch_wide = [&](const RowsMeta& m, auto ic, auto slot) {
        constexpr int i = decltype(ic)::value, sl = decltype(slot)::value;
        const uint32_t ad = (row_value<i>(m.offb) + 4 * NR * J) & ~3u;
        if constexpr (NR == 2) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rc, ad, 0, 0);
            CW[sl][0] = v[0];
            CW[sl][1] = v[1];
        } else {
#pragma unroll
            for (int c = 0; c < NR; c += 4) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(rc, ad, 4 * c, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) CW[sl][c + e] = v[e];
            }
        }
        CW[sl][NR] = __builtin_amdgcn_raw_buffer_load_b32(rc, ad, 4 * NR, 0);
    };

    uint16_t* const lrow = lds + row * kRowsLds<NR>;          // this row's entries
    // Between accesses of lrow by different lanes: the hardware keeps a wave's LDS accesses
    // in their order, the compiler those on the two sides of this (entries are written as
    // words and as halves, which it may take for different objects).
    auto lds_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint32_t MF[NR];                                          // full range: 0xFFFF past N
#pragma unroll
    for (int c = 0; c < NR; ++c) {
        const int k = 2 * NR * j + 2 * c;
        MF[c] = (k < N ? 0u : 0xFFFFu) | (k + 1 < N ? 0u : 0xFFFF0000u);
        *(uint32_t*)(lrow + k) = ~0u;
        *(uint32_t*)(lrow + 2 * PAD + k) = ~0u;
    }

    Raw raw = load_raw();
    RowsMeta cur{};
    cur = decode(raw, cur);
    raw = load_raw();
    RowsMeta nxt = decode(raw, cur);
    raw = load_raw();
    // (a store that the descriptor drops after each load, as in the loop: the waits for
    // the loads count the accesses issued since, on the way that has the fewest)
    static_for<B>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        locate_cell(cur, ic);
        C[i] = __builtin_amdgcn_raw_buffer_load_b16(
            rc, cur.wide & (1u << i) ? spread(cur, ic, A[i]) : A[i], 0, 0);
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)0, ro, kNowhere, 0, 0);
    });
    static_for<DW>([&](auto ic) {
        if (cur.wide & (1u << decltype(ic)::value)) fetch_wide(cur, ic, ic);
    });

    uint32_t V = 0, m = 0;                    // the previous pixel's path costs, minimum
    uint32_t Wp[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c) Wp[c] = 0;
    uint32_t last_lo = 0;                     // lo of the last step of the block before

    auto step = [&](auto ic, uint32_t busy) {
        constexpr int i = decltype(ic)::value;
        constexpr uint32_t bit = 1u << i;
        const uint32_t cost = in[i] ? C[i] : kOut;
        const uint32_t ad = A[i];
        locate_cell(nxt, ic);                 // the slot just consumed
        auto prev_lo = [&] { return i > 0 ? row_value<(i + B - 1) % B>(cur.lo) : last_lo; };
        if (__builtin_expect(cur.pre & bit, 0)) {
            const uint32_t flags = row_value<i>(cur.flags);
            const uint32_t lo = row_value<i>(cur.lo), pl = prev_lo();
            const bool moved = lo - 1 + ((J + 1 - lo) & 15u) != pl + ((J - pl) & 15u);
            if (moved && (flags & kRowJump)) V = kOut;
            if (flags & kRowStart) {          // so that L = C
                V = 0;
                m = 0;
#pragma unroll
                for (int c = 0; c < NR; ++c) Wp[c] = 0;
            }
        }
        const uint32_t side = V + P1;
        const uint32_t nbr = min(row_prev(side), row_next(side));
        const uint32_t t = min(min(V, nbr), m + P2);
        const uint32_t L = t + (cost - m);
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)L, ro, ad, 0, 0);   // or nowhere
        uint32_t Vn = L, rmin = L;
        uint32_t next = A[i];
        if (__builtin_expect(busy & bit, 0)) {
          if (cur.wide & bit) {
            const uint32_t flags = row_value<i>(cur.flags);
            if (flags & kRowWide) {
                const uint32_t offb = row_value<i>(cur.offb), lo = row_value<i>(cur.lo);
                const uint32_t w = row_value<i>(cur.hi) - lo;
                // the previous path costs from this window's first hypothesis on, and
                // the one before it (at the start of a path: zeros)
                uint32_t below = 0xFFFF0000u;
                if (__builtin_expect(cur.conv & bit, 0) && (flags & kRowConv)) {
                    const bool pw = (flags & kRowAfterWide) != 0;
                    const uint32_t pl = prev_lo();
                    uint32_t* const own = (uint32_t*)(lrow + PAD + 2 * NR * j);
#pragma unroll
                    for (int c = 0; c < NR; ++c) own[c] = pw ? Wp[c] : ~0u;
                    lds_order();
                    if (!pw && V < 0x10000u) lrow[PAD + ((J - pl) & 15u)] = (uint16_t)V;
                    lds_order();
                    const int d = clampi((int)lo - (int)pl, 1 - PAD, PAD - 1);
                    __builtin_memcpy(Wp, lrow + PAD + d + 2 * NR * j, 4 * NR);
                    below = (uint32_t)lrow[PAD + d - 1] << 16;
                    lds_order();
                }
                const uint32_t P11 = P1 | P1 << 16, mP2 = m + P2;
                const uint32_t m2 = mP2 | mP2 << 16, mm2 = m | m << 16;
                uint32_t Xw[NR], nb[NR + 1];
#pragma unroll
                for (int c = 0; c < NR; ++c) Xw[c] = pk_add_sat(Wp[c], P11);
                nb[0] = pk_next(dpp<0x111>(pk_add_sat(below, P11), Xw[NR - 1]), Xw[0]);
#pragma unroll
                for (int c = 1; c < NR; ++c) nb[c] = pk_next(Xw[c - 1], Xw[c]);
                nb[NR] = pk_next(Xw[NR - 1], dpp<0x101>(~0u, Xw[0]));
                const uint32_t shift = (offb & 2u) * 8;
                uint32_t out[NR], wm = ~0u;
#pragma unroll
                for (int c = 0; c < NR; ++c) out[c] = MF[c];
                const bool part = __builtin_expect((cur.part & bit) != 0, 0);
                if (part) {
#pragma unroll
                    for (int c = 0; c < NR; ++c) {
                        const uint32_t k = 2 * NR * J + 2 * c;
                        out[c] = (k <= w ? 0u : 0xFFFFu) | (k + 1 <= w ? 0u : 0xFFFF0000u);
                    }
                }
#pragma unroll
                for (int c = 0; c < NR; ++c) {
                    const uint32_t cw = __builtin_amdgcn_alignbit(CW[i % DW][c + 1],
                                                                  CW[i % DW][c], shift);
                    const uint32_t tt = pk_min(pk_min(Wp[c], m2), pk_min(nb[c], nb[c + 1]));
                    Wp[c] = pk_add(tt, pk_sub(cw, mm2)) | out[c];
                    wm = pk_min(wm, Wp[c]);
                }
                rmin = min(wm & 0xFFFFu, wm >> 16);
                // 2 NR cells per lane, the last lane's in pieces of 8, 4, 2, 1; of how
                // many cells is wave-uniform unless some row is not at its full range
                const uint32_t to = offb + 4 * NR * J;
                auto store_cells = [&](int left, int last) {
                    if (left >= 2 * NR) {
                        if constexpr (NR == 2) {
                            __builtin_amdgcn_raw_buffer_store_b64(u32x2{Wp[0], Wp[1]}, ro, to, 0,
                                                                  0);
                        } else {
#pragma unroll
                            for (int c = 0; c < NR; c += 4)
                                __builtin_amdgcn_raw_buffer_store_b128(
                                    u32x4{Wp[c], Wp[c + 1], Wp[c + 2], Wp[c + 3]}, ro, to, 4 * c,
                                    0);
                        }
                    }
                    const bool end = left > 0 && left < 2 * NR;
                    uint32_t v[NR], at = to;
#pragma unroll
                    for (int e = 0; e < NR; ++e) v[e] = Wp[e];
                    static_for<NR == 8 ? 3 : NR == 4 ? 2 : 1>([&](auto h) {
                        constexpr int n = (NR >> 1) >> decltype(h)::value;    // registers
                        if (last & (2 * n)) {
                            if (end) {
                                if constexpr (n == 4)
                                    __builtin_amdgcn_raw_buffer_store_b128(
                                        u32x4{v[0], v[1], v[2], v[3]}, ro, at, 0, 0);
                                else if constexpr (n == 2)
                                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{v[0], v[1]}, ro,
                                                                          at, 0, 0);
                                else
                                    __builtin_amdgcn_raw_buffer_store_b32(v[0], ro, at, 0, 0);
                            }
                            at += 4 * n;
#pragma unroll
                            for (int e = 0; e < n; ++e) v[e] = v[e + n];
                        }
                    });
                    if (last & 1)
                        if (end)
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)v[0], ro, at, 0, 0);
                };
                if (part) store_cells((int)w + 1 - 2 * NR * j, (int)w + 1 - 2 * NR * j);
                else store_cells(N - 2 * NR * j, N);
                if (__builtin_expect(cur.leave & bit, 0)) {   // a row's next pixel is narrow
                    const uint32_t nl = row_value<(i + 1) % B>(i + 1 < B ? cur.lo : nxt.lo);
                    uint32_t* const own = (uint32_t*)(lrow + PAD + 2 * NR * j);
#pragma unroll
                    for (int c = 0; c < NR; ++c) own[c] = Wp[c];
                    lds_order();
                    // hypotheses lo' - 1 .. lo' + 14 of the next window
                    const int d = (int)(nl - 1 + ((J + 1 - nl) & 15u) - lo);
                    Vn = lrow[PAD + clampi(d, -PAD, 2 * PAD - 1)];
                    lds_order();
                }
            }
          }
          if (nxt.wide & bit) next = spread(nxt, ic, next);
          const RowsMeta& ahead = i + DW < B ? cur : nxt;
          if (ahead.wide & (1u << (i + DW) % B))
              fetch_wide(ahead, std::integral_constant<int, (i + DW) % B>(),
                         std::integral_constant<int, i % DW>());
        }
        C[i] = __builtin_amdgcn_raw_buffer_load_b16(rc, next, 0, 0);
        V = Vn;
        m = row_min(rmin);
    };
    for (int base = 0; base < steps; base += B) {
        // steps that are at a wide pixel or prefetch for one
        const uint32_t busy = cur.wide | nxt.wide | cur.wide >> DW | nxt.wide << (B - DW);
        static_for<B>([&](auto ic) {
            step(ic, busy);
        });
        last_lo = row_value<B - 1>(cur.lo);
        cur = nxt;
        nxt = decode(raw, cur);
        raw = load_raw();
    }
}

__device__ __forceinline__ bool rows_suit(const RowsArgs& a) {
    const int16_t* __restrict__ plo = a.lo;
    const int16_t* __restrict__ phi = a.hi;
    const uint32_t HW = (uint32_t)a.H * a.W;
    int16_t lo[4][4], hi[4][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // multiples of the golden section: even over the image, whatever its width
        const uint32_t i = ((threadIdx.x & 63) + 64 * e) * 2654435769u;
        const uint32_t p = 4 * (uint32_t)(((uint64_t)i * (HW / 4)) >> 32);
        __builtin_memcpy(lo[e], plo + p, 8);
        __builtin_memcpy(hi[e], phi + p, 8);
    }
    const int64_t cells = min(a.off[HW], (int64_t)a.dir_stride);
    int part = 0, full = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        bool some = false, all = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int l = clampi(lo[e][q], 0, a.N - 1), h = clampi(hi[e][q], l, a.N - 1);
            const bool wide = h - l >= kRowsNarrow, whole = h - l == a.N - 1;
            some |= wide && !whole;
            all |= wide && whole;
        }
        part += __popcll(__builtin_amdgcn_ballot_w64(some));
        full += __popcll(__builtin_amdgcn_ballot_w64(all && !some));
    }
    return (float)part + a.choice.full * (float)full <=
           256.0f * (a.choice.limit + a.choice.slope * ((float)cells / (float)HW));
}

template <class Src, int NR>
__global__ __launch_bounds__(64 * kWavesPerBlock, NR <= 4 ? 4 : 2) void sgm_bounded_rows_kernel(Src src) {
    __shared__ __align__(16) uint16_t lds[kWavesPerBlock * 4 * kRowsLds<NR>];
    uint32_t b;
    const RowsArgs& a = member(src, blockIdx.x, b);
    if (a.choice.on && !rows_suit(a)) {               // uniform
        for (uint32_t p = b * 256 + threadIdx.x; p < (uint32_t)a.H * a.W; p += a.nblk * 256)
            a.meta[p] = pix_meta(a.off[p], a.lo[p], a.hi[p], a.N);
        return;
    }
    if (b == 0 && threadIdx.x == 0) a.meta[0].rows = 1;
    const int wv = threadIdx.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(b * kWavesPerBlock + wv);
    if (w >= a.wbase[kMaxPaths]) return;              // wave-uniform
    bounded_rows_wave<NR>(a, w, lds + wv * 4 * kRowsLds<NR>);
}

// csum[c] = sum_r Lbuf[r][c] over the cells of the CSR volume; each of a light
// field's nblk workgroups strides over its device-side cell count.
struct BsumArgs {
    gptr<const uint16_t> Lbuf;     // [npaths][dir_stride]
    size_t dir_stride;
    gptr<const int64_t> total;     // device-side cell count
    gptr<void> csum;
    uint32_t nblk;
};

template <class Src, typename SumT, int kPaths>
__global__ __launch_bounds__(256) void bounded_sum_kernel(Src src) {
    for (uint32_t vb = blockIdx.x; vb < src.total; vb += gridDim.x) {
        uint32_t b;
        const BsumArgs& a = member(src, vb, b);
        // the device-side count, never past the buffers (offsets that are not the
        // prefix sum of in-range widths would otherwise run past them)
        const int64_t n = min(*a.total, (int64_t)a.dir_stride);
        const uint16_t* __restrict__ L = a.Lbuf;
        SumT* __restrict__ csum = (SumT*)a.csum;
        for (int64_t c = (int64_t)b * 256 + threadIdx.x; c < n; c += (int64_t)a.nblk * 256) {
            uint32_t x[kPaths];
#pragma unroll
            for (int r = 0; r < kPaths; ++r)
                x[r] = __builtin_nontemporal_load(L + (size_t)r * a.dir_stride + c);
            uint32_t s = 0;
#pragma unroll
            for (int r = 0; r < kPaths; ++r) s += x[r];
            csum[c] = (SumT)s;
        }
    }
}

// --- host-side dispatch of the kernel variants ---------------------------------
template <int K, typename LT, bool kPad>
hipError_t dense_variant(Runner& r, const std::vector<DenseArgs>& args,
                         const std::vector<uint32_t>& blocks) {
    switch (r.tune.dense_depth) {
        case 4:
            return launch(r, kStInitPaths, sgm_dense_paths_kernel<Single<DenseArgs>, K, LT, 4, kPad>,
                          sgm_dense_paths_kernel<Group<DenseArgs>, K, LT, 4, kPad>, args, blocks,
                          64 * kWavesPerBlock);
        case 16:
            return launch(r, kStInitPaths, sgm_dense_paths_kernel<Single<DenseArgs>, K, LT, 16, kPad>,
                          sgm_dense_paths_kernel<Group<DenseArgs>, K, LT, 16, kPad>, args, blocks,
                          64 * kWavesPerBlock);
        default:
            return launch(r, kStInitPaths, sgm_dense_paths_kernel<Single<DenseArgs>, K, LT, 8, kPad>,
                          sgm_dense_paths_kernel<Group<DenseArgs>, K, LT, 8, kPad>, args, blocks,
                          64 * kWavesPerBlock);
    }
}

// v: 0 8-bit path costs, 1 16-bit, 2 8-bit with the padded rows standing in for
// kInf (K = 2 only: up to 64 hypotheses take four lines per wave)
hipError_t dense_k(Runner& r, int K, int v, const std::vector<DenseArgs>& args,
                   const std::vector<uint32_t>& blocks) {
    if (v == 2) return dense_variant<2, uint8_t, true>(r, args, blocks);
    if (v == 1) {
        switch (K) {
            case 1: return dense_variant<1, uint16_t, false>(r, args, blocks);
            case 2: return dense_variant<2, uint16_t, false>(r, args, blocks);
            case 3: return dense_variant<3, uint16_t, false>(r, args, blocks);
            default: return dense_variant<4, uint16_t, false>(r, args, blocks);
        }
    }
    switch (K) {
        case 1: return dense_variant<1, uint8_t, false>(r, args, blocks);
        case 2: return dense_variant<2, uint8_t, false>(r, args, blocks);
        case 3: return dense_variant<3, uint8_t, false>(r, args, blocks);
        default: return dense_variant<4, uint8_t, false>(r, args, blocks);
    }
}

template <int K, int D>
hipError_t bounded_depth_variant(Runner& r, const std::vector<BoundedArgs>& args,
                                 const std::vector<uint32_t>& blocks, bool buf) {
    if (buf)
        return launch(r, kStSgmFinal, sgm_bounded_paths_kernel<Single<BoundedArgs>, K, D, true>,
                      sgm_bounded_paths_kernel<Group<BoundedArgs>, K, D, true>, args, blocks,
                      64 * kWavesPerBlock);
    return launch(r, kStSgmFinal, sgm_bounded_paths_kernel<Single<BoundedArgs>, K, D, false>,
                  sgm_bounded_paths_kernel<Group<BoundedArgs>, K, D, false>, args, blocks,
                  64 * kWavesPerBlock);
}

template <int K>
hipError_t bounded_variant(Runner& r, const std::vector<BoundedArgs>& args,
                           const std::vector<uint32_t>& blocks) {
    // 32-bit buffer offsets when every volume of the launch is below 2^31 bytes
    bool buf = r.tune.bounded_offsets == 32;
    for (const BoundedArgs& a : args)
        buf = buf && (a.dir_stride + a.N) * 2 <= (size_t)INT32_MAX &&
              (size_t)a.H * a.W * sizeof(PixMeta) <= (size_t)INT32_MAX;
    const int d = r.tune.bounded_depth;
    if (d == 4) return bounded_depth_variant<K, 4>(r, args, blocks, buf);
    if (d == 8) return bounded_depth_variant<K, 8>(r, args, blocks, buf);
    return bounded_depth_variant<K, 16>(r, args, blocks, buf);
}

template <int NR>
hipError_t bounded_rows(Runner& r, const std::vector<RowsArgs>& args) {
    std::vector<uint32_t> blocks;
    for (const RowsArgs& a : args) blocks.push_back(a.nblk);
    return launch(r, kStSgmFinal, sgm_bounded_rows_kernel<Single<RowsArgs>, NR>,
                  sgm_bounded_rows_kernel<Group<RowsArgs>, NR>, args, blocks,
                  64 * kWavesPerBlock);
}

template <int NR>
hipError_t dense_rows(Runner& r, const std::vector<DenseRowsArgs>& args) {
    std::vector<uint32_t> blocks;
    for (const DenseRowsArgs& a : args) blocks.push_back(a.wblocks * a.nv);
    return launch(r, kStInitPaths, sgm_dense_rows_kernel<Single<DenseRowsArgs>, NR>,
                  sgm_dense_rows_kernel<Group<DenseRowsArgs>, NR>, args, blocks,
                  64 * kWavesPerBlock);
}

hipError_t bounded_k(Runner& r, int K, const std::vector<BoundedArgs>& args,
                     const std::vector<uint32_t>& blocks) {
    switch (K) {
        case 1: return bounded_variant<1>(r, args, blocks);
        case 2: return bounded_variant<2>(r, args, blocks);
        case 3: return bounded_variant<3>(r, args, blocks);
        default: return bounded_variant<4>(r, args, blocks);
    }
}


// Which bounded SGM kernel: four lines per wave, one, or (both set) the four-line kernel
// with the choice, and the other after it.
struct Form {
    bool rows, one;
    RowsChoice choice;
};

// A step of four lines costs the GPU less than half of what four steps of one do, but takes
// about twice as long as one of those (every pixel of a wave waits for its widest), so it
// needs lines enough beside the longest one: all path steps over the steps of the longest
// line (`many`).  Bounded paths in us, one line per wave against four, 12 % full-range
// pixels: 512x512, N = 100 on the benchmark bounds (4,096) 199 / 219; 640x640 (5,120) 299 /
// 202; 512x512 with 16 paths (8,192) 382 / 254; 1080x1920, N = 96 (8,640) 1468 / 664.
// Beyond 128 hypotheses a lane of the one-line form holds three or four: N = 200, 256x256
// (2,048) 94 / 95, 384x384 (3,072) 190 / 141, 375x450 with 16 paths 458 / 181.
//
// With windows of 15 hypotheses and more nearly every step of four lines is a wide one.
// Call of lf_sgm_aggregate in us, one line against four, windows of 15 everywhere: 640x640,
// N = 64 229 / 440, N = 96 334 / 562; 900x1000 (7,200) 601 / 645, 743 / 812; 1300x1300
// (10,400), N = 96 1303 / 1402, 1500x1500 (12,000) 1677 / 1631; 640x640, N = 140 410 / 767,
// N = 200 482 / 770; 600x640 with 16 paths (9,600), N = 200 871 / 815; 1080x1920, N = 140
// 1867 / 2364.  Windows of 33: 640x640, N = 64 261 / 460; 1080x1920 1828 / 1538.  Full
// ranges everywhere: 640x640, N = 16 230 / 344, N = 64 350 / 420, N = 96 602 / 551; 800x800
// (6,400), N = 16 497 / 432.  So between the sizes where four lines never pay and those
// where they always do, the ranges decide (RowsChoice; lines fitted to these times and to
// those of windows of 21, 64 and N and of 7 with a tenth to three quarters of full ranges,
// at the same sizes: at most 3 % above the better form, 1 to 5 us of them the choice).
Form bounded_form(const Tuning& tune, int N, bool full_range, uint64_t many) {
    const int c = (N - 1) / 64;
    constexpr uint64_t sure[4] = {11000, 11000, 16000, 9000};
    if (tune.bounded_lanes) return {tune.bounded_lanes < 64, tune.bounded_lanes == 64, {}};
    if ((many > 4500 && N <= kRowsNarrow) || many > sure[c]) return {true, false, {}};
    if (many <= (N > 128 ? 2300 : 4500)) return {false, true, {}};
    constexpr float limit[3][4] = {{0.30f, 0.34f, 0.20f, 0.54f},
                                   {0.73f, 0.60f, 0.60f, 0.78f},
                                   {0.74f, 0.74f, 0.60f, 0.78f}};
    constexpr float slope[3][4] = {{0.0048f, 0.0080f, 0.0041f, 0.0043f},
                                   {0.0080f, 0.0105f, 0.0065f, 0.0070f},
                                   {0.0125f, 0.0125f, 0.0065f, 0.0070f}};
    const int more = many >= 8500 ? 2 : many >= 6000 ? 1 : 0;
    RowsChoice ch{1, limit[more][c], slope[more][c],
                  N > 128 ? 0.45f + 0.0032f * N : 0.6f + 0.005f * N};
    if (!full_range) return {true, true, ch};
    const bool rows = ch.full <= ch.limit + ch.slope * N;
    return {rows, !rows, {}};
}

// The path steps of some light fields.  Those with up to 128 hypotheses count, and run,
// together: a launch takes its longest line's time at least (six light fields, N = 33 .. 96,
// of 89x197 to 317x414: 336 us by two launches of one line per wave, 411 us by two of four,
// 263 us by one of four).
struct BoundedLines {
    uint64_t steps[2] = {0, 0}, longest[2] = {1, 1};  // up to 128 hypotheses, more
    int widest = 0;                                   // of the former
    explicit BoundedLines(const Jobs& jobs) {
        for (const Job* j : jobs) {
            const int big = j->N > 128;
            steps[big] += (uint64_t)j->H * j->W * j->prm.sgm_final.npaths;
            longest[big] = std::max(longest[big], (uint64_t)std::max(j->H, j->W));
            if (!big) widest = std::max(widest, j->N);
        }
    }
    uint64_t many(int N) const { return steps[N > 128] / longest[N > 128]; }
};

}  // namespace

int dense_np(int N) { return (N + 3) / 4 * 4; }

// Row stride (elements) of the initial path costs: rows longer than 64 bytes
// take whole 128-byte cache lines, so that the path kernel's non-temporal
// copy-out writes full lines; shorter ones stay packed (4-byte multiples).
int dense_lnp(int N, int elem_bytes) {
    const int rb = dense_np(N) * elem_bytes;
    return rb <= 64 ? dense_np(N) : (rb + 127) / 128 * 128 / elem_bytes;
}

// Row stride of the initial Census cost volume: room for two bytes of 255 after
// the N costs (hypotheses past N read them), within the 256-byte LDS tile rows.
int dense_cvol_np(int N) { return min(dense_np(N + 2), LF_MAX_HYPOTHESES); }

size_t sgm_dense_scratch_bytes(int nv, int H, int W, int N, int npaths, int bits, int P2) {
    const size_t lt = bits + P2 <= 255 ? 1 : 2;
    const size_t cv = round256((size_t)nv * H * W * dense_cvol_np(N));
    // + 256: the row-wise sum reads up to 128 bytes past the last pixel's row
    return cv + (size_t)npaths * nv * H * W * dense_lnp(N, (int)lt) * lt + 256;
}

size_t sgm_bounded_scratch_bytes(int H, int W, int N, int npaths) {
    const size_t meta = round256((size_t)H * W * sizeof(PixMeta));
    return meta + (size_t)npaths * H * W * N * sizeof(uint16_t);
}

namespace {

// Four lines per wave, or one (8-bit path costs with the bound of kPad; paths in us, one
// line against four).  Up to 64 hypotheses four are the faster at nearly every size tried:
// 4 views of 512x512, N = 40, 256 / 147, of 96x96, N = 32, 24 / 18; 2 of 24x1900, N = 60,
// 196 / 189, of 1080x1920, N = 64, 1259 / 902 (but 500x2000 with 16 paths 928 / 1092).  With
// more, a step of a line takes longer than in the one-line form, so there have to be lines
// enough beside the longest one, counted as all path steps over that one's: 32x400, 16
// paths, N = 128 (2,048) 76 / 76; 128x128, N = 100 (4,096) 35 / 23; 512x512, N = 100, 313 /
// 281.  With 2 views and 8 paths the longest lines of a thin image are left alone all the
// same: 200x600 98 / 96, 200x700 105 / 120, 275x1650 297 / 361.  And as the lines of all
// directions are walked at once, the Census costs have to stay in the 256 MB cache beside
// the path costs: 256x1024, N = 65 (71 MB) 312 / 252; 2 views of 600x1000, N = 100 (125 MB)
// 395 / 375, of 720x1280, N = 96 (181 MB) 554 / 551, of 1080x1920 (415 MB) 1366 / 1451; 4 of
// 1080x1080, N = 80 (392 MB) 1543 / 1533.
struct DenseLines {
    uint64_t steps = 0, longest = 1;               // of those with more than 64 hypotheses
    static bool fits(const Job* j) {
        const int bits = j->C * census_bits(j->prm.census);
        const int np = std::max(dense_cvol_np(j->N), dense_lnp(j->N, 1));
        const int64_t HW = (int64_t)j->H * j->W;
        const bool thin = std::max(j->H, j->W) > 3 * std::min(j->H, j->W) &&
                          j->nv * j->prm.sgm_init.npaths < 32;
        return j->N <= 128 && bits + j->prm.sgm_init.P2 <= 255 &&
               bits + 2 * j->prm.sgm_init.P2 <= 255 + j->prm.sgm_init.P1 &&
               HW * np <= (int64_t)kRowsVolume &&
               (j->N <= 64 ||
                (!thin && j->nv * HW * dense_cvol_np(j->N) <= (int64_t)128 << 20));
    }
    explicit DenseLines(const Jobs& jobs) {
        for (const Job* j : jobs)
            if (j->N > 64 && fits(j)) {
                steps += (uint64_t)j->nv * j->H * j->W * j->prm.sgm_init.npaths;
                longest = std::max(longest, (uint64_t)std::max(j->H, j->W));
            }
    }
    bool four(const Job* j) const { return fits(j) && (j->N <= 64 || steps > 2048 * longest); }
};

}  // namespace

bool uses_dense_depth(const Jobs& jobs) {
    Jobs bounded;                                  // the others have no initial stage
    for (const Job* j : jobs)
        if (j->prm.lambda >= 0) bounded.push_back(j);
    const DenseLines lines(bounded);
    return std::any_of(bounded.begin(), bounded.end(),
                       [&](const Job* j) { return !lines.four(j); });
}

int default_bounded_lanes(const Jobs& jobs) {
    const BoundedLines lines(jobs);
    bool rows = true, one = true;
    for (const Job* j : jobs) {
        const Form f = bounded_form(Tuning{}, j->N, j->full_range, lines.many(j->N));
        rows &= !f.one;
        one &= !f.rows;
    }
    return rows ? 16 : one ? 64 : 0;
}

hipError_t stage_sgm_initial(Runner& r, const Jobs& jobs, int part) {
    std::vector<CcvArgs> ccv[2];                   // [gray/colour]
    std::vector<uint32_t> ccv_blocks[2];
    // variants: K in 1..4 x (8-bit, 16-bit, 8-bit with padded rows)
    std::vector<DenseArgs> dense[4][3];
    std::vector<uint32_t> dense_blocks[4][3];
    std::vector<DenseRowsArgs> drows[2];           // up to 64, 128 hypotheses
    std::vector<SumWtaArgs> sums[2][2];            // [8/16-bit path costs][8/16 paths]
    std::vector<uint32_t> sum_blocks[2][2];
    std::vector<SumWtaArgs> rows[2];               // 8-bit rows <= 128 B: [8/16 paths]
    std::vector<uint32_t> row_blocks[2];
    std::vector<ExportArgs> ex_cost, ex_sum;       // outputs for checking
    std::vector<uint32_t> ex_cost_blocks, ex_sum_blocks;
    const DenseLines lines(jobs);
    for (const Job* j : jobs) {
        const int H = j->H, W = j->W, N = j->N, NPc = dense_cvol_np(N);
        const size_t HW = (size_t)H * W;
        const lf_sgm_params& sp = j->prm.sgm_init;
        const int bits = j->C * census_bits(j->prm.census);
        const int lt = bits + sp.P2 <= 255 ? 0 : 1;
        const int NP = dense_lnp(N, 1 << lt);
        uint8_t* cvol = (uint8_t*)j->paths;
        void* Lbuf = (char*)j->paths + round256((size_t)j->nv * HW * NPc);
        const int sh = (j->S - 1) / 2, th = (j->T - 1) / 2;

        CcvArgs c{};
        c.cref = j->census;
        c.cview = j->census + (size_t)j->C * HW;
        c.hyp = j->hyp;
        for (int i = 0; i < j->nv; ++i) {
            c.cs4 |= (uint64_t)(uint16_t)(int16_t)(sh - j->st[2 * i]) << (16 * i);
            c.ct4 |= (uint64_t)(uint16_t)(int16_t)(th - j->st[2 * i + 1]) << (16 * i);
        }
        c.nv = j->nv;
        c.H = H;
        c.W = W;
        c.N = N;
        c.NP = NPc;
        c.tiles = div_up(HW, kTilePix);
        c.cvol = cvol;
        const int col = j->C == 3 ? 1 : 0;
        ccv[col].push_back(c);
        ccv_blocks[col].push_back(c.tiles * j->nv);

        DenseArgs d{};
        d.cvol = cvol;
        d.Lbuf = Lbuf;
        d.lines = make_lines(H, W, sp.npaths);
        d.nv = j->nv;
        d.H = H;
        d.W = W;
        d.N = N;
        d.NP = NP;
        d.NPc = NPc;
        d.P1 = (uint32_t)sp.P1;
        d.P2 = (uint32_t)sp.P2;
        d.units = make_units(d.lines, H, W);
        d.wblocks = div_up(d.units.nunits, kWavesPerBlock);
        const int K = (N + 63) / 64 - 1;
        const int v = lt == 0 && K <= 1 && bits + 2 * sp.P2 <= 255 + sp.P1 ? 2 : lt;
        if (lines.four(j)) {
            DenseRowsArgs w{};
            w.cvol = cvol;
            w.Lbuf = (uint8_t*)Lbuf;
            w.nv = j->nv;
            w.H = H;
            w.W = W;
            w.N = N;
            w.NP = NP;
            w.NPc = NPc;
            w.P1 = d.P1;
            w.P2 = d.P2;
            w.npaths = sp.npaths;
            rows_waves(H, W, sp.npaths, w.wbase);
            w.wblocks = div_up(w.wbase[kMaxPaths], kWavesPerBlock);
            drows[K].push_back(w);
        } else {
            dense[K][v].push_back(d);
            dense_blocks[K][v].push_back(d.wblocks * j->nv);
        }

        SumWtaArgs s{};
        s.Lbuf = Lbuf;
        s.HW = (int64_t)HW;
        s.nv = j->nv;
        s.N = N;
        s.NP = NP;
        s.dmap = j->maps;
        const uint32_t ex_blocks = div_up((uint64_t)j->nv * HW * N, 256);
        if (j->ccv_out) {
            ex_cost.push_back(ExportArgs{cvol, j->ccv_out, (int64_t)(j->nv * HW), N, NPc,
                                         sp.npaths, 1});
            ex_cost_blocks.push_back(ex_blocks);
        }
        if (j->csum_init_out) {
            ex_sum.push_back(ExportArgs{Lbuf, j->csum_init_out, (int64_t)(j->nv * HW), N, NP,
                                        sp.npaths, 1 << lt});
            ex_sum_blocks.push_back(ex_blocks);
        }
        const int np16 = sp.npaths == 16 ? 1 : 0;
        if (lt == 0 && NP <= 128) {
            rows[np16].push_back(s);
            row_blocks[np16].push_back(div_up((uint64_t)j->nv * HW, 16));
        } else {
            sums[lt][np16].push_back(s);
            sum_blocks[lt][np16].push_back(div_up((uint64_t)j->nv * HW, 4));
        }
    }
    hipError_t e = hipSuccess;
    using EA = ExportArgs;
    if (part == 0) {
        if (!ccv[0].empty())
            e = launch(r, kStInitCost, census_cost_volume_kernel<Single<CcvArgs>, 1>,
                       census_cost_volume_kernel<Group<CcvArgs>, 1>, ccv[0], ccv_blocks[0], 256);
        if (e == hipSuccess && !ccv[1].empty())
            e = launch(r, kStInitCost, census_cost_volume_kernel<Single<CcvArgs>, 3>,
                       census_cost_volume_kernel<Group<CcvArgs>, 3>, ccv[1], ccv_blocks[1], 256);
        if (e == hipSuccess && !ex_cost.empty())
            e = launch(r, kStInitCost, initial_export_kernel<Single<EA>, false>,
                       initial_export_kernel<Group<EA>, false>, ex_cost, ex_cost_blocks, 256);
        return e;
    }
    if (part == 2 && !ex_sum.empty() &&
        (e = launch(r, kStInitSum, initial_export_kernel<Single<EA>, true>,
                    initial_export_kernel<Group<EA>, true>, ex_sum, ex_sum_blocks, 256)) !=
            hipSuccess)
        return e;
    if (part == 1) {
        for (int K = 0; K < 4; ++K)
            for (int v = 0; v < 3; ++v) {
                if (dense[K][v].empty()) continue;
                if ((e = dense_k(r, K + 1, v, dense[K][v], dense_blocks[K][v])) != hipSuccess)
                    return e;
            }
        if (!drows[0].empty() && (e = dense_rows<2>(r, drows[0])) != hipSuccess) return e;
        if (!drows[1].empty() && (e = dense_rows<4>(r, drows[1])) != hipSuccess) return e;
        return hipSuccess;
    }
    // the row-wise sums: one workgroup per 16 pixels (measured faster than
    // persistent workgroups); the others: persistent, each workgroup walks pixels
    constexpr uint32_t kSumGrid = 8192;
    using SA = SumWtaArgs;
    if (!rows[0].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_rows_kernel<Single<SA>, 8>,
                    dense_sum_wta_rows_kernel<Group<SA>, 8>, rows[0], row_blocks[0], 256)) !=
            hipSuccess)
        return e;
    if (!rows[1].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_rows_kernel<Single<SA>, 16>,
                    dense_sum_wta_rows_kernel<Group<SA>, 16>, rows[1], row_blocks[1], 256)) !=
            hipSuccess)
        return e;
    if (!sums[0][0].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_kernel<Single<SA>, uint8_t, 8>,
                    dense_sum_wta_kernel<Group<SA>, uint8_t, 8>, sums[0][0], sum_blocks[0][0],
                    256, kSumGrid)) != hipSuccess)
        return e;
    if (!sums[1][0].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_kernel<Single<SA>, uint16_t, 8>,
                    dense_sum_wta_kernel<Group<SA>, uint16_t, 8>, sums[1][0], sum_blocks[1][0],
                    256, kSumGrid)) != hipSuccess)
        return e;
    if (!sums[0][1].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_kernel<Single<SA>, uint8_t, 16>,
                    dense_sum_wta_kernel<Group<SA>, uint8_t, 16>, sums[0][1], sum_blocks[0][1],
                    256, kSumGrid)) != hipSuccess)
        return e;
    if (!sums[1][1].empty() &&
        (e = launch(r, kStInitSum, dense_sum_wta_kernel<Single<SA>, uint16_t, 16>,
                    dense_sum_wta_kernel<Group<SA>, uint16_t, 16>, sums[1][1], sum_blocks[1][1],
                    256, kSumGrid)) != hipSuccess)
        return e;
    return hipSuccess;
}

hipError_t stage_sgm_final(Runner& r, const Jobs& jobs) {
    std::vector<MetaArgs> meta;
    std::vector<uint32_t> meta_blocks;
    std::vector<BoundedArgs> paths[4];
    std::vector<uint32_t> path_blocks[4];
    std::vector<RowsArgs> rows[3];                 // up to 64, 128, 256 hypotheses
    std::vector<BsumArgs> sums[2][2];              // [16/32-bit sums][8/16 paths]
    std::vector<uint32_t> sum_blocks[2][2];
    const BoundedLines lines(jobs);
    for (const Job* j : jobs) {
        const int H = j->H, W = j->W, N = j->N;
        const size_t HW = (size_t)H * W;
        const lf_sgm_params& sp = j->prm.sgm_final;
        PixMeta* pm = (PixMeta*)j->sgm_ws;
        uint16_t* Lbuf = (uint16_t*)((char*)j->sgm_ws + round256(HW * sizeof(PixMeta)));
        const size_t dir_stride = HW * N;          // worst-case cells per direction

        const int big = N > 128;
        Form form = bounded_form(r.tune, N, j->full_range, lines.many(N));
        if (r.tune.bounded_offsets != 32 || dir_stride * 2 + 4 > (size_t)INT32_MAX)
            form.one = true, form.rows = false;
        if (form.rows) {
            RowsArgs w{};
            w.cost = j->cost;
            w.off = j->offsets;
            w.lo = j->lo;
            w.hi = j->hi;
            w.Lbuf = Lbuf;
            w.dir_stride = dir_stride;
            w.H = H;
            w.W = W;
            w.N = N;
            w.P1 = (uint32_t)sp.P1;
            w.P2 = (uint32_t)sp.P2;
            w.npaths = sp.npaths;
            rows_waves(H, W, sp.npaths, w.wbase);
            w.meta = pm;
            w.nblk = div_up(w.wbase[kMaxPaths], kWavesPerBlock);
            w.choice = form.choice;
            rows[big ? 2 : lines.widest <= 64 ? 0 : 1].push_back(w);
        } else {
            meta.push_back(MetaArgs{j->offsets, j->lo, j->hi, pm, (int)HW, N});
            meta_blocks.push_back(div_up(HW, 256));
        }
        if (form.one) {
            BoundedArgs b{};
            b.cost = j->cost;
            b.meta = pm;
            b.Lbuf = Lbuf;
            b.dir_stride = dir_stride;
            b.lines = make_lines(H, W, sp.npaths);
            b.units = make_units(b.lines, H, W);
            b.H = H;
            b.W = W;
            b.N = N;
            b.P1 = (uint32_t)sp.P1;
            b.P2 = (uint32_t)sp.P2;
            b.chosen = form.rows;
            const int K = (N + 63) / 64 - 1;
            paths[K].push_back(b);
            path_blocks[K].push_back(div_up(b.units.nunits, kWavesPerBlock));
        }

        BsumArgs s{};
        s.Lbuf = Lbuf;
        s.dir_stride = dir_stride;
        s.total = j->offsets + HW;
        s.csum = j->csum;
        s.nblk = std::min<uint32_t>(2048, std::max<uint32_t>(1, div_up(dir_stride, 4096)));
        const int sb = j->prm.sum_bits == 16 ? 0 : 1;
        const int np16 = sp.npaths == 16 ? 1 : 0;
        sums[sb][np16].push_back(s);
        sum_blocks[sb][np16].push_back(s.nblk);
    }
    hipError_t e = hipSuccess;
    if (!meta.empty() &&
        (e = launch(r, kStSgmFinal, pix_meta_kernel<Single<MetaArgs>>,
                    pix_meta_kernel<Group<MetaArgs>>, meta, meta_blocks, 256)) != hipSuccess)
        return e;
    if (!rows[0].empty() && (e = bounded_rows<2>(r, rows[0])) != hipSuccess) return e;
    if (!rows[1].empty() && (e = bounded_rows<4>(r, rows[1])) != hipSuccess) return e;
    if (!rows[2].empty() && (e = bounded_rows<8>(r, rows[2])) != hipSuccess) return e;
    for (int K = 0; K < 4; ++K) {
        if (paths[K].empty()) continue;
        e = bounded_k(r, K + 1, paths[K], path_blocks[K]);
        if (e != hipSuccess) return e;
    }
    using BA = BsumArgs;
    if (!sums[0][0].empty() &&
        (e = launch(r, kStSgmFinal, bounded_sum_kernel<Single<BA>, uint16_t, 8>,
                    bounded_sum_kernel<Group<BA>, uint16_t, 8>, sums[0][0], sum_blocks[0][0],
                    256)) != hipSuccess)
        return e;
    if (!sums[1][0].empty() &&
        (e = launch(r, kStSgmFinal, bounded_sum_kernel<Single<BA>, uint32_t, 8>,
                    bounded_sum_kernel<Group<BA>, uint32_t, 8>, sums[1][0], sum_blocks[1][0],
                    256)) != hipSuccess)
        return e;
    if (!sums[0][1].empty() &&
        (e = launch(r, kStSgmFinal, bounded_sum_kernel<Single<BA>, uint16_t, 16>,
                    bounded_sum_kernel<Group<BA>, uint16_t, 16>, sums[0][1], sum_blocks[0][1],
                    256)) != hipSuccess)
        return e;
    if (!sums[1][1].empty() &&
        (e = launch(r, kStSgmFinal, bounded_sum_kernel<Single<BA>, uint32_t, 16>,
                    bounded_sum_kernel<Group<BA>, uint32_t, 16>, sums[1][1], sum_blocks[1][1],
                    256)) != hipSuccess)
        return e;
    return hipSuccess;
}

}  // namespace lf
