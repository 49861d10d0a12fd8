// k_2d.hip -- the paper's two-dimensional Tsallis thresholding (Tsallis-
// entropy section, the 2D form): the 3x3 average image g = floor(mean of the
// 3x3 gray levels, edge pixels repeated), the 2D histogram h(i, j) of
// (gray level, average gray level), the classes {i <= t, j <= s} and
// {i > t, j > s} (quadrants 1 and 3) and the arg max over (t, s) of the
// pseudo-additive objective.  Only t thresholds the image (ts_label, k = 1).
//
// k_hist2d: one workgroup per CU; each counts whole images and stores their
// planes, and the images left over are split into parts by rows, which add to
// theirs.  Small images take smaller workgroups, several per CU, an image each.
// The whole L x L plane is counted in LDS as 16-bit cells (two per word; 128 KiB
// at L = 256).  A lane holds 8 neighbouring columns and walks down the rows:
// gray levels, row sums of three and the sums of three rows stay in
// registers as packed 16-bit pairs, the neighbours' edge columns come by lane
// moves, and LDS sees nothing but one atomic per pixel.  Lanes whose 8 pixels
// all lie in a clamp corner ((0, 0) or (L-1, L-1), a large share of the pixels
// under a narrow window) count in a register instead of one hot address.
//
// k_search2d: one workgroup per (q index, problem); the rows holding counts
// are split into blocks, one per wavefront, four columns per lane.  Class 2
// sums are accumulated bottom-up over rows and class 1 sums top-down; a
// wavefront starts its block from the carried sums of the blocks before it in
// that direction (every block's column totals, added up over the blocks in
// both directions and summed along s, exchanged through LDS), so all walk
// their rows at once.  FP32 keys of every pair, then an FP64 re-check of the
// rows whose best key is within the keys' error bound of the maximum, from the
// same sums; the first best FP64 pair wins (t outermost).  Sums along s are
// fixed-order scans, and an empty cell (or an empty column of the totals)
// takes the sum of the last occupied one, so a whole empty column or row
// leaves every class sum unchanged bit for bit and the pairs it separates tie
// exactly.  q = 1 is the Shannon limit, as in the one-dimensional search.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace ts {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int H2_THREADS = 1024;
constexpr int H2_MAX_W = 4096;    // widest row
constexpr int H2_MAX_L = 256;     // 2D histograms up to 256 x 256
constexpr int H2_MIN_ROWS = 16;   // rows a workgroup takes at least
constexpr int H2_MIN_PIX = 4096;  // pixels of an image that is not split
constexpr int H2_SMALL = 16384;   // pixels of a small image
constexpr size_t H2_LDS = 160 * 1024;
constexpr int S2_CPL = 4;         // columns per lane (L <= 256)
constexpr int S2_TAB = 1024;      // p^q (or p ln p) of counts below this from an LDS table
constexpr int S2_RING = 2;        // rows of counts in flight ahead of the row being summed

// ------------------------------------------------------------------ histogram

// 8 pixels at any pixel address (gfx950 takes unaligned global loads)
typedef v4i v4i_any __attribute__((aligned(2)));

__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b));
}

// The pair (high half of a, low half of b): the window one pixel later.
__device__ __forceinline__ uint32_t pair_mid(uint32_t a, uint32_t b) { return __builtin_amdgcn_alignbit(b, a, 16); }

// Cross-lane moves within the wavefront (DPP): lanes without a source, or in
// rows masked off, receive 0, the identity of the sums below.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    // where every row takes part the move itself fills in the zeros
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, ROWS == 0xf);
}

// How the rows are laid over a workgroup: row groups of 1 << gsh lanes (8
// columns each), nch chunks of columns per row, nrun rows walked at once.
struct Hist2dShape {
    int gsh, nch, nrun;
};

// Words of the plane: word w holds cell w in its high half and the cell
// hist2d_words later in its low half, so that a wavefront's words are
// neighbouring cells twice.
__host__ __device__ inline int hist2d_words(int L) { return (L + 1) / 2 * L; }

// Bounded by its vector operations (24 per pixel, 51 when the gray levels were
// staged in LDS as bytes and summed one by one), then by adding up the planes:
// 300 images of 512 x 512 at 256 levels 214 -> 88 us (of 48 us of vector issue
// at one wavefront instruction per four clocks), 37 of 301 x 415 at 200 levels
// 53 -> 25 us, 120 residue images of 512 x 512 115 -> 48 us.  Before, 65535
// pixels were counted between two additions of a plane's cells to the cleared
// histogram, and one band of an image per workgroup left the last round of
// workgroups short.  A row loop that copied its loaded registers at the end
// waited there for the load: 99 us.
template <int KIND, bool RAGGED, int REPS>
__global__ void __launch_bounds__(H2_THREADS) k_hist2d(const int16_t *const *__restrict__ vox, int nseg, int whole,
                                                       int parts, int H, int W, Hist2dShape sh, BinMap bm, uint32_t mul24,
                                                       uint32_t *__restrict__ hist)
{
    // [REPS copies of the plane's words | two corner sums | the sweep's per-wavefront maxima]
    extern __shared__ uint32_t sm[];
    const int L = bm.L, nw2 = hist2d_words(L);
    uint32_t *plane = sm;
    const int nw4 = (nw2 + 3) & ~3; // the words past the plane stay 0
    uint4 *plane4 = reinterpret_cast<uint4 *>(sm);
    const int nall = nw4 * REPS;
    uint32_t *corner = plane + nall, *wmax = corner + 2;
    const int lane = threadIdx.x & 63;
    uint32_t *mine = plane + (lane & (REPS - 1)) * nw4; // the copy this lane counts into
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // this lane's row group: chunk of columns and run of rows
    const int grp = (wv << (6 - sh.gsh)) + (lane >> sh.gsh);
    const int chunk = grp % sh.nch, runid = grp / sh.nch; // runid >= nrun: idle (nch need not divide the groups)
    const int x0 = (chunk << (sh.gsh + 3)) + ((lane & ((1 << sh.gsh) - 1)) << 3);
    const int nv = runid < sh.nrun ? min(8, W - x0) : 0; // columns of this lane (<= 0: none)
    const bool at_left = x0 == 0, at_right = x0 + 8 >= W;
    const int xl = nv > 0 ? x0 : 0;                               // column this lane loads
    const bool g_first = (lane & ((1 << sh.gsh) - 1)) == 0, g_last = ((lane + 1) & ((1 << sh.gsh) - 1)) == 0;
    const int xe = min(max(g_first ? xl - 1 : xl + 8, 0), W - 1); // and beside its chunk (nch > 1)
    const int edge = (W - 1) & 7; // last column's place in its lane
    const int64_t npix = (int64_t)H * W;
    const u16x2 half2 = {(unsigned short)((L + 1) / 2), (unsigned short)((L + 1) / 2)};
    const uint32_t fmul = (uint32_t)L << 15, top = 9u * (uint32_t)(L - 1) * 0x10001u;

    for (int i = threadIdx.x; i < nall / 4; i += blockDim.x)
        plane4[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < 2 + H2_THREADS / 64) // and the maxima, of which a small workgroup writes a part
        corner[threadIdx.x] = 0u;
    __syncthreads();

    // the largest cell of the plane, for the whole workgroup
    auto plane_max = [&]() {
        u16x2 m = {0, 0};
        for (int i = threadIdx.x; i < nall / 4; i += blockDim.x) {
            const uint4 w4 = plane4[i];
            m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w4.x));
            m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w4.y));
            m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w4.z));
            m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w4.w));
        }
        uint32_t mx = max((uint32_t)m[0], (uint32_t)m[1]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
        if (lane == 0)
            wmax[wv] = mx;
        __syncthreads();
        for (int v = 0; v < H2_THREADS / 64; ++v)
            mx = max(mx, wmax[v]);
        __syncthreads(); // wmax is read before the next call writes it
        return mx;
    };

    // rows [ra, rb) of image s counted into the plane and added to (or, for a
    // whole image, stored as) its histogram; the plane is zero before and after
    auto process = [&](int s, int ra, int rb, bool store) {
        const TS_GLOBAL int16_t *img = gp(vox[s]);
        uint32_t *hs = hist + (int64_t)s * L * L;
        const int run = (rb - ra + sh.nrun - 1) / sh.nrun;
        const int y0 = ra + runid * run, y1 = min(rb, y0 + run); // this lane's rows
        const int ya = y0 - 2, steps_all = run + 2; // two rows before them fill the running sums
        auto load = [&](int y, v4i &raw, int &ext) {
            const int64_t at = (int64_t)min(max(y, 0), H - 1) * W;
            const int64_t p = min(at + xl, npix - 8); // not past the image's end
            raw = *reinterpret_cast<const TS_GLOBAL v4i_any *>(img + p);
            if (RAGGED) {
                const int sh16 = (int)(at + xl - p); // pixels to shift out: the image's last rows only
                if (__any(sh16)) {
                    uint32_t e[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        e[j] = (uint32_t)raw[j];
#pragma unroll
                    for (int n = 4; n >= 1; n >>= 1) {
                        const bool on = sh16 & n;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t up = n == 1 ? (j < 3 ? pair_mid(e[j], e[j + 1]) : e[3] >> 16)
                                                       : (j + n / 2 < 4 ? e[(j + n / 2) & 3] : 0u);
                            e[j] = on ? up : e[j];
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        raw[j] = (int)e[j];
                }
            }
            ext = 0;
            if (sh.nch > 1) // the columns beside the chunk, for its end lanes
                ext = img[at + xe];
        };
        // gray levels and row sums of three of a loaded row
        auto sums = [&](const v4i &raw, int ext, uint32_t(&l)[4], uint32_t(&h)[4]) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                l[j] = levels2<KIND>((uint32_t)raw[j], bm, mul24);
            // all four formed here: raw is free for the next load, which must not
            // wait for a copy of it at the loop's end
            asm volatile("" : "+v"(l[0]), "+v"(l[1]), "+v"(l[2]), "+v"(l[3]));
            if (RAGGED) { // columns past the row's end repeat its last
                uint32_t prev = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t a = 2 * j <= edge ? l[j] & 0xffffu : prev;
                    prev = 2 * j + 1 <= edge ? l[j] >> 16 : a;
                    l[j] = at_right ? a | prev << 16 : l[j];
                }
            }
            uint32_t before = dpp32<0x138, 0xf>(l[3]), after = dpp32<0x130, 0xf>(l[0]); // lane - 1, lane + 1
            if (sh.nch > 1) {
                const uint32_t e = levels2<KIND>((uint32_t)ext & 0xffffu, bm, mul24) & 0xffffu;
                before = g_first ? e << 16 : before;
                after = g_last ? e : after;
            }
            before = at_left ? l[0] << 16 : before;
            after = at_right ? l[3] >> 16 : after;
            uint32_t m[5];
            m[0] = pair_mid(before, l[0]);
#pragma unroll
            for (int j = 1; j < 4; ++j)
                m[j] = pair_mid(l[j - 1], l[j]);
            m[4] = pair_mid(l[3], after);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                h[j] = pk_add(pk_add(m[j], l[j]), m[j + 1]);
        };
        uint32_t hot0 = 0, hot1 = 0;
        uint32_t h2[4] = {}, hc[4] = {}, lc[4] = {}; // row sums of rows y-1 and y together, of row y; levels at y
        v4i raw[2];
        int ext[2];
        load(y0 - 1, raw[0], ext[0]);
        load(y0, raw[1], ext[1]);
        // one row: the row below arrives in raw (row y + 3 is loaded in its
        // place), its sums complete the 3 x 3 sums of row y.  The two rows
        // before the first only fill the running sums.
        auto row = [&](int y, v4i &rw, int &ex) {
            uint32_t ln[4], hn[4], t[4];
            sums(rw, ex, ln, hn);
            load(y + 3, rw, ex);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                t[j] = pk_add(h2[j], hn[j]);
            if (nv > 0 && y >= y0 && y < y1) {
                if ((t[0] | t[1] | t[2] | t[3]) == 0u && (!RAGGED || nv == 8)) {
                    hot0 += 8;
                } else if (((t[0] ^ top) | (t[1] ^ top) | (t[2] ^ top) | (t[3] ^ top)) == 0u && (!RAGGED || nv == 8)) {
                    hot1 += 8;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // levels from half on move to the low halves: f - half, which
                        // wraps past 2^15 for the levels below (kept as they are, by
                        // the unsigned minimum), whose increments shift by 16
                        const u16x2 l2 = __builtin_bit_cast(u16x2, lc[j]), x2 = l2 - half2;
                        const uint32_t f = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(l2, x2));
                        const uint32_t up = __builtin_bit_cast(uint32_t, x2 >> (u16x2){11, 11}) & 0x100010u;
                        // word f L + floor(sum / 9) in units of 2^-15: 3641 / 2^15 is
                        // 1/9 closely enough for every sum up to 9 * 255
                        const uint32_t c0 = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, t[j]), (u16x2){3641, 0},
                                                                   __umul24(f & 0xffffu, fmul), false);
                        const uint32_t c1 = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, t[j]), (u16x2){0, 3641},
                                                                   __umul24(f >> 16, fmul), false);
                        if (!RAGGED || 2 * j < nv)
                            atomicAdd(mine + (c0 >> 15), 1u << (up & 0xffffu));
                        if (!RAGGED || 2 * j + 1 < nv)
                            atomicAdd(mine + (c1 >> 15), 1u << (up >> 16));
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                h2[j] = pk_add(hc[j], hn[j]);
                hc[j] = hn[j];
                lc[j] = ln[j];
            }
        };
        // Every cell is at most 65535 minus the budget before each stretch of
        // rows, and the workgroup counts at most nrun * W <= 8192 pixels per
        // row step, so no half-word overflows.
        uint32_t budget = 65535u;
        for (int i0 = 0;;) {
            const int steps = min((int)(budget / (uint32_t)(sh.nrun * W)), steps_all - i0); // >= 4 or the rest
            for (int i = 0; i + 1 < steps; i += 2) {
                row(ya + i0 + i, raw[0], ext[0]);
                row(ya + i0 + i + 1, raw[1], ext[1]);
            }
            i0 += steps;
            if (steps & 1) { // the row after it is in raw[1]
                row(ya + i0 - 1, raw[0], ext[0]);
                const v4i rt = raw[0];
                const int et = ext[0];
                raw[0] = raw[1];
                ext[0] = ext[1];
                raw[1] = rt;
                ext[1] = et;
            }
            __syncthreads();
            if (i0 >= steps_all)
                break;
            uint32_t mx = (uint32_t)__builtin_amdgcn_readfirstlane((int)plane_max());
            if (mx >= 32768u) { // rare: cells from there up move to the histogram
                if (store) { // which is not cleared yet for a whole image
                    for (int i = threadIdx.x; i < L * L; i += blockDim.x)
                        hs[i] = 0u;
                    __threadfence();
                    store = false;
                    __syncthreads();
                }
                for (int i = threadIdx.x; i < nall; i += blockDim.x) {
                    const uint32_t w2 = plane[i];
                    const int cell = REPS > 1 ? i % nw4 : i; // a copy's last words stay 0
                    uint32_t keep = w2;
                    if (w2 & 0x8000u) {
                        atomicAdd(&hs[nw2 + cell], w2 & 0xffffu);
                        keep &= 0xffff0000u;
                    }
                    if (w2 & 0x80000000u) {
                        atomicAdd(&hs[cell], w2 >> 16);
                        keep &= 0xffffu;
                    }
                    if (keep != w2)
                        plane[i] = keep;
                }
                mx = 32767u;
                __syncthreads();
            }
            budget = 65535u - mx;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            hot0 += __shfl_xor(hot0, o, 64);
            hot1 += __shfl_xor(hot1, o, 64);
        }
        if (lane == 0) {
            atomicAdd(&corner[0], hot0);
            atomicAdd(&corner[1], hot1);
        }
        __syncthreads();
        const int last = L * L - 1;
        if (store) {
            const bool vec = (nw2 & 3) == 0 && (L & 1) == 0 && ((uintptr_t)hs & 15) == 0;
            for (int i = threadIdx.x; i < nw4 / 4; i += blockDim.x) { // 4 words: 4 cells of each half
                const uint4 w4 = plane4[i];
                plane4[i] = make_uint4(0u, 0u, 0u, 0u);
                uint32_t c[4] = {w4.x >> 16, w4.y >> 16, w4.z >> 16, w4.w >> 16};
                uint32_t d[4] = {w4.x & 0xffffu, w4.y & 0xffffu, w4.z & 0xffffu, w4.w & 0xffffu};
                for (int r = 1; r < REPS; ++r) {
                    const uint4 x4 = plane4[r * (nw4 / 4) + i];
                    plane4[r * (nw4 / 4) + i] = make_uint4(0u, 0u, 0u, 0u);
                    const uint32_t x[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        c[j] += x[j] >> 16;
                        d[j] += x[j] & 0xffffu;
                    }
                }
                c[0] += i == 0 ? corner[0] : 0u;
                if ((last - nw2) >> 2 == i) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        d[j] += ((last - nw2) & 3) == j ? corner[1] : 0u;
                }
                if (vec) {
                    *reinterpret_cast<uint4 *>(hs + 4 * i) = make_uint4(c[0], c[1], c[2], c[3]);
                    *reinterpret_cast<uint4 *>(hs + nw2 + 4 * i) = make_uint4(d[0], d[1], d[2], d[3]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (4 * i + j < nw2)
                            hs[4 * i + j] = c[j];
                        if (4 * i + j < nw2 && nw2 + 4 * i + j <= last)
                            hs[nw2 + 4 * i + j] = d[j];
                    }
                }
            }
        } else {
            for (int i = threadIdx.x; i < nw2; i += blockDim.x) {
                uint32_t hi = 0u, lo = 0u;
                for (int r = 0; r < REPS; ++r) {
                    const uint32_t w2 = plane[r * nw4 + i];
                    plane[r * nw4 + i] = 0u;
                    hi += w2 >> 16;
                    lo += w2 & 0xffffu;
                }
                if (hi)
                    atomicAdd(&hs[i], hi);
                if (lo) // a half past the last cell counts nothing
                    atomicAdd(&hs[nw2 + i], lo);
            }
            if (threadIdx.x < 2 && corner[threadIdx.x])
                atomicAdd(&hs[threadIdx.x ? last : 0], corner[threadIdx.x]);
        }
        __syncthreads();
        if (threadIdx.x < 2)
            corner[threadIdx.x] = 0u;
        __syncthreads();
    };
    // whole images first, then a share of the rest's rows: an equal part of
    // one image, or of all their rows in turn
    const int64_t rest = (int64_t)(nseg - whole) * H;
    int64_t r, r1;
    if (parts > 0) {
        const int s = blockIdx.x / parts, j = blockIdx.x % parts;
        r = min(rest, (int64_t)s * H + (int64_t)H * j / parts);
        r1 = min(rest, (int64_t)s * H + (int64_t)H * (j + 1) / parts);
    } else {
        r = rest * blockIdx.x / gridDim.x;
        r1 = rest * (blockIdx.x + 1) / gridDim.x;
    }
    for (int i = blockIdx.x;; i += gridDim.x) {
        const bool all = i < whole;
        if (!all && r >= r1)
            break;
        const int s = all ? i : (int)(whole + r / H), ra = all ? 0 : (int)(r % H);
        const int rb = all ? H : (int)min((int64_t)H, ra + (r1 - r));
        process(s, ra, rb, all);
        r += all ? 0 : rb - ra;
    }
}

// Images of fewer than 8 pixels: one thread per pixel.
__global__ void __launch_bounds__(256) k_hist2d_tiny(const int16_t *const *__restrict__ vox, int nseg, int H, int W,
                                                     BinMap bm, uint32_t *__restrict__ hist)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int s = (int)(i >> 3), p = (int)(i & 7);
    if (s >= nseg || p >= H * W)
        return;
    const TS_GLOBAL int16_t *img = gp(vox[s]);
    const int y = p / W, x = p % W;
    int sum = 0;
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx)
            sum += bin_of(img[min(max(y + dy, 0), H - 1) * W + min(max(x + dx, 0), W - 1)], bm);
    atomicAdd(&hist[(int64_t)s * bm.L * bm.L + bin_of(img[p], bm) * bm.L + sum / 9], 1u);
}

ts_status launch_hist2d(const ts_batch &b, int H, int W, const BinMap &bm, uint32_t *hist, hipStream_t st)
{
    if (W > H2_MAX_W || bm.L > H2_MAX_L)
        return fail(TS_ERR_INVALID_ARG, "ts_histogram2d: width or nbins beyond the LDS layout");
    if ((int64_t)H * W < 8) { // no 8 pixels to load together
        ts_status e = launch_fill_u32(hist, (int64_t)b.nseg * bm.L * bm.L, st);
        if (e != TS_OK)
            return e;
        hipLaunchKernelGGL(k_hist2d_tiny, dim3((unsigned)(((int64_t)b.nseg * 8 + 255) / 256)), dim3(256), 0, st, b.vox,
                           b.nseg, H, W, bm, hist);
        return check_launch("ts_histogram2d");
    }
    // Few levels and many pixels: copies of the plane by lane, since a wavefront's
    // counts then meet in a handful of words (300 images of 512 x 512, 16 levels
    // over the whole CT range: 158 us with one copy, 69 with eight).
    const int reps = bm.L <= 32 && b.total >= (1 << 24) ? 8 : 1;
    const size_t lds = ((size_t)((hist2d_words(bm.L) + 3) & ~3) * reps + 2 + H2_THREADS / 64) * 4;
    const int lanes = (W + 7) / 8;
    // Many small images whose planes share a CU: workgroups of 512 or 256 threads,
    // as many as the LDS or 2048 threads hold, since clearing, counting and adding
    // up follow each other within one.  64 levels, 2000 images of 16 x 16 38 -> 12
    // us, 1000 of 64 x 64 22 -> 10; 600 of 128 x 96 at 128 levels, four planes per
    // CU, are better off with one workgroup (28 against 33).
    const int cus = device_cu_count(), fit = (int)std::min<size_t>(8, H2_LDS / lds);
    const bool tiny = (int64_t)H * W <= H2_SMALL;
    const int per = !tiny || b.nseg <= cus ? 1 : b.nseg <= 2 * cus ? (fit > 1 ? 2 : 1)
                    : fit == 8 || (fit > 1 && (int64_t)H * W <= H2_MIN_PIX) ? 4 : 1; // of H2_THREADS
    const int threads = lanes * per <= H2_THREADS ? H2_THREADS / per : H2_THREADS;
    // Row groups of 16, 32 or 64 lanes, or of fewer where they hold a row: those
    // that leave the fewest lanes without columns, several chunks per row counted
    // a sixteenth dearer (the columns beside a chunk are loaded apart).  552
    // columns are 69 lanes: 12 rows of five 16-lane chunks at once keep 828 of
    // 1024 lanes, 8 rows of two wavefronts 552.  300 images of 4096 x 8 at 64
    // levels: 93 us with groups of 16 lanes, 20 with one lane a row.
    Hist2dShape sh{6, 1, 1};
    for (int g = 6, best = 0; g >= 0; --g) {
        const int nch = (lanes + (1 << g) - 1) >> g, nrun = (threads >> g) / nch;
        const int score = nrun * lanes * (nch > 1 ? 15 : 16);
        if (score > best && (g >= 4 || nch == 1)) {
            best = score;
            sh = Hist2dShape{g, nch, nrun};
        }
    }
    // Workgroups: one per CU (small images: as many as fit), each with an image
    // of its own or at least H2_MIN_ROWS rows (clearing and adding up the plane
    // takes as long as counting about as many; images of H2_MIN_PIX pixels are not
    // split, which would need the clearing launch), and below one per CU equal
    // parts of every image.  300 images of 1 x 4096 at 64 levels: 69 us by rows
    // alone, 7 with a workgroup each.
    const int64_t most = (int64_t)cus * (threads < H2_THREADS ? std::min(fit, 2048 / threads) : 1);
    int64_t want = (int64_t)b.nseg * ((int64_t)H * W <= H2_MIN_PIX ? 1 : std::max(1, H / H2_MIN_ROWS));
    if (want > most)
        want = std::min<int64_t>(most, tiny && b.nseg >= cus ? b.nseg : std::max<int64_t>(b.nseg, (int64_t)b.nseg * H / H2_MIN_ROWS));
    const int nwg = (int)want;
    // Whole images first, as many as fill every workgroup equally: those store
    // their histograms; the rest's rows are split evenly and added to cleared
    // histograms.  A second round of small images takes less than the clearing
    // launch and the split.
    const int whole = tiny && b.nseg >= nwg && b.nseg < 2 * nwg ? b.nseg : b.nseg / nwg * nwg;
    // A workgroup whose rows cross into another image adds up two planes, 5 to
    // 10 us each: parts that keep to one image, unless they leave more than an
    // eighth of the workgroups idle.
    const int rest = b.nseg - whole;
    const int parts = rest && nwg / rest * rest * 8 >= nwg * 7 ? nwg / rest : 0;
    if (whole < b.nseg) {
        ts_status e = launch_fill_u32(hist + (int64_t)whole * bm.L * bm.L, (int64_t)(b.nseg - whole) * bm.L * bm.L, st);
        if (e != TS_OK)
            return e;
    }
    const uint32_t mul24 = binmap_mul24(bm);
    const int kind = levels_kind(bm);
    const dim3 g((unsigned)nwg), blk(threads);
#define TS_H2(K, R, C)                                                                                              \
    allow_dynamic_lds((const void *)k_hist2d<K, R, C>, lds);                                                      \
    hipLaunchKernelGGL((k_hist2d<K, R, C>), g, blk, lds, st, b.vox, b.nseg, whole, parts, H, W, sh, bm, mul24, hist)
#define TS_H2K(R, C)                                                                                                \
    if (kind == 0) { TS_H2(0, R, C); } else if (kind == 1) { TS_H2(1, R, C); } else { TS_H2(2, R, C); }
    if (W % 8 == 0) {
        if (reps == 1) { TS_H2K(false, 1) } else { TS_H2K(false, 8) }
    } else {
        if (reps == 1) { TS_H2K(true, 1) } else { TS_H2K(true, 8) }
    }
#undef TS_H2K
#undef TS_H2
    return check_launch("ts_histogram2d");
}

// ------------------------------------------------------------------ search

struct Q2List {
    double q[TS_MAX_Q];
};

// With p_ij = c_ij / N the class term sgn(1-q) (ln Q - q ln w) equals
// sgn(1-q) (ln sum c^q - q ln C) for a class of C pixels, and the Shannon
// term ln w - E / w equals ln C - (sum c ln c) / C: N cancels, so the search
// works on raw counts.  cterm(c) is c^q (c ln c for q = 1), 0 for c = 0.
__device__ __forceinline__ double cterm(uint32_t c, double q)
{
    if (!c)
        return 0.0;
    const double x = (double)c;
    return q == 1.0 ? x * log(x) : pow(x, q);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp64(uint64_t v)
{
    const uint32_t lo = dpp32<CTRL, ROWS>((uint32_t)v), hi = dpp32<CTRL, ROWS>((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dppv(T v)
{
    if constexpr (std::is_same<T, double>::value)
        return __longlong_as_double((long long)dpp64<CTRL, ROWS>((uint64_t)__double_as_longlong(v)));
    else if constexpr (sizeof(T) == 4)
        return (T)dpp32<CTRL, ROWS>((uint32_t)v);
    else
        return (T)dpp64<CTRL, ROWS>((uint64_t)v);
}

// Exclusive sum over the lanes of the wavefront in a fixed order: a
// Hillis-Steele scan within each row of 16 lanes, then the rows carried by
// broadcasts of lanes 15 and 31, then a shift by one lane.
template <typename T>
__device__ __forceinline__ T wave_excl_sum(T v)
{
    v = v + dppv<0x111, 0xf>(v); // row_shr:1
    v = v + dppv<0x112, 0xf>(v); // row_shr:2
    v = v + dppv<0x114, 0xf>(v); // row_shr:4
    v = v + dppv<0x118, 0xf>(v); // row_shr:8
    v = v + dppv<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
    v = v + dppv<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
    return dppv<0x138, 0xf>(v);  // wave_shr:1: lane 0 gets 0
}

// Sums along s of one 2D histogram row, S2_CPL cells per lane: scan position
// p = S2_CPL * lane + u (u = 0 .. S2_CPL-1) is column p (prefix order) or
// column L-1-p (suffix order); c the counts, t their terms.  For every position
// the exact count sum and the FP64 sum of cterm up to it: within the lane sequentially, after the
// lane's exclusive base.  An empty position takes the value at the nearest
// occupied position before it in scan order, so an all-empty column never
// changes a class sum (bit for bit) and the pairs it separates tie.
template <typename CT>
__device__ __forceinline__ void row_sums(const uint32_t (&c)[S2_CPL], const double (&t)[S2_CPL], CT (&rc)[S2_CPL],
                                         double (&rq)[S2_CPL])
{
    const int lane = threadIdx.x & 63;
    CT lc = 0;
    double lq = 0.0;
    int first = S2_CPL; // first occupied position of this lane
    CT pc[S2_CPL];
    double pq[S2_CPL];
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        lc += (CT)c[u];
        lq = lq + t[u]; // an empty cell adds +0.0: bits unchanged
        pc[u] = lc;
        pq[u] = lq;
        if (c[u] && first == S2_CPL)
            first = u;
    }
    const uint64_t occ = __ballot(lc != 0);
    const CT bc = wave_excl_sum<CT>(lc);
    const double bq = wave_excl_sum<double>(lq);
    const double last = bq + lq; // the value at this lane's last occupied position
    const uint64_t before = occ & ((1ull << lane) - 1ull);
    const int src = before ? 63 - __clzll((long long)before) : lane;
    const double prev_raw = __shfl(last, src, 64);
    const double prev = before ? prev_raw : 0.0;
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        rc[u] = bc + pc[u];
        rq[u] = u >= first ? bq + pq[u] : prev;
    }
}

// The same scan for per-position values given directly (cc counts, cq sums
// of cterm; a block's column totals): exact count prefix, FP64 prefix in
// the lane then after its exclusive base, an empty position taking the
// value at the nearest occupied position before it.
template <typename CT>
__device__ __forceinline__ void pos_sums(const CT (&cc)[S2_CPL], const double (&cq)[S2_CPL], CT (&rc)[S2_CPL],
                                         double (&rq)[S2_CPL])
{
    const int lane = threadIdx.x & 63;
    CT lc = 0;
    double lq = 0.0;
    int first = S2_CPL;
    CT pc[S2_CPL];
    double pq[S2_CPL];
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        lc += cc[u];
        lq = lq + cq[u];
        pc[u] = lc;
        pq[u] = lq;
        if (cc[u] && first == S2_CPL)
            first = u;
    }
    const uint64_t occ = __ballot(lc != 0);
    const CT bc = wave_excl_sum<CT>(lc);
    const double bq = wave_excl_sum<double>(lq);
    const double last = bq + lq;
    const uint64_t before = occ & ((1ull << lane) - 1ull);
    const int src = before ? 63 - __clzll((long long)before) : lane;
    const double prev_raw = __shfl(last, src, 64);
    const double prev = before ? prev_raw : 0.0;
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        rc[u] = bc + pc[u];
        rq[u] = u >= first ? bq + pq[u] : prev;
    }
}

// FP64 class term from the class sums: sgn(1-q) (ln S - q ln C) for Tsallis,
// ln C - S / C for q = 1 (S = sum of cterm, C = pixels); -inf for an empty
// class; clamped to [0, hmax].
__device__ __forceinline__ double class_term2(uint64_t c, double sumq, double q, double sgn, double hmax)
{
    if (c == 0)
        return -INFINITY;
    const double C = (double)c;
    const double h = sgn == 0.0 ? log(C) - sumq / C : sgn * (log(sumq) - q * log(C));
    return fmin(fmax(h, 0.0), hmax);
}

// A value that is the same in every lane, held in scalar registers.
__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform(double v)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Per-problem constants of the search.
struct S2 {
    const uint32_t *h; // the L x L histogram
    int L;
    bool vec;          // rows load as 16-byte vectors (L % 4 == 0, aligned)
    double q, sgn, hmax;
    const double *tab; // cterm of counts below S2_TAB
    double *big;       // cterm of the cells with larger counts, [L][L] (workspace, t2's place until pass 3)
    float mq;          // -q rounded to FP32 (Tsallis)
    float sg;          // sgn(1-q) as +-1 (Tsallis)
    float gmax;        // hmax / ln 2 rounded up
};

// The same class term in log2 units in FP32, from the FP64 class sums: the
// key of the search.  Its error against class_term2 / ln 2 is bounded in
// s2_delta.  sgn(1-q) (log2 S - q log2 C) is formed as the fma
// log2 S - q log2 C times +-1 (exact).
template <typename CT>
__device__ __forceinline__ float class_key32(CT c, double sumq, const S2 &p)
{
    const float lc = __builtin_amdgcn_logf((float)c);
    float g;
    if (p.sgn == 0.0) { // Shannon: log2 C - (S / C) log2 e
        const float r = (float)(sumq / (double)c);
        g = fmaf(r, -1.44269504f, lc);
    } else {
        g = fmaf(p.mq, lc, __builtin_amdgcn_logf((float)sumq)) * p.sg;
    }
    g = __builtin_amdgcn_fmed3f(g, 0.0f, p.gmax);
    return c ? g : -INFINITY;
}

// Bound on |key32 - key64 / ln 2| for every pair of one problem (key32 the
// sum of the two FP32 class keys, key64 the FP64 sum of class_term2 from the
// same class sums) for an image of N pixels.  Per class: the casts of C and
// S (or S / C) to FP32 (2^-24 relative each, 1.5 * 2^-24 after the log2),
// v_log_f32 (LOG2_ERR_UNITS * 2^-24 * max(1, |log2 x|)), q or log2 e rounded
// to FP32, the fma; then the FP32 sum of the two clamped terms, and the
// clamp at gmax instead of hmax / ln 2.  Magnitudes: 1 <= C <= N; a class of
// m <= L^2 occupied cells has 1 <= S <= max(C^q, m^(1-q) C^q), so
// 0 <= log2 S <= q log2 N + 2 |1-q| log2 L; 0 <= S / C <= ln N for q = 1.
// Infinity when S could leave the FP32 range: every pair is then re-checked
// in FP64.
__device__ __forceinline__ double s2_delta(const S2 &p, double N)
{
    const double u = 0x1p-24;
    const double lN = log2(N) * 1.0001 + 1e-6;
    const double q = p.q;
    double e1;
    if (p.sgn == 0.0) {
        const double r = lN * 0.6931471805599453 * 1.0001; // S / C <= ln N
        e1 = 1.5 * u + LOG2_ERR_UNITS * u * fmax(1.0, lN) + 2.0 * u * 1.4426950408889634 * r +
             u * (lN + 1.4426950408889634 * r);
    } else {
        const double Ux = q * lN + 2.0 * fabs(1.0 - q) * log2((double)p.L) * 1.0001 + 1e-6, Vy = lN;
        if (Ux > 120.0)
            return INFINITY;
        e1 = 1.5 * u * (1.0 + q) + LOG2_ERR_UNITS * u * (fmax(1.0, Ux) + q * fmax(1.0, Vy)) + u * q * Vy +
             u * (Ux + q * Vy);
    }
    return (2.0 * e1 + 2.0 * u * (double)p.gmax + 2.0 * 0x1p-20 * (double)p.gmax) * 1.01 + 1e-12;
}

// Counts of row t in the lane's scan positions (DIR = +1: column
// S2_CPL * lane + u; DIR = -1: column L-1-(S2_CPL * lane + u)); zero past
// the row's ends.  t must be a valid row.  The loads are unconditional
// (clamped addresses, masked values) so that several rows' loads can be in
// flight at once.
template <int DIR>
__device__ __forceinline__ void load_row(const uint32_t *h, int L, bool vec, int t, int jlo, int jhi,
                                         uint32_t (&c)[S2_CPL])
{
    const int lane = threadIdx.x & 63;
    const uint32_t *row = h + (int64_t)t * L;
    // columns outside [jlo, jhi] hold no counts: those lanes load nothing
    const int c0 = DIR > 0 ? S2_CPL * lane : L - S2_CPL - S2_CPL * lane; // the lane's lowest column (vec)
    if (vec) {
        const bool ok = S2_CPL * lane < L && c0 <= jhi && c0 + S2_CPL - 1 >= jlo;
        const uint4 v = ok ? *reinterpret_cast<const uint4 *>(row + c0) : make_uint4(0u, 0u, 0u, 0u);
        if (DIR > 0) {
            c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
        } else {
            c[0] = v.w; c[1] = v.z; c[2] = v.y; c[3] = v.x;
        }
    } else {
#pragma unroll
        for (int u = 0; u < S2_CPL; ++u) {
            const int col = DIR > 0 ? S2_CPL * lane + u : L - 1 - (S2_CPL * lane + u);
            const bool ok = col >= 0 && col < L && col >= jlo && col <= jhi;
            c[u] = ok ? row[col] : 0u;
        }
    }
}

// Element u of an array in registers.
template <typename T>
__device__ __forceinline__ T pick(const T (&v)[S2_CPL], int u)
{
    return u == 0 ? v[0] : u == 1 ? v[1] : u == 2 ? v[2] : v[3];
}

// A listed row: the row | the lowest column of its band << 8 | the highest <<
// 16 (levels are below 256), read once as a scalar.
struct S2Row {
    int t, lo, hi;
};
__device__ __forceinline__ S2Row listed(const uint32_t *rows, int k)
{
    const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)rows[k]);
    return S2Row{(int)(v & 0xffu), (int)((v >> 8) & 0xffu), (int)(v >> 16)};
}
template <int DIR>
__device__ __forceinline__ void load_row(const S2 &p, const S2Row &r, uint32_t (&c)[S2_CPL])
{
    load_row<DIR>(p.h, p.L, p.vec, r.t, r.lo, r.hi, c);
}

// The terms of a row's counts: from the table for small counts (which holds
// the identical expression, so both give the same bits), else from what
// block_totals left in the workspace, or formed anew (POW).
template <int DIR, bool POW>
__device__ __forceinline__ void row_terms(const S2 &p, int t, const uint32_t (&c)[S2_CPL], double (&term)[S2_CPL])
{
    bool big = false;
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        term[u] = p.tab[min(c[u], (uint32_t)S2_TAB - 1u)];
        big |= c[u] >= (uint32_t)S2_TAB;
    }
    if (__ballot(big)) {
        if (POW) {
#pragma unroll 1
            for (int u = 0; u < S2_CPL; ++u) {
                const double x = cterm(pick(c, u), p.q);
#pragma unroll
                for (int v = 0; v < S2_CPL; ++v)
                    term[v] = v == u && c[v] >= (uint32_t)S2_TAB ? x : term[v];
            }
        } else {
            const int pos = S2_CPL * (threadIdx.x & 63);
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u)
                if (c[u] >= (uint32_t)S2_TAB)
                    term[u] = p.big[t * p.L + (DIR > 0 ? pos + u : p.L - 1 - (pos + u))];
        }
    }
}

// Visits n >= 0 rows of the compacted list of rows holding counts, rows[k0],
// rows[k0 + DIR], ..., with each row's sums along s (row_sums, in DIR's scan
// order) and S2_CPL auxiliary values aux(k, .) per lane (stored keys the row
// needs); the counts and auxiliary values of the next S2_RING rows are in
// flight meanwhile.  Past the last row the ring reloads the last row and its
// sums are discarded.
template <int DIR, typename CT, typename A, typename F>
__device__ __forceinline__ void for_rows(const S2 &p, const uint32_t *rows, int k0, int n, A &&aux, F &&f)
{
    if (n <= 0)
        return;
    uint32_t ring[S2_RING][S2_CPL];
    float xr[S2_RING][S2_CPL];
#pragma unroll
    for (int d = 0; d < S2_RING; ++d) {
        const int kk = k0 + DIR * min(d, n - 1);
        load_row<DIR>(p, listed(rows, kk), ring[d]);
        aux(kk, xr[d]);
    }
    for (int i0 = 0; i0 < n; i0 += S2_RING) {
#pragma unroll
        for (int d = 0; d < S2_RING; ++d) {
            const int i = i0 + d;
            if (i < n) { // uniform over the wavefront
                uint32_t c[S2_CPL];
                float x[S2_CPL];
#pragma unroll
                for (int u = 0; u < S2_CPL; ++u) {
                    c[u] = ring[d][u];
                    x[u] = xr[d][u];
                }
                const int kk = k0 + DIR * min(i + S2_RING, n - 1);
                load_row<DIR>(p, listed(rows, kk), ring[d]);
                aux(kk, xr[d]);
                CT rc[S2_CPL];
                double rq[S2_CPL], t[S2_CPL];
                row_terms<DIR, false>(p, listed(rows, k0 + DIR * i).t, c, t);
                row_sums<CT>(c, t, rc, rq);
                f(k0 + DIR * i, rc, rq, x);
            }
        }
    }
}

// Column totals of the listed rows rows[k0 .. k0 + n - 1] for the lane's
// columns S2_CPL * lane + u: count sums and sums of cterm; leaves the terms of
// the counts past the table in p.big for the later walks.
template <typename CT>
__device__ __forceinline__ void block_totals(const S2 &p, const uint32_t *rows, int k0, int n, CT (&cc)[S2_CPL],
                                             double (&cq)[S2_CPL])
{
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        cc[u] = 0;
        cq[u] = 0.0;
    }
    if (n <= 0)
        return;
    uint32_t ring[S2_RING][S2_CPL];
#pragma unroll
    for (int d = 0; d < S2_RING; ++d)
        load_row<1>(p, listed(rows, k0 + min(d, n - 1)), ring[d]);
    for (int i0 = 0; i0 < n; i0 += S2_RING) {
#pragma unroll
        for (int d = 0; d < S2_RING; ++d) {
            const int i = i0 + d;
            if (i < n) {
                uint32_t c[S2_CPL];
                double t[S2_CPL];
                bool big = false;
#pragma unroll
                for (int u = 0; u < S2_CPL; ++u) {
                    c[u] = ring[d][u];
                    big |= c[u] >= (uint32_t)S2_TAB;
                }
                load_row<1>(p, listed(rows, k0 + min(i + S2_RING, n - 1)), ring[d]);
                if (__ballot(big)) {
                    const int at = listed(rows, k0 + i).t * p.L + S2_CPL * (threadIdx.x & 63);
#pragma unroll 1
                    for (int u = 0; u < S2_CPL; ++u) {
                        const uint32_t x = pick(c, u);
                        if (x >= (uint32_t)S2_TAB) // skipped where no lane's u is
                            p.big[at + u] = cterm(x, p.q);
                    }
                }
                row_terms<1, false>(p, listed(rows, k0 + i).t, c, t);
#pragma unroll
                for (int u = 0; u < S2_CPL; ++u) {
                    cc[u] += c[u];
                    cq[u] = cq[u] + t[u];
                }
            }
        }
    }
}

// Maximum over the wavefront by DPP moves (no LDS round trips): within rows
// of 16 lanes, then carried by the broadcasts of lanes 15 and 31; lanes
// without a source read -inf.  The result is read from lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_max_step(float v)
{
    const int ninf = __float_as_int(-INFINITY);
    const float o = __int_as_float(__builtin_amdgcn_update_dpp(ninf, __float_as_int(v), CTRL, ROWS, 0xf, false));
    return fmaxf(v, o);
}

__device__ __forceinline__ float wave_max_f32(float v)
{
    v = dpp_max_step<0x111, 0xf>(v); // row_shr:1
    v = dpp_max_step<0x112, 0xf>(v); // row_shr:2
    v = dpp_max_step<0x114, 0xf>(v); // row_shr:4
    v = dpp_max_step<0x118, 0xf>(v); // row_shr:8
    v = dpp_max_step<0x142, 0xa>(v); // row_bcast:15
    v = dpp_max_step<0x143, 0xc>(v); // row_bcast:31
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// LDS of one (q index, problem).
template <int NW, typename CT>
struct S2Lds {
    double tab[S2_TAB];               // cterm of counts below S2_TAB
    double tq[2][NW][H2_MAX_L];       // per block and column: sums of cterm of the blocks before ([0]) and after ([1])
    CT tc[NW + 1][H2_MAX_L];          // count sums of the blocks before (exact: those after are the rest)
    uint32_t rows[H2_MAX_L];          // rows holding counts, increasing, as listed rows (S2Row)
    float rmax[H2_MAX_L];             // best pair key of each listed row
    float wm[NW];                     // per-wavefront maxima
    double wb[NW];                    // per-wavefront best FP64 pair
    long long wcode[NW];
    int nrows;
};

// The class sums carried into block w in DIR's scan positions: class 1 (DIR =
// +1) from the blocks above, class 2 (DIR = -1) from those below.
template <int DIR, int NW, typename CT>
__device__ __forceinline__ void carry_in(const S2Lds<NW, CT> &sh, int L, int w, CT (&ac)[S2_CPL],
                                         double (&aq)[S2_CPL])
{
    CT cc[S2_CPL];
    double cq[S2_CPL];
#pragma unroll
    for (int u = 0; u < S2_CPL; ++u) {
        const int pos = S2_CPL * (threadIdx.x & 63) + u, col = DIR > 0 ? pos : L - 1 - pos;
        const bool ok = col >= 0 && col < L;
        const CT n = DIR > 0 ? sh.tc[w][ok ? col : 0] : (CT)(sh.tc[NW][ok ? col : 0] - sh.tc[w + 1][ok ? col : 0]);
        cc[u] = ok ? n : 0;
        cq[u] = ok ? sh.tq[DIR > 0 ? 0 : 1][w][ok ? col : 0] : 0.0;
    }
    pos_sums<CT>(cc, cq, ac, aq);
}

typedef float v4f __attribute__((ext_vector_type(4)));
typedef v4f v4f_any __attribute__((aligned(4)));

// Bounded by its vector operations, about 190 per row, wavefront and pass (a
// third of them the FP64 sums along s), four clocks each: 900 problems
// of 256 levels (132 rows with counts) 288 -> 201 us with the row pass, 37 of
// 200 levels 103 -> 55 us.  What changed: one walk for both directions' column
// totals, rows' terms past the table kept instead of formed by calls in the
// walks, constants of a problem in scalar registers (128 vector registers: four
// wavefronts per SIMD), two or four times the wavefronts per problem.
//
// One (q index, problem) per workgroup of NW wavefronts; CT is the type of
// count sums (uint32_t when the image holds fewer than 2^32 pixels).  R >= 1
// rows hold counts, listed in rows[] in increasing order, in NW blocks.  A row
// without counts (t >= 1) leaves the class 1 sums unchanged and
// B(t+1, .) = B(t, .): its pairs tie exactly with those of row t-1, which
// come first, so only listed rows are visited, and the class 2 partner of
// the listed row rows[k] is rows[k+1].
//  0. column totals of every block, then those of all blocks before and after
//     each block;
//  1. class 2 keys, bottom-up: B(t, s) = sums over {i >= t, j >= s} (scan
//     position p is column L-1-p), each block started from the totals of the
//     blocks below it; FP32 key of every listed row t >= 1 into k2
//     (workspace, [L][L] floats);
//  2. class 1, top-down: A(t, s) = sums over {i <= t, j <= s}, the listed
//     rows up to R - 2, each block started from the totals of the blocks above
//     it; the pair key is the FP32 class 1 key plus k2 at (rows[k+1], s+1);
//     row maxima rmax[k] and the maximum M;
//  3. rows with rmax >= M - 2 delta (the FP64 arg max is among them): the
//     FP64 class 2 terms of their partner rows into t2 (workspace, doubles),
//     from the same sums as in 1;
//  4. the FP64 value of every pair of those rows whose key is >= M - 2
//     delta, from the same sums as in 2; the first best pair (t outermost).
template <int NW, typename CT>
__device__ __forceinline__ void search2d_body(const S2 &p, double N, int R, S2Lds<NW, CT> &sh, float *k2, double *t2,
                                              int32_t *thr_t, int32_t *thr_s, double *obj_p, int32_t *status_p)
{
    const int lane = threadIdx.x & 63, L = p.L;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t *rows = sh.rows;
    float *rmax = sh.rmax;
    const int posl = S2_CPL * lane; // the lane's first scan position
    const int colB0 = L - 1 - posl; // its column in suffix order; position u's is colB0 - u (negative: none)
    const int kB = listed(rows, 0).t == 0 ? 1 : 0; // class 2 starts at row 1 at the earliest
    const int b0 = R * w / NW, b1 = R * (w + 1) / NW; // this wavefront's block
    const int bb = max(b0, kB), nb = b1 - bb;         // its class 2 rows (nb <= 0: none)
    const int na = min(b1, R - 1) - b0;               // its rows with pairs (rows[k] <= L - 2 follows)
    auto none = [](int, float(&)[S2_CPL]) {};
    // the stored class 2 keys at (rows[k + 1], s + 1) for the lane's columns
    // s; past the row the next one's (or what follows the keys), masked below
    auto partner = [&](int k, float(&x)[S2_CPL]) {
        const float *row2 = k2 + (int64_t)listed(rows, k + 1).t * L; // k <= R - 2 in the pass that uses it
        if (p.vec) {
            const v4f v = *reinterpret_cast<const v4f_any *>(row2 + min(posl, L - S2_CPL) + 1);
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u)
                x[u] = v[u];
        } else {
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u)
                x[u] = row2[min(posl + u + 1, L - 1)];
        }
    };

    // 0. block totals, then per column the sums before and after every block
    {
        CT cc[S2_CPL];
        double cq[S2_CPL];
        block_totals<CT>(p, rows, b0, b1 - b0, cc, cq);
#pragma unroll
        for (int u = 0; u < S2_CPL; ++u) {
            sh.tc[w + 1][posl + u] = cc[u];
            sh.tq[0][w][posl + u] = cq[u];
        }
    }
    __syncthreads();
    if (threadIdx.x < H2_MAX_L) {
        const int c = threadIdx.x;
        double aq = 0.0;
#pragma unroll
        for (int v = NW - 1; v >= 0; --v) {
            sh.tq[1][v][c] = aq;
            aq = aq + sh.tq[0][v][c];
        }
        CT ac = 0;
        aq = 0.0;
        sh.tc[0][c] = 0;
#pragma unroll
        for (int v = 0; v < NW; ++v) {
            const double y = sh.tq[0][v][c];
            sh.tq[0][v][c] = aq;
            aq = aq + y;
            ac += sh.tc[v + 1][c];
            sh.tc[v + 1][c] = ac;
        }
    }
    __syncthreads();
    // the sums carried into this wavefront's block are formed again at the
    // start of each walk rather than held in registers across the passes

    // 1. class 2 keys
    {
        CT bc[S2_CPL];
        double bq[S2_CPL];
        carry_in<-1>(sh, L, w, bc, bq);
        for_rows<-1, CT>(p, rows, b1 - 1, nb, none, [&](int k, const CT(&rc)[S2_CPL], const double(&rq)[S2_CPL],
                                                        const float(&)[S2_CPL]) {
            float *row = k2 + (int64_t)listed(rows, k).t * L;
            v4f key;
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u) {
                bc[u] += rc[u];
                bq[u] = bq[u] + rq[u];
                key[S2_CPL - 1 - u] = class_key32(bc[u], bq[u], p);
            }
            if (p.vec) {
                if (colB0 >= 0)
                    *reinterpret_cast<v4f_any *>(row + colB0 - (S2_CPL - 1)) = key;
            } else {
#pragma unroll
                for (int u = 0; u < S2_CPL; ++u)
                    if (colB0 - u >= 0)
                        row[colB0 - u] = key[S2_CPL - 1 - u];
            }
        });
    }
    __syncthreads();
    // 2. pair keys, row maxima
    {
        float M = -INFINITY;
        CT ac[S2_CPL];
        double aq[S2_CPL];
        carry_in<1>(sh, L, w, ac, aq);
        for_rows<1, CT>(p, rows, b0, na, partner, [&](int k, const CT(&rc)[S2_CPL], const double(&rq)[S2_CPL],
                                                      const float(&x)[S2_CPL]) {
            float m = -INFINITY;
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u) {
                ac[u] += rc[u];
                aq[u] = aq[u] + rq[u];
                const float key = class_key32(ac[u], aq[u], p) + x[u];
                m = posl + u <= L - 2 ? fmaxf(m, key) : m;
            }
            m = wave_max_f32(m);
            if (lane == 0)
                rmax[k] = m;
            M = fmaxf(M, m);
        });
        if (lane == 0)
            sh.wm[w] = M;
    }
    __syncthreads();
    float M = -INFINITY;
    for (int v = 0; v < NW; ++v)
        M = fmaxf(M, sh.wm[v]);
    M = uniform(M);
    const double delta = s2_delta(p, N);
    const bool all = !(uniform(delta) < INFINITY);
    if (!all && !(M > -INFINITY)) { // every key finite for a valid pair: none is valid
        if (threadIdx.x == 0) {
            *thr_t = *thr_s = -1;
            *obj_p = NAN;
            *status_p = TS_PROBLEM_DEGENERATE;
        }
        return;
    }
    const double T = uniform(all ? -INFINITY : (double)M - 2.0 * delta);
    // candidate rows of this block, and rows whose partner is one: bit l is row
    // b0 + l (a block has at most 256 / NW rows).  Both walks stop at the rows
    // they evaluate, so that the loads in flight do not hold registers beside
    // the logarithms.
    auto candidate = [&](int k) { return all || (double)rmax[k] >= T; };
    uint64_t m4 = __ballot(lane < na && candidate(b0 + min(lane, max(na - 1, 0))));
    const uint64_t m3 = __ballot(b0 + lane >= 1 && lane < b1 - b0 && candidate(max(b0 + lane - 1, 0)));
    // 3. FP64 class 2 terms of the rows in m3, from the block's bottom up to
    // the highest of them
    if (m3) {
        CT bc[S2_CPL];
        double bq[S2_CPL];
        carry_in<-1>(sh, L, w, bc, bq);
        int k = b1 - 1;
        for (uint64_t m = m3; m;) {
            const int l = 63 - __clzll((long long)m), ke = b0 + l;
            m &= ~(1ull << l);
            for_rows<-1, CT>(p, rows, k, k - ke + 1, none,
                             [&](int, const CT(&rc)[S2_CPL], const double(&rq)[S2_CPL], const float(&)[S2_CPL]) {
#pragma unroll
                                 for (int u = 0; u < S2_CPL; ++u) {
                                     bc[u] += rc[u];
                                     bq[u] = bq[u] + rq[u];
                                 }
                             });
            k = ke - 1;
            double *row = t2 + (int64_t)listed(rows, ke).t * L;
#pragma unroll 1
            for (int u = 0; u < S2_CPL; ++u)
                if (colB0 - u >= 0)
                    row[colB0 - u] = class_term2(pick(bc, u), pick(bq, u), p.q, p.sgn, p.hmax);
        }
    }
    __syncthreads();
    // 4. FP64 values of the candidate pairs of this wavefront's block; rows in
    // m3 form the terms of counts past the table anew (3 wrote over them)
    double best = -INFINITY;
    long long code = 0x7fffffffffffffffLL;
    if (m4) {
        CT ac[S2_CPL];
        double aq[S2_CPL];
        carry_in<1>(sh, L, w, ac, aq);
        auto add = [&](int, const CT(&rc)[S2_CPL], const double(&rq)[S2_CPL], const float(&)[S2_CPL]) {
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u) {
                ac[u] += rc[u];
                aq[u] = aq[u] + rq[u];
            }
        };
        for (int l = 0; m4;) {
            int le = __ffsll((long long)m4) - 1; // the next candidate
            if ((m3 >> l) & 1u) {
                uint32_t c[S2_CPL];
                double t[S2_CPL], rq[S2_CPL];
                CT rc[S2_CPL];
                const float x[S2_CPL] = {};
                const S2Row r = listed(rows, b0 + l);
                load_row<1>(p, r, c);
                row_terms<1, true>(p, r.t, c, t);
                row_sums<CT>(c, t, rc, rq);
                add(b0 + l, rc, rq, x);
                if (l != le) {
                    ++l;
                    continue;
                }
            } else {
                const uint64_t over = m3 >> l; // bit 0 is clear
                const int stop = over ? l + __ffsll((long long)over) - 2 : 63;
                const bool reach = le <= stop;
                const int last = reach ? le : stop;
                for_rows<1, CT>(p, rows, b0 + l, last - l + 1, none, add);
                l = last;
                if (!reach) {
                    ++l;
                    continue;
                }
            }
            m4 &= m4 - 1;
            const int k = b0 + le, t = listed(rows, k).t, r2 = listed(rows, k + 1).t;
            const float *row2 = k2 + (int64_t)r2 * L;
            const double *row2d = t2 + (int64_t)r2 * L;
#pragma unroll 1
            for (int u = 0; u < S2_CPL; ++u) {
                const int col = posl + u;
                if (col <= L - 2) {
                    const CT c = pick(ac, u);
                    const double q = pick(aq, u);
                    const float key = class_key32(c, q, p) + row2[col + 1];
                    if (all || (double)key >= T) {
                        const double lam = class_term2(c, q, p.q, p.sgn, p.hmax) + row2d[col + 1];
                        const long long cd = ((long long)t << 12) | col;
                        if (lam > -INFINITY && (lam > best || (lam == best && cd < code))) {
                            best = lam;
                            code = cd;
                        }
                    }
                }
            }
            l = le + 1;
        }
    }
    // first best pair of the wavefront, then of the workgroup
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const double b2 = __shfl_xor(best, o, 64);
        const long long c2 = __shfl_xor(code, o, 64);
        if (b2 > best || (b2 == best && c2 < code)) {
            best = b2;
            code = c2;
        }
    }
    if (lane == 0) {
        sh.wb[w] = best;
        sh.wcode[w] = code;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 0; v < NW; ++v)
            if (sh.wb[v] > best || (sh.wb[v] == best && sh.wcode[v] < code)) {
                best = sh.wb[v];
                code = sh.wcode[v];
            }
        if (!(best > -INFINITY)) {
            *thr_t = *thr_s = -1;
            *obj_p = NAN;
            *status_p = TS_PROBLEM_DEGENERATE;
        } else {
            *thr_t = (int32_t)(code >> 12);
            *thr_s = (int32_t)(code & 4095);
            *obj_p = p.sgn == 0.0 ? best : expm1(p.sgn * best) / (1.0 - p.q);
            *status_p = TS_PROBLEM_OK;
        }
    }
}

// Which rows of each image hold counts, the image's pixel count and each
// row's band of columns holding counts: one wavefront per group of 16 rows,
// all 16 rows' loads in flight together (bounded by reading the histograms
// once).  mask[s][g] bit d: row 16 g + d holds counts; cnt[s][g]: its pixels;
// band[s][t]: the first column of the lowest lane holding counts in row t | the
// last of the highest << 16 (0xffff | 0 << 16 for an empty row).
__global__ void __launch_bounds__(64) k_rows2d(const uint32_t *__restrict__ hist, int L, int groups,
                                               uint16_t *__restrict__ mask, uint64_t *__restrict__ cnt,
                                               uint32_t *__restrict__ band)
{
    const int s0 = blockIdx.x / groups, g = blockIdx.x % groups, lane = threadIdx.x & 63;
    const uint32_t *h = hist + (int64_t)s0 * L * L;
    const bool vec = (L % S2_CPL) == 0 && ((uintptr_t)h & 15) == 0;
    uint32_t c[16][S2_CPL];
#pragma unroll
    for (int d = 0; d < 16; ++d) // rows past L reload row L-1 and count as empty
        load_row<1>(h, L, vec, min(16 * g + d, L - 1), 0, L - 1, c[d]);
    uint32_t bits = 0, mine = 0xffffu; // lane d < 16 keeps row d's band
    uint64_t n = 0;
#pragma unroll
    for (int d = 0; d < 16; ++d) {
        const bool in = 16 * g + d < L;
        const uint64_t occ = __ballot((c[d][0] | c[d][1] | c[d][2] | c[d][3]) != 0u && in);
        if (in) {
#pragma unroll
            for (int u = 0; u < S2_CPL; ++u)
                n += c[d][u];
        }
        if (occ) {
            bits |= 1u << d;
            const uint32_t lo = S2_CPL * (__ffsll((long long)occ) - 1);
            const uint32_t hi = S2_CPL * (63 - __clzll((long long)occ)) + S2_CPL - 1;
            mine = lane == d ? lo | hi << 16 : mine;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        n += __shfl_xor(n, o, 64);
    if (lane < 16 && 16 * g + lane < L)
        band[(int64_t)s0 * L + 16 * g + lane] = mine;
    if (threadIdx.x == 0) {
        mask[(int64_t)s0 * 16 + g] = (uint16_t)bits;
        cnt[(int64_t)s0 * 16 + g] = n;
    }
}

// Workgroup b takes image s0 = 8 (b / 8 / nq) + b % 8 and q index (b / 8) %
// nq: the nq workgroups of an image are 8 apart, so they land on the same XCD
// (workgroups go to the 8 XCDs in turn) and share its L2 for the image's
// rows; workgroups with s0 >= nseg do nothing.
template <int NW>
__global__ void __launch_bounds__(64 * NW, NW == 8 ? 4 : 1)
    k_search2d(const uint32_t *__restrict__ hist, int nseg, int nq, int L, Q2List ql, float *__restrict__ k2all,
               double *__restrict__ t2all, const uint16_t *__restrict__ mask, const uint64_t *__restrict__ cnt,
               const uint32_t *__restrict__ band, int32_t *__restrict__ thr, double *__restrict__ obj,
               int32_t *__restrict__ status)
{
    extern __shared__ double s2_lds[]; // S2Lds of either count type
    S2Lds<NW, uint32_t> &sh = *reinterpret_cast<S2Lds<NW, uint32_t> *>(s2_lds);
    S2Lds<NW, uint64_t> &sh64 = *reinterpret_cast<S2Lds<NW, uint64_t> *>(s2_lds);
    const int lane = threadIdx.x & 63;
    const int slot = blockIdx.x >> 3, s0 = (slot / nq) * 8 + (blockIdx.x & 7), j = slot % nq;
    if (s0 >= nseg)
        return;
    const int prob = j * nseg + s0;
    // the image's pixel count (every wavefront)
    const int groups = (L + 15) / 16;
    uint64_t n = lane < groups ? cnt[(int64_t)s0 * 16 + lane] : 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        n += __shfl_xor(n, o, 64);
    // thr is [nq][2][nseg]: t at row 0, s at row 1 of this q
    int32_t *thr_t = thr + (int64_t)(2 * j) * nseg + s0, *thr_s = thr_t + nseg;
    if (n == 0) {
        if (threadIdx.x == 0) {
            *thr_t = *thr_s = -1;
            obj[prob] = NAN;
            status[prob] = TS_PROBLEM_EMPTY;
        }
        return;
    }
    S2 p;
    p.h = hist + (int64_t)s0 * L * L;
    p.L = L;
    p.vec = (L % S2_CPL) == 0 && ((uintptr_t)p.h & 15) == 0;
    p.q = ql.q[j];
    p.sgn = uniform(p.q == 1.0 ? 0.0 : (p.q < 1.0 ? 1.0 : -1.0));
    p.hmax = uniform((p.q == 1.0 ? 1.0 : fabs(1.0 - p.q)) * 2.0 * log((double)L)); // a class holds at most L^2 cells
    p.mq = uniform((float)(-p.q));
    p.sg = uniform(p.q < 1.0 ? 1.0f : -1.0f);
    p.gmax = uniform((float)(p.hmax * 1.4426950408889634 * (1.0 + 0x1p-20)));
    float *k2 = k2all + (int64_t)prob * L * L;
    double *t2 = t2all + (int64_t)prob * L * L;
    p.big = t2;
    // the rows holding counts, in increasing order (wavefront 0): lane l looks
    // at rows 4l .. 4l+3 (groups past the last hold no rows below L); the
    // table of terms and the rows' bands
    auto setup = [&](auto &sl) {
        p.tab = sl.tab;
        if (threadIdx.x < 64) {
            const uint32_t g16 = (4 * lane) / 16 < groups ? mask[(int64_t)s0 * 16 + (4 * lane) / 16] : 0u;
            uint32_t nib = (g16 >> ((4 * lane) % 16)) & 0xfu;
            if (4 * lane + 4 > L)
                nib &= (4 * lane < L) ? (1u << (L - 4 * lane)) - 1u : 0u;
            uint32_t w = wave_excl_sum<uint32_t>((uint32_t)__popc(nib));
#pragma unroll
            for (int d = 0; d < 4; ++d)
                if (nib & (1u << d)) {
                    const uint32_t bd = band[(int64_t)s0 * L + 4 * lane + d];
                    sl.rows[w++] = (uint32_t)(4 * lane + d) | (bd & 0xffu) << 8 | (bd >> 16) << 16;
                }
            if (lane == 63)
                sl.nrows = (int)w;
        }
#pragma unroll 1
        for (int i = threadIdx.x; i < S2_TAB; i += blockDim.x)
            sl.tab[i] = cterm((uint32_t)i, p.q);
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(sl.nrows);
    };
    if (n >> 32) {
        const int R = setup(sh64);
        search2d_body<NW, uint64_t>(p, (double)n, R, sh64, k2, t2, thr_t, thr_s, obj + prob, status + prob);
    } else {
        const int R = setup(sh);
        search2d_body<NW, uint32_t>(p, (double)n, R, sh, k2, t2, thr_t, thr_s, obj + prob, status + prob);
    }
}

// Workspace: FP64 terms [nprob][L][L], FP32 keys [nprob][L][L], row masks
// uint16 [nseg][16], pixel counts uint64 [nseg][16] and row bands uint32
// [nseg][L], each part starting 256-byte aligned (the workspace itself must
// be 8-byte aligned).
static size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t search2d_workspace_bytes(int nseg, int nq, int L)
{
    const size_t cells = (size_t)nseg * nq * L * L;
    return up256(cells * sizeof(double)) + up256(cells * sizeof(float)) + up256((size_t)nseg * 16 * 2) +
           up256((size_t)nseg * 16 * 8) + (size_t)nseg * L * 4;
}

ts_status launch_search2d(const uint32_t *hist, int nseg, int L, int nq, const double *q, void *ws, int32_t *thr,
                          double *obj, int32_t *status, hipStream_t st)
{
    Q2List ql;
    for (int i = 0; i < TS_MAX_Q; ++i)
        ql.q[i] = q[i < nq ? i : 0];
    const size_t cells = (size_t)nseg * nq * L * L;
    char *w = (char *)ws;
    double *t2 = (double *)w;
    float *k2 = (float *)(w + up256(cells * sizeof(double)));
    uint16_t *mask = (uint16_t *)(w + up256(cells * sizeof(double)) + up256(cells * sizeof(float)));
    uint64_t *cnt = (uint64_t *)((char *)mask + up256((size_t)nseg * 16 * 2));
    uint32_t *band = (uint32_t *)((char *)cnt + up256((size_t)nseg * 16 * 8));
    const int groups = (L + 15) / 16;
    hipLaunchKernelGGL(k_rows2d, dim3((unsigned)(nseg * groups)), dim3(64), 0, st, hist, L, groups, mask, cnt, band);
    const unsigned nblk = (unsigned)((nseg + 7) / 8 * 8 * nq);
    // Sixteen wavefronts per problem while every problem then has a CU of its
    // own, eight (two problems per CU) beyond: 37 problems of 200 levels 56
    // against 62 us, 120 of 256 levels 86 against 99, 900 of 256 levels 266
    // against 212 (with the row pass).
    const bool few = (int64_t)nseg * nq <= device_cu_count();
#define TS_S2(NW)                                                                                                   \
    const size_t lds = sizeof(S2Lds<NW, uint64_t>);                                                               \
    allow_dynamic_lds((const void *)k_search2d<NW>, lds);                                                         \
    hipLaunchKernelGGL(k_search2d<NW>, dim3(nblk), dim3(64 * NW), lds, st, hist, nseg, nq, L, ql, k2, t2, mask,   \
                       cnt, band, thr, obj, status)
    if (few) {
        TS_S2(16);
    } else {
        TS_S2(8);
    }
#undef TS_S2
    return check_launch("ts_threshold_search2d");
}

} // namespace ts
