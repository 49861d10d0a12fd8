// k_label.hip -- the thresholding kernel function (Algorithm 1) generalised
// to k thresholds, fused with the bin map: label(v) = #{j : b(v) > t_j}.
//
// No bin index is materialised.  For the window rule of ts_binning,
// b(v) > t  <=>  v >= cut(t) = lo + ceil((t + 1) * W / L)   (W = hi - lo + 1),
// which also covers values outside the window (below lo: bin 0, never above a
// threshold; above hi: bin L-1, above every threshold since cut(t) <= hi + 1).
// So each voxel costs k integer compares; on the vector path two voxels
// share each operation (packed 16-bit arithmetic).  One-shot grid over tiles
// of the flattened batch; 16-byte loads of 8 voxels and 8-byte stores of 8
// labels at any alignment.
//
// Bound by HBM: 2 B read and NS B written per voxel.  300 slices, k = 2:
// 512 x 512 with three sets 67 us (5.9 TB/s), with one 39 us; 511 x 511 (every
// slice and output starts at another alignment) with three sets 65 us (6.0
// TB/s; 221 us when such tiles went voxel by voxel), with one 41 us (49).
#include <algorithm>

#include "common.h"
#include "label_dev.h"

namespace ts {

// Cut values of problem s for every set, one lane per (set, threshold): lane KM
// u + j holds cut j of set u.  (t+1) W <= 4095 * 65536 < 2^32, so the ceiling
// division is exact in uint32.  NS * KM <= 64 lanes.
template <int NS, int KM>
__device__ __forceinline__ int wave_cuts(const LabelSets &sets, int s, int k, const BinMap &bm)
{
    static_assert(NS * KM <= 64, "one lane per (set, threshold)");
    const int lane = threadIdx.x & 63;
    const int u = lane / KM, j = lane % KM;
    const int32_t *row = sets.thr[0];
#pragma unroll
    for (int u2 = 1; u2 < NS; ++u2)
        row = u == u2 ? sets.thr[u2] : row;
    // one load per lane, whatever k: the row's order is checked against the
    // neighbour lane's value, so a tile waits for one round trip (with a loop
    // over the row, which waited for k of them, two sets of four thresholds
    // over 300 512 x 512 slices took 78 us instead of 55)
    const bool have = u < NS && j < k;
    const int t = have ? row[(int64_t)s * k + j] : 0;
    const int before = __builtin_amdgcn_update_dpp(0, t, 0x138, 0xf, 0xf, false); // wave_shr:1
    const bool good = !have || (t >= 0 && t <= bm.L - 2 && (j == 0 || t > before));
    const unsigned long long bal = __ballot(good);
    // the whole row must be a strictly ascending tuple in [0, L-2]
    const bool ok = have && ((bal >> (u * KM)) & ((1ull << KM) - 1ull)) == (1ull << KM) - 1ull;
    const uint32_t W = (uint32_t)((int64_t)bm.hi - bm.lo + 1);
    return ok ? bm.lo + (int)(((uint32_t)(t + 1) * W + (uint32_t)bm.L - 1) / (uint32_t)bm.L) : 0x7fffffff;
}

// Set u's cuts from the lanes that hold them, uniform over the wavefront.
template <int KM>
__device__ __forceinline__ PCuts<KM> set_cuts(int c, int u)
{
    Cuts<KM> cuts;
#pragma unroll
    for (int j = 0; j < KM; ++j)
        cuts.c[j] = __builtin_amdgcn_readlane(c, KM * u + j);
    return pack_cuts(cuts);
}

// The n <= blockDim * 8 * U voxels at src (one piece of one problem): 16-byte
// loads of 8 voxels, every load of a thread in flight before the first is
// used, 8-byte stores per set; the last n mod 8 voxel by voxel.  AL: src is
// 16-byte and every dst 8-byte aligned (else any alignment).
// Above eight cuts one set after the other, so that one set's cuts are held at a
// time (all 48 of three sets spilled: 20000 problems of 1000 voxels, 751 -> 908
// us, now 741).
template <int NS, int U, int KM, bool AL>
__device__ __forceinline__ void label_piece(const TS_GLOBAL int16_t *src, TS_GLOBAL uint8_t *const (&dst)[NS], int n,
                                            int c)
{
    constexpr bool ALL = KM <= 8; // every set's cuts at once
    PCuts<KM> pc[ALL ? NS : 1];
    if constexpr (ALL) {
#pragma unroll
        for (int u = 0; u < NS; ++u)
            pc[u] = set_cuts<KM>(c, u);
    }
    const TS_GLOBAL v4i_any *vp = reinterpret_cast<const TS_GLOBAL v4i_any *>(src);
    const int nvec = n >> 3, tb = nvec << 3;
    v4i w[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int i = threadIdx.x + j * blockDim.x;
        w[j] = i < nvec ? (v4i)__builtin_nontemporal_load(vp + i) : v4i{0, 0, 0, 0};
    }
    if constexpr (ALL) {
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = threadIdx.x + j * blockDim.x;
            if (i < nvec) {
#pragma unroll
                for (int u = 0; u < NS; ++u)
                    store_lab8(dst[u], i, lab8(w[j], pc[u]), AL);
            }
        }
        if ((int)threadIdx.x < n - tb) {
            const int v = src[tb + threadIdx.x];
#pragma unroll
            for (int u = 0; u < NS; ++u)
                dst[u][tb + threadIdx.x] = (uint8_t)lab1p(v, pc[u]);
        }
    } else {
        const int v = (int)threadIdx.x < n - tb ? src[tb + threadIdx.x] : 0;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            pc[0] = set_cuts<KM>(c, u);
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int i = threadIdx.x + j * blockDim.x;
                if (i < nvec)
                    store_lab8(dst[u], i, lab8(w[j], pc[0]), AL);
            }
            if ((int)threadIdx.x < n - tb)
                dst[u][tb + threadIdx.x] = (uint8_t)lab1p(v, pc[0]);
        }
    }
}

// Problems a tile may span and still be labelled piece by piece.
constexpr int LABEL_MAX_PIECES = 4;

// One workgroup per tile of blockDim * 8 * U voxels of the flattened batch,
// one pass over the voxels for NS threshold sets (up to TS_MAX_LABEL_SETS):
// each 16-byte load of 8 voxels feeds one 8-byte store per set.  A tile that
// spans up to LABEL_MAX_PIECES problems is labelled one piece after the other
// with vector accesses, at any alignment; a tile over more (tiny problems,
// whose pieces would each cost a round trip for a few voxels) voxel by voxel.
// A one-shot grid keeps the voxels in flight at any time in one window of
// HBM, which streams faster on MI355X than long per-workgroup ranges.
template <int NS, int U, int KM>
__global__ void __launch_bounds__(1024) k_label(const int16_t *const *__restrict__ vox,
                                                const int64_t *__restrict__ offs, int nseg, int64_t total, BinMap bm,
                                                LabelSets sets, int k)
{
    const int64_t T = (int64_t)blockDim.x * 8 * U;
    const int64_t t0 = (int64_t)blockIdx.x * T;
    const int64_t t1 = min(total, t0 + T);
    // everything the tile needs from the guessed segment is loaded in one
    // round trip; a wrong guess (uneven segments) is corrected afterwards
    int s = guess_segment(nseg, total, t0);
    int64_t o0 = offs[s], o1 = offs[s + 1];
    const int16_t *vs = vox[s];
    uint8_t *os[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u)
        os[u] = sets.out[u][s];
    int cuts = wave_cuts<NS, KM>(sets, s, k, bm);
    if (!(o0 <= t0 && t0 < o1)) {
        s = find_segment(offs, nseg, t0);
        while (s + 1 < nseg && offs[s + 1] <= t0) // skip empty segments
            ++s;
        o0 = offs[s];
        o1 = offs[s + 1];
        vs = vox[s];
#pragma unroll
        for (int u = 0; u < NS; ++u)
            os[u] = sets.out[u][s];
        cuts = wave_cuts<NS, KM>(sets, s, k, bm);
    }
    if (t1 <= o1) { // the whole tile in one problem
        const TS_GLOBAL int16_t *src = gp(vs) + (t0 - o0);
        bool al = ((uintptr_t)src & 15u) == 0;
        TS_GLOBAL uint8_t *dst[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            dst[u] = gpw(os[u]) + (t0 - o0);
            al = al && ((uintptr_t)dst[u] & 7u) == 0;
        }
        if (al) {
            label_piece<NS, U, KM, true>(src, dst, (int)(t1 - t0), cuts);
            return;
        }
    }
    if (t1 <= o1 || t1 <= offs[min(s + LABEL_MAX_PIECES, nseg)]) { // offs[s] <= t0 < offs[s + 1]: at most LABEL_MAX_PIECES problems
        int64_t pos = t0;
        for (;;) {
            const int64_t end = min(t1, o1);
            TS_GLOBAL uint8_t *dst[NS];
#pragma unroll
            for (int u = 0; u < NS; ++u)
                dst[u] = gpw(os[u]) + (pos - o0);
            label_piece<NS, U, KM, false>(gp(vs) + (pos - o0), dst, (int)(end - pos), cuts);
            if (end >= t1)
                return;
            pos = end; // the next problem (an empty one gives an empty piece)
            ++s;
            o0 = o1;
            o1 = offs[s + 1];
            vs = vox[s];
#pragma unroll
            for (int u = 0; u < NS; ++u)
                os[u] = sets.out[u][s];
            cuts = wave_cuts<NS, KM>(sets, s, k, bm);
        }
    }
    // many problems in the tile: voxel by voxel, segments walked forward
    for (int64_t pos = t0 + threadIdx.x; pos < t1; pos += blockDim.x) {
        int sv = s;
        while (offs[sv + 1] <= pos)
            ++sv;
        const int64_t i = pos - offs[sv];
        const int v = gp(vox[sv])[i];
#pragma unroll
        for (int u = 0; u < NS; ++u)
            gpw(sets.out[u][sv])[i] = (uint8_t)lab1(v, make_cuts<KM>(sets.thr[u] + (int64_t)sv * k, k, bm));
    }
}

template <int NS, int KM>
static void launch_label_ns(int U, dim3 g, dim3 blk, hipStream_t st, const ts_batch &b, const BinMap &bm,
                            const LabelSets &sets, int k)
{
    if (U == 1)
        hipLaunchKernelGGL((k_label<NS, 1, KM>), g, blk, 0, st, b.vox, b.offs, b.nseg, b.total, bm, sets, k);
    else if (U == 2)
        hipLaunchKernelGGL((k_label<NS, 2, KM>), g, blk, 0, st, b.vox, b.offs, b.nseg, b.total, bm, sets, k);
    else
        hipLaunchKernelGGL((k_label<NS, 4, KM>), g, blk, 0, st, b.vox, b.offs, b.nseg, b.total, bm, sets, k);
}

template <int KM>
static void launch_label_km(int nsets, int U, dim3 g, dim3 blk, hipStream_t st, const ts_batch &b, const BinMap &bm,
                            const LabelSets &sets, int k)
{
    switch (nsets) {
    case 1: launch_label_ns<1, KM>(U, g, blk, st, b, bm, sets, k); break;
    case 2: launch_label_ns<2, KM>(U, g, blk, st, b, bm, sets, k); break;
    case 3: launch_label_ns<3, KM>(U, g, blk, st, b, bm, sets, k); break;
    default: launch_label_ns<4, KM>(U, g, blk, st, b, bm, sets, k); break;
    }
}

ts_status launch_label(const ts_batch &b, const BinMap &bm, const LabelSets &sets, int nsets, int k, const Tune &t,
                       hipStream_t st)
{
    if (b.total == 0)
        return TS_OK;
    const int64_t T = (int64_t)t.label_block * 8 * t.label_vecs;
    const int64_t grid = (b.total + T - 1) / T;
    if (grid > 0x7fffffff)
        return fail(TS_ERR_INVALID_ARG, "ts_label: batch too large for one launch");
    const dim3 g((unsigned)grid), blk(t.label_block);
    // as many cut values as thresholds up to 4, then the next of 6, 8 and 16:
    // every cut costs three packed operations per voxel pair and set, used or
    // not, and past about six of them per set the pass is bound by these
    // instead of HBM (300 512 x 512 slices, two sets: k = 4 55 us, 148 us with
    // 16 cuts; k = 6 66 us, 152 us with 16)
    switch (k) {
    case 1: launch_label_km<1>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    case 2: launch_label_km<2>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    case 3: launch_label_km<3>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    case 4: launch_label_km<4>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    case 5:
    case 6: launch_label_km<6>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    case 7:
    case 8: launch_label_km<8>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    default: launch_label_km<LABEL_MAX_K>(nsets, t.label_vecs, g, blk, st, b, bm, sets, k); break;
    }
    return check_launch("ts_label");
}

} // namespace ts
