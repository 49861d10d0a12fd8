// k_dp.hip -- exact multilevel threshold search by dynamic programming over
// the class boundaries, for any k up to TS_DP_MAX_K (Tsallis-entropy section:
// the objective of k thresholds is 1 + (1-q) S = prod_j Q_j / w_j^q, so the
// arg max of S is the arg max of the sum of the class terms
// g(a..b) = sgn(1-q) (ln Q_[a,b] - q ln w_[a,b]), or of the class Shannon
// entropies for q = 1; a sum over consecutive classes is separable).
//
// Completion values, for a threshold at t and m more thresholds after it:
//   V_0(t) = g(t+1 .. L-1)
//   V_m(t) = max over t < u <= L-2 of g(t+1 .. u) + V_{m-1}(u)
// and the maximum M = max over t of g(0 .. t) + V_{k-1}(t).  FP64 addition is
// monotone, so M is exactly the largest of the per-tuple sums formed right
// to left.  The tuple is rebuilt from the left: t_1 is the smallest t whose
// value equals M, then t_j the smallest u > t_{j-1} reaching V_{k-j+1}(t_{j-1})
// (kept by the level kernels; found again by k_dp_block, whose recomputed
// values equal the maxima exactly), so the tuple is the first
// (lexicographically) of those reaching M.  A class with zero mass has g = -inf.  Empty bins repeat
// P and Q bit for bit (ts_prefix), so tuples that differ inside a run of
// empty bins tie exactly, as in the exhaustive search.
//
// Only bins that change P or Q can be thresholds: where bin u repeats P and Q
// of bin u-1, every class ending at u equals the one ending at u-1, every
// class starting after u the one starting after u-1, and the class {u} is
// empty.  V_m(u) is then V_m(u-1) bit for bit, its tuples tie with those of
// u-1, and the first of them holds u-1.  So both forms leave such bins out.
//
// Work: n (n-1) / 2 class terms (two FP64 logarithms each) per problem and
// level, n the bins left, against C(L-1, k) tuples for the exhaustive search.
// k_dp_block (a whole problem per workgroup) forms each term once for all k
// levels.
#include <math.h>

#include "common.h"

namespace ts {

constexpr int DP_THREADS = 256;
constexpr int DP_FINAL_THREADS = 1024;
constexpr int DP_FINAL_LDS = 16384; // first indices staged by k_dp_final
constexpr int DP_BLOCK_BINS = 256; // levels of a problem that one workgroup takes whole
constexpr int DP_BLOCK_WAVES = 8;  // of such a workgroup, at most
constexpr int DP_ROWS = 4;         // rows of a workgroup of k_dp_rows

struct DPQ {
    double q[TS_MAX_Q];
};

struct DPArgs {
    const double *P, *Q;
    int nseg, nprob, L, k;
    DPQ qs;
    // Workspace of k planes of nprob L doubles: V_m in plane m & 1 (V_0 is not
    // kept), then the levels' first indices.
    double *V;
};

// Row of V_m, m >= 1, of problem s.
__device__ __forceinline__ double *dp_v(const DPArgs &a, int m, int s)
{
    return a.V + ((int64_t)(a.k > 2 ? m & 1 : 0) * a.nprob + s) * a.L;
}

// Row of level m's first indices, 1 <= m < k, of problem s: after the planes
// of V (one for k = 2, two for k > 2), of 2 (k - 1) bytes per bin in all,
// which the remaining k - 1 or k - 2 planes of 8 bytes hold.
__device__ __forceinline__ uint16_t *dp_next(const DPArgs &a, int m, int s)
{
    uint16_t *rows = (uint16_t *)(a.V + (int64_t)(a.k > 2 ? 2 : 1) * a.nprob * a.L);
    return rows + ((int64_t)(m - 1) * a.nprob + s) * a.L;
}

__device__ __forceinline__ void dp_consts(double q, int L, double &sgn, double &hmax)
{
    sgn = q == 1.0 ? 0.0 : (q < 1.0 ? 1.0 : -1.0);
    hmax = (q == 1.0 ? 1.0 : fabs(1.0 - q)) * log((double)L); // a class holds at most L bins
}

// Class term from the class's differences of P and Q; -inf if the class has
// zero mass; clamped to [0, hmax].
__device__ __forceinline__ double dp_h(double dP, double dQ, double q, double sgn, double hmax)
{
    const double h = sgn == 0.0 ? log(dP) - dQ / dP : sgn * (log(dQ) - q * log(dP));
    return dP > 0.0 ? fmin(fmax(h, 0.0), hmax) : -INFINITY;
}

// Bin u repeats the prefix sums of the bin before it (of nothing for u = 0).
__device__ __forceinline__ bool dp_repeats(const double *P, const double *Q, int u)
{
    const double pa = u ? P[u - 1] : 0.0, qa = u ? Q[u - 1] : 0.0;
    return P[u] == pa && Q[u] == qa;
}

__device__ __forceinline__ double wave_max_d(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

__device__ __forceinline__ double readlane_d(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// V_m(t) and the first u reaching it for one (problem, t) per workgroup: the
// threads split u.  Bounded by one round of loads and the two logarithms of
// its terms; rows and terms of repeating bins are left out (their V is never
// read).  FIRST is m = 1, which forms V_0(u) itself: four logarithms per term
// of one level take less than the launch of a kernel for V_0.
template <bool FIRST>
__global__ void __launch_bounds__(DP_THREADS) k_dp_level(DPArgs a, int m)
{
    __shared__ double red[DP_THREADS / 64];
    __shared__ int redu[DP_THREADS / 64];
    const int L = a.L;
    const int s = blockIdx.x / (L - 1), t = blockIdx.x % (L - 1);
    const double q = a.qs.q[s / a.nseg];
    const double *P = a.P + (int64_t)(s % a.nseg) * L, *Q = a.Q + (int64_t)s * L;
    const double *Vp = dp_v(a, m - 1, s); // not read by FIRST
    const bool skip = dp_repeats(P, Q, t);
    const double pt = P[t], qt = Q[t], PL = P[L - 1], QL = Q[L - 1];
    int u = t + 1 + threadIdx.x; // u - 1 >= 0; past the row's end its last bin is read and not used
    auto at = [&](int i) { return min(i, L - 1); };
    double pu = P[at(u)], qu = Q[at(u)], pb = P[at(u) - 1], qb = Q[at(u) - 1], vu = FIRST ? 0.0 : Vp[at(u)];
    if (skip)
        return;
    double sgn, hmax;
    dp_consts(q, L, sgn, hmax);
    double best = -INFINITY;
    int bu = 0x7fffffff;
    while (__any(u <= L - 2)) {
        const bool use = u <= L - 2 && !(pu == pb && qu == qb);
        const int cu = u;
        const double cp = pu, cq = qu, cv = vu;
        u += blockDim.x;
        pu = P[at(u)], qu = Q[at(u)], pb = P[at(u) - 1], qb = Q[at(u) - 1], vu = FIRST ? 0.0 : Vp[at(u)];
        if (use) {
            const double v = FIRST ? dp_h(PL - cp, QL - cq, q, sgn, hmax) : cv;
            const double x = dp_h(cp - pt, cq - qt, q, sgn, hmax) + v;
            if (x > best) {
                best = x;
                bu = cu;
            }
        }
    }
    const double wbest = wave_max_d(best);
    bu = best == wbest ? bu : 0x7fffffff;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        bu = min(bu, __shfl_xor(bu, o, 64));
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = wbest;
        redu[threadIdx.x >> 6] = bu;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        best = wbest;
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (red[w] > best || (red[w] == best && redu[w] < bu)) {
                best = red[w];
                bu = redu[w];
            }
        dp_v(a, m, s)[t] = best;
        dp_next(a, m, s)[t] = (uint16_t)bu; // not read where the best is -inf
    }
}

// The same for DP_ROWS neighbouring t per workgroup, for calls whose workgroups
// fill the chip several times over: bounded by the logarithms of the class terms,
// of which FIRST forms two more per u for V_0 (half of all with one row per
// workgroup), and by the workgroups' own loads and reductions.  The level before
// leaves -inf for bins that repeat, so theirs are not compared again.  30 problems
// of 1024 levels, counts in every bin: k = 2 161 us, 240 by k_dp_level; k = 6 637
// against 754, and 319 against 367 on CT volumes.
template <bool FIRST>
__global__ void __launch_bounds__(DP_THREADS) k_dp_rows(DPArgs a, int m)
{
    constexpr int T = DP_ROWS;
    __shared__ double red[T][DP_THREADS / 64];
    __shared__ int redu[T][DP_THREADS / 64];
    const int L = a.L, nt = (L - 1 + T - 1) / T;
    const int s = blockIdx.x / nt, t0 = blockIdx.x % nt * T;
    const double q = a.qs.q[s / a.nseg];
    const double *P = a.P + (int64_t)(s % a.nseg) * L, *Q = a.Q + (int64_t)s * L;
    const double *Vp = dp_v(a, m - 1, s); // not read by FIRST
    double *V = dp_v(a, m, s);
    double pt[T], qt[T];
    bool row[T], some = false; // rows that can hold a threshold
#pragma unroll
    for (int j = 0; j < T; ++j) {
        const int t = min(t0 + j, L - 2);
        pt[j] = P[t];
        qt[j] = Q[t];
        row[j] = t0 + j <= L - 2 && !dp_repeats(P, Q, t);
        some = some || row[j];
    }
    const double PL = P[L - 1], QL = Q[L - 1];
    int u = t0 + 1 + threadIdx.x; // u - 1 >= 0; past the row's end its last bin is read and not used
    auto at = [&](int i) { return min(i, L - 1); };
    double pu = P[at(u)], qu = Q[at(u)];
    double pb = FIRST ? P[at(u) - 1] : 0.0, qb = FIRST ? Q[at(u) - 1] : 0.0, vu = FIRST ? 0.0 : Vp[at(u)];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < T; ++j)
            if (t0 + j <= L - 2 && !row[j])
                V[t0 + j] = -INFINITY;
    }
    if (!some)
        return;
    double sgn, hmax;
    dp_consts(q, L, sgn, hmax);
    double best[T];
    int bu[T];
#pragma unroll
    for (int j = 0; j < T; ++j) {
        best[j] = -INFINITY;
        bu[j] = 0x7fffffff;
    }
    while (__any(u <= L - 2)) {
        const bool use = u <= L - 2 && (FIRST ? !(pu == pb && qu == qb) : vu > -INFINITY);
        const int cu = u;
        const double cp = pu, cq = qu, cv = vu;
        u += blockDim.x;
        pu = P[at(u)], qu = Q[at(u)];
        if (FIRST)
            pb = P[at(u) - 1], qb = Q[at(u) - 1];
        else
            vu = Vp[at(u)];
        if (use) {
            const double v = FIRST ? dp_h(PL - cp, QL - cq, q, sgn, hmax) : cv;
#pragma unroll
            for (int j = 0; j < T; ++j) {
                if (row[j]) {
                    const double x = dp_h(cp - pt[j], cq - qt[j], q, sgn, hmax) + v;
                    if (x > best[j] && (j == 0 || cu > t0 + j)) {
                        best[j] = x;
                        bu[j] = cu;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < T; ++j) {
        const double wbest = wave_max_d(best[j]);
        int wu = best[j] == wbest ? bu[j] : 0x7fffffff;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            wu = min(wu, __shfl_xor(wu, o, 64));
        if ((threadIdx.x & 63) == 0) {
            red[j][threadIdx.x >> 6] = wbest;
            redu[j][threadIdx.x >> 6] = wu;
        }
    }
    __syncthreads();
    if (threadIdx.x < T) {
        const int j = threadIdx.x, t = t0 + j;
        double b = red[j][0];
        int ub = redu[j][0];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (red[j][w] > b || (red[j][w] == b && redu[j][w] < ub)) {
                b = red[j][w];
                ub = redu[j][w];
            }
        if (t <= L - 2) { // a repeating bin's is -inf (again)
            V[t] = b;
            dp_next(a, m, s)[t] = (uint16_t)ub; // not read where the best is -inf
        }
    }
}

// LDS of dp_tuple: two stages' exchange, by stage parity (one barrier each).
struct DPTupleLds {
    double d[2][4][DP_BLOCK_WAVES];
    int c[2][DP_BLOCK_WAVES];
};

// Result of a problem whose maximum is M (-inf: no tuple), its thresholds
// already written; by one thread.
__device__ __forceinline__ void dp_result(double M, bool ok, int k, double q, double sgn, double last, int32_t *out,
                                          double *obj, int32_t *status)
{
    if (ok) {
        *obj = sgn == 0.0 ? M : expm1(sgn * M) / (1.0 - q);
        *status = TS_PROBLEM_OK;
    } else {
        for (int j = 0; j < k; ++j)
            out[j] = -1;
        *obj = NAN;
        *status = last > 0.0 ? TS_PROBLEM_DEGENERATE : TS_PROBLEM_EMPTY;
    }
}

// The maximum and the first tuple reaching it, by the whole workgroup, from
// candidates c = 0 .. n-1, one per thread: bins bin[c], increasing, prefix
// sums Pc[c], Qc[c] and V[m][c].  The recomputed values equal the stored
// maxima bit for bit, so an index is always found; should one not be, the
// problem is reported degenerate rather than indexing past the row.  The
// thread that owns a stage's threshold hands its values on.
__device__ __forceinline__ void dp_tuple(DPTupleLds &sh, int n, int k, double q, double sgn, double hmax,
                                         double last, const int *bin, const double *Pc, const double *Qc,
                                         const double (*V)[DP_BLOCK_BINS], int32_t *out, double *obj,
                                         int32_t *status)
{
    const int c = threadIdx.x, lane = c & 63, w = c >> 6, waves = blockDim.x >> 6;
    constexpr int NONE = 0x7fffffff;
    const bool use = c < n;
    const double pc = use ? Pc[c] : 0.0, qc = use ? Qc[c] : 0.0;
    double v = use ? V[k - 1][c] : -INFINITY;
    double val = use ? dp_h(pc, qc, q, sgn, hmax) + v : -INFINITY;
    double M = wave_max_d(val);
    if (lane == 0)
        sh.d[1][0][w] = M;
    __syncthreads();
    for (int x = 0; x < waves; ++x)
        M = fmax(M, sh.d[1][0][x]);
    bool ok = M > -INFINITY;
    double target = M, pb = 0.0, qb = 0.0;
    int c0 = 0; // candidates from here on
    for (int j = 0; j < k && ok; ++j) {
        const bool in = use && c >= c0;
        if (j && in)
            val = dp_h(pc - pb, qc - qb, q, sgn, hmax) + v;
        const uint64_t hit = __ballot(in && val == target);
        const int par = j & 1;
        if (hit ? lane == __ffsll((long long)hit) - 1 : lane == 0) {
            sh.c[par][w] = hit ? c : NONE;
            sh.d[par][1][w] = v;
            sh.d[par][2][w] = pc;
            sh.d[par][3][w] = qc;
        }
        if (j + 1 < k && use)
            v = V[k - 2 - j][c];
        __syncthreads();
        int bw = 0;
        for (int x = 1; x < waves; ++x)
            if (sh.c[par][x] < sh.c[par][bw])
                bw = x;
        const int first = sh.c[par][bw];
        target = sh.d[par][1][bw];
        pb = sh.d[par][2][bw];
        qb = sh.d[par][3][bw];
        ok = first != NONE;
        if (ok && c == 0)
            out[j] = bin[first];
        c0 = first + 1; // unused once not ok
    }
    if (c == 0)
        dp_result(M, ok, k, q, sgn, last, out, obj, status);
}

// One workgroup per problem: the maximum over t_1 (smallest t_1 reaching it),
// then the thresholds after it from the levels' first indices, a chain of
// k - 1 dependent reads: of LDS where the rows of all levels fit.  (Found
// again by recomputing every stage's values it took 15 us at 1024 bins, k = 6:
// 2 (k - 1) logarithms per thread on one CU.)
__global__ void __launch_bounds__(DP_FINAL_THREADS) k_dp_final(DPArgs a, int32_t *__restrict__ thr,
                                                               double *__restrict__ obj,
                                                               int32_t *__restrict__ status)
{
    constexpr int NONE = 0x7fffffff;
    __shared__ uint16_t snext[DP_FINAL_LDS];
    __shared__ double redv[DP_FINAL_THREADS / 64];
    __shared__ int redt[DP_FINAL_THREADS / 64];
    const int s = blockIdx.x, L = a.L, k = a.k;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double q = a.qs.q[s / a.nseg];
    double sgn, hmax;
    dp_consts(q, L, sgn, hmax);
    const double *P = a.P + (int64_t)(s % a.nseg) * L, *Q = a.Q + (int64_t)s * L;
    const double PL = P[L - 1], QL = Q[L - 1];
    const bool staged = (k - 1) * L <= DP_FINAL_LDS;
    if (staged)
        for (int m = 1; m < k; ++m)
            for (int t = threadIdx.x; t < L - 1; t += blockDim.x) // rows of repeating bins: never written, never used
                snext[(m - 1) * L + t] = dp_next(a, m, s)[t];
    const double *Vk = dp_v(a, k - 1, s); // k = 1: V_0 is formed here
    double M = -INFINITY;
    int t1 = NONE;
    for (int t = threadIdx.x; t <= L - 2; t += blockDim.x) {
        const double p = P[t], x = Q[t], v = k > 1 ? Vk[t] : 0.0;
        if (dp_repeats(P, Q, t))
            continue;
        const double val = dp_h(p, x, q, sgn, hmax) + (k > 1 ? v : dp_h(PL - p, QL - x, q, sgn, hmax));
        if (val > M) {
            M = val;
            t1 = t;
        }
    }
    const double wM = wave_max_d(M);
    t1 = M == wM ? t1 : NONE;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        t1 = min(t1, __shfl_xor(t1, o, 64));
    if (lane == 0) {
        redv[w] = wM;
        redt[w] = t1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        M = wM;
        for (int x = 1; x < (int)(blockDim.x >> 6); ++x)
            if (redv[x] > M || (redv[x] == M && redt[x] < t1)) {
                M = redv[x];
                t1 = redt[x];
            }
        int32_t *out = thr + (int64_t)s * k;
        const bool ok = M > -INFINITY;
        if (ok) {
            out[0] = t1;
            int t = t1;
            for (int j = 1; j < k; ++j) {
                const int m = k - j; // t_{j+1} completes m thresholds after t_j
                t = min(staged ? (int)snext[(m - 1) * L + t] : (int)dp_next(a, m, s)[t], L - 2);
                out[j] = t;
            }
        }
        dp_result(M, ok, k, q, sgn, PL, out, obj + s, status + s);
    }
}

// A whole problem per workgroup, for L <= DP_BLOCK_BINS and k <= KM.  The
// bins that can be thresholds are compacted (candidates 0 .. n-1); thread c
// owns candidate c and holds V_m(c) as running maxima, and the candidates u
// are pushed to those before them from the last to the first,
// V_m(t) = max(V_m(t), g(t+1 .. u) + V_{m-1}(u)),
// so that a class term is formed once for all levels.  The terms do not
// depend on V: NW candidates u at a time, wavefront w forms those of the w-th
// for every t into an LDS tile, one step ahead of its use.  A step:
//   apply the NW u of the step before (V from LDS) to the wavefronts below
//   them; the wavefront owning this step's NW pushes them one by one, V(u)
//   read from its lane, and stores their V; the next step's tile; one
//   barrier (three tiles in turn).
// Bounded by the logarithms (about 95 FP64 instructions each, a dependent
// chain): 600 problems of 256 levels, about 130 candidates, k = 4: 88 us
// (three level launches and the tuple's took 733); one problem 36 us with eight
// wavefronts, 46 with four.  With the terms formed by each candidate's own
// wavefront, where the wavefronts wait for each other in turn, 115 and 102 us.
template <int KM, int NW>
__global__ void __launch_bounds__(64 * NW) k_dp_block(DPArgs a, int32_t *__restrict__ thr,
                                                      double *__restrict__ obj, int32_t *__restrict__ status)
{
    constexpr int DP_STEP = NW; // candidates pushed per step, one per wavefront
    __shared__ double sP[DP_BLOCK_BINS], sQ[DP_BLOCK_BINS]; // prefix sums of the candidates
    __shared__ double sV[KM][DP_BLOCK_BINS];
    extern __shared__ double sgdyn[]; // dp_block_lds
    double(*sg)[DP_STEP][DP_BLOCK_BINS] = reinterpret_cast<double(*)[DP_STEP][DP_BLOCK_BINS]>(sgdyn);
    __shared__ int sbin[DP_BLOCK_BINS];
    __shared__ int wcount[DP_STEP];
    __shared__ DPTupleLds sh;
    const int s = blockIdx.x, L = a.L, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double q = a.qs.q[s / a.nseg];
    double sgn, hmax;
    dp_consts(q, L, sgn, hmax);
    const double *P = a.P + (int64_t)(s % a.nseg) * L, *Q = a.Q + (int64_t)s * L;
    const double PL = P[L - 1], QL = Q[L - 1];
    const bool cand = tid <= L - 2 && !dp_repeats(P, Q, tid);
    const uint64_t bal = __ballot(cand);
    if (lane == 0)
        wcount[w] = __popcll(bal);
    __syncthreads();
    int base = 0, n = 0;
    for (int v = 0; v < DP_STEP; ++v) {
        base += v < w ? wcount[v] : 0;
        n += wcount[v];
    }
    n = __builtin_amdgcn_readfirstlane(n);
    if (cand) {
        const int c = base + __popcll(bal & ((1ull << lane) - 1ull));
        sP[c] = P[tid];
        sQ[c] = Q[tid];
        sbin[c] = tid;
    }
    __syncthreads();
    // the terms of u = 4 b + w for the candidates t of the chunks up to the
    // step's; -inf where t does not precede u
    auto tile = [&](int b, int buf) {
        const int u = DP_STEP * b + w;
        if (u >= n)
            return;
        const double pu = sP[u], qu = sQ[u];
        for (int t = lane; t < DP_STEP * (b + 1); t += 64) {
            const int tc = min(t, n - 1);
            const double g = dp_h(pu - sP[tc], qu - sQ[tc], q, sgn, hmax);
            sg[buf][w][t] = t < u ? g : -INFINITY;
        }
    };
    double acc[KM]; // V_m(tid); threads past the candidates stay at -inf
    acc[0] = tid < n ? dp_h(PL - sP[tid], QL - sQ[tid], q, sgn, hmax) : -INFINITY;
#pragma unroll
    for (int m = 1; m < KM; ++m)
        acc[m] = -INFINITY;
    const int nb = (n + DP_STEP - 1) / DP_STEP;
    int cur = 0, prv = 2, nxt = 1; // tiles of this step, of the one before, of the next
    if (nb > 0)
        tile(nb - 1, cur);
    __syncthreads();
    for (int b = nb - 1; b >= 0; --b) {
        const int u0 = DP_STEP * b, own = u0 >> 6;
        if (b + 1 < nb && w < (u0 + DP_STEP) >> 6) {
#pragma unroll
            for (int d = DP_STEP - 1; d >= 0; --d) {
                const int u = u0 + DP_STEP + d;
                if (u < n) {
                    const double g = sg[prv][d][tid];
#pragma unroll
                    for (int m = 1; m < KM; ++m)
                        acc[m] = fmax(acc[m], g + sV[m - 1][u]);
                }
            }
        }
        if (w == own) {
            // lanes past the tile's width hold candidates after u: no term
#pragma unroll
            for (int d = DP_STEP - 1; d >= 0; --d) {
                if (u0 + d < n) {
                    const double g = tid < u0 + d ? sg[cur][d][tid] : -INFINITY;
                    double vu[KM];
#pragma unroll
                    for (int m = 0; m < KM - 1; ++m)
                        vu[m] = readlane_d(acc[m], (u0 + d) & 63);
#pragma unroll
                    for (int m = 1; m < KM; ++m)
                        acc[m] = fmax(acc[m], g + vu[m - 1]);
                }
            }
            if (tid >= u0 && tid < u0 + DP_STEP) {
#pragma unroll
                for (int m = 0; m < KM; ++m)
                    sV[m][tid] = acc[m];
            }
        }
        if (b > 0)
            tile(b - 1, nxt);
        __syncthreads();
        const int x = prv;
        prv = cur;
        cur = nxt;
        nxt = x;
    }
    dp_tuple(sh, n, a.k, q, sgn, hmax, PL, sbin, sP, sQ, sV, thr + (int64_t)s * a.k, obj + s, status + s);
}

size_t dp_workspace_bytes(int nprob, int L, int k) { return (size_t)k * nprob * L * sizeof(double); }

ts_status launch_dp(const double *P, const double *Q, int nseg, int L, int k, int nq, const double *q, void *ws,
                    int32_t *thr, double *obj, int32_t *status, hipStream_t st)
{
    DPArgs a;
    a.P = P;
    a.Q = Q;
    a.nseg = nseg;
    a.nprob = nseg * nq;
    a.L = L;
    a.k = k;
    for (int j = 0; j < TS_MAX_Q; ++j)
        a.qs.q[j] = q[j < nq ? j : 0];
    a.V = (double *)ws;
    // One workgroup per problem takes as long for one problem as for the chip
    // full of them (a chain over the candidates); a level takes about 4.5 us and
    // more with every problem.  The lines below are fitted to both, measured over
    // 8 to 256 levels, 1 to 300 problems and k = 2 .. 16, between histograms with
    // counts in every bin and CT slices with counts in half of them, in us (one
    // workgroup / levels): 64 levels, 1 problem, k = 2 16 / 10 and 12 / 10, k = 4
    // 18 / 22 and 14 / 18; 128 levels, 24 problems, k = 4 35 / 37 and 20 / 32; 256
    // levels, 24 problems, k = 4 83 / 64 and 37 / 45, 60 problems 84 / 104 and 37 /
    // 83, k = 2 82 / 43 and 35 / 34.  Eight wavefronts per problem while every
    // problem has a CU of its own (256 levels, k = 4, 60 problems 111 -> 83 us) and
    // while two share one where a step has enough terms (257 problems, k = 2, 256
    // levels 160 -> 141 and, CT, 51 -> 47; 128 levels 58 -> 53 and 24 -> 24; k = 6, 256
    // levels 188 -> 170 and 64 -> 62, but 128 levels 72 -> 69 and 31 -> 33), four
    // beyond (900 problems of 128 levels with eight 56 us, 50 with four), below 32
    // levels and past 8 thresholds, where the chain itself bounds it.
    const double level = 6.0 + (k - 1) * (4.5 + 0.0018 * a.nprob * L);
    const double block = L * (k <= 4 ? 0.22 : k <= 8 ? 0.32 : 0.46);
    if (L <= DP_BLOCK_BINS && k > 1 && level >= block) {
        const int per_cu = L >= (k <= 4 ? 128 : 192) ? 2 : 1;
        const bool eight = a.nprob <= per_cu * device_cu_count() && L >= 32;
#define TS_DP(KM, NW)                                                                                               \
    const size_t lds = sizeof(double) * 3 * NW * DP_BLOCK_BINS;                                                   \
    allow_dynamic_lds((const void *)k_dp_block<KM, NW>, lds);                                                     \
    hipLaunchKernelGGL((k_dp_block<KM, NW>), dim3((unsigned)a.nprob), dim3(64 * NW), lds, st, a, thr, obj, status)
        if (k <= 4 && eight) {
            TS_DP(4, 8);
        } else if (k <= 4) {
            TS_DP(4, 4);
        } else if (k <= 8 && eight) {
            TS_DP(8, 8);
        } else if (k <= 8) {
            TS_DP(8, 4);
        } else {
            TS_DP(16, 4);
        }
#undef TS_DP
        return check_launch("ts_threshold_search_dp");
    }
    // four rows per workgroup where that leaves 1792 or more of them, seven per
    // CU: 30 problems of 300 levels, k = 6, 125 us against 140 (CT 78 against 85),
    // 12 of 512 levels 90 against 97, but 102 against 83 on CT volumes
    if ((int64_t)a.nprob * (L - 1) >= 7168) {
        const dim3 g((unsigned)((int64_t)a.nprob * ((L - 1 + DP_ROWS - 1) / DP_ROWS)));
        for (int m = 1; m < k; ++m)
            hipLaunchKernelGGL(m == 1 ? k_dp_rows<true> : k_dp_rows<false>, g, dim3(DP_THREADS), 0, st, a, m);
    } else {
        const dim3 g((unsigned)((int64_t)a.nprob * (L - 1)));
        for (int m = 1; m < k; ++m)
            hipLaunchKernelGGL(m == 1 ? k_dp_level<true> : k_dp_level<false>, g, dim3(DP_THREADS), 0, st, a, m);
    }
    hipLaunchKernelGGL(k_dp_final, dim3((unsigned)a.nprob), dim3(DP_FINAL_THREADS), 0, st, a, thr, obj, status);
    return check_launch("ts_threshold_search_dp");
}

} // namespace ts
