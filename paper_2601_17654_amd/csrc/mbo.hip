// Scores and batch selection of the multi-pass Bayesian optimisation (Section 4.3,
// Algorithm 1; reference point from Appendix C).
//
// Exploitation scores.  For each partition and each energy variant (total E, dynamic
// E - p_static * T, static p_static * T) a block turns the measured points into their
// staircase (strictly increasing T, strictly decreasing energy) and its hypervolume
// against r = 1.1 x the worst measured values.  The score kernel then stages a
// partition's three staircases in LDS and gives every candidate y its hypervolume
// improvement directly as the area that y adds: the part of [y.T, rT] x [y.E, rE] that
// no staircase step covers, summed strip by strip from y.T rightwards until a step at or
// below y.E closes it.  That is exact in real arithmetic and never forms the difference
// of two large hypervolumes.
//
// Selection.  Every pass is a top-k by (score descending, index ascending) over the
// partition's unmeasured candidates, with k <= 64.  A wave keeps its best entries sorted
// across its lanes; new candidates are compared against the k-th of them, and those that
// beat it are collected, sorted (by counting better ones) and merged in (reverse, lane-wise
// better, bitonic merge) 64 at a time.  Tiles of a partition reduce to one sorted list per
// pass; one block per partition merges the tile lists and assembles the batch in pass order.
#include <math.h>

#include "kr_device.h"
#include "kr_launch.h"

namespace kr {

__device__ __forceinline__ double energy_variant(int v, double t, double e, double ps)
{
    if (v == 0) return e;
    if (v == 1) return e - ps * t;  // no contraction: the library is built without it
    return ps * t;
}

struct HvMaxF64 {
    __device__ __forceinline__ double operator()(double a, double b) const { return b > a ? b : a; }
};
struct SumI32x {
    __device__ __forceinline__ int32_t operator()(int32_t a, int32_t b) const { return a + b; }
};

// One block per partition and variant: reference point, the variant's staircase and its HV.
// Bound by latency (a few hundred points): the three variants run side by side, and the
// pairwise tests read four points at a time without an early exit, so that the LDS reads
// overlap (64 partitions of 96 points: 62 us with one block per partition and a data-
// dependent loop, 16.5 us now).
__global__ void __launch_bounds__(KR_BLOCK) hvi_prep_kernel(HviArgs a)
{
    // points outside the box are stored as (+inf, +inf): they beat nothing
    __shared__ double sT[KR_HVI_MAX_OBS], sV[KR_HVI_MAX_OBS];
    __shared__ double fT[KR_HVI_MAX_OBS], fE[KR_HVI_MAX_OBS];
    __shared__ double red[2][KR_WAVES];
    __shared__ int32_t ired[KR_WAVES];
    const int g = blockIdx.x, v = blockIdx.y, tid = threadIdx.x;
    const int64_t o0 = a.obs_off[g], no64 = a.obs_off[g + 1] - o0;
    if (no64 < 1 || no64 > KR_HVI_MAX_OBS) {
        if (tid == 0) {
            a.fr_n[g * 3 + v] = -1;
            a.hv[g * 3 + v] = NAN;
            a.ref[g * 4 + 1 + v] = NAN;
            if (v == 0) a.ref[g * 4] = NAN;
        }
        return;
    }
    const int no = (int)no64;
    constexpr int kPer = KR_HVI_MAX_OBS / KR_BLOCK;
    double t[kPer], e[kPer];
    double mt = -INFINITY, me = -INFINITY;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * KR_BLOCK;
        t[q] = i < no ? a.T_obs[o0 + i] : INFINITY;
        e[q] = i < no ? energy_variant(v, t[q], a.E_obs[o0 + i], a.p_static) : INFINITY;
        if (i < no) {
            mt = t[q] > mt ? t[q] : mt;
            me = e[q] > me ? e[q] : me;
        }
    }
    const double rT = 1.1 * block_reduce(mt, (double)-INFINITY, HvMaxF64(), red[0]);
    const double rE = 1.1 * block_reduce(me, (double)-INFINITY, HvMaxF64(), red[1]);
    const int no4 = (no + 3) & ~3;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * KR_BLOCK;
        const bool in = t[q] < rT && e[q] < rE;
        if (i < no4) {
            sT[i] = in ? t[q] : INFINITY;
            sV[i] = in ? e[q] : INFINITY;
        }
    }
    __syncthreads();
    // a point opens a staircase step iff it is inside the box and no point inside the
    // box is at least as good in both and earlier in (T, energy, index) order
    bool keep[kPer];
    int32_t mine = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * KR_BLOCK;
        bool beaten = false;
        if (i < no) {
#pragma unroll 4
            for (int j = 0; j < no4; ++j) {
                const double tj = sT[j], ej = sV[j];
                beaten = beaten || (tj <= t[q] && ej <= e[q] &&
                                    (tj < t[q] || ej < e[q] || j < i));
            }
        }
        keep[q] = i < no && t[q] < rT && e[q] < rE && !beaten;
        mine += keep[q];
    }
    const int32_t s = block_reduce(mine, 0, SumI32x(), ired);
    // only the steps keep their times, so a step's rank is the number of smaller ones
    // (step times are distinct)
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * KR_BLOCK;
        if (i < no4 && !keep[q]) sT[i] = INFINITY;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int i = tid + q * KR_BLOCK;
        if (!keep[q]) continue;
        int r = 0;
#pragma unroll 4
        for (int j = 0; j < no4; ++j) r += sT[j] < t[q] ? 1 : 0;
        fT[r] = t[q];
        fE[r] = e[q];
        a.fr_T[(int64_t)v * a.n_obs + o0 + r] = t[q];
        a.fr_E[(int64_t)v * a.n_obs + o0 + r] = e[q];
    }
    __syncthreads();
    if (tid == 0) {
        double hv = 0.0;
        for (int r = 0; r < s; ++r) {
            const double next = r + 1 < s ? fT[r + 1] : rT;
            hv = hv + (next - fT[r]) * (rE - fE[r]);
        }
        a.hv[g * 3 + v] = hv;
        a.ref[g * 4 + 1 + v] = rE;
        if (v == 0) a.ref[g * 4] = rT;
        a.fr_n[g * 3 + v] = s;
    }
}

// Area that y = (t, e) adds to the staircase (fT, fE)[0, s) inside the box below (rT, rE).
__device__ __forceinline__ double hvi_one(const double *fT, const double *fE, int s, double rT,
                                          double rE, double t, double e)
{
    if (!(t < rT) || !(e < rE)) return 0.0;
    int lo = 0, hi = s;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (fT[mid] <= t) lo = mid + 1;
        else hi = mid;
    }
    double level = lo == 0 ? rE : fE[lo - 1];
    if (level <= e) return 0.0;  // a step at or before t is at or below e
    double area = 0.0, start = t;
    int i = lo;
    while (i < s && fE[i] > e) {
        area = area + (fT[i] - start) * (level - e);
        start = fT[i];
        level = fE[i];
        ++i;
    }
    const double end = i < s ? fT[i] : rT;
    return area + (end - start) * (level - e);
}

// Flat tiles of KR_HVI_TILE candidates; a tile visits every partition it overlaps.  One block
// more turns the preparation's verdicts into the status word and returns: a store ahead of the
// tiles' uniform loads would take those off the scalar cache (138 M candidates: 956 us; with
// block 0 doing both, 1,086).
__global__ void __launch_bounds__(KR_BLOCK) hvi_score_kernel(HviArgs a)
{
    __shared__ double fT[3][KR_HVI_MAX_OBS], fE[3][KR_HVI_MAX_OBS];
    const int tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        bool bad = false;
        for (int g = tid; g < a.n_seg; g += KR_BLOCK) bad = bad || a.fr_n[g * 3] < 0;
        bad = __syncthreads_or(bad);
        if (tid == 0) *a.status = bad ? KR_EINVAL : KR_OK;
        return;
    }
    const int64_t t0 = (int64_t)blockIdx.x * KR_HVI_TILE;
    const int64_t t1 = t0 + KR_HVI_TILE < a.n_cand ? t0 + KR_HVI_TILE : a.n_cand;
    // last partition starting at or before t0 (uniform binary search)
    int lo = 0, hi = a.n_seg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (a.cand_off[mid] <= t0) lo = mid;
        else hi = mid;
    }
    for (int g = lo; g < a.n_seg && a.cand_off[g] < t1; ++g) {
        const int64_t c0 = a.cand_off[g], c1 = a.cand_off[g + 1];
        if (c1 <= t0) continue;
        const int64_t o0 = a.obs_off[g];
        int s[3];
        bool bad = false;
        for (int v = 0; v < 3; ++v) {
            s[v] = a.fr_n[g * 3 + v];
            bad = bad || s[v] < 0;
        }
        __syncthreads();
        if (!bad)
            for (int v = 0; v < 3; ++v)
                for (int i = tid; i < s[v]; i += KR_BLOCK) {
                    fT[v][i] = a.fr_T[(int64_t)v * a.n_obs + o0 + i];
                    fE[v][i] = a.fr_E[(int64_t)v * a.n_obs + o0 + i];
                }
        __syncthreads();
        const double rT = a.ref[g * 4];
        const double rE[3] = {a.ref[g * 4 + 1], a.ref[g * 4 + 2], a.ref[g * 4 + 3]};
        const int64_t x0 = c0 > t0 ? c0 : t0, x1 = c1 < t1 ? c1 : t1;
        // all of this thread's candidates of the partition are loaded before any is
        // scored, so their loads are in flight together
        constexpr int kPer = KR_HVI_TILE / KR_BLOCK;
        double t[kPer], e[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t x = x0 + tid + (int64_t)j * KR_BLOCK;
            t[j] = x < x1 ? __builtin_nontemporal_load(a.T_hat + x) : 0.0;
            e[j] = x < x1 ? __builtin_nontemporal_load(a.E_hat + x) : 0.0;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t x = x0 + tid + (int64_t)j * KR_BLOCK;
            if (x >= x1) break;
#pragma unroll
            for (int v = 0; v < 3; ++v) {
                const double h = bad ? NAN
                                     : hvi_one(fT[v], fE[v], s[v], rT, rE[v], t[j],
                                               energy_variant(v, t[j], e[j], a.p_static));
                __builtin_nontemporal_store(h, a.hvi + (int64_t)v * a.n_cand + x);
            }
        }
    }
}

// ev: optional start/stop events around the score kernel (null entries: none).
static void mark(hipEvent_t *ev, int which, hipStream_t st)
{
    if (ev && ev[0] && ev[1]) (void)hipEventRecord(ev[which], st);
}

hipError_t launch_hvi(const HviArgs &a, hipEvent_t *ev, hipStream_t st)
{
    hipLaunchKernelGGL(hvi_prep_kernel, dim3(a.n_seg, 3), dim3(KR_BLOCK), 0, st, a);
    const int64_t blocks = (a.n_cand + KR_HVI_TILE - 1) / KR_HVI_TILE;
    mark(ev, 0, st);
    hipLaunchKernelGGL(hvi_score_kernel, dim3((unsigned)(blocks + 1)), dim3(KR_BLOCK), 0, st, a);
    mark(ev, 1, st);
    return hipGetLastError();
}

// Population standard deviation of the members' T plus that of their E.  With M a
// compile-time count the members stay in registers between the mean and the deviations;
// the generic form reads them twice.
template <int MC>
__global__ void __launch_bounds__(KR_BLOCK) unc_kernel(int M_rt, int64_t n, const double *Tm,
                                                     const double *Em, double *unc)
{
    const int M = MC > 0 ? MC : M_rt;
    const int64_t stride = (int64_t)gridDim.x * KR_BLOCK;
    if constexpr (MC > 0) {
        // two candidates per step, all their members loaded before either is reduced
        for (int64_t x = (int64_t)blockIdx.x * KR_BLOCK + threadIdx.x; x < n; x += 2 * stride) {
            const int64_t xs[2] = {x, x + stride < n ? x + stride : x};
            double t[2][MC], e[2][MC];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int m = 0; m < MC; ++m) {
                    t[j][m] = __builtin_nontemporal_load(Tm + (int64_t)m * n + xs[j]);
                    e[j][m] = __builtin_nontemporal_load(Em + (int64_t)m * n + xs[j]);
                }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                double st = 0.0, se = 0.0;
#pragma unroll
                for (int m = 0; m < MC; ++m) {
                    st = st + t[j][m];
                    se = se + e[j][m];
                }
                const double mt = st / M, me = se / M;
                double vt = 0.0, ve = 0.0;
#pragma unroll
                for (int m = 0; m < MC; ++m) {
                    const double dt = t[j][m] - mt, de = e[j][m] - me;
                    vt = vt + dt * dt;
                    ve = ve + de * de;
                }
                if (j == 0 || x + stride < n)
                    __builtin_nontemporal_store(sqrt(vt / M) + sqrt(ve / M), unc + xs[j]);
            }
        }
        return;
    }
    for (int64_t x = (int64_t)blockIdx.x * KR_BLOCK + threadIdx.x; x < n; x += stride) {
        double st = 0.0, se = 0.0;
        {
            for (int m = 0; m < M; ++m) {
                st = st + Tm[(int64_t)m * n + x];
                se = se + Em[(int64_t)m * n + x];
            }
            const double mt = st / M, me = se / M;
            double vt = 0.0, ve = 0.0;
            for (int m = 0; m < M; ++m) {
                const double dt = Tm[(int64_t)m * n + x] - mt, de = Em[(int64_t)m * n + x] - me;
                vt = vt + dt * dt;
                ve = ve + de * de;
            }
            unc[x] = sqrt(vt / M) + sqrt(ve / M);
        }
    }
}

hipError_t launch_uncertainty(int M, int64_t n, const double *Tm, const double *Em, double *unc,
                              hipEvent_t *ev, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    const int64_t blocks = (n + KR_BLOCK - 1) / KR_BLOCK;
    const unsigned grid = (unsigned)(blocks < 8192 ? blocks : 8192);
    const dim3 g(grid), b(KR_BLOCK);
    mark(ev, 0, st);
    switch (M) {
    case 1: hipLaunchKernelGGL(unc_kernel<1>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 2: hipLaunchKernelGGL(unc_kernel<2>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 3: hipLaunchKernelGGL(unc_kernel<3>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 4: hipLaunchKernelGGL(unc_kernel<4>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 5: hipLaunchKernelGGL(unc_kernel<5>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 6: hipLaunchKernelGGL(unc_kernel<6>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 7: hipLaunchKernelGGL(unc_kernel<7>, g, b, 0, st, M, n, Tm, Em, unc); break;
    case 8: hipLaunchKernelGGL(unc_kernel<8>, g, b, 0, st, M, n, Tm, Em, unc); break;
    default: hipLaunchKernelGGL(unc_kernel<0>, g, b, 0, st, M, n, Tm, Em, unc); break;
    }
    mark(ev, 1, st);
    return hipGetLastError();
}

// ---- selection -----------------------------------------------------------------------

// Order key of a score: larger key = larger score; -0 and +0 share one key.  Key 0 is
// below every score and marks an empty list entry.
__device__ __forceinline__ uint64_t score_key(double s)
{
    if (s == 0.0) s = 0.0;
    const uint64_t u = dbits(s);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ __forceinline__ double key_score(uint64_t k)
{
    return bitsd((k >> 63) ? k ^ 0x8000000000000000ull : ~k);
}

struct Entry {
    uint64_t key;
    int32_t idx;
};

__device__ __forceinline__ bool better(const Entry &a, const Entry &b)
{
    return a.key > b.key || (a.key == b.key && a.idx < b.idx);
}

__device__ __forceinline__ Entry shfl_entry(const Entry &e, int src)
{
    Entry r;
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)e.key, src, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(e.key >> 32), src, 64);
    r.key = ((uint64_t)hi << 32) | lo;
    r.idx = __shfl(e.idx, src, 64);
    return r;
}

// One compare-exchange step with lane ^ j: the lower lane of a pair keeps the better entry.
__device__ __forceinline__ Entry cmpx(const Entry &e, int lane, int j)
{
    const Entry p = shfl_entry(e, lane ^ j);
    const bool take = (lane & j) == 0 ? better(p, e) : better(e, p);
    return take ? p : e;
}

// The wave's first n entries (distinct), best first, through the LDS room key/idx[64]; the
// lanes from n on get empty ones.  An entry's place is the number of better ones, counted
// over lane reads: fewer instructions than a bitonic network and no chain of shuffles, whose
// latency (21 stages) was most of the selection's time.
__device__ __forceinline__ Entry wave_sort(const Entry &e, int n, int lane, uint64_t *key,
                                           int32_t *idx)
{
    int rank = 0;
#pragma unroll 4
    for (int y = 0; y < n; ++y) {
        Entry c;
        c.key = lane_u64(e.key, y);
        c.idx = lane_i32(e.idx, y);
        rank += better(c, e) ? 1 : 0;
    }
    if (lane < n) {
        key[rank] = e.key;
        idx[rank] = e.idx;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
    Entry r;
    r.key = lane < n ? key[lane] : 0;
    r.idx = lane < n ? idx[lane] : INT32_MAX;
    return r;
}

// Best 64 of two best-first lists, best first.
__device__ __forceinline__ Entry wave_merge(const Entry &list, const Entry &sorted, int lane)
{
    const Entry r = shfl_entry(sorted, 63 - lane);
    Entry e = better(list, r) ? list : r;
#pragma unroll
    for (int j = 32; j > 0; j >>= 1) e = cmpx(e, lane, j);
    return e;
}

// A wave's best candidates of one pass: the list (best first), the threshold a candidate has
// to beat, and a buffer of candidates that did, in LDS (key/idx [KR_SEL_LIST]).
struct Best {
    Entry list;
    double tv;  // the k-th best seen, or a bound from elsewhere (uniform); ties by index
    int32_t ti;
    int cnt;      // candidates in the buffer
    bool listed;  // the list holds something

    __device__ __forceinline__ void init(double v, int32_t i)
    {
        list.key = 0;
        list.idx = INT32_MAX;
        tv = v;
        ti = i;
        cnt = 0;
        listed = false;
    }

    __device__ __forceinline__ bool beats(double v, int32_t x) const
    {
        return v > tv || (v == tv && x < ti);
    }

    // Sorts the buffer into the list and raises the threshold to its k-th entry (k >= 1).
    __device__ __forceinline__ void flush(int k, int lane, uint64_t *key, int32_t *idx)
    {
        Entry e;
        e.key = key[lane];
        e.idx = idx[lane];
        e = wave_sort(e, cnt, lane, key, idx);
        list = listed ? wave_merge(list, e, lane) : e;
        listed = true;
        cnt = 0;
        const uint64_t tk = lane_u64(list.key, k - 1);
        if (tk == 0) return;  // fewer than k so far
        const double v = key_score(tk);
        const int32_t x = lane_i32(list.idx, k - 1);
        if (v > tv || (v == tv && x < ti)) {
            tv = v;
            ti = x;
        }
    }

    // Offers one candidate per lane (`in`: there is one).
    __device__ __forceinline__ void offer(bool in, double v, int32_t x, int k, int lane,
                                          uint64_t *key, int32_t *idx)
    {
        bool pass = in && beats(v, x);
        uint64_t m = __ballot(pass);
        if (m == 0) return;
        if (cnt + __popcll(m) > KR_SEL_LIST) {
            flush(k, lane, key, idx);
            pass = in && beats(v, x);
            m = __ballot(pass);
        }
        if (pass) {
            const int pos = cnt + (int)__builtin_amdgcn_mbcnt_hi(
                                      (uint32_t)(m >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            key[pos] = score_key(v);
            idx[pos] = x;
        }
        cnt += __popcll(m);
    }
};

// Scores of pass p over the partition whose candidates start at c0.
__device__ __forceinline__ const double *pass_scores(const SelArgs &a, int p, int64_t c0)
{
    return (p < 3 ? a.score + (int64_t)p * a.n_cand : (p < a.npass ? a.unc : a.score)) + c0;
}

// Block g < n_seg, one wave per pass: about the k_p-th best unmeasured candidate of a sample
// of the partition (pieces of 8, evenly spread, as good scores come in clusters).  At least
// k_p candidates of the partition are as good, so nothing below it can be selected, and it
// is the threshold that the tiles start with.  Without one every wave had to find its own
// among its first candidates, and those sorts were most of the tile kernel.
// Block n_seg: the tiles of each partition, and a cleared NaN flag.
#define KR_SEL_SAMPLE 32  // rows of eight pieces sampled
__global__ void __launch_bounds__(KR_BLOCK) sel_plan_kernel(SelArgs a)
{
    __shared__ int64_t red[KR_WAVES];
    __shared__ uint32_t excl[KR_SEL_SAMPLE * 2];  // measured candidates of the sample
    static_assert(KR_WAVES == 4, "one wave per pass");
    const int tid = threadIdx.x, lane = tid & 63;
    const int p = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (blockIdx.x == a.n_seg) {
        int64_t carry = 0;
        for (int64_t base = 0; base < a.n_seg; base += KR_BLOCK) {
            const int64_t g = base + tid;
            const int64_t n = g < a.n_seg ? a.cand_off[g + 1] - a.cand_off[g] : 0;
            const int64_t tile = a.rows * KR_BLOCK, tiles = (n + tile - 1) / tile;
            int64_t total;
            const int64_t ex = block_exclusive(tiles, (int64_t)0, SumI64(), red, &total);
            if (g < a.n_seg) {
                a.tile_off[g] = carry + ex;
                for (int64_t t = 0; t < tiles; ++t) a.tile_seg[carry + ex + t] = (int32_t)g;
            }
            carry += total;
        }
        if (tid == 0) {
            a.tile_off[a.n_seg] = carry;
            *a.flag = 0;
        }
        return;
    }
    const int g = blockIdx.x;
    const int64_t c0 = a.cand_off[g], n = a.cand_off[g + 1] - c0;
    // piece i of the sample is the partition's piece i * step (n < 2^31); a small partition
    // is sampled whole
    const uint32_t n8 = (uint32_t)((n + 7) / 8);
    const uint32_t step = max(1u, (n8 + KR_SEL_SAMPLE * 8 - 1) / (KR_SEL_SAMPLE * 8));
    const uint32_t np8 = (n8 + step - 1) / step;  // sampled pieces
    auto at = [&](int r) {  // this lane's candidate of row r, or n
        const uint32_t piece = r * 8 + (lane >> 3);
        return piece < np8 ? min(n, (int64_t)piece * step * 8 + (lane & 7)) : n;
    };
    const int k = a.k[p];
    const bool on = p < a.npass && k > 0;
    const double *const src = pass_scores(a, p, c0);
    double v[KR_SEL_SAMPLE];  // loaded together, before the measured set is read
#pragma unroll
    for (int r = 0; r < KR_SEL_SAMPLE; ++r) v[r] = on && at(r) < n ? src[at(r)] : 0.0;
    if (tid < KR_SEL_SAMPLE * 2) excl[tid] = 0;
    __syncthreads();
    for (int64_t i = a.obs_off[g] + tid; i < a.obs_off[g + 1]; i += KR_BLOCK) {
        const int64_t x = a.obs_idx[i];
        if (x < 0 || x >= n) continue;
        const uint32_t x8 = (uint32_t)x / 8, piece = x8 / step;
        if (piece * step != x8) continue;
        const uint32_t pos = piece * 8 + ((uint32_t)x & 7);
        atomicOr(&excl[pos >> 5], 1u << (pos & 31));
    }
    __syncthreads();
    // Each lane's best of its column of the sample; the k-th best of those is at or below
    // the k-th best of the sample, and takes one rank count instead of a top-k.
    double bv = -INFINITY;
    int32_t bx = INT32_MAX;
#pragma unroll
    for (int r = 0; r < KR_SEL_SAMPLE; ++r) {
        const int64_t x = at(r);
        const bool in = on && x < n && !(excl[2 * r + (lane >> 5)] >> (lane & 31) & 1);
        const bool up = in && (v[r] > bv || (v[r] == bv && bx == INT32_MAX));
        bv = up ? v[r] : bv;  // rows come in ascending index order: ties keep the first
        bx = up ? (int32_t)x : bx;
    }
    int rank = 0;  // lanes with a better best
#pragma unroll 4
    for (int y = 0; y < 64; ++y) {
        const double yv = bitsd(lane_u64(dbits(bv), y));
        const int32_t yx = lane_i32(bx, y);
        rank += yv > bv || (yv == bv && yx < bx) ? 1 : 0;
    }
    // the k-th itself still passes; with fewer candidates everything does, and an empty
    // pass takes nothing
    const uint64_t kth = __ballot(bx != INT32_MAX && rank == k - 1);
    const int y = kth ? __ffsll((long long)kth) - 1 : 0;
    if (lane == y) {
        a.floor_v[g * 4 + p] = k == 0 ? INFINITY : kth ? bv : -INFINITY;
        a.floor_i[g * 4 + p] = k == 0 ? INT32_MIN : kth ? bx + 1 : INT32_MAX;
    }
}

// One block per tile: each pass's best unmeasured candidates of the tile, in one sweep over
// the scores of all passes.  Pass p takes k_p candidates of the partition (the exploration
// pass at most k: its first k hold enough that are not in C already), so only a candidate
// that beats the sample's k_p-th best and the k_p-th best that the wave has seen can matter.
// Such candidates are compacted into an LDS buffer, which is sorted and merged into the
// wave's list when the next row would overflow it.  Bound by reading the scores (32 bytes a
// candidate) and by the row's few compares and ballots a pass.  17.3 M candidates: 295 us
// with the 64th best as every pass's threshold and no sample, 146 us now.
// A list holds the exact best k_p of its candidates; entries behind those are in order but
// need not be the next best.
template <int G>
__global__ void __launch_bounds__(KR_BLOCK) sel_tile_kernel(SelArgs a)
{
    __shared__ uint64_t excl[KR_SEL_ROWS_MAX * KR_WAVES];  // measured candidates of each row
    __shared__ uint64_t bkey[KR_WAVES][4][KR_SEL_LIST];
    __shared__ int32_t bidx[KR_WAVES][4][KR_SEL_LIST];
    const int64_t b = blockIdx.x;
    if (b >= a.tile_off[a.n_seg]) return;
    const int g = a.tile_seg[b];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = a.rows, tile = rows * KR_BLOCK;
    const int64_t c0 = a.cand_off[g], ng = a.cand_off[g + 1] - c0;
    const int64_t l0 = (b - a.tile_off[g]) * tile;  // local index of the tile start
    const int len = (int)min((int64_t)tile, ng - l0);
    const int np = a.npass;
    const double *src[4];
    Best best[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        src[p] = pass_scores(a, p, c0 + l0);
        best[p].init(a.floor_v[g * 4 + p], a.floor_i[g * 4 + p]);
    }
    // Rows of 64 candidates are visited in bit-reversed order.  Scores trend along the
    // index (it runs over frequencies slowest), and in index order late rows would keep
    // beating the threshold and force merges; the result does not depend on the order,
    // since (score, index) is a total order.
    const int bits = 31 - __clz(rows);
    auto row = [&](int r) { return wave * rows + (int)(__brev((uint32_t)r) >> (32 - bits)); };
    // G rows at a time, the next ones' loads in flight meanwhile
    double cur[G][4], nxt[G][4];
    auto load = [&](double (&v)[G][4], int r0) {
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int off = row(r0 + q) * 64 + lane;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                v[q][p] = p < np && off < len ? __builtin_nontemporal_load(src[p] + off) : 0.0;
        }
    };
    load(cur, 0);
    for (int i = tid; i < rows * KR_WAVES; i += KR_BLOCK) excl[i] = 0;
    __syncthreads();
    for (int64_t i = a.obs_off[g] + tid; i < a.obs_off[g + 1]; i += KR_BLOCK) {
        const int64_t x = a.obs_idx[i] - l0;
        if (x >= 0 && x < len) atomicOr((unsigned long long *)&excl[x >> 6], 1ull << (x & 63));
    }
    __syncthreads();
    bool nan_seen = false;
    for (int r0 = 0; r0 < rows; r0 += G) {
        if (r0 + G < rows) load(nxt, r0 + G);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const int rw = row(r0 + q), off = rw * 64 + lane;
            const bool in = off < len && !((excl[rw] >> lane) & 1);
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if (p >= np) break;
                const double v = cur[q][p];  // 0 past the tile's end
                nan_seen = nan_seen || v != v;
                best[p].offer(in, v, (int32_t)l0 + off, a.k[p], lane, bkey[wave][p],
                              bidx[wave][p]);
            }
        }
#pragma unroll
        for (int q = 0; q < G; ++q)
#pragma unroll
            for (int p = 0; p < 4; ++p) cur[q][p] = nxt[q][p];
    }
    // a wave's buffers are its own until here; wave p merges pass p's lists
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (p >= np) break;
        if (best[p].cnt > 0) best[p].flush(a.k[p], lane, bkey[wave][p], bidx[wave][p]);
        bkey[wave][p][lane] = best[p].list.key;
        bidx[wave][p][lane] = best[p].list.idx;
    }
    __syncthreads();
    if (wave < np) {
        Entry list;
        for (int w = 0; w < KR_WAVES; ++w) {
            Entry o;
            o.key = bkey[w][wave][lane];
            o.idx = bidx[w][wave][lane];
            list = w == 0 ? o : wave_merge(list, o, lane);
        }
        const int64_t slot = (b * np + wave) * KR_SEL_LIST + lane;
        a.part_key[slot] = list.key;
        a.part_idx[slot] = list.idx;
    }
    if (nan_seen) *a.flag = 1;
}

// One block per partition: merge its tile lists per pass (four waves a pass) and assemble
// the batch.
__global__ void __launch_bounds__(1024) sel_final_kernel(SelArgs a)
{
    __shared__ uint64_t lkey[4][4][KR_SEL_LIST];
    __shared__ int32_t lidx[4][4][KR_SEL_LIST];
    const int g = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int p = __builtin_amdgcn_readfirstlane(tid >> 8), w = (tid >> 6) & 3;
    const bool bad = *a.flag != 0;
    if (g == 0 && tid == 0) *a.status = bad ? KR_EINVAL : KR_OK;
    if (bad) {
        if (tid == 0) a.count[g] = 0;
        return;
    }
    const int64_t tb = a.tile_off[g], te = a.tile_off[g + 1];
    Entry list;
    list.key = 0;
    list.idx = INT32_MAX;
    if (p < a.npass)
        for (int64_t t = tb + w; t < te; t += 16) {
            Entry o[4];  // loaded together
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = t + 4 * q < te;
                const int64_t slot = ((in ? t + 4 * q : t) * a.npass + p) * KR_SEL_LIST + lane;
                o[q].key = a.part_key[slot];
                o[q].idx = a.part_idx[slot];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t + 4 * q < te) list = q == 0 && t == tb + w ? o[0] : wave_merge(list, o[q], lane);
        }
    lkey[p][w][lane] = list.key;
    lidx[p][w][lane] = list.idx;
    __syncthreads();
    if (w == 0) {
        const int nl = (int)min((int64_t)4, te - tb);  // waves that had a list
        for (int q = 1; q < nl; ++q) {
            Entry o;
            o.key = lkey[p][q][lane];
            o.idx = lidx[p][q][lane];
            list = wave_merge(list, o, lane);
        }
        lkey[p][0][lane] = list.key;
        lidx[p][0][lane] = list.idx;
    }
    __syncthreads();
    if (tid >= 64) return;
    // the batch: lane i holds its i-th member
    int32_t mine = -1;
    int cnt = 0;
    const int k = a.k[3];
    for (int q = 0; q < a.npass; ++q) {
        const uint64_t key = lkey[q][0][lane];
        const int32_t idx = lidx[q][0][lane];
        const int want = q < 3 ? a.k[q] : k;
        for (int r = 0; r < want && cnt < k; ++r) {
            if (lane_u64(key, r) == 0) break;
            const int32_t x = lane_i32(idx, r);
            if (__ballot(lane < cnt && mine == x) != 0) continue;
            if (lane == cnt) mine = x;
            ++cnt;
        }
    }
    if (lane < cnt) a.sel[(int64_t)g * k + lane] = mine;
    if (lane == 0) a.count[g] = cnt;
}

hipError_t launch_select(const SelArgs &a, hipEvent_t *ev, hipStream_t st)
{
    hipLaunchKernelGGL(sel_plan_kernel, dim3(a.n_seg + 1), dim3(KR_BLOCK), 0, st, a);
    mark(ev, 0, st);
    if (a.max_tiles > 0)
        hipLaunchKernelGGL(sel_tile_kernel<4>, dim3((unsigned)a.max_tiles), dim3(KR_BLOCK), 0, st,
                           a);
    mark(ev, 1, st);
    hipLaunchKernelGGL(sel_final_kernel, dim3(a.n_seg), dim3(1024), 0, st, a);
    return hipGetLastError();
}

}  // namespace kr
