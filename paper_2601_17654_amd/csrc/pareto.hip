// Segmented GetFrontier (Algorithm 1's return value, Algorithm 2's last step).
//
// Rule: within a segment, sort points by (T, E, index) and keep a point iff its E is
// strictly below every E before it -- the non-dominated set, exact duplicates
// resolved to the smallest index.  The rule is decomposable: the frontier of a union
// is the frontier of the union of the parts' frontiers.
//
// Work split: every segment is cut into units with a slot each.  A tile of points leaves
// its exact frontier there (SegLayout::exact); the frequency range of a fused workgroup
// leaves the frontiers of its chunks or tiles one behind another, and a frequency of a
// microbatch its configurations, in no order that the merge relies on.
// The union of a segment's units is then sorted by a merge sort in LDS and
// scanned: a 256-thread block per segment of up to 512 points, a 1024-thread block
// for the few segments of up to 4096, and beyond that LDS-sized chunks whose
// frontiers are merged pairwise in device memory; with up to KR_FUSED_SEGS segments one
// launch does all of this and copies out (finalize_fused_kernel).  A pairwise merge of two
// staircases needs no sort: an element's rank in the partner comes from a binary search, and it
// survives iff the partner element just before it in key order has a larger E.
#include "kr_filter.h"
#include "kr_launch.h"

namespace kr {

// The layout kernels also clear lists[0], the count of segments that the first merge
// stage passes on (or the ticket of the fused one), the segments' counts and the input
// check's verdict (so that none of them needs a launch of its own).
__global__ void uniform_layout_kernel(int64_t *seg_off, int64_t *unit_base, int n_seg,
                                      int64_t seg_len, int64_t units_per_seg, int32_t *lists,
                                      int32_t *fcnt, int32_t *status)
{
    const int g = blockIdx.x * KR_BLOCK + threadIdx.x;
    if (g < n_seg) fcnt[g] = 0;
    if (g == 0) lists[0] = 0;
    if (g == 0 && status) *status = KR_OK;
    if (g > n_seg) return;
    seg_off[g] = (int64_t)g * seg_len;
    unit_base[g] = (int64_t)g * units_per_seg;
}

hipError_t launch_uniform_layout(int64_t *seg_off, int64_t *unit_base, int n_seg,
                                 int64_t seg_len, int64_t units_per_seg, int32_t *lists,
                                 int32_t *fcnt, int32_t *status, hipStream_t st)
{
    hipLaunchKernelGGL(uniform_layout_kernel, dim3((n_seg + 1 + KR_BLOCK - 1) / KR_BLOCK),
                       dim3(KR_BLOCK), 0, st, seg_off, unit_base, n_seg, seg_len, units_per_seg,
                       lists, fcnt, status);
    return hipGetLastError();
}

// unit_base = exclusive prefix sum of ceil(len_g / tile); one block, of as many threads as
// there are (4,096 segments: 18 us with 256 threads, 9 us with 1,024).
#define KR_LAYOUT_NT 1024
__global__ void __launch_bounds__(KR_LAYOUT_NT)
tile_layout_kernel(const int64_t *seg_off, int64_t *unit_base, int n_seg, int tile,
                   int32_t *lists, int32_t *fcnt, int32_t *status)
{
    __shared__ int64_t sc[KR_LAYOUT_NT / 64];
    for (int g = threadIdx.x; g < n_seg; g += KR_LAYOUT_NT) fcnt[g] = 0;
    if (threadIdx.x == 0) lists[0] = 0;
    if (threadIdx.x == 0 && status) *status = KR_OK;
    int64_t carry = 0;
    for (int g0 = 0; g0 < n_seg; g0 += KR_LAYOUT_NT) {
        const int g = g0 + threadIdx.x;
        int64_t nt = 0;
        if (g < n_seg) {
            const int64_t len = seg_off[g + 1] - seg_off[g];
            nt = len > 0 ? (len + tile - 1) / tile : 0;
        }
        int64_t tot;
        const int64_t ex = block_exclusive<int64_t, SumI64, KR_LAYOUT_NT / 64>(
            nt, (int64_t)0, SumI64(), sc, &tot);
        if (g < n_seg) unit_base[g] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) unit_base[n_seg] = carry;
}

hipError_t launch_tile_layout(const int64_t *seg_off, int64_t *unit_base, int n_seg, int tile,
                              int32_t *lists, int32_t *fcnt, int32_t *status, hipStream_t st)
{
    hipLaunchKernelGGL(tile_layout_kernel, dim3(1), dim3(KR_LAYOUT_NT), 0, st, seg_off, unit_base,
                       n_seg, tile, lists, fcnt, status);
    return hipGetLastError();
}

// Segment holding global unit w (unit_base is non-decreasing).
__device__ __forceinline__ int find_segment(const int64_t *unit_base, int n_seg, int64_t w)
{
    int lo = 0, hi = n_seg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (unit_base[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Exact frontier of one tile of up to KR_TILE consecutive points of a segment.  The
// first pass holds KR_SURV_CAP survivors in LDS and defers (count -1) a tile with more;
// the second pass takes only deferred tiles, with LDS for the whole tile, and sorts
// their survivors.
template <bool BIG>
__global__ void __launch_bounds__(KR_BLOCK)
pareto_tile_kernel(const double *T, const double *E, SegLayout L, UnitOut o, int32_t *status)
{
    static_assert(KR_TILE == 8 * KR_BLOCK, "a tile is 8 points per thread");
    extern __shared__ double tile_lds[];
    __shared__ FilterShared fsh;
    const int64_t w = blockIdx.x;
    if (w >= L.unit_base[L.n_seg]) return;
    if (BIG && o.cnt[w] >= 0) return;  // done by the first pass
    const int g = find_segment(L.unit_base, L.n_seg, w);
    const int64_t s0 = L.seg_off[g];
    const int64_t start = s0 + (w - L.unit_base[g]) * L.unit_stride;
    const int64_t end = min(start + L.unit_stride, L.seg_off[g + 1]);
    FilterLds fl;
    fl.sh = &fsh;
    fl.sT = (uint64_t *)tile_lds;
    fl.sE = fl.sT + KR_SURV_CAP;
    fl.sI = (int32_t *)(fl.sE + KR_SURV_CAP);
    if (BIG) {
        fl.bT = (uint64_t *)tile_lds;
        fl.bE = fl.bT + KR_TILE;
        fl.bI = (int32_t *)(fl.bE + KR_TILE);
        fl.big_cap = KR_TILE;
    } else {
        fl.defer = true;
    }
    double vT[8], vE[8];
    int32_t vI[8];
    bool ok[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int64_t x = start + threadIdx.x + q * KR_BLOCK;
        ok[q] = x < end;
        // + 0.0 maps -0.0 to +0.0, so that the bit patterns order like the values
        vT[q] = ok[q] ? T[x] + 0.0 : 0.0;
        vE[q] = ok[q] ? E[x] + 0.0 : 0.0;
        vI[q] = (int32_t)(x - s0);
    }
    if (!BIG && status) {  // every point is in one tile, and the first pass reads them all
        uint32_t worst = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) worst = max(worst, max(raw_hi(vT[q]), raw_hi(vE[q])));
        report_values(status, worst >= KR_BAD_HI);
    }
    int parity = 0;
    const int n = tile_frontier<8>(vT, vE, vI, ok, fl, parity, o.T + start, o.E + start,
                                   o.I + start);
    if (threadIdx.x == 0) o.cnt[w] = n;
}

hipError_t launch_pareto_tiles(const double *T, const double *E, const SegLayout &L,
                               int64_t n_units_bound, const UnitOut &o, int32_t *status,
                               hipStream_t st)
{
    if (n_units_bound == 0) return hipSuccess;
    const size_t lds = (size_t)KR_SURV_CAP * 20, lds_big = (size_t)KR_TILE * 20;
    hipLaunchKernelGGL(pareto_tile_kernel<false>, dim3((unsigned)n_units_bound), dim3(KR_BLOCK),
                       lds, st, T, E, L, o, status);
    hipLaunchKernelGGL(pareto_tile_kernel<true>, dim3((unsigned)n_units_bound), dim3(KR_BLOCK),
                       lds_big, st, T, E, L, o, status);
    return hipGetLastError();
}

// Loads that bypass the CU's L1, for data this block wrote earlier in the same launch.
__device__ __forceinline__ double ld_l2(const double *p)
{
    return bitsd(__hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ int32_t ld_l2(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint8_t ld_l2(const uint8_t *p)
{
    const uint32_t word = __hip_atomic_load((const uint32_t *)((uintptr_t)p & ~(uintptr_t)3),
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (uint8_t)(word >> (8 * ((uintptr_t)p & 3)));
}

// Rank of key (t, e, i) in the sorted staircase b[0..n): number of elements before it.
__device__ __forceinline__ int rank_in(const double *bT, const double *bE, const int32_t *bI,
                                       int n, uint64_t t, uint64_t e, int32_t i)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key_less(dbits(ld_l2(bT + mid)), dbits(ld_l2(bE + mid)), ld_l2(bI + mid), t, e, i))
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// Merge staircases a = in[sa, sa+na) and b = in[sb, sb+nb) into out[sa ...); returns
// the merged frontier's size.  Every thread of the block must call.  beat() is called every
// now and then (see finalize_fused_kernel).
template <int NT, typename Beat>
__device__ inline int merge_pair(PointBufs in, PointBufs out, uint8_t *flags,
                                 int64_t sa, int na, int64_t sb, int nb, const Beat &beat)
{
    __shared__ int32_t sc[NT / 64];
    const double *aT = in.T + sa, *aE = in.E + sa, *bT = in.T + sb, *bE = in.E + sb;
    const int32_t *aI = in.I + sa, *bI = in.I + sb;
    for (int x = threadIdx.x; x < na + nb; x += NT) {
        if (x / NT % 256 == 0) beat();
        const bool fromA = x < na;
        const int y = fromA ? x : x - na;
        const double t = ld_l2(fromA ? aT + y : bT + y);
        const double e = ld_l2(fromA ? aE + y : bE + y);
        const int32_t id = ld_l2(fromA ? aI + y : bI + y);
        const int r = fromA ? rank_in(bT, bE, bI, nb, dbits(t), dbits(e), id)
                            : rank_in(aT, aE, aI, na, dbits(t), dbits(e), id);
        const double *oE = fromA ? bE : aE;
        const bool alive = !(r > 0 && ld_l2(oE + r - 1) <= e);
        const int64_t dst = sa + y + r;
        out.T[dst] = t;
        out.E[dst] = e;
        out.I[dst] = id;
        flags[dst] = alive;
    }
    __syncthreads();
    const int n = na + nb;
    int base = 0;
    for (int c0 = 0; c0 < n; c0 += NT) {
        if (c0 / NT % 256 == 0) beat();
        const int x = c0 + threadIdx.x;
        const bool has = x < n;
        double t = 0.0, e = 0.0;
        int32_t id = 0;
        int f = 0;
        if (has) {
            t = ld_l2(out.T + sa + x);
            e = ld_l2(out.E + sa + x);
            id = ld_l2(out.I + sa + x);
            f = ld_l2(flags + sa + x);
        }
        __syncthreads();
        int tot;
        const int pos = block_exclusive<int, SumI32, NT / 64>(f, 0, SumI32(), sc, &tot);
        if (has && f) {
            out.T[sa + base + pos] = t;
            out.E[sa + base + pos] = e;
            out.I[sa + base + pos] = id;
        }
        base += tot;
        __syncthreads();
    }
    return base;
}

struct FinLds {
    uint64_t sT[KR_FIN_CAP], sE[KR_FIN_CAP];
    int32_t sI[KR_FIN_CAP];
    int32_t upre[KR_FIN_UNITS + 1];
};

// ----------------------------------------------------------------------------
// Union of a segment's unit frontiers -> the segment's frontier in `fin` at the
// segment start, its size in fcnt[g].  `buf` holds the unit slots (free to be
// overwritten once they are gathered).
//
// Segments of at most NT * PER points in at most NT units: one block of NT threads
// per segment sorts the union in LDS by merging.  Thread t gathers points t * PER ..
// t * PER + PER - 1 and sorts them in registers; the sorted runs are then merged
// pairwise, one level per doubling of the run width, every thread forming PER outputs of a
// level (merge path: a search for where they start, then a merge in registers).  The
// levels move (T, 16-bit point id) pairs between two buffers; E and the index stay in
// place and are read on a tie in T only.  A strict prefix-minimum scan of E over the
// sorted order gives the frontier.
//
// Three stages: every segment first meets the small instance (a block per segment);
// what it cannot take goes on a list for the large instance (one block per listed
// segment, looping), and what that cannot take on a second list for the chunked
// fallback at the end of this section.
#define KR_FM_SMALL_NT 256
#define KR_FM_SMALL_PER 2
#define KR_FM_LARGE_NT 1024
#define KR_FM_LARGE_PER 4

template <int NT, int PER>
struct MergeLds {
    static constexpr int CAP = NT * PER;
    uint64_t T[2][CAP];
    uint16_t id[2][CAP];
    uint64_t E[CAP];
    int32_t I[CAP];
    int32_t upre[NT + 1];  // upre[u] = points in units before u
    int32_t sc32[NT / 64];
    uint64_t sc64[NT / 64];
};

struct MKey {
    uint64_t t, e;
    int32_t i;
};

__device__ __forceinline__ bool mk_less(const MKey &a, const MKey &b)
{
    return key_less(a.t, a.e, a.i, b.t, b.e, b.i);
}

// Key of the point at a level position (T there, id -> E and index) below another's.
__device__ __forceinline__ bool pos_less(uint64_t ta, int xa, uint64_t tb, int xb,
                                         const uint64_t *E, const int32_t *I)
{
    if (ta != tb) return ta < tb;
    const uint64_t ea = E[xa], eb = E[xb];
    if (ea != eb) return ea < eb;
    return I[xa] < I[xb];
}

// Stage entry: unit prefix of segment g into sh.upre and the point count n, or false
// when the segment has more than NT units or NT * PER points.  Block-uniform.
template <int NT, int PER>
__device__ __forceinline__ bool merge_prefix(int g, const SegLayout &L, const int32_t *ucnt,
                                             MergeLds<NT, PER> &sh, int &n)
{
    const int tid = threadIdx.x;
    const int64_t u0 = L.unit_base[g];
    const int nu = (int)(L.unit_base[g + 1] - u0);
    if (nu > NT) return false;
    const int ex = block_exclusive<int, SumI32, NT / 64>(tid < nu ? ucnt[u0 + tid] : 0, 0,
                                                         SumI32(), sh.sc32, &n);
    if (n > MergeLds<NT, PER>::CAP) return false;
    if (tid < nu) sh.upre[tid] = ex;
    if (tid == 0) sh.upre[nu] = n;
    return true;
}

// The points of a segment's up to NU units (upre as merge_prefix leaves it): load(q, key) for q
// in [q0, q1).
template <int NU, int PER>
struct UnitPoints {
    const int32_t *upre;
    const PointBufs &buf;
    int64_t s0, stride;
    int nu;

    __device__ __forceinline__ void operator()(int q0, int q1, MKey (&k)[PER]) const
    {
        int u = 0;  // unit holding point q0: the last u < nu with upre[u] <= q0
#pragma unroll
        for (int step = NU / 2; step >= 1; step >>= 1)
            if (u + step < nu && upre[u + step] <= q0) u += step;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int x = q0 + j;
            if (x < q1) {
                while (upre[u + 1] <= x) ++u;  // skip ended and empty units (x < upre[nu])
                const int64_t src = s0 + (int64_t)u * stride + (x - upre[u]);
                k[j] = MKey{dbits(buf.T[src]), dbits(buf.E[src]), buf.I[src]};
            }
        }
    }
};

// Sorts n points (read by `points`) and writes their frontier to (oT, oE, oI)[d0 ...], where
// d0 = place(count) is asked for once the count is known, up to element cap.
template <int NT, int PER, typename Points, typename Place>
__device__ __forceinline__ void merge_segment(int n, const Points &points, MergeLds<NT, PER> &sh,
                                              double *oT, double *oE, int32_t *oI, int64_t cap,
                                              const Place &place)
{
    static_assert(NT * PER <= 65536 && (PER & (PER - 1)) == 0, "16-bit ids, power-of-two runs");
    const int tid = threadIdx.x;
    lds_barrier();  // upre
    const int q0 = min(n, tid * PER), q1 = min(n, q0 + PER);
    MKey k[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j)
        k[j] = MKey{~0ull, ~0ull, 0x7FFFFFFF};  // beyond the segment: sorts last, dropped
    points(q0, q1, k);
#pragma unroll
    for (int w = 2; w <= PER; w <<= 1)
#pragma unroll
        for (int j = w >> 1; j > 0; j >>= 1)
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int l = i ^ j;
                if (l > i && ((i & w) == 0 ? mk_less(k[l], k[i]) : mk_less(k[i], k[l]))) {
                    const MKey x = k[i];
                    k[i] = k[l];
                    k[l] = x;
                }
            }
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (q0 + j < q1) {
            sh.T[0][q0 + j] = k[j].t;
            sh.id[0][q0 + j] = (uint16_t)(q0 + j);
            sh.E[q0 + j] = k[j].e;
            sh.I[q0 + j] = k[j].i;
        }
    lds_barrier();
    // Sorted runs of width w -> width 2w by merge path: the thread owning output
    // positions [q0, q0 + PER) of a pair of runs (A, then B) finds how many of the first
    // q0 - base outputs come from A (a binary search along that diagonal of the merge),
    // then merges its PER outputs from there, holding the next key of each run.
    int cur = 0;
    for (int w = PER; w < n; w <<= 1) {
        const uint64_t *inT = sh.T[cur];
        const uint16_t *inI = sh.id[cur];
        if (q0 < q1) {
            const int base = q0 & ~(2 * w - 1);
            const int la = min(w, n - base), lb = max(0, min(w, n - base - w));
            const uint64_t *AT = inT + base, *BT = inT + base + w;
            const uint16_t *AI = inI + base, *BI = inI + base + w;
            const int d = q0 - base;
            int lo = max(0, d - lb), hi = min(d, la);
            while (lo < hi) {  // the least i with A[i] after B[d - 1 - i]
                const int mid = (lo + hi) >> 1;
                const int jb = d - 1 - mid;
                if (pos_less(AT[mid], AI[mid], BT[jb], BI[jb], sh.E, sh.I)) lo = mid + 1;
                else hi = mid;
            }
            int i = lo, j = d - lo;
            uint64_t at = i < la ? AT[i] : 0, bt = j < lb ? BT[j] : 0;
            int ai = i < la ? AI[i] : 0, bi = j < lb ? BI[j] : 0;
            uint64_t *const oT = sh.T[cur ^ 1] + q0;
            uint16_t *const oI = sh.id[cur ^ 1] + q0;
            for (int u = 0; u < q1 - q0; ++u) {
                const bool fromA = i < la && (j >= lb || pos_less(at, ai, bt, bi, sh.E, sh.I));
                if (fromA) {
                    oT[u] = at;
                    oI[u] = (uint16_t)ai;
                    ++i;
                    if (i < la) {
                        at = AT[i];
                        ai = AI[i];
                    }
                } else {
                    oT[u] = bt;
                    oI[u] = (uint16_t)bi;
                    ++j;
                    if (j < lb) {
                        bt = BT[j];
                        bi = BI[j];
                    }
                }
            }
        }
        cur ^= 1;
        lds_barrier();
    }
    // keep a point iff its E is below every E before it in key order
    const uint16_t *ord = sh.id[cur];
    uint64_t e[PER];
    uint64_t m = KR_INF_BITS;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        e[j] = q0 + j < q1 ? sh.E[ord[q0 + j]] : KR_INF_BITS;
        m = e[j] < m ? e[j] : m;
    }
    uint64_t all;
    const uint64_t best0 =
        block_exclusive<uint64_t, MinU64, NT / 64>(m, KR_INF_BITS, MinU64(), sh.sc64, &all);
    uint64_t best = best0;
    int nkeep = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (e[j] < best) {
            ++nkeep;
            best = e[j];
        }
    int count;
    int opos = block_exclusive<int, SumI32, NT / 64>(nkeep, 0, SumI32(), sh.sc32, &count);
    best = best0;
    const int64_t d0 = place(count);
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (e[j] < best) {
            const int q = q0 + j;
            if (d0 + opos < cap) {
                oT[d0 + opos] = bitsd(sh.T[cur][q]);
                oE[d0 + opos] = bitsd(e[j]);
                oI[d0 + opos] = sh.I[ord[q]];
            }
            ++opos;
            best = e[j];
        }
}

// The union of segment g's n unit points into `fin` at the segment's start.
template <int NT, int PER>
__device__ __forceinline__ void merge_units(int g, int n, const SegLayout &L, const PointBufs &buf,
                                            const PointBufs &fin, int32_t *fcnt,
                                            MergeLds<NT, PER> &sh)
{
    const int64_t s0 = L.seg_off[g];
    const UnitPoints<NT, PER> points{sh.upre, buf, s0, L.unit_stride,
                                     (int)(L.unit_base[g + 1] - L.unit_base[g])};
    merge_segment(n, points, sh, fin.T, fin.E, fin.I, INT64_MAX, [&](int count) {
        if (threadIdx.x == 0) fcnt[g] = count;
        return s0;
    });
}

// Stage 1: a block per segment.  lists[0] counts the segments passed on (zero on
// entry), lists[2 ...] holds them; lists[1] (the second list's count) is cleared here.
__global__ void __launch_bounds__(KR_FM_SMALL_NT)
finalize_small_kernel(SegLayout L, PointBufs buf, const int32_t *ucnt, PointBufs fin,
                      int32_t *fcnt, int32_t *lists)
{
    __shared__ MergeLds<KR_FM_SMALL_NT, KR_FM_SMALL_PER> sh;
    const int g = blockIdx.x;
    if (g == 0 && threadIdx.x == 0) lists[1] = 0;
    int n;
    const int64_t u0 = L.unit_base[g];
    if (L.exact && L.unit_base[g + 1] - u0 == 1) {  // one unit: its frontier is the segment's
        const int64_t s0 = L.seg_off[g];
        n = ucnt[u0];
        for (int64_t x = s0 + threadIdx.x; x < s0 + n; x += KR_FM_SMALL_NT) {
            fin.T[x] = buf.T[x];
            fin.E[x] = buf.E[x];
            fin.I[x] = buf.I[x];
        }
        if (threadIdx.x == 0) fcnt[g] = n;
        return;
    }
    if (merge_prefix(g, L, ucnt, sh, n)) merge_units(g, n, L, buf, fin, fcnt, sh);
    else if (threadIdx.x == 0) lists[2 + atomicAdd(&lists[0], 1)] = g;
}

// Stage 2: the listed segments, a block each (blocks loop over the list); those it
// cannot take go on the second list (count lists[1], entries from lists[2 + n_seg]).
__global__ void __launch_bounds__(KR_FM_LARGE_NT)
finalize_large_kernel(SegLayout L, PointBufs buf, const int32_t *ucnt, PointBufs fin,
                      int32_t *fcnt, int32_t *lists)
{
    __shared__ MergeLds<KR_FM_LARGE_NT, KR_FM_LARGE_PER> sh;
    const int cnt = lists[0];
    for (int i = blockIdx.x; i < cnt; i += gridDim.x) {
        const int g = lists[2 + i];
        int n;
        if (merge_prefix(g, L, ucnt, sh, n)) merge_units(g, n, L, buf, fin, fcnt, sh);
        else if (threadIdx.x == 0) lists[2 + L.n_seg + atomicAdd(&lists[1], 1)] = g;
        __syncthreads();  // LDS reuse by the next segment
    }
}

// Stage 3, the segments on the second list: one block per segment (blocks loop over the list).
// The union is sorted in LDS when it fits; otherwise it is cut into LDS-sized chunks whose
// frontiers are merged pairwise in device memory.

// A segment's union in chunks; returns the frontier's size.  upre: NT + 1 entries; cap: points
// per chunk, at least KR_FIN_CAP; chunk(x, n) replaces the n points at element x of `fin` by
// their frontier and returns its size, in every thread.
template <int NT, typename Beat, typename Chunk>
__device__ __forceinline__ int finalize_chunks(int g, const SegLayout &L, const PointBufs &buf,
                                               const int32_t *ucnt, const PointBufs &fin,
                                               int32_t *runcnt, uint8_t *flags, int32_t *upre,
                                               int32_t *sc, int cap, const Beat &beat,
                                               const Chunk &chunk)
{
    const int64_t s0 = L.seg_off[g];
    const int64_t u0 = L.unit_base[g];
    const int nu = (int)(L.unit_base[g + 1] - u0);
    int64_t total = 0;
    for (int c0 = 0; c0 < nu; c0 += NT) {
        const int k = c0 + threadIdx.x;
        total += block_reduce<int, SumI32, NT / 64>(k < nu ? ucnt[u0 + k] : 0, 0, SumI32(), sc);
    }
    // Gather contiguously into fin.  A wave takes a unit, or the block where the units have
    // many points: the block took 1.5 us for a unit however few they were (512 frequencies of
    // a microbatch, 20 configurations each: 773 us).
    const int per = total < (int64_t)nu * (NT / 2) ? 64 : NT;  // threads to a unit
    int64_t pre = s0;
    for (int k0 = 0; k0 < nu; k0 += NT) {
        const int k = k0 + threadIdx.x;
        int tot;
        const int ex = block_exclusive<int, SumI32, NT / 64>(k < nu ? ucnt[u0 + k] : 0, 0, SumI32(),
                                                             sc, &tot);
        upre[threadIdx.x] = ex;
        if (threadIdx.x == 0) upre[NT] = tot;
        __syncthreads();
        for (int j = threadIdx.x / per; j < min(NT, nu - k0); j += NT / per) {
            const int at = upre[j], n = upre[j + 1] - at;
            const int64_t src = s0 + (int64_t)(k0 + j) * L.unit_stride, dst = pre + at;
            for (int x = threadIdx.x % per; x < n; x += per) {
                fin.T[dst + x] = buf.T[src + x];
                fin.E[dst + x] = buf.E[src + x];
                fin.I[dst + x] = buf.I[src + x];
            }
        }
        pre += tot;
        __syncthreads();
    }
    // reduce the chunks in place, then merge their staircases pairwise (fin <-> buf)
    int32_t *rc = runcnt + s0 / KR_FIN_CAP + g;
    const int nchunks = (int)((total + cap - 1) / cap);
    for (int c = 0; c < nchunks; ++c) {
        beat();
        const int64_t c0 = (int64_t)c * cap;
        const int cnt = chunk(s0 + c0, (int)min((int64_t)cap, total - c0));
        if (threadIdx.x == 0) rc[c] = cnt;
        __syncthreads();
    }
    PointBufs cur = fin, other = buf;
    for (int span = 1; span < nchunks; span <<= 1) {
        for (int r = 0; r < nchunks; r += 2 * span) {
            const int64_t sa = s0 + (int64_t)r * cap;
            const int na = ld_l2(rc + r);
            int merged;
            if (r + span < nchunks) {
                const int64_t sb = s0 + (int64_t)(r + span) * cap;
                merged = merge_pair<NT>(cur, other, flags, sa, na, sb, ld_l2(rc + r + span),
                                        beat);
            } else {
                for (int x = threadIdx.x; x < na; x += NT) {
                    other.T[sa + x] = ld_l2(cur.T + sa + x);
                    other.E[sa + x] = ld_l2(cur.E + sa + x);
                    other.I[sa + x] = ld_l2(cur.I + sa + x);
                }
                merged = na;
            }
            __syncthreads();
            if (threadIdx.x == 0) rc[r] = merged;
            __syncthreads();
        }
        const PointBufs t = cur;
        cur = other;
        other = t;
    }
    const int n = nchunks > 0 ? ld_l2(rc) : 0;
    if (cur.T != fin.T) {
        for (int x = threadIdx.x; x < n; x += NT) {
            fin.T[s0 + x] = ld_l2(cur.T + s0 + x);
            fin.E[s0 + x] = ld_l2(cur.E + s0 + x);
            fin.I[s0 + x] = ld_l2(cur.I + s0 + x);
        }
    }
    return n;
}

// A union of up to KR_FIN_CAP points in up to KR_FIN_UNITS units; -1 if it is larger.
__device__ __forceinline__ int finalize_few(int g, const SegLayout &L, const PointBufs &buf,
                                            const int32_t *ucnt, const PointBufs &fin, FinLds &sh,
                                            int32_t *sc)
{
    const int64_t s0 = L.seg_off[g];
    const int64_t u0 = L.unit_base[g];
    const int nu = (int)(L.unit_base[g + 1] - u0);
    if (nu > KR_FIN_UNITS) return -1;
    int64_t total = 0;
    for (int c0 = 0; c0 < nu; c0 += KR_BLOCK) {
        const int k = c0 + threadIdx.x;
        int tot;
        const int ex = block_exclusive(k < nu ? ucnt[u0 + k] : 0, 0, SumI32(), sc, &tot);
        if (k < nu) sh.upre[k] = (int)total + ex;
        total += tot;
    }
    __syncthreads();
    if (total > KR_FIN_CAP) return -1;
    const int n = (int)total;
    for (int x = threadIdx.x; x < n; x += KR_BLOCK) {
        int lo = 0, hi = nu - 1;  // unit holding element x
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sh.upre[mid] <= x) lo = mid;
            else hi = mid - 1;
        }
        const int64_t src = s0 + (int64_t)lo * L.unit_stride + (x - sh.upre[lo]);
        sh.sT[x] = dbits(buf.T[src]);
        sh.sE[x] = dbits(buf.E[src]);
        sh.sI[x] = buf.I[src];
    }
    __syncthreads();
    lds_sort_keys(sh.sT, sh.sE, sh.sI, n);
    return lds_frontier_scan(sh.sT, sh.sE, sh.sI, n, fin.T + s0, fin.E + s0, fin.I + s0);
}

__global__ void __launch_bounds__(KR_BLOCK)
finalize_block_kernel(SegLayout L, PointBufs buf, const int32_t *ucnt, PointBufs fin,
                      int32_t *fcnt, int32_t *runcnt, uint8_t *flags, const int32_t *lists)
{
    __shared__ FinLds sh;
    __shared__ int32_t sc[KR_WAVES];
    const int cnt = lists[1];
    for (int i = blockIdx.x; i < cnt; i += gridDim.x) {
        const int g = lists[2 + L.n_seg + i];
        int n = finalize_few(g, L, buf, ucnt, fin, sh, sc);
        if (n < 0) {
            __syncthreads();
            auto chunk = [&](int64_t x0, int m) {
                for (int x = threadIdx.x; x < m; x += KR_BLOCK) {
                    sh.sT[x] = dbits(ld_l2(fin.T + x0 + x));
                    sh.sE[x] = dbits(ld_l2(fin.E + x0 + x));
                    sh.sI[x] = ld_l2(fin.I + x0 + x);
                }
                __syncthreads();
                lds_sort_keys(sh.sT, sh.sE, sh.sI, m);
                return lds_frontier_scan(sh.sT, sh.sE, sh.sI, m, fin.T + x0, fin.E + x0,
                                         fin.I + x0);
            };
            n = finalize_chunks<KR_BLOCK>(g, L, buf, ucnt, fin, runcnt, flags, sh.upre, sc,
                                          KR_FIN_CAP, [] {}, chunk);
        }
        if (threadIdx.x == 0) fcnt[g] = n;
        __syncthreads();  // LDS reuse by the next segment
    }
}

// ----------------------------------------------------------------------------
// All of the merge in one launch, for up to KR_FUSED_SEGS segments (one block of 1,024
// threads each, which then fit on the chip together): a block merges its segment in LDS, or
// in chunks when it is larger, publishes its count, and writes the frontier to its final
// place as soon as the counts before it are known.  Blocks take their segments by ticket, so
// a block waits only for segments of blocks that started before it.  Waits are bounded all the
// same, for two calls that use one workspace at the same time: a count that neither comes nor
// changes for o.polls polls is given up, the block writes nothing, and the status word (if
// there is one) says KR_EHIP.  fcnt[g] is 0 until segment g's block has its count (then
// count + 1); a block that merges in chunks, which can take seconds, counts down from 0
// meanwhile, so that the others see it at work.  Four launches of which
// most blocks do nothing cost more than the merge itself where segments are few (4 to 256
// partitions; the 1,518 configurations of a microbatch: 193 us a call, 126 us so).
// RAW: the points come straight from (T, E), with no unit frontiers before (all segments
// together hold at most the LDS capacity, so any of them fits).
#define KR_FUSED_SEGS 256
constexpr int kFusedCap = KR_FM_LARGE_NT * KR_FM_LARGE_PER;

template <bool RAW>
__global__ void __launch_bounds__(KR_FM_LARGE_NT)
finalize_fused_kernel(const double *T, const double *E, int64_t n_total, SegLayout L,
                      PointBufs buf, const int32_t *ucnt, PointBufs fin, int32_t *fcnt,
                      int32_t *runcnt, uint8_t *flags, int32_t *lists, FrontierOut o)
{
    constexpr int NT = KR_FM_LARGE_NT, PER = KR_FM_LARGE_PER;
    union Lds {
        MergeLds<NT, PER> merge;
        MergeLds<KR_FM_SMALL_NT, KR_FM_SMALL_PER> small;  // below merge.upre
        int32_t upre[NT + 1];
        __device__ Lds() {}
    };
    __shared__ Lds sh;
    __shared__ int32_t s_seg;
    __shared__ int32_t sc32[NT / 64];
    __shared__ int64_t sc64[NT / 64], sc_small[KR_FM_SMALL_NT / 64];
    static_assert(sizeof(sh.small) <= 32 * NT * PER, "the prefix stays clear of it");
    const int tid = threadIdx.x;
    int g = 0;
    if (L.n_seg > 1) {
        if (tid == 0) s_seg = atomicAdd(&lists[0], 1);
        __syncthreads();
        g = s_seg;
        if (g < 0 || g >= L.n_seg) return;  // another call's ticket
    }
    int32_t beats = 0;
    auto beat = [&] {
        if (L.n_seg > 1 && threadIdx.x == 0)
            __hip_atomic_store(fcnt + g, --beats, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // the first output element of segment g, which holds `count` points (cap: a wait was given
    // up).  A count given up makes the sum of up to KR_FUSED_SEGS counts negative.
    constexpr int64_t kLost = -((int64_t)1 << 50);
    auto place = [&](int count, auto &sc) -> int64_t {  // sc: a word per wave of the block
        int64_t d0 = 0;
        if (L.n_seg > 1) {
            static_assert(KR_FUSED_SEGS <= KR_FM_SMALL_NT, "a thread per earlier segment");
            constexpr int NW = sizeof(sc) / sizeof(sc[0]);
            if (tid == 0)
                __hip_atomic_store(fcnt + g, count + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            int64_t before = 0;
            if (tid < g) {
                int32_t c, seen = 0;
                for (int n = 0; (c = ld_l2(fcnt + tid)) <= 0;) {
                    if (c != seen) n = 0;
                    else if (++n > o.polls) break;
                    seen = c;
                    __builtin_amdgcn_s_sleep(1);
                }
                before = c > 0 ? c - 1 : kLost;
            }
            d0 = block_reduce<int64_t, SumI64, NW>(before, (int64_t)0, SumI64(), sc);
            if (d0 < 0) {
                if (tid == 0) {
                    if (o.status) __hip_atomic_store(o.status, (int32_t)KR_EHIP, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                    o.off[g] = 0;
                    if (g == L.n_seg - 1) o.off[L.n_seg] = 0;
                }
                return o.cap;
            }
        }
        if (tid == 0) {
            o.off[g] = d0;
            if (g == L.n_seg - 1) o.off[L.n_seg] = d0 + count;
        }
        return d0;
    };
    if (RAW) {
        const int64_t s0 = L.seg_off[g];
        const int n = (int)max((int64_t)0, min(L.seg_off[g + 1] - s0, n_total - s0));
        uint32_t worst = 0;
        auto points = [&](int q0, int q1, MKey (&k)[PER]) {
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (q0 + j < q1) {
                    // + 0.0 maps -0.0 to +0.0, so that the bit patterns order like the values
                    const double t = T[s0 + q0 + j] + 0.0, e = E[s0 + q0 + j] + 0.0;
                    worst = max(worst, max(raw_hi(t), raw_hi(e)));
                    k[j] = MKey{dbits(t), dbits(e), q0 + j};
                }
        };
        merge_segment(n, points, sh.merge, o.T, o.E, o.idx, o.cap,
                      [&](int count) { return place(count, sc64); });
        if (o.status) {
            if (L.n_seg > 1) {
                report_values(o.status, worst >= KR_BAD_HI);  // KR_OK before the launch
            } else {
                const int bad = __syncthreads_or(worst >= KR_BAD_HI);
                if (tid == 0) *o.status = bad ? KR_ENONFINITE : KR_OK;
            }
        }
        return;
    }
    int n;
    if (merge_prefix(g, L, ucnt, sh.merge, n)) {
        const int nu = (int)(L.unit_base[g + 1] - L.unit_base[g]);
        __syncthreads();  // upre
        if (n <= KR_FM_SMALL_NT * KR_FM_SMALL_PER) {
            // Few points: four waves, the others end (a barrier waits for no ended wave).  256
            // segments of 100 points took 120 us a call with all sixteen, 115 so, and 112 with
            // launches of their own.
            if (tid >= KR_FM_SMALL_NT) return;
            const UnitPoints<NT, KR_FM_SMALL_PER> points{sh.merge.upre, buf, L.seg_off[g],
                                                         L.unit_stride, nu};
            merge_segment(n, points, sh.small, o.T, o.E, o.idx, o.cap,
                          [&](int count) { return place(count, sc_small); });
            return;
        }
        const UnitPoints<NT, PER> points{sh.merge.upre, buf, L.seg_off[g], L.unit_stride, nu};
        merge_segment(n, points, sh.merge, o.T, o.E, o.idx, o.cap,
                      [&](int count) { return place(count, sc64); });
        return;
    }
    __syncthreads();
    // Chunks of the merge sort's capacity, sorted by it: a union of about 5,000 points 87 us, with
    // bitonic chunks of 2,560 198 us (and with tile frontiers in front 135).
    auto chunk = [&](int64_t x0, int m) {
        auto points = [&](int q0, int q1, MKey (&k)[PER]) {
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (q0 + j < q1) {
                    const int64_t x = x0 + q0 + j;
                    k[j] = MKey{dbits(ld_l2(fin.T + x)), dbits(ld_l2(fin.E + x)), ld_l2(fin.I + x)};
                }
        };
        int kept = 0;
        merge_segment(m, points, sh.merge, fin.T, fin.E, fin.I, INT64_MAX, [&](int count) {
            kept = count;
            return x0;
        });
        return kept;
    };
    n = finalize_chunks<NT>(g, L, buf, ucnt, fin, runcnt, flags, sh.upre, sc32, kFusedCap, beat,
                            chunk);
    __syncthreads();  // the block's stores to fin are read back below
    const int64_t d0 = place(n, sc64), src0 = L.seg_off[g];
    for (int64_t x = tid; x < n && d0 + x < o.cap; x += NT) {
        o.idx[d0 + x] = ld_l2(fin.I + src0 + x);
        o.T[d0 + x] = ld_l2(fin.T + src0 + x);
        o.E[d0 + x] = ld_l2(fin.E + src0 + x);
    }
}

bool pareto_raw(int64_t n_total, int n_seg)
{
    return n_seg >= 1 && n_seg <= KR_FUSED_SEGS && n_total <= kFusedCap;
}

hipError_t launch_pareto_raw(const double *T, const double *E, int64_t n_total, const SegLayout &L,
                             int32_t *fcnt, int32_t *lists, const FrontierOut &o, hipStream_t st)
{
    const PointBufs none{nullptr, nullptr, nullptr};
    hipLaunchKernelGGL(finalize_fused_kernel<true>, dim3(L.n_seg), dim3(KR_FM_LARGE_NT), 0, st, T,
                       E, n_total, L, none, (const int32_t *)nullptr, none, fcnt,
                       (int32_t *)nullptr, (uint8_t *)nullptr, lists, o);
    return hipGetLastError();
}

// out_off = exclusive prefix sum of the per-segment frontier sizes; one block.
__global__ void __launch_bounds__(KR_BLOCK)
count_scan_kernel(int n_seg, const int32_t *fcnt, int64_t *out_off)
{
    __shared__ int64_t sc[KR_WAVES];
    int64_t carry = 0;
    for (int g0 = 0; g0 < n_seg; g0 += KR_BLOCK) {
        const int g = g0 + threadIdx.x;
        const int64_t c = g < n_seg ? fcnt[g] : 0;
        int64_t tot;
        const int64_t ex = block_exclusive(c, (int64_t)0, SumI64(), sc, &tot);
        if (g < n_seg) out_off[g] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) out_off[n_seg] = carry;
}

__global__ void __launch_bounds__(KR_BLOCK)
copy_out_kernel(SegLayout L, PointBufs fin, const int64_t *out_off, int64_t cap,
                int32_t *out_idx, double *out_T, double *out_E)
{
    const int g = blockIdx.x;
    const int64_t dst0 = out_off[g], n = out_off[g + 1] - dst0;
    const int64_t src0 = L.seg_off[g];
    for (int64_t x = threadIdx.x; x < n; x += KR_BLOCK) {
        const int64_t d = dst0 + x;
        if (d >= cap) break;
        out_idx[d] = fin.I[src0 + x];
        out_T[d] = fin.T[src0 + x];
        out_E[d] = fin.E[src0 + x];
    }
}

// Up to KR_OUT_SCAN segments: each block forms its segment's output offset itself (the
// sum of the counts before it, in integers, so equal to the scan's) and copies the
// segment, with no separate scan launch.
#define KR_OUT_SCAN 4096
__global__ void __launch_bounds__(KR_BLOCK)
copy_out_scan_kernel(SegLayout L, PointBufs fin, const int32_t *fcnt, int64_t *out_off,
                     int64_t cap, int32_t *out_idx, double *out_T, double *out_E)
{
    __shared__ int64_t sc[KR_WAVES];
    const int g = blockIdx.x;
    int64_t part = 0;
    for (int h = threadIdx.x; h < g; h += KR_BLOCK) part += fcnt[h];
    const int64_t dst0 = block_reduce(part, (int64_t)0, SumI64(), sc);
    const int64_t n = fcnt[g];
    if (threadIdx.x == 0) {
        out_off[g] = dst0;
        if (g == L.n_seg - 1) out_off[L.n_seg] = dst0 + n;
    }
    const int64_t src0 = L.seg_off[g];
    for (int64_t x = threadIdx.x; x < n; x += KR_BLOCK) {
        const int64_t d = dst0 + x;
        if (d >= cap) break;
        out_idx[d] = fin.I[src0 + x];
        out_T[d] = fin.T[src0 + x];
        out_E[d] = fin.E[src0 + x];
    }
}

static hipError_t launch_finalize(const SegLayout &L, const PointBufs &buf, const int32_t *ucnt,
                           const PointBufs &fin, int32_t *fcnt, int32_t *runcnt, uint8_t *flags,
                           int32_t *lists, hipStream_t st)
{
    if (L.n_seg == 0) return hipSuccess;
    const dim3 loop_grid(min(L.n_seg, 256));
    hipLaunchKernelGGL(finalize_small_kernel, dim3(L.n_seg), dim3(KR_FM_SMALL_NT), 0, st, L, buf,
                       ucnt, fin, fcnt, lists);
    hipLaunchKernelGGL(finalize_large_kernel, loop_grid, dim3(KR_FM_LARGE_NT), 0, st, L, buf,
                       ucnt, fin, fcnt, lists);
    hipLaunchKernelGGL(finalize_block_kernel, loop_grid, dim3(KR_BLOCK), 0, st, L, buf, ucnt,
                       fin, fcnt, runcnt, flags, lists);
    return hipGetLastError();
}

static hipError_t launch_output(const SegLayout &L, const PointBufs &fin, const int32_t *fcnt,
                         int64_t cap, int64_t *out_off, int32_t *out_idx, double *out_T,
                         double *out_E, hipStream_t st)
{
    if (L.n_seg > 0 && L.n_seg <= KR_OUT_SCAN) {
        hipLaunchKernelGGL(copy_out_scan_kernel, dim3(L.n_seg), dim3(KR_BLOCK), 0, st, L, fin,
                           fcnt, out_off, cap, out_idx, out_T, out_E);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(count_scan_kernel, dim3(1), dim3(KR_BLOCK), 0, st, L.n_seg, fcnt, out_off);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || L.n_seg == 0) return e;
    hipLaunchKernelGGL(copy_out_kernel, dim3(L.n_seg), dim3(KR_BLOCK), 0, st, L, fin, out_off, cap,
                       out_idx, out_T, out_E);
    return hipGetLastError();
}

hipError_t launch_merge(const SegLayout &L, const PointBufs &buf, const int32_t *ucnt,
                        const PointBufs &fin, int32_t *fcnt, int32_t *runcnt, uint8_t *flags,
                        int32_t *lists, const FrontierOut &o, hipStream_t st)
{
    if (L.n_seg >= 1 && L.n_seg <= KR_FUSED_SEGS) {
        hipLaunchKernelGGL(finalize_fused_kernel<false>, dim3(L.n_seg), dim3(KR_FM_LARGE_NT), 0, st,
                           (const double *)nullptr, (const double *)nullptr, (int64_t)0, L, buf,
                           ucnt, fin, fcnt, runcnt, flags, lists, o);
        return hipGetLastError();
    }
    const hipError_t e = launch_finalize(L, buf, ucnt, fin, fcnt, runcnt, flags, lists, st);
    if (e != hipSuccess) return e;
    return launch_output(L, fin, fcnt, o.cap, o.off, o.idx, o.T, o.E, st);
}

}  // namespace kr
