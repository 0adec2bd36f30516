// Launch-timing frontier of two operation sequences (Appendix B's dynamic program), one
// instance per 64-lane workgroup.
//
// The cells P(i, j) (suffixes from S1[i] and S2[j]) are filled from (I, J) back to
// (0, 0), row by row, so every successor is ready.  Per cell:
//   * one lane per decision slot (S1 op alone, S2 op alone, S1's communication
//     overlapped with k of S2's computations, the same swapped) prices its group with
//     the fluid overlap walk and checks that it is allowed; the allowed slots, in that
//     order, become the cell's sources;
//   * the candidates are (group + successor point) over the sources, in source order
//     and then the successor's order; their index is their generation order;
//   * a candidate is kept iff no candidate before it in (T, E, index) order has energy at
//     or below its own (GetFrontier with exact duplicates to the first), decided by
//     comparing against every candidate (cells hold tens of candidates, so this beats
//     sorting): with at most 64 candidates one per lane, through lane reads; otherwise
//     through LDS broadcast reads; a kept point's rank is the number of kept points
//     with a smaller time;
//   * the kept points go to an LDS arena with their back-pointer (source, point).
// The schedules of P(0, 0) are then walked back one lane per point.
//
// Most cells have a handful of candidates (4 on average on two 11-op sequences, 98.9 % have
// at most 16), so the first pass packs four instances into a wave, one per row of 16 lanes:
// the cells, their slots and their order are the same for all of them, only the counts
// differ.  Sources, scans and comparisons stay inside a row and use its DPP broadcasts.
// The instances that need more than their share are solved again, one per wave as above.
#include <math.h>

#include <type_traits>
#include <utility>

#include "kr_device.h"
#include "kr_launch.h"

namespace kr {

namespace {

constexpr int kSlots = 2 + 2 * KR_DP_MAX_K;

// Value of lane `src` (per-lane index) for a 64-bit quantity.
__device__ __forceinline__ uint64_t shfl_u64(uint64_t x, int src)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)x, src, 64);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(x >> 32), src, 64);
    return ((uint64_t)hi << 32) | lo;
}

// An instance is one wave, whose LDS accesses execute in order: ordering them for the
// compiler is all the synchronisation a cell needs.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ void dp_alone(const double *op, double ps, double *T, double *E)
{
    const double t = op[0], p = op[1];
    *T = t;
    *E = t * p + ps * t;
}

// A communication `c` with the computations ops[r0], ops[r0 + 1], ... ops[r0 + k - 1].
__device__ __forceinline__ void dp_group(const double *ops, int c, int r0, int k, double ps,
                                         double *T, double *E)
{
    const double tc = ops[4 * c], pc = ops[4 * c + 1];
    double tau = 0.0, e = 0.0;
    for (int r = 0; r < k; ++r) {
        const double *o = ops + 4 * (r0 + r);
        const double t0 = o[0], p0 = o[1], t1 = o[2], p1 = o[3];
        if (tau < tc) {
            const double nt = tau + t1;
            if (nt <= tc) {
                e = e + t1 * p1;
                tau = nt;
            } else {
                const double dt = tc - tau;
                const double rem = 1.0 - dt / t1;
                const double ta = rem * t0;
                e = e + dt * p1;
                e = e + ta * p0;
                tau = tc + ta;
            }
        } else {
            e = e + t0 * p0;
            tau = tau + t0;
        }
    }
    const double t = tau > tc ? tau : tc;
    *T = t;
    *E = (e + tc * pc) + ps * t;
}

struct Slots {
    int va, vb, nc, nd;  // allowed: S1 alone, S2 alone, overlaps of each kind
};

__device__ __forceinline__ Slots dp_slots(const DpArgs &a, int i, int j)
{
    Slots s;
    s.va = i < a.I;
    s.vb = j < a.J;
    s.nc = i < a.I && a.kind[i] == 1 ? min(a.kmax, (int)a.run2[j]) : 0;
    s.nd = j < a.J && a.kind[a.I + j] == 1 ? min(a.kmax, (int)a.run1[i]) : 0;
    return s;
}

// Source r of cell (i, j) -> decision code (case * 32 + k) and successor cell.
__device__ __forceinline__ int dp_decode(const DpArgs &a, int i, int j, int r, int *ni, int *nj)
{
    const Slots s = dp_slots(a, i, j);
    if (r < s.va) {
        *ni = i + 1;
        *nj = j;
        return 0;
    }
    r -= s.va;
    if (r < s.vb) {
        *ni = i;
        *nj = j + 1;
        return 32;
    }
    r -= s.vb;
    if (r < s.nc) {
        *ni = i + 1;
        *nj = j + r + 1;
        return 64 + r + 1;
    }
    r -= s.nc;
    *ni = i + r + 1;
    *nj = j + 1;
    return 96 + r + 1;
}

// Whether a walk back goes on from cell (i, j).  Kept points are strictly ordered in time
// unless a time is not a number; then a place behind the others stays unwritten and the
// back-pointer read there may be anything, so the walk ends outside the table as well.
__device__ __forceinline__ bool dp_inside(const DpArgs &a, int i, int j)
{
    return i <= a.I && j <= a.J && !(i == a.I && j == a.J);
}

// Byte offsets of the LDS sections of one instance (all 8-byte aligned).
struct DpLds {
    int ops, arT, arE, cT, cE, sT, sE, soff, sstart, arB, cstart, ccnt, csrc, keep, bytes;
};

__host__ __device__ inline DpLds dp_lds(int nops, int ncell, int arena, int cand)
{
    DpLds l;
    int o = 0;
    auto take = [&](int bytes) {
        const int at = o;
        o += (bytes + 7) / 8 * 8;
        return at;
    };
    l.ops = take(32 * nops);
    l.arT = take(8 * arena);
    l.arE = take(8 * arena);
    l.cT = take(8 * cand);
    l.cE = take(8 * cand);
    l.sT = take(8 * kSlots);
    l.sE = take(8 * kSlots);
    l.soff = take(4 * (kSlots + 1));
    l.sstart = take(4 * kSlots);
    l.arB = take(2 * arena);
    l.cstart = take(2 * ncell);
    l.ccnt = take(2 * ncell);
    l.csrc = take(cand);
    l.keep = take(cand);
    l.bytes = o;
    return l;
}

// One instance by one wave, with an arena of `arena` points and `cand` candidates per
// cell; false (nothing written) if the instance needs more.
__device__ bool dp_solve(const DpArgs &a, int64_t inst, char *lds, int arena, int cand)
{
    const int lane = threadIdx.x;
    const int nops = a.I + a.J, W = a.J + 1;
    const DpLds L = dp_lds(nops, (a.I + 1) * W, arena, cand);
    double *ops = (double *)(lds + L.ops);
    double *arT = (double *)(lds + L.arT), *arE = (double *)(lds + L.arE);
    double *cT = (double *)(lds + L.cT), *cE = (double *)(lds + L.cE);
    double *sT = (double *)(lds + L.sT), *sE = (double *)(lds + L.sE);
    int32_t *soff = (int32_t *)(lds + L.soff), *sstart = (int32_t *)(lds + L.sstart);
    int16_t *arB = (int16_t *)(lds + L.arB);
    int16_t *cstart = (int16_t *)(lds + L.cstart), *ccnt = (int16_t *)(lds + L.ccnt);
    uint8_t *keep = (uint8_t *)(lds + L.keep);
    uint8_t *csrc = (uint8_t *)(lds + L.csrc);  // source of each candidate of the cell
    for (int x = lane; x < 4 * nops; x += 64) ops[x] = a.ops[inst * 4 * nops + x];
    if (lane == 0) {
        const int last = a.I * W + a.J;
        arT[0] = 0.0;
        arE[0] = 0.0;
        arB[0] = -1;
        cstart[last] = 0;
        ccnt[last] = 1;
    }
    wave_sync();
    int used = 1;  // arena points in use (uniform)
    bool ok = true;
    for (int i = a.I; i >= 0 && ok; --i) {
        for (int j = a.J; j >= 0 && ok; --j) {
            if (i == a.I && j == a.J) continue;
            const Slots s = dp_slots(a, i, j);
            // lane = decision slot in canonical order; allowed slots become sources
            bool allowed = false;
            double gT = 0.0, gE = 0.0;
            int ni = 0, nj = 0;
            if (lane == 0 && s.va) {
                allowed = true;
                dp_alone(ops + 4 * i, a.p_static, &gT, &gE);
                ni = i + 1;
                nj = j;
            } else if (lane == 1 && s.vb) {
                allowed = true;
                dp_alone(ops + 4 * (a.I + j), a.p_static, &gT, &gE);
                ni = i;
                nj = j + 1;
            } else if (lane >= 2 && lane < 2 + KR_DP_MAX_K && lane - 1 <= s.nc) {
                const int k = lane - 1;
                allowed = true;
                dp_group(ops, i, a.I + j, k, a.p_static, &gT, &gE);
                ni = i + 1;
                nj = j + k;
            } else if (lane >= 2 + KR_DP_MAX_K && lane < kSlots &&
                       lane - 1 - KR_DP_MAX_K <= s.nd) {
                const int k = lane - 1 - KR_DP_MAX_K;
                allowed = true;
                dp_group(ops, a.I + j, i, k, a.p_static, &gT, &gE);
                ni = i + k;
                nj = j + 1;
            }
            const uint64_t m = __ballot(allowed);
            const int ns = __popcll(m);
            const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const int n_succ = allowed ? ccnt[ni * W + nj] : 0;
            // exclusive prefix of the successor counts in source order
            int inc = n_succ;
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(inc, d, 64);
                if (lane >= d) inc += y;
            }
            const int C = __shfl(inc, 63, 64);
            if (C > cand) {
                ok = false;
                break;
            }
            const int ex = inc - n_succ;  // first candidate of this lane's source
            const int st = allowed ? (int)cstart[ni * W + nj] : 0;
            int kept;
            if (C <= 64) {
                // one candidate per lane; its source found and read through lane reads
                const bool live = lane < C;
                int sl = 0, sr = 0, rk = 0;
                for (uint64_t mm = m; mm; mm &= mm - 1) {
                    const int l = __ffsll((long long)mm) - 1;
                    if (__builtin_amdgcn_readlane(ex, l) <= lane) {
                        sl = l;
                        sr = rk;
                    }
                    ++rk;
                }
                const double sgT = bitsd(shfl_u64(dbits(gT), sl));
                const double sgE = bitsd(shfl_u64(dbits(gE), sl));
                const int q = lane - __shfl(ex, sl, 64);
                const int sst = __shfl(st, sl, 64);
                double t = INFINITY, e = INFINITY;
                const int lo = sr;
                if (live) {
                    t = sgT + arT[sst + q];
                    e = sgE + arE[sst + q];
                }
                bool k = live;
                for (int y = 0; y < C; ++y) {
                    const double ty = bitsd(lane_u64(dbits(t), y));
                    const double ey = bitsd(lane_u64(dbits(e), y));
                    const bool before = ty < t || (ty == t && (ey < e || (ey == e && y < lane)));
                    if (before && ey <= e) k = false;
                }
                uint64_t km = __ballot(k);
                kept = __popcll(km);
                if (kept > KR_DP_CELL_CAP || used + kept > arena) {
                    ok = false;
                    break;
                }
                int rank = 0;  // kept points are strictly ordered in time
                while (km) {
                    const int y = __ffsll((long long)km) - 1;
                    km &= km - 1;
                    rank += bitsd(lane_u64(dbits(t), y)) < t ? 1 : 0;
                }
                if (k) {
                    arT[used + rank] = t;
                    arE[used + rank] = e;
                    arB[used + rank] = (int16_t)(lo * 64 + q);
                }
            } else {
                if (allowed) {
                    sT[r] = gT;
                    sE[r] = gE;
                    soff[r] = ex;
                    sstart[r] = st;
                    for (int q = 0; q < n_succ; ++q) csrc[ex + q] = (uint8_t)r;
                }
                if (lane == 0) soff[ns] = C;
                wave_sync();
                for (int c = lane; c < C; c += 64) {
                    const int lo = csrc[c];
                    const int q = c - soff[lo];
                    cT[c] = sT[lo] + arT[sstart[lo] + q];
                    cE[c] = sE[lo] + arE[sstart[lo] + q];
                }
                wave_sync();
                int kept_here = 0;
                for (int c = lane; c < C; c += 64) {
                    const double t = cT[c], e = cE[c];
                    bool k = true;
#pragma unroll 4
                    for (int y = 0; y < C; ++y) {
                        const double ty = cT[y], ey = cE[y];
                        const bool before = ty < t || (ty == t && (ey < e || (ey == e && y < c)));
                        if (before && ey <= e) k = false;
                    }
                    keep[c] = k;
                    kept_here += k;
                }
                wave_sync();
                kept = kept_here;
                for (int d = 32; d > 0; d >>= 1) kept += __shfl_xor(kept, d, 64);
                if (kept > KR_DP_CELL_CAP || used + kept > arena) {
                    ok = false;
                    break;
                }
                for (int c = lane; c < C; c += 64) {
                    if (!keep[c]) continue;
                    const double t = cT[c];
                    int rank = 0;
#pragma unroll 4
                    for (int y = 0; y < C; ++y) rank += keep[y] && cT[y] < t;
                    const int lo = csrc[c];
                    arT[used + rank] = t;
                    arE[used + rank] = cE[c];
                    arB[used + rank] = (int16_t)(lo * 64 + (c - soff[lo]));
                }
            }
            if (lane == 0) {
                cstart[i * W + j] = (int16_t)used;
                ccnt[i * W + j] = (int16_t)kept;
            }
            used += kept;
            wave_sync();
        }
    }
    if (!ok) return false;
    const int n0 = ccnt[0];
    if (lane == 0) a.out_n[inst] = n0;
    const int q = lane;
    if (q < n0 && q < a.out_cap) {
        const int64_t o = inst * a.out_cap + q;
        a.out_T[o] = arT[cstart[0] + q];
        a.out_E[o] = arE[cstart[0] + q];
        if (a.out_sched) {
            int32_t *sc = a.out_sched + o * nops;
            int ci = 0, cj = 0, cq = q, d = 0;
            while (dp_inside(a, ci, cj) && d < nops) {
                const int b = arB[min(cstart[ci * W + cj] + cq, arena - 1)];
                int ni, nj;
                sc[d++] = dp_decode(a, ci, cj, b >> 6, &ni, &nj);
                ci = ni;
                cj = nj;
                cq = b & 63;
            }
            for (; d < nops; ++d) sc[d] = -1;
        }
    }
    return true;
}

// ---- four instances per wave -----------------------------------------------------------

// Lane Y of every row of 16, in all lanes of the row.
template <int Y>
__device__ __forceinline__ int row_bcast(int x)
{
    // row_newbcast; every lane has a source, so no old value is set up (VALU issue bounds the
    // kernel, and that move doubled the broadcasts)
    return __builtin_amdgcn_mov_dpp(x, 0x150 + Y, 0xF, 0xF, false);
}
template <int Y>
__device__ __forceinline__ double row_bcast(double x)
{
    const uint64_t b = dbits(x);
    const uint32_t lo = (uint32_t)row_bcast<Y>((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)row_bcast<Y>((int)(uint32_t)(b >> 32));
    return bitsd(((uint64_t)hi << 32) | lo);
}
template <int D>
__device__ __forceinline__ int row_add_below(int x)  // x plus lane - D's x (0 past the row)
{
    return x + __builtin_amdgcn_update_dpp(0, x, 0x110 + D, 0xF, 0xF, false);  // row_shr
}

// f(0), f(1), ... f(15) with compile-time arguments, as long as they are below n (uniform).
template <typename F, int... Y>
__device__ __forceinline__ void row_for(int n, F f, std::integer_sequence<int, Y...>)
{
    ((Y < n && (f(std::integral_constant<int, Y>()), true)) && ...);
}
template <typename F>
__device__ __forceinline__ void row_for(int n, F f)
{
    row_for(n, f, std::make_integer_sequence<int, 16>());
}

// Byte offsets of the LDS of one wave of four instances: their operations, the points of
// all their cells (one pool) and each cell's (first point << 8 | points).
struct DpQuadLds {
    int ops, arT, arE, arB, cell, bytes;
};

__host__ __device__ inline DpQuadLds dp_quad_lds(int nops, int ncell, int pool)
{
    DpQuadLds l;
    int o = 0;
    auto take = [&](int bytes) {
        const int at = o;
        o += (bytes + 7) / 8 * 8;
        return at;
    };
    l.ops = take(4 * 32 * nops);
    l.arT = take(8 * pool);
    l.arE = take(8 * pool);
    l.cell = take(4 * 4 * ncell);
    l.arB = take(2 * pool);
    l.bytes = o;
    return l;
}

// Keeps candidate c (this lane's, `mine`) unless one before it in (T, E, index) order has
// energy at or below its own; y is the other one's index.
__device__ __forceinline__ bool dp_beaten(double ty, double ey, int y, double t, double e, int c)
{
    return ty <= t && ey <= e && !(ty == t && ey == e && y >= c);
}

// The points of four instances fill up to 40 KB of LDS, so only four such groups share a
// compute unit, and a cell is one chain of LDS reads, row scans and compares.  The cells of an
// antidiagonal need only later antidiagonals, so KR_DP_QW waves share the group's LDS and
// take them in turn, a barrier between antidiagonals.  65,536 instances of two 11-op
// sequences: 6.8 ms with one instance per wave, 2.7 ms with one wave per four, 1.3 ms so.
#define KR_DP_QW 4

struct QuadShared {
    int32_t used;  // pool points in use (may pass the pool's end)
    int32_t dead;  // bit q: instance q needs more than its share
};

// The instances of group `grp`: 4 * grp .. 4 * grp + 3 of all, or of the first queue; the
// ones that need more (points than the pool or KR_DP_ARENA holds, or more than 64 candidates in
// a cell; 128 from the queue) go on the first queue, or from there on the second.
template <bool QUEUED>
__device__ __forceinline__ void dp_quad(const DpArgs &a, int64_t grp, int64_t n, int pool,
                                        char *lds, QuadShared &sh)
{
    const int lane = threadIdx.x & 63, row = lane >> 4, r = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int H = QUEUED ? 8 : 4;  // candidates per lane at most
    const int nops = a.I + a.J, W = a.J + 1, ncell = (a.I + 1) * W;
    const DpQuadLds L = dp_quad_lds(nops, ncell, pool);
    double *const ops4 = (double *)(lds + L.ops);
    double *const arT = (double *)(lds + L.arT), *const arE = (double *)(lds + L.arE);
    int16_t *const arB = (int16_t *)(lds + L.arB);
    int32_t *const cell = (int32_t *)(lds + L.cell) + row * ncell;
    const int64_t inst0 = grp * 4;
    const bool there = inst0 + row < n;  // row-uniform
    const int64_t inst = !there ? 0 : QUEUED ? a.retry[inst0 + row] : inst0 + row;
    const double *const ops = ops4 + 4 * nops * row;
    {
        // a row with no instance solves a copy of another's numbers, and writes nothing
        const double *const src = a.ops + inst * 4 * nops;
        for (int x = wave * 16 + r; x < 4 * nops; x += 16 * KR_DP_QW)
            ops4[4 * nops * row + x] = src[x];
    }
    if (threadIdx.x == 0) {
        arT[0] = 0.0;
        arE[0] = 0.0;
        arB[0] = -1;
        sh.used = 1;
        sh.dead = 0;
    }
    if (wave == 0 && r == 0) cell[ncell - 1] = 1;  // P(I, J) = {(0, 0)}, one point for all four
    // lane o: kind and run of op o of each sequence (reading them from the arguments by a
    // varying index would be a memory access per cell)
    const int seq1 = lane < a.I ? a.kind[lane] | a.run1[lane] << 1 : 0;
    const int seq2 = lane < a.J ? a.kind[a.I + lane] | a.run2[lane] << 1 : 0;
    bool dead = !there;  // row-uniform
    const uint64_t row_bits = 0xFFFFull << (16 * row);
    for (int d = a.I + a.J - 1; d >= 0; --d) {
        __syncthreads();  // the later antidiagonals' cells are in LDS
        dead = dead || (sh.dead >> row & 1);
        const int i1 = min(a.I, d);
        for (int i = max(0, d - a.J) + wave; i <= i1; i += KR_DP_QW) {
            const int j = d - i;
            const int k1 = lane_i32(seq1, i), k2 = lane_i32(seq2, j);
            Slots s;
            s.va = i < a.I;
            s.vb = j < a.J;
            s.nc = k1 & 1 ? min(a.kmax, k2 >> 1) : 0;
            s.nd = k2 & 1 ? min(a.kmax, k1 >> 1) : 0;
            const int ns = s.va + s.vb + s.nc + s.nd;  // at most 16 (the launch checks)
            // lane r of a row = source r, in canonical order (nc and nd are never both set)
            double gT = 0.0, gE = 0.0;
            int succ = 0;
            {
                const bool isb = r >= s.va;  // the alone op of S2, and overlaps below
                const int k = r - s.va - s.vb + 1;
                const int ni = k >= 1 ? (s.nc ? i + 1 : i + k) : (isb ? i : i + 1);
                const int nj = k >= 1 ? (s.nc ? j + k : j + 1) : (isb ? j + 1 : j);
                if (r < ns) succ = cell[ni * W + nj];
                if (k < 1)
                    dp_alone(ops + 4 * (isb ? a.I + j : i), a.p_static, &gT, &gE);
                else if (r < ns)
                    dp_group(ops, s.nc ? i : a.I + j, s.nc ? a.I + j : i, k, a.p_static, &gT, &gE);
            }
            const int n_succ = dead ? 0 : succ & 0xFF, st = succ >> 8;
            int inc = row_add_below<1>(n_succ);
            inc = row_add_below<2>(inc);
            inc = row_add_below<4>(inc);
            inc = row_add_below<8>(inc);
            const int ex = inc - n_succ;  // first candidate of this lane's source
            int C = row_bcast<15>(inc);   // candidates of this row's cell
            if (C > 16 * H) {
                dead = true;
                C = 0;
            }
            const int Cm = max(max(lane_i32(C, 0), lane_i32(C, 16)),
                               max(lane_i32(C, 32), lane_i32(C, 48)));
            // up to NH candidates per lane: c = r, r + 16, ...
            auto solve = [&](auto nh) {
                constexpr int NH = decltype(nh)::value;
                const int rb = lane & 48;
                double t[NH], e[NH];
                int lo[NH], q[NH], at[NH];
#pragma unroll
                for (int h = 0; h < NH; ++h) lo[h] = q[h] = at[h] = 0;
                if constexpr (NH <= 2) {
                    row_for(ns, [&](auto y) {
                        constexpr int Y = decltype(y)::value;
                        const int exy = row_bcast<Y>(ex), sty = row_bcast<Y>(st);
                        const double Ty = row_bcast<Y>(gT), Ey = row_bcast<Y>(gE);
#pragma unroll
                        for (int h = 0; h < NH; ++h)
                            if (exy <= r + 16 * h) {
                                lo[h] = Y;
                                q[h] = r + 16 * h - exy;
                                at[h] = sty;
                                t[h] = Ty;
                                e[h] = Ey;
                            }
                    });
                } else {
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        if (16 * h >= Cm) break;
                        for (int y = 0; y < ns; ++y) {
                            const int exy = __shfl(ex, rb + y, 64);
                            if (exy <= r + 16 * h) {
                                lo[h] = y;
                                q[h] = r + 16 * h - exy;
                            }
                        }
                        t[h] = bitsd(shfl_u64(dbits(gT), rb + lo[h]));
                        e[h] = bitsd(shfl_u64(dbits(gE), rb + lo[h]));
                        at[h] = __shfl(st, rb + lo[h], 64);
                    }
                }
                bool k[NH];
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    k[h] = r + 16 * h < C;
                    t[h] = k[h] ? t[h] + arT[at[h] + q[h]] : INFINITY;
                    e[h] = k[h] ? e[h] + arE[at[h] + q[h]] : INFINITY;
                }
                // f(T, E, index) of every candidate of the row
                auto each = [&](const double (&u)[NH], const double (&v)[NH], auto f) {
#pragma unroll
                    for (int g = 0; g < NH; ++g) {
                        if constexpr (NH <= 2)
                            row_for(Cm - 16 * g, [&](auto y) {
                                constexpr int Y = decltype(y)::value;
                                f(row_bcast<Y>(u[g]), row_bcast<Y>(v[g]), 16 * g + Y);
                            });
                        else
                            for (int y = 0; y < 16 && 16 * g + y < Cm; ++y)
                                f(bitsd(shfl_u64(dbits(u[g]), rb + y)),
                                  bitsd(shfl_u64(dbits(v[g]), rb + y)), 16 * g + y);
                    }
                };
                each(t, e, [&](double ty, double ey, int y) {
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        if (16 * h >= Cm) break;  // uniform
                        if (dp_beaten(ty, ey, y, t[h], e[h], r + 16 * h)) k[h] = false;
                    }
                });
                // pool places: rows in order, kept points of a row by time (distinct)
                int kept = 0, before = 0, total = 0;
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    const uint64_t km = __ballot(k[h]);
                    kept += __popcll(km & row_bits);
                    before += __popcll(km & ((1ull << (16 * row)) - 1));
                    total += __popcll(km);
                }
                int used = 0;
                if (lane == 0) used = atomicAdd(&sh.used, total);
                double tk[NH];
                int rank[NH];
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    tk[h] = k[h] ? t[h] : INFINITY;
                    rank[h] = 0;
                }
                each(tk, tk, [&](double ty, double, int) {
#pragma unroll
                    for (int h = 0; h < NH; ++h) {
                        if (16 * h >= Cm) break;
                        rank[h] += ty < t[h] ? 1 : 0;
                    }
                });
                const int b = lane_i32(used, 0) + before;
                const bool fits = kept <= KR_DP_CELL_CAP && b + kept <= pool;
                if (!fits) dead = true;
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    if (k[h] && fits) {
                        arT[b + rank[h]] = t[h];
                        arE[b + rank[h]] = e[h];
                        arB[b + rank[h]] = (int16_t)(lo[h] * 64 + q[h]);
                    }
                if (r == 0) cell[i * W + j] = fits ? b << 8 | kept : 0;
            };
            if (Cm <= 16) solve(std::integral_constant<int, 1>());
            else if (Cm <= 32) solve(std::integral_constant<int, 2>());
            else solve(std::integral_constant<int, H>());
            if (dead && r == 0 && there) atomicOr(&sh.dead, 1 << row);
        }
    }
    __syncthreads();
    if (!there) return;
    // The pool is shared, but the limit of KR_DP_ARENA points over all cells is an
    // instance's own: with the pool above it the row counts its points (every wave its four
    // rows alike), so that no verdict depends on the instances beside it.
    dead = sh.dead >> row & 1;
    if (sh.used > KR_DP_ARENA) {
        int points = 0;
        for (int x = r; x < ncell; x += 16) points += cell[x] & 0xFF;
        for (int m = 8; m > 0; m >>= 1) points += __shfl_xor(points, m, 64);
        dead = dead || points > KR_DP_ARENA;
    }
    if (dead) {
        if (wave == 0 && r == 0) {
            a.out_n[inst] = -1;
            int32_t *const queue = a.retry + (QUEUED ? a.n_inst : 0);
            queue[atomicAdd(a.retry_n + (QUEUED ? 1 : 0), 1)] = (int32_t)inst;
        }
        return;
    }
    const int n0 = cell[0] & 0xFF;
    if (wave == 0 && r == 0) a.out_n[inst] = n0;
    for (int p = wave * 16 + r; p < min(n0, a.out_cap); p += 16 * KR_DP_QW) {
        const int64_t o = inst * a.out_cap + p;
        a.out_T[o] = arT[(cell[0] >> 8) + p];
        a.out_E[o] = arE[(cell[0] >> 8) + p];
        if (a.out_sched) {
            int32_t *sc = a.out_sched + o * nops;
            int ci = 0, cj = 0, cq = p, d = 0;
            while (dp_inside(a, ci, cj) && d < nops) {
                const int b = arB[min((cell[ci * W + cj] >> 8) + cq, pool - 1)];
                int ni, nj;
                sc[d++] = dp_decode(a, ci, cj, b >> 6, &ni, &nj);
                ci = ni;
                cj = nj;
                cq = b & 63;
            }
            for (; d < nops; ++d) sc[d] = -1;
        }
    }
}

__global__ void __launch_bounds__(64 * KR_DP_QW) dp_quad_kernel(DpArgs a, int pool)
{
    extern __shared__ double dp_smem[];
    __shared__ QuadShared sh;
    dp_quad<false>(a, blockIdx.x, a.n_inst, pool, (char *)dp_smem, sh);
}

// The queued instances, four to a block with a larger pool (a block for an instance alone
// would take as long).
__global__ void __launch_bounds__(64 * KR_DP_QW) dp_quad_retry_kernel(DpArgs a, int pool)
{
    extern __shared__ double dp_smem[];
    __shared__ QuadShared sh;
    const int64_t n = a.retry_n[0];
    for (int64_t grp = blockIdx.x; grp * 4 < n; grp += gridDim.x) {
        dp_quad<true>(a, grp, n, pool, (char *)dp_smem, sh);
        __syncthreads();
    }
}

__global__ void dp_init_kernel(int32_t *status, int32_t *retry_n)
{
    *status = KR_OK;
    retry_n[0] = 0;
    retry_n[1] = 0;
}

// Every instance with the small on-chip budget; the ones that need more are queued.
__global__ void __launch_bounds__(64) dp_first_kernel(DpArgs a)
{
    extern __shared__ double dp_smem[];
    const int64_t inst = blockIdx.x;
    if (!dp_solve(a, inst, (char *)dp_smem, a.arena_s, a.cand_s) && threadIdx.x == 0) {
        a.out_n[inst] = -1;
        a.retry[atomicAdd(a.retry_n, 1)] = (int32_t)inst;
    }
}

// The instances of queue `tier` (0 or 1) with a larger budget (persistent grid over the
// queue); the ones that still do not fit go to the next queue, or are reported after
// the last tier.
__global__ void __launch_bounds__(64) dp_retry_kernel(DpArgs a, int tier, int arena, int cand)
{
    extern __shared__ double dp_smem[];
    const int n = a.retry_n[tier];
    const int32_t *q = a.retry + (int64_t)tier * a.n_inst;
    for (int r = blockIdx.x; r < n; r += gridDim.x) {
        const int64_t inst = q[r];
        if (!dp_solve(a, inst, (char *)dp_smem, arena, cand) && threadIdx.x == 0) {
            a.out_n[inst] = -1;
            if (tier == 0)
                a.retry[a.n_inst + atomicAdd(a.retry_n + 1, 1)] = (int32_t)inst;
            else
                *a.status = KR_ECAPACITY;
        }
        wave_sync();
    }
}

}  // namespace

hipError_t launch_dp(const DpArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(dp_init_kernel, dim3(1), dim3(1), 0, st, a.status, a.retry_n);
    if (a.n_inst > 0) {
        const int nops = a.I + a.J, ncell = (a.I + 1) * (a.J + 1);
        // a cell has at most two lone ops and one run of overlaps as its sources: a row of
        // 16 lanes takes runs of up to 14
        int run = 0;
        for (int i = 0; i <= a.I; ++i) run = a.run1[i] > run ? a.run1[i] : run;
        for (int j = 0; j <= a.J; ++j) run = a.run2[j] > run ? a.run2[j] : run;
        const int64_t g2 = a.n_inst < 512 ? a.n_inst : 512;
        if (2 + (a.kmax < run ? a.kmax : run) <= 16) {
            // As many points as let the four groups that the registers allow share a compute
            // unit (40 KB each); what does not fit is solved again with 64 KB.  Two 11-op
            // sequences: 796 points a group on average, 1,969 at most of 1,500 groups.  A
            // pool of 1,296 sent 2 % of the instances to one-wave solvers, which took 0.76 ms
            // however few they were.
            const int fixed = 64 + dp_quad_lds(nops, ncell, 0).bytes;
            const int room = (40 * 1024 - fixed) / 18 & ~3, most = (64 * 1024 - fixed) / 18 & ~3;
            const int pool = room < 1024 ? 1024 : room < 16 * ncell ? room : 16 * ncell;
            const int64_t groups = (a.n_inst + 3) / 4;
            hipLaunchKernelGGL(dp_quad_kernel, dim3((unsigned)groups), dim3(64 * KR_DP_QW),
                               dp_quad_lds(nops, ncell, pool).bytes, st, a, pool);
            hipLaunchKernelGGL(dp_quad_retry_kernel, dim3((unsigned)(groups < 512 ? groups : 512)),
                               dim3(64 * KR_DP_QW), dp_quad_lds(nops, ncell, most).bytes, st, a,
                               most);
        } else {
            const int small = dp_lds(nops, ncell, a.arena_s, a.cand_s).bytes;
            hipLaunchKernelGGL(dp_first_kernel, dim3((unsigned)a.n_inst), dim3(64), small, st, a);
            // middle budget: still several instances per compute unit; then the full one
            const int am = KR_DP_ARENA / 2, cm = KR_DP_CAND / 4;
            const int mid = dp_lds(nops, ncell, am, cm).bytes;
            const int64_t g1 = a.n_inst < 2048 ? a.n_inst : 2048;
            hipLaunchKernelGGL(dp_retry_kernel, dim3((unsigned)g1), dim3(64), mid, st, a, 0, am, cm);
        }
        const int big = dp_lds(nops, ncell, KR_DP_ARENA, KR_DP_CAND).bytes;
        hipLaunchKernelGGL(dp_retry_kernel, dim3((unsigned)g2), dim3(64), big, st, a, 1,
                           KR_DP_ARENA, KR_DP_CAND);
    }
    return hipGetLastError();
}

}  // namespace kr
