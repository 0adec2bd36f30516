// Two-comm candidate evaluation and frontier filter, a few waves per slab (gfx950).
//
// With two comm kernels the candidates of a (partition, frequency) slab are the
// launch-position pairs p1 <= p2 times the SM choices (s1, s2) (Sections 4.1, 4.5).  The
// waves of a block share one slab's tables in LDS and split its launch positions p1;
// lane s1 * S + s2 takes SM choices (s1, s2) (at most 8 SM choices, so S * S <= 64) and
// steps through a wave's pairs in candidate order, one pair per round for every lane.
//
// The walk of the partition cost model (fluid SM-share reading of Sections 3.2, 4.2
// and 4.5; the comm kernels share one stream in launch order) falls into phases whose
// inputs repeat across many candidates:
//  - compute in the all-SM state up to kernel p1, then the first comm phase (state
//    s1 + 1 for tc1 seconds), depend on (p1, s1) only;
//  - if compute has not reached kernel p2 when the first comm kernel ends, it runs in
//    the all-SM state up to p2 and the second comm phase starts there with kernel p2
//    untouched: that phase and the all-SM rest after it depend on (p2, s2) only, and
//    are tabled in LDS once per slab;
//  - otherwise the second comm kernel starts as soon as the first ends and continues
//    the first phase's progress: that phase depends on (p1, s1, s2), and each lane
//    forms it once per p1.
// Most candidates need no evaluation at all:
//  - every second launch position that compute has passed by the time the first comm kernel
//    ends (p2 <= j1) gives the same walk, so of those only p2 = p1, the first in candidate
//    order, can be kept;
//  - a later one (p2 > j1) adds its own part, which depends on (p2, s2) only: X = A0[p2] +
//    tc2 + rest to the time and Z = static power * X + its energies to the energy.  A pair
//    q = (p2, s2) whose X and Z both exceed those of another pair with the same or a later
//    position is worse in every candidate that could hold it (the other one is available
//    there too), and is dropped for the slab.  X and Z must differ by more than the roundings
//    of a candidate's sums can undo (KR_PAIR_MARGIN), so what is dropped is strictly worse
//    in the rounded results as well, and the frontier is the same, point for point.
// Of the two-comm workload's 264 pairs per slab 9 are left on average, and a launch position
// and SM choice take 8 + 9 evaluations instead of 264 to 8 (kernel 931 us with all of them,
// 370 us without).
// Of what is evaluated, most is beaten in time and energy by the wave's best candidate of the
// slab so far (least E + mean power T); the rest gathers in the wave's scratch, 64 candidates to
// a frontier, instead of taking a frontier per launch position (with the end of the first comm
// phase tabled and a slab's frontiers merged one point per lane: 373 -> 268 us, up to 287 on
// other boxes).  What is left is latency: of those 268 us the sums, the table and the pruning take about 65, the
// positions' phases about 100.
// A phase is kept as the values it adds to the energy sum and to the time, in the
// order the walk adds them.  A candidate applies them to its own sums in that order,
// so every candidate gets the roundings of the plain walk, operation for operation.
// A step the walk skips is stored as +0: the energy and time sums are never -0 (they
// start from +0 or a positive value and only non-negative terms are added), so adding
// +0 leaves them unchanged.
#include "kr_filter.h"
#include "kr_launch.h"
#include "kr_wave.h"

namespace kr {

// What a second comm phase and the all-SM rest after it add: energy terms ea (the
// kernel that was in progress), eb (whole kernels), ec (the kernel the phase ends in),
// a4 (the rest finishing that kernel), b4 (the rest's whole kernels), and the rest's
// time el4.  All +0 where the walk adds nothing (ea of a phase starting at a kernel
// boundary; a4, b4, el4 when compute finishes before the comm kernel does).
struct alignas(16) PairRec {
    double ea, eb, ec, a4, b4, el4;
};

// Largest j in [i0, N] with A[j][s] - base <= rb, where base = A[i0][s] and rb >= 0:
// galloping, then bisection.  The predicate is monotone in j (the running sums never
// decrease and rounding is monotone), so this is the j at which a left-to-right scan
// of whole kernels stops.
// hint: a guess at j, the search starts there if it is no overshoot (launch positions come
// in ascending order, so a phase ends at or after the kernel where the one before did).
__device__ __forceinline__ int pair_scan(const ColRec *AB, int S1, int s, int i0, int N,
                                         double base, double rb, int hint = 0)
{
    int lo = i0, step = 1;
    if (hint > i0 && AB[hint * S1 + s].a - base <= rb) lo = hint;
    while (lo + step <= N && AB[(lo + step) * S1 + s].a - base <= rb) {
        lo += step;
        step <<= 1;
    }
    int hi = min(N, lo + step - 1);
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (AB[mid * S1 + s].a - base <= rb) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Second comm phase in SM state s for tc seconds, from kernel i with unfinished
// fraction w (w = 1: kernel i not started), then the rest in the all-SM state; i < N.
// The lines are the walk's: finish the interrupted kernel if the budget allows (else
// spend the whole budget on it), whole kernels while they fit, the part of the next one
// the budget leaves; then the rest of the interrupted kernel and the remaining kernels.
__device__ __forceinline__ PairRec pair_phase(const double *Lt, const double *Lp,
                                              const ColRec *AB, int S1, int N, int s, int i,
                                              double w, double tc, int &hint)
{
    PairRec o{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    double used = 0.0;
    bool fin = false, spent = false;
    if (w < 1.0) {
        const double tk = Lt[i * S1 + s];
        const double need = w * tk;
        if (need <= tc) {
            o.ea = Lp[i * S1 + s] * need;
            used = need;
            i = i + 1;
            w = 1.0;
        } else {  // the budget ends inside the interrupted kernel
            o.ea = Lp[i * S1 + s] * tc;
            w = w - tc / tk;
            if (w < 0.0) w = 0.0;
            spent = true;
        }
    }
    if (!spent) {
        const double rb = tc - used;
        const ColRec zi = AB[i * S1 + s];
        const int j = pair_scan(AB, S1, s, i, N, zi.a, rb, hint);
        hint = j;
        const ColRec zj = AB[j * S1 + s];
        o.eb = zj.b - zi.b;
        if (j == N) {
            fin = true;
        } else {
            const double r = rb - (zj.a - zi.a);
            o.ec = Lp[j * S1 + s] * r;
            w = 1.0 - r / Lt[j * S1 + s];
            if (w < 0.0) w = 0.0;
            i = j;
        }
    }
    if (!fin) {  // the rest in the all-SM state (column 0)
        double u = 0.0;
        if (w < 1.0) {
            const double need = w * Lt[i * S1];
            o.a4 = Lp[i * S1] * need;
            u = need;
            i = i + 1;
        }
        const ColRec zN = AB[N * S1], zi = AB[i * S1];
        o.b4 = zN.b - zi.b;
        o.el4 = u + (zN.a - zi.a);
    }
    return o;
}

// Sorts n keys (T bits, E bits, index) ascending in LDS by one wave: a bitonic network
// whose comparators all put the smaller key at the lower index (the first stage of each
// merge compares mirrored positions); entries from n on act as +inf and never move.
__device__ inline void wave_sort_keys(uint64_t *sT, uint64_t *sE, int32_t *sI, int n)
{
    int m = 1, lm = 0;
    while (m < n) {
        m <<= 1;
        ++lm;
    }
    for (int lk = 1; lk <= lm; ++lk) {
        const int k = 1 << lk;
        for (int lj = lk - 1; lj >= 0; --lj) {
            const int j = 1 << lj;
            for (int q = threadIdx.x & 63; q < (m >> 1); q += 64) {
                int lo, hi;
                if (lj == lk - 1) {
                    const int blk = q >> lj, r = q & (j - 1);
                    lo = blk * k + r;
                    hi = blk * k + (k - 1 - r);
                } else {
                    lo = ((q >> lj) << (lj + 1)) + (q & (j - 1));
                    hi = lo + j;
                }
                if (hi < n) {
                    const uint64_t ta = sT[lo], ea = sE[lo], tb = sT[hi], eb = sE[hi];
                    const int32_t ia = sI[lo], ib = sI[hi];
                    if (key_less(tb, eb, ib, ta, ea, ia)) {
                        sT[lo] = tb;
                        sE[lo] = eb;
                        sI[lo] = ib;
                        sT[hi] = ta;
                        sE[hi] = ea;
                        sI[hi] = ia;
                    }
                }
            }
            wave_lds_fence();
        }
    }
}

// GetFrontier's strict prefix minimum over n keys sorted by (T, E, index), by one wave:
// writes the keys whose E is below every earlier E to o*[0 ..) in order and returns
// their count (uniform).  Lane l scans a contiguous block of the keys.
__device__ inline int wave_frontier_scan(const uint64_t *sT, const uint64_t *sE, const int32_t *sI,
                                         int n, double *oT, double *oE, int32_t *oI)
{
    const int lane = threadIdx.x & 63;
    const int per = (n + 63) / 64;
    const int q0 = min(n, lane * per), q1 = min(n, q0 + per);
    uint64_t m = KR_INF_BITS;
    for (int q = q0; q < q1; ++q) m = min(m, sE[q]);
    unsigned long long inc = m;  // least E of lanes 0 .. lane
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long y = __shfl_up(inc, d, 64);
        if (lane >= d) inc = min(inc, y);
    }
    unsigned long long best0 = __shfl_up(inc, 1, 64);  // least E of the lanes before
    if (lane == 0) best0 = KR_INF_BITS;
    uint64_t best = best0;
    int nk = 0;
    for (int q = q0; q < q1; ++q)
        if (sE[q] < best) {
            ++nk;
            best = sE[q];
        }
    int pos = nk;  // kept keys of lanes 0 .. lane
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(pos, d, 64);
        if (lane >= d) pos += y;
    }
    const int total = __builtin_amdgcn_readlane(pos, 63);
    pos -= nk;
    best = best0;
    for (int q = q0; q < q1; ++q) {
        const uint64_t e = sE[q];
        if (e < best) {
            oT[pos] = bitsd(sT[q]);
            oE[pos] = bitsd(e);
            oI[pos] = sI[q];
            ++pos;
            best = e;
        }
    }
    return total;
}

// The wave of a block of NW waves that takes launch position p1 (snake order).
__host__ __device__ __forceinline__ int pair_owner(int p1, int NW)
{
    const int r = p1 % (2 * NW);
    return r < NW ? r : 2 * NW - 1 - r;
}

// Copy n doubles from global memory into LDS by the block's NW waves, W bytes per lane
// and instruction (W = 16 needs n even and both addresses 16-byte aligned).
template <int W, int NW>
__device__ __forceinline__ void copy_to_lds_nw(const double *g, double *l, int n)
{
    const int units = n * 8 / W;
    const int lane = threadIdx.x & 63, w0 = threadIdx.x & ~63;
    for (int u0 = w0; u0 < units; u0 += 64 * NW) {
        const int u = u0 + lane;
        if (u < units) {
            const void *src = (const char *)g + (size_t)u * W;
            lds_void *dst = (lds_void *)((char *)l + (size_t)u0 * W);
            if constexpr (W == 16)
                __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
            else
                __builtin_amdgcn_global_load_lds(src, dst, 4, 0, 0);
        }
    }
}

// Roundings: a time is at most 5 operations on values up to Tm from its parts, X 2; an
// energy 9 and 5 of the time's (times static power) on values up to Em, Z 8 and 2.  With
// u = 2^-53 two candidates keep the order of their parts when those differ by 14 u Tm and
// 48 u Em; the margins are twice that and more.
#define KR_PAIR_MARGIN_T (32 * 0x1p-53)
#define KR_PAIR_MARGIN_E (128 * 0x1p-53)

// Pair (p2, s2)'s own part of the time and energy of the candidates that start it fresh.
struct alignas(16) PairPart {
    double x, z;
};

// Wave maximum of two non-NaN doubles (every lane active; uniform).
__device__ __forceinline__ void wave_max2_f64(double &x, double &y)
{
    x = -x;
    y = -y;
    wave_min2_f64(x, y);
    x = -x;
    y = -y;
}

// Block (p, b): NW waves sharing the slabs of partition p, frequencies [b*fb,
// min(F, (b+1)*fb)), one slab at a time.  LDS (in doubles): t slab [N][S1] at 0, pw slab
// at q_pw, running sums {A, B} [N + 1][S1] at q_ab (column 0 the all-SM state), the
// fresh second-phase table [n_pos][S] at q_f, the pairs' own parts [n_pos][S] at q_c, each
// wave's filter scratch at q_sc (the
// positions' champions before that), the list of the pairs kept at q_l, after the second
// comm kernel's times and energies [2][S].  Launch positions p1 go to the waves in
// snake order (0, 1, .., NW - 1, NW - 1, .., 0, 0, 1, .., see pair_owner); a wave is a unit of its own (slot
// and count), so waves never share output.
// Lane (s1, s2) evaluates, for each p1, the candidate that continues with s2, then every
// S-th of the kept pairs from the s2-th on.  Frontiers of up to 64 gathered candidates go to
// the wave's slot; if a slab wrote more than one, its points are read back at the end and
// replaced in place by their frontier: up to 64 one per lane, more by a sort in the
// second-phase tables, idle by then, when they fit there.  SC > 0 fixes the number of
// SM choices at compile time (four blocks share a compute unit then, by registers and LDS:
// 370 us against 444 us with three, before candidates were gathered); FN also fixes the
// two-comm workload's 48 kernels and 33 launch positions.
template <int R, int W, int NW, int SC, bool FN>
__global__ void __launch_bounds__(64 * NW, SC > 0 ? 4 : 3) eval_filter_pair_kernel(EvalArgs a, UnitOut o)
{
    extern __shared__ __attribute__((aligned(16))) double lds[];
    static_assert(!FN || SC > 0, "the fixed shape fixes the SM choices too");
    const int N = FN ? 48 : a.N, S = SC > 0 ? SC : a.S, S1 = S + 1, SS = S * S, slab = N * S1;
    const int np = FN ? 33 : a.n_pos;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double *const Lt = lds, *const Lp = lds + a.q_pw;
    ColRec *const AB = (ColRec *)(lds + a.q_ab);
    PairRec *const Fr = (PairRec *)(lds + a.q_f);
    double *const scw = lds + a.q_sc + 160 * wave;
    const Scratch sc{scw, scw + 64, (int32_t *)(scw + 128), 64};
    const int p = blockIdx.x / a.nfb, fbk = blockIdx.x - p * a.nfb;
    const int f0 = fbk * a.fb, f1 = min(a.F, f0 + a.fb);
    const bool live = lane < SS;
    const int s1 = live ? lane / S : 0, s2 = live ? lane - (lane / S) * S : 0;
    // rows of the fresh table this thread forms: SM choice sF, positions g, g + G, ...
    const int G = 64 * NW / S, g = tid / S, sF = tid - g * S;
    const int64_t unit = (int64_t)blockIdx.x * NW + wave;
    const size_t slot0 = (size_t)p * a.useg + (size_t)(unit - (int64_t)p * a.uper) * a.ustride;
    double *const oT = o.T + slot0, *const oE = o.E + slot0;
    int32_t *const oI = o.I + slot0;
    int count = 0;
    uint32_t worst = 0;  // largest high word read (input check)
    const double p_static = a.p_static;
    __shared__ int32_t s_kept;  // pairs kept
    PairPart *const part = (PairPart *)(lds + a.q_c);        // [np][S]
    int16_t *const champ = (int16_t *)(lds + a.q_sc);        // [np][2]
    double *const ltc = lds + a.q_l, *const lct = ltc + S;   // [S] each
    int16_t *const list = (int16_t *)(lds + a.q_l + 2 * S);  // [np * S]
    const int npS = np * S;
    int16_t *const first = list + npS;  // [np * S]: where the first comm phase ends
    // sort room of the slab-end reduction: this wave's share of the fresh table and the pairs'
    // own parts
    const int scap = a.pair_scap;
    uint64_t *const sT = (uint64_t *)(lds + a.q_f) + (size_t)wave * ((a.q_sc - a.q_f) / NW);
    uint64_t *const sE = sT + scap;
    int32_t *const sI = (int32_t *)(sE + scap);

    for (int f = f0; f < f1; ++f) {
        const size_t pf = (size_t)p * a.F + f;
        const int cs = count;  // first output of this slab
        // every LDS read of the previous slab has returned (all waves: the barrier
        // after the reduction, or none yet)
        copy_to_lds_nw<W, NW>(a.t + pf * slab, Lt, slab);
        copy_to_lds_nw<W, NW>(a.pw + pf * slab, Lp, slab);
        const double *const cm = a.tc + pf * 2 * S, *const cpw = a.pc + pf * 2 * S;
        const double tc1 = cm[s1], tc2 = cm[S + s2], tcF = cm[S + sF], tcF1 = cm[sF];
        const double pc1 = cpw[s1], pc2 = cpw[S + s2];
        const double ct1 = pc1 * tc1, ct2 = pc2 * tc2;
        worst = max(worst, max(max(value_hi(tc1), value_hi(tc2)), max(value_hi(pc1), value_hi(pc2))));
        __builtin_amdgcn_s_waitcnt(KR_WAIT_VM0);  // this wave's part of slab f is in LDS
        __syncthreads();                          // and the other waves' parts

        // Running sums, thread c < S1 forming column c left to right (8 rows of loads
        // ahead of the additions).
        if (tid < S1) {
            double sa = 0.0, sb = 0.0;
            const uint32_t seen = worst;  // of what came before this column
            AB[tid] = ColRec{0.0, 0.0};
            for (int i0 = 0; i0 < N; i0 += 8) {
                double vt[8], vw[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int i = min(i0 + q, N - 1);
                    vt[q] = Lt[i * S1 + tid];
                    vw[q] = Lp[i * S1 + tid];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (i0 + q < N) {
                        worst = max(worst, max(raw_hi(vt[q]), raw_hi(vw[q])));
                        sa = sa + vt[q];
                        sb = sb + vw[q] * vt[q];
                        AB[(i0 + q + 1) * S1 + tid] = ColRec{sa, sb};
                    }
            }
            // raw words also stop at -0.0: such a column is looked at again
            if (worst >= KR_BAD_HI) {
                worst = seen;
                for (int i = 0; i < N; ++i)
                    worst = max(worst, max(value_hi(Lt[i * S1 + tid]), value_hi(Lp[i * S1 + tid])));
            }
        }
        __syncthreads();
        // Second comm phases that start fresh at kernel q.  Row q = N (a comm kernel
        // launched after the last compute kernel) adds nothing: all +0.
        if (g < G) {
            const double ctF = cpw[S + sF] * tcF;
            if (g == 0) {
                ltc[sF] = tcF;
                lct[sF] = ctF;
            }
            int hint = 0, hint1 = 0;
            for (int q = g; q < np; q += G) {
                const PairRec o = q < N ? pair_phase(Lt, Lp, AB, S1, N, sF + 1, q, 1.0, tcF, hint)
                                        : PairRec{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                if (q < N)
                    hint1 = pair_scan(AB, S1, sF + 1, q, N, AB[q * S1 + sF + 1].a, tcF1, hint1);
                first[q * S + sF] = (int16_t)(q < N ? hint1 : N);
                const ColRec z = AB[q * S1];
                const double x = (z.a + tcF) + o.el4;
                Fr[q * S + sF] = o;
                part[q * S + sF] = PairPart{
                    x, (p_static * x + ((((z.b + o.eb) + o.ec) + o.a4) + o.b4)) + ctF};
            }
        }
        // bounds of the slab's times and energies, for the margins (any wave's lanes cover
        // every SM choice and state)
        double mt1 = tc1, mt2 = tc2, mc = ct1 + ct2;
        double mb = lane < S1 ? AB[N * S1 + lane].b : 0.0;
        wave_max2_f64(mt1, mt2);
        wave_max2_f64(mc, mb);
        const ColRec zall = AB[N * S1];
        const double Tm = 2.0 * zall.a + (mt1 + mt2), Em = p_static * Tm + (10.0 * mb + mc);
        const double dT = KR_PAIR_MARGIN_T * Tm, dE = KR_PAIR_MARGIN_E * Em;
        if (tid == 0) s_kept = 0;
        __syncthreads();
        // Champions: per position the pair at it or later with the least Z + c X, for two
        // weights c around the slab's mean power (a time-leaning and an energy-leaning one).
        // Testing every pair against these two keeps 9 of 264, against all of them 7.  A
        // lane starts from its position's own first pair: where the sums overflow that one
        // stays, and any pair at or after a position may stand there.
        const double mean = zall.a > 0.0 ? p_static + zall.b / zall.a : p_static;
        const double c0 = 0.25 * mean, c1 = 4.0 * mean;
        if (wave == 0) {
            double l0 = INFINITY, l1 = INFINITY;  // least of the later positions (uniform)
            int a0 = 0, a1 = 0;
            for (int base = (np - 1) / 64 * 64; base >= 0; base -= 64) {
                double g0 = INFINITY, g1 = INFINITY;
                const int own = min(base + lane, np - 1) * S;
                int i0 = own, i1 = own;
                if (base + lane < np)
                    for (int c = 0; c < S; ++c) {
                        const int q = own + c;
                        const PairPart y = part[q];
                        const double v0 = y.z + c0 * y.x, v1 = y.z + c1 * y.x;
                        i0 = v0 < g0 ? q : i0;
                        g0 = v0 < g0 ? v0 : g0;
                        i1 = v1 < g1 ? q : i1;
                        g1 = v1 < g1 ? v1 : g1;
                    }
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {  // least of lanes lane ..
                    const double y0 = __shfl_down(g0, d, 64), y1 = __shfl_down(g1, d, 64);
                    const int j0 = __shfl_down(i0, d, 64), j1 = __shfl_down(i1, d, 64);
                    if (lane + d < 64 && y0 < g0) {
                        g0 = y0;
                        i0 = j0;
                    }
                    if (lane + d < 64 && y1 < g1) {
                        g1 = y1;
                        i1 = j1;
                    }
                }
                if (l0 < g0) {
                    g0 = l0;
                    i0 = a0;
                }
                if (l1 < g1) {
                    g1 = l1;
                    i1 = a1;
                }
                if (base + lane < np) {
                    champ[2 * (base + lane)] = (int16_t)i0;
                    champ[2 * (base + lane) + 1] = (int16_t)i1;
                }
                l0 = bitsd(lane_u64(dbits(g0), 0));
                l1 = bitsd(lane_u64(dbits(g1), 0));
                a0 = lane_i32(i0, 0);
                a1 = lane_i32(i1, 0);
            }
        }
        __syncthreads();
        for (int q0 = 64 * wave; q0 < npS; q0 += 64 * NW) {
            const int q = q0 + lane;
            bool keep = q < npS;
            if (keep) {
                const PairPart y = part[q];
                const int p2 = q / S;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const PairPart b = part[champ[2 * p2 + h]];
                    if (b.x + dT < y.x && b.z + dE < y.z) keep = false;
                }
            }
            const uint64_t m = __ballot(keep);
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_kept, __popcll(m));
            at = lane_i32(at, 0) + lane_rank(m);
            if (keep) list[at] = (int16_t)q;
        }
        __syncthreads();
        const int nk = s_kept;

        // What the candidates of launch position p1 and this lane's SM choices share.
        struct First {
            int j1;             // the first comm phase ends in kernel j1
            double Ec1, tau1;   // energy and time at its end
            double Eca, used2;  // and with the interrupted kernel finished, and its time
            ColRec zi2;         // running sums from there on, in the all-SM state
            PairRec rec;        // the second phase that continues at once
        };
        int hint2 = 0;
        auto first_phase = [&](int p1) {
            First o;
            const int sa1 = s1 + 1;
            const ColRec z0 = AB[p1 * S1], zp = AB[p1 * S1 + sa1];
            const int j1 = first[p1 * S + s1];
            const ColRec zj = AB[j1 * S1 + sa1];
            o.j1 = j1;
            o.Ec1 = z0.b + (zj.b - zp.b);
            o.tau1 = z0.a + tc1;
            double w1 = 1.0;
            if (j1 < N) {
                const double r1 = tc1 - (zj.a - zp.a);
                o.Ec1 = o.Ec1 + Lp[j1 * S1 + sa1] * r1;
                w1 = 1.0 - r1 / Lt[j1 * S1 + sa1];
                if (w1 < 0.0) w1 = 0.0;
            }
            // compute on to p2 in the all-SM state (candidates with j1 < p2)
            o.Eca = o.Ec1;
            o.used2 = 0.0;
            int i2 = j1;
            if (j1 < N && w1 < 1.0) {
                const double need = w1 * Lt[j1 * S1];
                o.Eca = o.Ec1 + Lp[j1 * S1] * need;
                o.used2 = need;
                i2 = j1 + 1;
            }
            o.zi2 = AB[i2 * S1];
            // the second comm phase continuing the first one's progress (p2 <= j1)
            o.rec = j1 < N ? pair_phase(Lt, Lp, AB, S1, N, s2 + 1, j1, w1, tc2, hint2)
                           : PairRec{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            return o;
        };
        // time and energy from a second phase: st2 its start, Ec the energy before it
        auto finish = [&](const PairRec &q, double st2, double Ec, double tcs, double cts,
                          double &T, double &E) {
            Ec = Ec + q.ea;
            Ec = Ec + q.eb;
            Ec = Ec + q.ec;
            Ec = Ec + q.a4;
            Ec = Ec + q.b4;
            T = (st2 + tcs) + q.el4;
            E = p_static * T;
            E = E + Ec;
            E = E + ct1;
            E = E + cts;
        };
        // The wave's best candidate of the slab so far, by E + mean T: what it beats in both
        // time and energy is on no frontier.  (Two of them, with the weights above: 361 us
        // against 333, for the registers and the second search.)
        double best = INFINITY, bestT = INFINITY, bestE = INFINITY;
        int nb = 0;     // candidates in the wave's scratch
        int parts = 0;  // frontiers written
        auto flush = [&]() {  // writes the scratch's frontier (nb > 0)
            wave_lds_fence();
            const int x = min(lane, nb - 1);
            const double xT = sc.T[x], xE = sc.E[x];
            const int32_t xI = sc.I[x];
            const double fT[1] = {lane < nb ? xT : INFINITY}, fE[1] = {lane < nb ? xE : INFINITY};
            wave_lds_fence();
            count += wave_frontier<1>(fT, fE, fT[0], fE[0], any_index([&](int) { return xI; }), sc,
                                      oT + count, oE + count, oI + count);
            nb = 0;
            ++parts;
        };
        // A chunk of R slots per position: the continuing candidate first, then rounds of kept
        // pairs.  Few slots, as few candidates are left to filter: R = 4 281 us, 3 281, 2 268, for
        // the registers that more take.
        for (int p1 = 0; p1 < np; ++p1) {
            if (pair_owner(p1, NW) != wave) continue;
            const First o = first_phase(p1);
            // pair rank of (p1, p2): ppb + p2
            const int ppb = p1 * np - p1 * (p1 - 1) / 2 - p1;
            const int i1 = f * a.Cf + s1 * S;
            for (int e0 = -S; e0 < nk; e0 += R * S) {
                double vT[R], vE[R];
                int32_t vI[R];
                double tl = INFINITY, el = INFINITY;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = e0 + r * S;  // this round's first list entry
                    vT[r] = INFINITY;
                    vE[r] = INFINITY;
                    vI[r] = 0;
                    if (e >= nk) continue;  // uniform
                    if (r == 0 && e < 0) {
                        finish(o.rec, o.tau1, o.Ec1, tc2, ct2, vT[r], vE[r]);
                        vI[r] = i1 + (ppb + p1) * SS + s2;
                        vT[r] = live ? vT[r] : INFINITY;
                        vE[r] = live ? vE[r] : INFINITY;
                    } else {
                        const bool in = live && e + s2 < nk;
                        const int q = in ? list[e + s2] : 0;
                        const int p2 = q / S, c = q - p2 * S;
                        const ColRec z2 = AB[p2 * S1];
                        const bool valid = in && o.j1 < p2;  // compute has not reached p2
                        double T, E;
                        finish(Fr[q], o.tau1 + (o.used2 + (z2.a - o.zi2.a)),
                               o.Eca + (z2.b - o.zi2.b), ltc[c], lct[c], T, E);
                        vI[r] = i1 + (ppb + p2) * SS + c;
                        vT[r] = valid ? T : INFINITY;
                        vE[r] = valid ? E : INFINITY;
                    }
                    const bool beaten = bestT < vT[r] && bestE < vE[r];
                    vT[r] = beaten ? INFINITY : vT[r];
                    vE[r] = beaten ? INFINITY : vE[r];
                    tl = vmin(tl, vT[r]);
                    el = vmin(el, vE[r]);
                }
                if (!__any(tl < INFINITY)) continue;
                double g = INFINITY, hT = 0.0, hE = 0.0;  // this lane's least E + mean T
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const double v = vE[r] + mean * vT[r];
                    hT = v < g ? vT[r] : hT;
                    hE = v < g ? vE[r] : hE;
                    g = v < g ? v : g;
                }
                double m0 = g, m1 = INFINITY;
                wave_min2_f64(m0, m1);
                if (m0 < best) {
                    const int L = __ffsll((long long)__ballot(g == m0)) - 1;
                    best = m0;
                    bestT = bitsd(lane_u64(dbits(hT), L));
                    bestE = bitsd(lane_u64(dbits(hE), L));
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const bool beaten = bestT < vT[r] && bestE < vE[r];
                        vT[r] = beaten ? INFINITY : vT[r];
                        vE[r] = beaten ? INFINITY : vE[r];
                    }
                }
                uint64_t ms[R];
                int tot = 0;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    ms[r] = __ballot(vT[r] < INFINITY);
                    tot += __popcll(ms[r]);
                }
                if (nb + tot > 64 && nb > 0) flush();
                if (tot > 64) {  // more than the scratch holds
                    tl = el = INFINITY;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        tl = vmin(tl, vT[r]);
                        el = vmin(el, vE[r]);
                    }
                    count += wave_frontier<R>(vT, vE, tl, el,
                                              any_index([&](int r) { return vI[r]; }), sc,
                                              oT + count, oE + count, oI + count);
                    ++parts;
                    continue;
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (ms[r]) {
                        if (vT[r] < INFINITY) {
                            const int q = nb + lane_rank(ms[r]);
                            sc.T[q] = vT[r];
                            sc.E[q] = vE[r];
                            sc.I[q] = vI[r];
                        }
                        nb += __popcll(ms[r]);
                    }
            }
        }
        if (nb > 0) flush();
        __syncthreads();  // every wave is done with the slab's tables
        const int ns = count - cs;
        if (parts > 1 && ns > 1 && ns <= scap) {
            // this wave's own stores, complete after the wait: plain loads see them
            __builtin_amdgcn_s_waitcnt(KR_WAIT_VM0);
            if (ns <= 64) {  // one point per lane
                const int x = cs + min(lane, ns - 1);
                const double xT = oT[x], xE = oE[x];
                const int32_t xI = oI[x];
                const double v1T[1] = {lane < ns ? xT : INFINITY}, v1E[1] = {lane < ns ? xE : INFINITY};
                count = cs + wave_frontier<1>(v1T, v1E, v1T[0], v1E[0],
                                              any_index([&](int) { return xI; }), sc, oT + cs,
                                              oE + cs, oI + cs);
            } else {
                for (int x = lane; x < ns; x += 64) {
                    sT[x] = dbits(oT[cs + x]);
                    sE[x] = dbits(oE[cs + x]);
                    sI[x] = oI[cs + x];
                }
                wave_lds_fence();
                wave_sort_keys(sT, sE, sI, ns);
                count = cs + wave_frontier_scan(sT, sE, sI, ns, oT + cs, oE + cs, oI + cs);
            }
        }
        __syncthreads();  // the sort room is free again, and Lt, Lp may be overwritten
    }
    if (a.status) report_values(a.status, worst >= KR_BAD_HI);
    if (lane == 0) o.cnt[unit] = count;
}

int pair_owner_host(int p1, int NW) { return pair_owner(p1, NW); }

// Instances: 8 SM choices at compile time (30 kernels, 31 positions: 84 us, general 106), and the
// two-comm workload's sizes (287 us, 303 with the SM choices alone, 391 general).
hipError_t launch_eval_filter_pair(const EvalArgs &a, const UnitOut &o, hipStream_t st)
{
    const size_t lds = (size_t)a.lds_doubles * sizeof(double);
    constexpr int NW = KR_PAIR_WAVES;
    const dim3 grid(a.P * a.nfb), block(64 * NW);
    if (a.dma16 && a.S == 8 && a.N == 48 && a.n_pos == 33)
        hipLaunchKernelGGL((eval_filter_pair_kernel<2, 16, NW, 8, true>), grid, block, lds, st, a, o);
    else if (a.dma16 && a.S == 8)
        hipLaunchKernelGGL((eval_filter_pair_kernel<2, 16, NW, 8, false>), grid, block, lds, st, a, o);
    else if (a.dma16)
        hipLaunchKernelGGL((eval_filter_pair_kernel<2, 16, NW, 0, false>), grid, block, lds, st, a, o);
    else
        hipLaunchKernelGGL((eval_filter_pair_kernel<2, 4, NW, 0, false>), grid, block, lds, st, a, o);
    return hipGetLastError();
}

}  // namespace kr
