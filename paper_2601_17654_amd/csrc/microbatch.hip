// Microbatch frontier (Section 4.4, Algorithm 2 with one GPU frequency per microbatch and
// one shared configuration per partition type).  One block per frequency composes its
// scaled type frontiers with the frontier composition's rules, walks every
// non-dominated bin back to its configuration and sums it exactly in execution order;
// the union over frequencies then goes to GetFrontier.  All frequencies take one launch.
#include "kr_launch.h"
#include "kr_device.h"

namespace kr {

#define KR_MB_WIN 4096   // offsets binned on chip per pass, bins of a composition kept there
#define KR_MB_NT 1024    // threads of a frequency's block
#define KR_MB_LIST 1024  // occupied offsets of a type kept on chip

struct MbMinF64 {
    __device__ __forceinline__ double operator()(double a, double b) const { return b < a ? b : a; }
};
struct MbMaxF64 {
    __device__ __forceinline__ double operator()(double a, double b) const { return b > a ? b : a; }
};

// Offset of a scaled time on frequency f's grid: floor((t - tmin) / delta), clamped to
// [0, M] (the composition's binning rule).
__device__ __forceinline__ int64_t mb_offset(double t, double tmin, double delta, int64_t M)
{
    const double x = floor((t - tmin) / delta);
    return !(x > 0.0) ? 0 : (x < (double)M ? (int64_t)x : M);
}

// Sums of one configuration per thread: partitions in execution order, then the components.
// val[u * stride], val[(Ku + u) * stride]: time and energy chosen for used type u (LDS).
__device__ __forceinline__ void mb_sum(const MbArgs &a, const uint8_t *seq, const double *val,
                                       int stride, int f, double *T, double *E)
{
    double Tm = 0.0, Em = 0.0;
    const int ne = a.Ku * stride;
#pragma unroll 8
    for (int i = 0; i < a.n_seq; ++i) {
        const double *const v = val + seq[i] * stride;
        Tm = Tm + v[0];
        Em = Em + v[ne];
    }
    for (int k = 0; k < a.n_comp; ++k) {
        Tm = Tm + a.comp_T[(int64_t)k * a.F + f];
        Em = Em + a.comp_E[(int64_t)k * a.F + f];
    }
    *T = Tm;
    *E = Em;
}

// One block per frequency f: the frequency's whole composition and walk, with the rules of
// kr_compose_frontiers applied to the used types' points scaled by their repeat counts
// (type order): the time range of each type, the bin width (ranges summed in type order
// on one thread, then nudged up one ulp at a time until the bins fit), each type's least
// energy per offset (ties: smallest point index) and its occupied offsets, the min-plus
// steps (ties: smallest offset), the bins strictly below every earlier bin, and for each
// of those the walk back to its configuration, summed exactly in execution order and then
// over the components.  The q-th configuration goes to slot f * B + q of `buf` (with the slot
// as its index), their number to ucnt[f]: the units of one segment, whose layout block 0
// writes.  A frequency whose composition fails (an empty type, a non-finite or negative
// value, or bins that do not fit) has none.
// Latency-bound: a chain of short passes over a few points and up to B bins on a chip with
// one busy block per frequency.  The composition stays in LDS while B <= KR_MB_WIN, and the
// sums read the chosen values from LDS; with 256 threads, the bins in memory and three
// dependent loads per summed partition the kernel took 97 us for 64 frequencies of 4 types,
// 4,096 bins and 64 partitions, 43 us now.
__global__ void __launch_bounds__(KR_MB_NT) mb_grid_kernel(MbArgs a, MbGridWs w)
{
    constexpr int NT = KR_MB_NT, NW = NT / 64;
    __shared__ double s_tmin[KR_MB_MAX_TYPES], s_range[KR_MB_MAX_TYPES], s_delta;
    __shared__ int64_t s_M[KR_MB_MAX_TYPES], s_L[KR_MB_MAX_TYPES], s_lo[KR_MB_MAX_TYPES];
    __shared__ int32_t s_n[KR_MB_MAX_TYPES];
    __shared__ int32_t s_status;
    __shared__ double scd[NW], s_red[2][KR_MB_MAX_TYPES][NW];
    __shared__ int32_t sci[NW];
    __shared__ uint64_t s_eb[KR_MB_WIN];
    __shared__ int32_t s_ea[KR_MB_WIN];
    __shared__ double s_F[2][KR_MB_WIN], s_oe[KR_MB_LIST];
    __shared__ int32_t s_ob[KR_MB_LIST], s_oa[KR_MB_LIST];
    __shared__ uint8_t s_seq[KR_MB_MAX_SEQ];
    const int f = blockIdx.x, tid = threadIdx.x, B = a.B, Ku = a.Ku;
    const int wave = tid >> 6;
    const size_t wb = (size_t)f * B;
    int32_t *const ob2 = w.ob2 + wb, *const oarg = w.oarg + wb;
    double *const oe = w.oe + wb;
    const bool onchip = B <= KR_MB_WIN;
    double *const F0 = onchip ? s_F[0] : w.F + (size_t)f * 2 * B;
    double *const F1 = onchip ? s_F[1] : w.F + (size_t)f * 2 * B + B;
    int32_t *const bp = w.bp + (size_t)f * a.K * B;
    int32_t *const stair = w.stair + (size_t)f * B;
    if (f == 0 && tid == 0) {
        w.seg_off[0] = 0;
        w.seg_off[1] = (int64_t)a.F * B;
        w.unit_base[0] = 0;
        w.unit_base[1] = a.F;
    }
    if (tid == 0) s_status = KR_OK;
    for (int i = tid; i < a.n_seq; i += NT) s_seq[i] = a.seq_u[i];
    if (tid < Ku) {
        const int64_t *const o = a.seg_off + a.used[tid] * a.F + f;
        s_lo[tid] = o[0];
        s_n[tid] = (int32_t)min(o[1] - o[0], (int64_t)0x7FFFFFFF);
    }
    __syncthreads();

    // time range of each type's scaled points; their times and energies are checked
    for (int u = 0; u < Ku; ++u) {
        const int64_t lo = s_lo[u];
        const int n = s_n[u];
        const double m = (double)a.count[u];
        double mn = INFINITY, mx = -INFINITY;
        bool bad = false;
        for (int j = tid; j < n; j += NT) {
            const double ts = m * a.T[lo + j], es = m * a.E[lo + j];
            mn = ts < mn ? ts : mn;
            mx = ts > mx ? ts : mx;
            bad = bad || !(dbits(fabs(ts)) < KR_INF_BITS) || !(dbits(es + 0.0) < KR_INF_BITS);
        }
        if (__ballot(bad) && (tid & 63) == 0) s_status = KR_ENONFINITE;
        if (wave * 64 < n) {  // wave-uniform: a wave with points
            for (int d = 32; d > 0; d >>= 1) {
                mn = MbMinF64()(mn, __shfl_xor(mn, d, 64));
                mx = MbMaxF64()(mx, __shfl_xor(mx, d, 64));
            }
        }
        if ((tid & 63) == 0) {
            s_red[0][u][wave] = mn;
            s_red[1][u][wave] = mx;
        }
    }
    __syncthreads();
    if (tid < Ku) {
        double mn = INFINITY, mx = -INFINITY;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            mn = MbMinF64()(mn, s_red[0][tid][q]);
            mx = MbMaxF64()(mx, s_red[1][tid][q]);
        }
        s_tmin[tid] = mn;
        s_range[tid] = mx - mn;
        if (s_n[tid] <= 0) s_status = KR_EINVAL;
    }
    __syncthreads();
    // bin width and the types' offset ranges M and reachable bins L
    if (tid == 0 && s_status == KR_OK) {
        double R = 0.0;
        for (int u = 0; u < Ku; ++u) R = R + s_range[u];
        double delta = R > 0.0 ? R / (double)(B - 1) : 1.0;
        for (int iter = 0;; ++iter) {
            int64_t tot = 0;
            for (int u = 0; u < Ku; ++u) {
                const double x = floor(s_range[u] / delta);
                const int64_t mm = x < (double)B ? (int64_t)x : (int64_t)B;
                s_M[u] = mm;
                tot += mm;
            }
            if (tot + 1 <= B) break;
            if (iter > 4096) {
                s_status = KR_ECAPACITY;
                break;
            }
            delta = __longlong_as_double(__double_as_longlong(delta) + 1);  // next double up
        }
        int64_t L = 1;
        for (int u = 0; u < Ku; ++u) {
            L += s_M[u];
            s_L[u] = L;
        }
        s_delta = delta;
    }
    __syncthreads();
    if (s_status != KR_OK) {
        if (tid == 0) w.ucnt[f] = 0;
        return;
    }
    const double delta = s_delta;

    for (int u = 0; u < Ku; ++u) {
        const int64_t lo = s_lo[u];
        const int n = s_n[u];
        const double m = (double)a.count[u], tmin = s_tmin[u];
        const int64_t M = s_M[u];
        // least energy per offset, then the smallest point index that has it, on
        // chip for a window of KR_MB_WIN offsets at a time; the occupied offsets
        // go to the block's list in ascending order (its start also on chip)
        int32_t occ = 0;
        for (int64_t c0 = 0; c0 <= M; c0 += KR_MB_WIN) {
            const int cn = (int)min((int64_t)KR_MB_WIN, M + 1 - c0);
            for (int b = tid; b < cn; b += NT) {
                s_eb[b] = KR_INF_BITS;
                s_ea[b] = 0x7FFFFFFF;
            }
            __syncthreads();
            for (int j = tid; j < n; j += NT) {
                const int64_t o = mb_offset(m * a.T[lo + j], tmin, delta, M) - c0;
                if (o >= 0 && o < cn)
                    atomicMin((unsigned long long *)&s_eb[o],
                              (unsigned long long)dbits(m * a.E[lo + j] + 0.0));
            }
            __syncthreads();
            for (int j = tid; j < n; j += NT) {
                const int64_t o = mb_offset(m * a.T[lo + j], tmin, delta, M) - c0;
                if (o >= 0 && o < cn && dbits(m * a.E[lo + j] + 0.0) == s_eb[o])
                    atomicMin(&s_ea[o], j);
            }
            __syncthreads();
            for (int b0 = 0; b0 < cn; b0 += NT) {
                const int b = b0 + tid;
                const int32_t arg = b < cn ? s_ea[b] : 0x7FFFFFFF;
                const int has = arg != 0x7FFFFFFF;
                int32_t tot;
                const int32_t pos =
                    occ + block_exclusive<int32_t, SumI32, NW>(has, 0, SumI32(), sci, &tot);
                if (has) {
                    const double e = bitsd(s_eb[b]);
                    if (pos < KR_MB_LIST) {
                        s_ob[pos] = (int32_t)(c0 + b);
                        s_oe[pos] = e;
                        s_oa[pos] = arg;
                    } else {
                        ob2[pos] = (int32_t)(c0 + b);
                        oe[pos] = e;
                        oarg[pos] = arg;
                    }
                }
                occ += tot;
            }
            __syncthreads();
        }
        const int near = min(occ, KR_MB_LIST);
        // F_1 = e_1, then F_u[b] = min over occupied b2 of F_{u-1}[b - b2] + e_u[b2]
        double *const Fc = (u & 1) ? F1 : F0;
        const double *const Fp = (u & 1) ? F0 : F1;
        int32_t *const bpu = bp + (size_t)u * B;
        const int Lu = (int)s_L[u], Lp = u > 0 ? (int)s_L[u - 1] : 0;
        for (int b = tid; b < B; b += NT) {
            double best = INFINITY;
            int32_t who = -1;
            auto offer = [&](int o, double e, int32_t arg) {
                const int src = b - o;
                if (src >= 0 && src < Lp) {
                    const double v = Fp[src] + e;
                    if (v < best) {
                        best = v;
                        who = arg;
                    }
                }
            };
            if (u > 0 && b < Lu) {
                for (int x = 0; x < near; ++x) offer(s_ob[x], s_oe[x], s_oa[x]);
                for (int x = near; x < occ; ++x) offer(ob2[x], oe[x], oarg[x]);
            }
            Fc[b] = best;
            bpu[b] = who;
        }
        __syncthreads();
        if (u == 0) {  // F_1 = e_1: the occupied offsets of the first type
            for (int x = tid; x < occ; x += NT) {
                const int o = x < near ? s_ob[x] : ob2[x];
                Fc[o] = x < near ? s_oe[x] : oe[x];
                bpu[o] = x < near ? s_oa[x] : oarg[x];
            }
            __syncthreads();
        }
    }
    // bins strictly below every earlier bin of F_Ku
    const double *const Fl = ((Ku - 1) & 1) ? F1 : F0;
    double before = INFINITY;
    int32_t nst = 0;
    const int Ll = (int)min(s_L[Ku - 1], (int64_t)B);  // nothing is reachable from there on
    for (int b0 = 0; b0 < Ll; b0 += NT) {
        const int b = b0 + tid;
        const double v = b < Ll ? Fl[b] : INFINITY;
        double call;
        const double wpre = block_exclusive<double, MbMinF64, NW>(v, (double)INFINITY, MbMinF64(),
                                                                  scd, &call);
        const int keep = v < MbMinF64()(before, wpre);
        int32_t tot;
        const int32_t pos = block_exclusive<int32_t, SumI32, NW>(keep, 0, SumI32(), sci, &tot);
        if (keep) stair[nst + pos] = b;
        nst += tot;
        before = MbMinF64()(before, call);
    }
    __syncthreads();

    // Each staircase bin walked back to its configuration and summed exactly, as many at a
    // time as the chosen values fit where the offsets were binned.  (The walk of a reachable
    // bin ends at offset 0; one that does not would be left out by its infinite values.)
    double *const val = (double *)s_eb;
    const int step = min(NT, KR_MB_WIN / (2 * Ku));
    for (int q0 = 0; q0 < nst; q0 += step) {
        const int q = q0 + tid;
        if (tid < step && q < nst) {
            const int64_t slot = (int64_t)f * B + q;
            int32_t *const ch = a.slot_choice + slot * a.K;
            for (int t = 0; t < a.K; ++t) ch[t] = -1;
            bool ok = true;
            int64_t b = stair[q];
            for (int u = Ku - 1; u >= 0 && ok; --u) {
                const int32_t j = bp[(size_t)u * B + b];
                ok = j >= 0;
                if (ok) {
                    const double t = a.T[s_lo[u] + j];
                    ch[a.used[u]] = j;
                    val[u * step + tid] = t;
                    val[(Ku + u) * step + tid] = a.E[s_lo[u] + j];
                    b -= mb_offset((double)a.count[u] * t, s_tmin[u], delta, s_M[u]);
                    ok = b >= 0;
                }
            }
            ok = ok && b == 0;
            double Tm = INFINITY, Em = INFINITY;
            if (ok) mb_sum(a, s_seq, val + tid, step, f, &Tm, &Em);
            w.buf.T[slot] = Tm;
            w.buf.E[slot] = Em;
            w.buf.I[slot] = (int32_t)slot;
        }
    }
    if (tid == 0) w.ucnt[f] = nst;
}

// Frequency and choices of the frontier points (slot indices), and their number.
__global__ void __launch_bounds__(KR_BLOCK) mb_gather_kernel(MbArgs a, const int64_t *front_off,
                                                           const int32_t *front_idx, int64_t cap,
                                                           int32_t *out_f, int32_t *out_choice,
                                                           int64_t *n_out)
{
    const int64_t n = front_off[1];
    const int64_t r = (int64_t)blockIdx.x * KR_BLOCK + threadIdx.x;
    if (r == 0) *n_out = n;
    if (r >= n || r >= cap) return;
    const int64_t slot = front_idx[r];
    out_f[r] = (int32_t)(slot / a.B);
    for (int t = 0; t < a.K; ++t) out_choice[r * a.K + t] = a.slot_choice[slot * a.K + t];
}

hipError_t launch_mb_grid(const MbArgs &a, const MbGridWs &w, hipStream_t st)
{
    hipLaunchKernelGGL(mb_grid_kernel, dim3(a.F), dim3(KR_MB_NT), 0, st, a, w);
    return hipGetLastError();
}

hipError_t launch_mb_gather(const MbArgs &a, const int64_t *front_off, const int32_t *front_idx,
                            int64_t cap, int32_t *out_f, int32_t *out_choice, int64_t *n_out,
                            hipStream_t st)
{
    const int64_t n = (int64_t)a.F * a.B;
    const int64_t m = cap < n ? cap : n;
    const int64_t blocks = (m > 0 ? m : 1) + KR_BLOCK - 1;
    hipLaunchKernelGGL(mb_gather_kernel, dim3((unsigned)(blocks / KR_BLOCK)), dim3(KR_BLOCK), 0, st,
                       a, front_off, front_idx, cap, out_f, out_choice, n_out);
    return hipGetLastError();
}

// ---- enumeration of every configuration (Algorithm 2 as written) ----------------------

// Configurations per frequency (product of the used types' point counts) and their
// running totals: base[f] .. base[f+1]-1 are frequency f's slots, seg = the one segment of
// all slots.  One block; fails with KR_ECAPACITY past the slots reserved.
__global__ void __launch_bounds__(KR_BLOCK) mb_count_kernel(MbArgs a, int64_t *base, int64_t *seg,
                                                          int64_t slots, int32_t *status)
{
    __shared__ int64_t sc[KR_WAVES];
    int64_t carry = 0;
    for (int f0 = 0; f0 < a.F; f0 += KR_BLOCK) {
        const int f = f0 + threadIdx.x;
        int64_t n = f < a.F ? 1 : 0;
        if (f < a.F)
            for (int u = 0; u < a.Ku; ++u) {
                const int64_t *const o = a.seg_off + a.used[u] * a.F + f;
                n *= o[1] - o[0];
            }
        int64_t tot;
        const int64_t ex = block_exclusive(n, (int64_t)0, SumI64(), sc, &tot);
        if (f < a.F) base[f] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) {
        base[a.F] = carry;
        seg[0] = 0;
        seg[1] = slots;
        *status = carry <= slots ? KR_OK : KR_ECAPACITY;
    }
}

// Frequency of slot x, and for each used type u (last first: the first is slowest)
// take(u, point, its index within its segment).
template <typename Take>
__device__ __forceinline__ int mb_decode(const MbArgs &a, const int64_t *base, int64_t x,
                                         const Take &take)
{
    int lo = 0, hi = a.F - 1;  // last f with base[f] <= x
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (base[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    const int f = lo;
    int64_t c = x - base[f];  // below 2^31, like the slots
    for (int u = a.Ku - 1; u >= 0; --u) {
        const int64_t s0 = a.seg_off[a.used[u] * a.F + f];
        const uint32_t n = (uint32_t)(a.seg_off[a.used[u] * a.F + f + 1] - s0);
        const uint32_t j = (uint32_t)c % n;
        take(u, s0 + j, (int32_t)j);
        c = (uint32_t)c / n;
    }
    return f;
}

// Time and energy of every configuration: partitions in execution order, then the
// components.  Slots past the total hold +inf.  The chosen values wait in LDS ([2 Ku]
// [threads]), then the sequence, so that a summed partition costs two LDS reads instead of
// three dependent loads.
__global__ void __launch_bounds__(KR_BLOCK) mb_enum_kernel(MbArgs a, const int64_t *base,
                                                         int64_t slots, const int32_t *status)
{
    extern __shared__ double mb_val[];
    const int NT = blockDim.x, tid = threadIdx.x;
    double *const val = mb_val + tid;
    uint8_t *const seq = (uint8_t *)(mb_val + 2 * a.Ku * NT);
    for (int i = tid; i < a.n_seq; i += NT) seq[i] = a.seq_u[i];
    __syncthreads();
    const int64_t total = *status == KR_OK ? base[a.F] : 0;
    for (int64_t x = (int64_t)blockIdx.x * NT + tid; x < slots; x += (int64_t)gridDim.x * NT) {
        double Tm = INFINITY, Em = INFINITY;
        if (x < total) {
            const int f = mb_decode(a, base, x, [&](int u, int64_t p, int32_t) {
                val[u * NT] = a.T[p];
                val[(a.Ku + u) * NT] = a.E[p];
            });
            mb_sum(a, seq, val, NT, f, &Tm, &Em);
        }
        a.slot_T[x] = Tm;
        a.slot_E[x] = Em;
    }
}

// Frequency and choices of the frontier slots, their number and the verdict.
__global__ void __launch_bounds__(KR_BLOCK) mb_enum_gather_kernel(
    MbArgs a, const int64_t *base, const int32_t *status, const int64_t *front_off,
    const int32_t *front_idx, int64_t cap, int32_t *out_f, int32_t *out_choice, int64_t *n_out,
    int32_t *status_out)
{
    const int64_t n = *status == KR_OK ? front_off[1] : 0;
    const int64_t r = (int64_t)blockIdx.x * KR_BLOCK + threadIdx.x;
    if (r == 0) {
        *n_out = n;
        *status_out = *status;
    }
    if (r >= n || r >= cap) return;
    int32_t *const ch = out_choice + r * a.K;
    for (int t = 0; t < a.K; ++t) ch[t] = -1;
    out_f[r] = mb_decode(a, base, front_idx[r],
                         [&](int u, int64_t, int32_t j) { ch[a.used[u]] = j; });
}

hipError_t launch_mb_enum(const MbArgs &a, int64_t *base, int64_t *seg, int64_t slots,
                          int32_t *status, hipStream_t st)
{
    hipLaunchKernelGGL(mb_count_kernel, dim3(1), dim3(KR_BLOCK), 0, st, a, base, seg, slots, status);
    const int nt = a.Ku <= 8 ? KR_BLOCK : 64;  // at most 32 KB of chosen values
    const size_t lds = (size_t)2 * a.Ku * nt * sizeof(double) + (a.n_seq + 7) / 8 * 8;
    const int64_t blocks = (slots + nt - 1) / nt;
    const unsigned grid = (unsigned)(blocks < 4096 ? (blocks > 0 ? blocks : 1) : 4096);
    hipLaunchKernelGGL(mb_enum_kernel, dim3(grid), dim3(nt), lds, st, a, base, slots,
                       (const int32_t *)status);
    return hipGetLastError();
}

hipError_t launch_mb_enum_gather(const MbArgs &a, const int64_t *base, const int32_t *status,
                                 const int64_t *front_off, const int32_t *front_idx, int64_t cap,
                                 int32_t *out_f, int32_t *out_choice, int64_t *n_out,
                                 int32_t *status_out, int64_t slots, hipStream_t st)
{
    const int64_t m = cap < slots ? cap : slots;
    const int64_t blocks = ((m > 0 ? m : 1) + KR_BLOCK - 1) / KR_BLOCK;
    hipLaunchKernelGGL(mb_enum_gather_kernel, dim3((unsigned)blocks), dim3(KR_BLOCK), 0, st, a,
                       base, status, front_off, front_idx, cap, out_f, out_choice, n_out,
                       status_out);
    return hipGetLastError();
}

}  // namespace kr
