// Learned warm start: per-point features of S, training targets of a finished run, and the
// warm initial availabilities (Eq. 2.2-2.3 evaluated at rho = 0 with a predicted base).
//
// Features of point i (HAP_WARM_FEATURES = 32 floats; a = |p_i|, p the level-1 preference):
//   [0,16)  the 16 largest off-diagonal s_ij of row i, descending (ties: lower j first), / a;
//           rows with fewer than 16 off-diagonal entries repeat the smallest one
//   16      p_i / a
//   17      #{j != i : s_ij > p_i} / (n - 1)
//   18      mean of the off-diagonal s_ij, / a
//   19      log(1 + #{j != i : s_ij > p_i}) / 10
//   20 + m log(1 + D_m(i)) / 10, D_m(i) = sum_{j != i} max(0, s_ij - 2^-m p_i) / a, m = 0..5
//   26 + m (D_m(i) - M_m(i)) / max(D_m(i), M_m(i)) (0 when both are 0), M_m(i) the largest
//           D_m over the 16 neighbours of the first block (all other points when n - 1 < 16)
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

#include "hap_internal.h"

namespace hap {

namespace {

constexpr int kTop = 16;
constexpr int kScales = 6;

// One workgroup per row.  A first pass over the row takes the largest value of every four threads and the
// sums; the sixteenth largest of these 64 maxima is at most the row's sixteenth largest value, so the
// row's top 16 are among the values that reach it, which a second pass collects in LDS and ranks by
// counting.  Usually they are a few dozen; where the nearest columns fall into few of the 64 groups, or are
// equal by the hundred, they can be thousands, and the bound is raised from a sample of them.
// Up to 256 NV vectors the row stays in registers between the passes (NV = 0: it is read again).
// 8192 FP32 points, the whole call: 124 us with points in random order, 281 us in a cyclic one (runs of 16
// columns in 1024; sixteen more reads of every such row took 1334 us), 234 us with four places for all
// points; a sorted list of sixteen per lane takes 387, 308 and 345 us.  The kernel's 110 us (2.4 TB/s) are
// bound by vector issue, busy two thirds of the time with four waves per SIMD: 42 instructions per element, of
// which the FP64 sums are about 20 and the passes' comparisons and the row's tail the rest.
constexpr int kFeatThreads = 256;
constexpr int kFeatCap = 512;   // collected values; more of them: the bound is raised until they fit

template <typename T, int NV>
__global__ __launch_bounds__(kFeatThreads) void warm_features_kernel(const T *__restrict__ S, int64_t lds,
                                                                     const T *__restrict__ pref, int n,
                                                                     float *__restrict__ F, int64_t ldf,
                                                                     int32_t *__restrict__ nbr,
                                                                     double *__restrict__ Dout) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N, NT = kFeatThreads, NW = NT / 64, NG = NT / 4;
    __shared__ __attribute__((aligned(16))) T maxima[NG];
    __shared__ __attribute__((aligned(16))) T cv[kFeatCap];
    __shared__ __attribute__((aligned(16))) int cj[kFeatCap];
    __shared__ T top_v[kTop];
    __shared__ int top_j[kTop];
    __shared__ double part[NW][kScales + 1];
    __shared__ int pcnt[NW];
    __shared__ T bound;
    __shared__ int bound_j;
    __shared__ int collected;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int i = blockIdx.x;
    const T *row = S + (int64_t)i * lds;
    const T p = pref[i];
    const double pd = (double)p, a = fabs(pd);
    const T ninf = neg_inf<T>(), nan = (T)__builtin_nanf("");
    double thr[kScales], D[kScales], sum = 0.0;
#pragma unroll
    for (int m = 0; m < kScales; ++m) {
        thr[m] = pd * (1.0 / (double)(1 << m));
        D[m] = 0.0;
    }
    int cnt = 0;
    T mx = ninf;
    // the diagonal and the columns past n become NaN, which no comparison takes; only a wave whose vectors
    // hold one of them looks for it
    auto first = [&](V &v, int w0, int j0) {
        V vd0 = v;
        if ((unsigned)(i - w0) < (unsigned)(64 * VW) || w0 + 64 * VW > n) {
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                const bool out = j0 + e >= n || j0 + e == i;
                v[e] = out ? nan : v[e];
                vd0[e] = out ? T(0) : vd0[e];
            }
        }
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            mx = v[e] > mx ? v[e] : mx;
            cnt += v[e] > p ? 1 : 0;
            const double vd = (double)v[e];
            sum += (double)vd0[e];
#pragma unroll
            for (int m = 0; m < kScales; ++m) D[m] += fmax(0.0, vd - thr[m]);
        }
    };
    const int wave0 = __builtin_amdgcn_readfirstlane(wid) * 64 * VW;
    V keep[NV > 0 ? NV : 1];
    if constexpr (NV > 0) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int j0 = (c * NT + tid) * VW;
            keep[c] = j0 < n ? __builtin_nontemporal_load((const V *)(row + j0)) : (V)(ninf);
        }
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            const int w0 = c * NT * VW + wave0;
            if (w0 < n) first(keep[c], w0, (c * NT + tid) * VW);
        }
    } else {
#pragma unroll 4
        for (int w0 = wave0; w0 < n; w0 += NT * VW) {
            const int j0 = w0 + lane * VW;
            V v = j0 < n ? *(const V *)(row + j0) : (V)(ninf);
            first(v, w0, j0);
        }
    }
    // maxima of groups of four threads
#pragma unroll
    for (int off = 2; off >= 1; off >>= 1) {
        const T o = __shfl_xor(mx, off, 64);
        mx = o > mx ? o : mx;
    }
    if ((lane & 3) == 0) maxima[tid >> 2] = mx;
    // row totals (a fixed order: lanes by butterfly, then the waves)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        cnt += __shfl_xor(cnt, off, 64);
        sum += __shfl_xor(sum, off, 64);
#pragma unroll
        for (int m = 0; m < kScales; ++m) D[m] += __shfl_xor(D[m], off, 64);
    }
    if (lane == 0) {
        pcnt[wid] = cnt;
        part[wid][kScales] = sum;
#pragma unroll
        for (int m = 0; m < kScales; ++m) part[wid][m] = D[m];
    }
    if (tid == 0) collected = 0;
    __syncthreads();
    // the sixteenth largest of them
    if (wid == 0) {
        const T mine = maxima[lane];
        int rank = 0;
#pragma unroll
        for (int k = 0; k < NG; k += VW) {
            const V o = *(const V *)&maxima[k];
#pragma unroll
            for (int e = 0; e < VW; ++e) rank += (o[e] > mine || (o[e] == mine && k + e < lane)) ? 1 : 0;
        }
        if (rank == kTop - 1) bound = mine;
    }
    __syncthreads();
    T lo = bound;
    int lo_j = INT_MAX;   // of the values equal to lo, the columns up to this one
    // The list takes what reaches the bound: a wave counts its own and reserves their places at once.
    auto collect = [&](const V &v, int j0) {
        bool take[VW];
        unsigned long long who[VW], any = 0;
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            const int j = j0 + e;
            take[e] = (v[e] > lo) | ((v[e] == lo) & (j <= lo_j));
            if constexpr (NV == 0) take[e] = take[e] & (j < n) & (j != i);
            any |= who[e] = __ballot(take[e]);
        }
        if (any == 0) return;
        int total = 0, first_at = 0;
#pragma unroll
        for (int e = 0; e < VW; ++e) total += __popcll(who[e]);
        if (lane == 0) first_at = atomicAdd(&collected, total);
        first_at = __builtin_amdgcn_readfirstlane(first_at);
#pragma unroll
        for (int e = 0; e < VW; ++e) {
            if (take[e]) {
                const int at = first_at + __builtin_amdgcn_mbcnt_hi((unsigned)(who[e] >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((unsigned)who[e], 0));
                // past the end, a slot of 0 .. at: the list stays a sample of all that came
                const int slot = at < kFeatCap ? at : (int)__umulhi((unsigned)at * 2654435761u, (unsigned)at + 1u);
                if (slot < kFeatCap) {
                    cv[slot] = v[e];
                    cj[slot] = j0 + e;
                }
            }
            first_at += __popcll(who[e]);
        }
    };
    auto collect_row = [&]() {
        if constexpr (NV > 0) {
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                const int j0 = (c * NT + tid) * VW;
                if (c * NT * VW + wave0 < n) collect(keep[c], j0);
            }
        } else {
            for (int w0 = wave0; w0 < n; w0 += 4 * NT * VW) {
                V v[4];   // four loads in flight
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j0 = w0 + u * NT * VW + lane * VW;
                    v[u] = j0 < n ? *(const V *)(row + j0) : (V)(nan);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) collect(v[u], w0 + u * NT * VW + lane * VW);
            }
        }
        __syncthreads();
        return collected;
    };
    // entries among the list's first m that come before (v, j): values descending, equal values by column
    auto before = [&](T v, int j, int m) {
        typedef int I4 __attribute__((ext_vector_type(4)));
        int c = 0;
#pragma unroll 2
        for (int k = 0; k < m; k += 4) {
            T o[4];
#pragma unroll
            for (int e = 0; e < 4; e += VW) *(V *)&o[e] = *(const V *)&cv[k + e];
            const I4 oj = *(const I4 *)&cj[k];
#pragma unroll
            for (int e = 0; e < 4; ++e) c += (int)((k + e < m) & ((o[e] > v) | ((o[e] == v) & (oj[e] < j))));
        }
        return c;
    };
    int found = collect_row();
    // More than the list holds: the sixteenth best of 256 entries of the list is the next bound, which leaves
    // out the other 240 at least and about 15 of 16 as a rule.
    for (int left = n / (NT - kTop) + 1; found > kFeatCap && left > 0; --left) {
        const int sj = cj[tid];
        const T sv = row[sj];   // two entries may have been written to a slot: the column decides
        cv[tid] = sv;
        __syncthreads();
        if (before(sv, sj, NT) == kTop - 1) {
            bound = sv;
            bound_j = sj;
        }
        if (tid == 0) collected = 0;
        __syncthreads();
        lo = bound;
        lo_j = bound_j;
        found = collect_row();
    }
    found = found < kFeatCap ? found : kFeatCap;
    const int avail = n - 1 < kTop ? n - 1 : kTop;
    for (int c = tid; c < found; c += NT) {
        const T v = cv[c];
        const int j = cj[c];
        const int at = before(v, j, found);
        if (at < kTop) {
            top_v[at] = v;
            top_j[at] = j;
        }
    }
    __syncthreads();
    float *Fi = F + (int64_t)i * ldf;
    const int have = found < avail ? found : avail;   // fewer only where the row holds NaN
    if (tid < kTop) {
        const int r = tid < have ? tid : have - 1;    // a short row repeats its smallest entry
        const T v = have > 0 ? top_v[r] : ninf;
        Fi[tid] = (float)((double)v / a);
        nbr[(int64_t)i * kTop + tid] = have > 0 ? top_j[r] : i;
    }
    if (tid < kScales) {
        double d = part[0][tid];
#pragma unroll
        for (int w = 1; w < NW; ++w) d += part[w][tid];
        const double dm = d / a;
        Dout[(int64_t)i * kScales + tid] = dm;
        Fi[20 + tid] = (float)(log1p(dm) / 10.0);
    }
    if (tid == 64) {
        int c = pcnt[0];
        double s = part[0][kScales];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            c += pcnt[w];
            s += part[w][kScales];
        }
        Fi[16] = (float)(pd / a);
        Fi[17] = (float)((double)c / (double)(n - 1));
        Fi[18] = (float)((s / (double)(n - 1)) / a);
        Fi[19] = (float)(log1p((double)c) / 10.0);
    }
}

// Neighbourhood comparison of the soft counts: sixteen lanes per point, one neighbour each.
__global__ __launch_bounds__(256) void warm_local_kernel(int n, const int32_t *__restrict__ nbr,
                                                         const double *__restrict__ D, float *__restrict__ F,
                                                         int64_t ldf) {
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), r = threadIdx.x & 15;
    if (i >= n) return;   // whole groups of sixteen lanes leave
    const int cnt = n - 1 < kTop ? n - 1 : kTop;
    double M[kScales];
    const int j = r < cnt ? nbr[(int64_t)i * kTop + r] : i;
#pragma unroll
    for (int m = 0; m < kScales; ++m) M[m] = r < cnt ? fmax(0.0, D[(int64_t)j * kScales + m]) : 0.0;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
        for (int m = 0; m < kScales; ++m) M[m] = fmax(M[m], __shfl_xor(M[m], off, 16));
    if (r < kScales) {
        double top = M[0];
#pragma unroll
        for (int m = 1; m < kScales; ++m) top = r == m ? M[m] : top;
        const double d = D[(int64_t)i * kScales + r];
        const double big = fmax(d, top);
        F[(int64_t)i * ldf + 26 + r] = big > 0.0 ? (float)((d - top) / big) : 0.0f;
    }
}

// Targets g((alpha^t_jj + rho^t_jj) / |p_j|), g(v) = sign(v) |v| / (sqrt(1 + |v|) + 1), where
// alpha^t finishes the damped availability update of the last sweep (as its next row pass
// would) when t >= 1.
template <typename T>
__global__ __launch_bounds__(256) void warm_targets_kernel(const T *__restrict__ R, const T *__restrict__ A,
                                                           const T *__restrict__ B, const T *__restrict__ pref, int n,
                                                           int64_t ldw, T lam, T oml, int t, float *__restrict__ out,
                                                           int64_t ldo) {
#pragma clang fp contract(off)
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const T r = R[(int64_t)j * ldw + j];
    T al = A[(int64_t)j * ldw + j];
    if (t >= 1) al = lam * al + oml * (B[j] - r);
    const double v = ((double)al + (double)r) / fabs((double)pref[j]);
    const double av = fabs(v);
    const double g = av / (sqrt(1.0 + av) + 1.0);
    out[(int64_t)j * ldo] = (float)(v < 0.0 ? -g : g);
}

// Bases B_j = sign(y) |y| (|y| + 2) |p_j| of the network outputs of one level.
template <typename T>
__global__ __launch_bounds__(256) void warm_bases_kernel(const float *__restrict__ Y, int64_t ldy,
                                                         const T *__restrict__ pref, int n, T *__restrict__ bases) {
#pragma clang fp contract(off)
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n) return;
    const double y = (double)Y[(int64_t)j * ldy];
    const double ay = fabs(y);
    const double g = ay * (ay + 2.0);
    const double b = (y < 0.0 ? -g : g) * fabs((double)pref[j]);
    bases[j] = (T)b;
}

// alpha_ij = min(0, B_j) (i != j), alpha_jj = B_j with B_j = bases[j * stride]; padding
// columns -inf.
template <typename T>
__global__ __launch_bounds__(256) void warm_fill_kernel(T *__restrict__ A, int n, int64_t ldw,
                                                        const T *__restrict__ bases, int64_t stride) {
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N;
    const int64_t per_row = ldw / VW;
    const int64_t total = (int64_t)n * per_row;
    const T zero = T(0), ninf = neg_inf<T>();
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
        const int64_t i = e / per_row;
        const int j0 = (int)((e % per_row) * VW);
        V out;
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            const int j = j0 + v;
            T x = ninf;
            if (j < n) {
                const T b = bases[(int64_t)j * stride];
                x = (j == i) ? b : fmin(zero, b);
            }
            out[v] = x;
        }
        *(V *)(A + i * ldw + j0) = out;
    }
}

}  // namespace

size_t warm_feature_scratch_bytes(int64_t n) { return (size_t)n * (kTop * sizeof(int32_t) + kScales * sizeof(double)); }

template <typename T>
hipError_t launch_warm_features(const T *S, int64_t lds, const T *pref, int n, float *F, int64_t ldf, void *scratch,
                                hipStream_t st) {
    if (n < 2) return hipErrorInvalidValue;
    double *D = (double *)scratch;
    int32_t *nbr = (int32_t *)((char *)scratch + (size_t)n * kScales * sizeof(double));
    // the row in registers (up to 64 of them), or read twice
    const int vecs = (n + kFeatThreads * Vec<T>::N - 1) / (kFeatThreads * Vec<T>::N);
#define HAP_FEATURES(NV)                                                                                               \
    hipLaunchKernelGGL((warm_features_kernel<T, NV>), dim3(n), dim3(kFeatThreads), 0, st, S, lds, pref, n, F, ldf, nbr, D)
    if (vecs <= 1) HAP_FEATURES(1);
    else if (vecs <= 2) HAP_FEATURES(2);
    else if (vecs <= 4) HAP_FEATURES(4);
    else if (vecs <= 8) HAP_FEATURES(8);
    else if (vecs <= 16) HAP_FEATURES(16);
    else HAP_FEATURES(0);
#undef HAP_FEATURES
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(warm_local_kernel, dim3((n + 15) / 16), dim3(256), 0, st, n, nbr, D, F, ldf);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_warm_targets(const LevelPtrs<T> &lv, int n, int64_t ldw, double lam, int t, float *out, int64_t ldo,
                               hipStream_t st) {
    hipLaunchKernelGGL((warm_targets_kernel<T>), dim3((n + 255) / 256), dim3(256), 0, st, lv.R, lv.A, lv.B, lv.pref, n,
                       ldw, (T)lam, (T)(1.0 - lam), t, out, ldo);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_warm_alpha(const LevelPtrs<T> &lv, int n, int64_t ldw, const float *Y, int64_t ldy, int col,
                             T *bases_scratch, hipStream_t st) {
    hipLaunchKernelGGL((warm_bases_kernel<T>), dim3((n + 255) / 256), dim3(256), 0, st, Y + col, ldy, lv.pref, n,
                       bases_scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_warm_fill<T>(lv, n, ldw, bases_scratch, 1, st);
}

template <typename T>
hipError_t launch_warm_fill(const LevelPtrs<T> &lv, int n, int64_t ldw, const T *bases, int64_t stride,
                            hipStream_t st) {
    const int64_t total = (int64_t)n * (ldw / Vec<T>::N);
    const int64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL((warm_fill_kernel<T>), dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, st, lv.A,
                       n, ldw, bases, stride);
    return hipGetLastError();
}

#define HAP_WARM_INSTANTIATE(T)                                                                                   \
    template hipError_t launch_warm_features<T>(const T *, int64_t, const T *, int, float *, int64_t, void *,      \
                                                hipStream_t);                                                      \
    template hipError_t launch_warm_targets<T>(const LevelPtrs<T> &, int, int64_t, double, int, float *, int64_t,  \
                                               hipStream_t);                                                       \
    template hipError_t launch_warm_alpha<T>(const LevelPtrs<T> &, int, int64_t, const float *, int64_t, int, T *, \
                                             hipStream_t);                                                         \
    template hipError_t launch_warm_fill<T>(const LevelPtrs<T> &, int, int64_t, const T *, int64_t, hipStream_t);
HAP_WARM_INSTANTIATE(float)
HAP_WARM_INSTANTIATE(double)

}  // namespace hap
