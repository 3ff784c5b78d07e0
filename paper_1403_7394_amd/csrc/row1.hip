// Row pass with one row per workgroup (the default up to 512 FP32 and 2048 FP64 points, whose column
// sums are then taken in row order).  There is nothing to overlap a row with, so the pass is a chain of
// latencies: every load (the row, the bases, the row's scalars, the iteration state) is issued before the
// first is waited for, nothing is staged, one barrier exchanges the waves' reductions and the row's
// contributions go straight to its partial row.  The arithmetic is flowpass.h's.  300 FP64 points:
// 6.1 us a launch with the scalars staged behind the state and two barriers, 4.0 us here.
#include "flowpass.h"

namespace hap {

namespace {

// cached stores where a level's matrices stay in the Infinity Cache (rows of 256 threads), as in flowpass.h
template <int NTG> constexpr int kRowAux = NTG == 256 ? 0 : kNT;

template <typename T, int NTG, bool FIRST, bool TAIL, int D>
__device__ __forceinline__ void one_row(const SweepArgs<T> &a, const int t, const int i,
                                        FlowRow<T, NTG, 4> &x, const typename Vec<T>::type (&Bv)[4], const T p_i,
                                        const T d_i, const T (&xi)[D > 0 ? D : 1], const int e_old, const bool has_tau,
                                        const T tau_i, T *sh_m1, T *sh_m2, T *sh_cv, int *sh_ck) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N, NCH = 4, NWG = NTG / 64;
    constexpr int CB = NTG * VW * (int)sizeof(T);
    const int ltid = threadIdx.x, lane = ltid & 63, wid = __builtin_amdgcn_readfirstlane(ltid >> 6);
    const int n = a.n;
    const int base = ltid * VW, voff = ltid * 16;
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * a.ldw, row_bytes);
    const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * a.ldw, row_bytes);
    T m1, m2, cv;
    int ck;
    flow_phase1<T, NTG, NCH, FIRST, TAIL, (D < 0), kRowAux<NTG>>(
        x, i, n, wid, base, a.lam, a.oml, p_i, d_i, rA, voff, m1, m2, cv, ck,
        [&](int c, V &s) {
            if constexpr (D > 0) {
#pragma unroll
                for (int v = 0; v < VW; ++v) {
                    const int j = c * NTG * VW + base + v;
                    double acc = 0.0;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        const double df = (double)xi[d] - (double)(j < n ? a.X[(int64_t)j * a.ldx + d] : T(0));
                        const double sq = df * df;
                        acc = acc + sq;
                    }
                    s[v] = (T)(-acc);
                }
            }
        },
        [&](int c) { return Bv[c]; });
    ck = (ck == INT_MAX) ? INT_MAX : ck + base;
    flow_reduce<T, !FIRST>(m1, m2, cv, ck);
    if constexpr (NWG > 1) {
        if (lane == 63) {
            sh_m1[wid] = m1;
            sh_m2[wid] = m2;
            sh_cv[wid] = cv;
            sh_ck[wid] = ck;
        }
        lds_settle();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        m1 = sh_m1[0];
        m2 = sh_m2[0];
#pragma unroll
        for (int w = 1; w < NWG; ++w) pair_merge(m1, m2, sh_m1[w], sh_m2[w]);
    } else {
        m1 = lane63(m1);
        m2 = lane63(m2);
    }
    flow_phase2<T, NTG, NCH, TAIL, kRowAux<NTG>>(x, i, n, wid, base, a.lam, a.oml, m1, has_tau ? fmin(tau_i, -m1) : -m1,
                                   has_tau ? fmin(tau_i, -m2) : -m2, rR, voff);
    const __amdgpu_buffer_rsrc_t rQ = row_rsrc(a.Qpart + (int64_t)blockIdx.x * a.ldw, row_bytes);
#pragma unroll
    for (int c = 0; c < NCH; ++c) buf_store<V, 0>(x.s[c], rQ, voff, c * CB);
    if (ltid == 63) {
        if constexpr (!FIRST) {
            if constexpr (NWG > 1) {
                cv = sh_cv[0];
                ck = sh_ck[0];
                for (int w = 1; w < NWG; ++w) argmax_merge(cv, ck, sh_cv[w], sh_ck[w]);
            }
            a.C[i] = cv;
            a.E[i] = ck;
            if (t >= 3 && e_old != ck) atomicOr(&a.ds->changed, 1);
        }
        if (a.phi_down && (!FIRST || a.mrhap)) a.phi_down[i] = m1;
        if (a.tau_store) a.tau_store[i] = has_tau ? tau_i : pos_inf<T>();
    }
}

template <typename T, int NTG, bool TAIL, int D>
__global__ __launch_bounds__(NTG) void sweep_row1_kernel(SweepArgs<T> a) {
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N, NCH = 4, NWG = NTG / 64;
    constexpr int CB = NTG * VW * (int)sizeof(T);
    __shared__ T sh_m1[NWG], sh_m2[NWG], sh_cv[NWG];
    __shared__ int sh_ck[NWG];
    const int ltid = threadIdx.x, n = a.n;
    const int i = blockIdx.x;
    const DevState *ds = a.ds;
    const int done = ds->done, t = ds->t + 1;
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * a.ldw, row_bytes);
    const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * a.ldw, row_bytes);
    const __amdgpu_buffer_rsrc_t rS = row_rsrc(a.S + (int64_t)i * a.lds, row_bytes);
    const __amdgpu_buffer_rsrc_t rB = row_rsrc(a.B, row_bytes);
    FlowRow<T, NTG, NCH> x;
    V Bv[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        if constexpr (D <= 0) x.s[c] = buf_load<V, 0>(rS, ltid * 16, c * CB);
        x.r[c] = buf_load<V, 0>(rR, ltid * 16, c * CB);
        x.a[c] = buf_load<V, 0>(rA, ltid * 16, c * CB);
        Bv[c] = buf_load<V, 0>(rB, ltid * 16, c * CB);
    }
    const T p_i = a.pref[i];
    const T d_i = D < 0 ? a.delta[i] : T(0);
    const int e_old = a.E[i];
    T xi[D > 0 ? D : 1] = {};
    if constexpr (D > 0) {
#pragma unroll
        for (int d = 0; d < D; ++d) xi[d] = a.X[(int64_t)i * a.ldx + d];
    }
    // the upward message (row_tau), loaded whether or not this iteration clips with it
    const bool mr = a.tau_c != nullptr;
    T tau_i = T(0);
    if (mr)
        tau_i = a.tau_c[i] + a.tau_q[i];
    else if (a.tau != nullptr)
        tau_i = a.tau[i];
    if (done) return;
    const bool has_tau = mr ? t >= 2 : a.tau != nullptr;
    if (t == 1)
        one_row<T, NTG, true, TAIL, D>(a, t, i, x, Bv, p_i, d_i, xi, e_old, has_tau, tau_i, sh_m1, sh_m2, sh_cv, sh_ck);
    else
        one_row<T, NTG, false, TAIL, D>(a, t, i, x, Bv, p_i, d_i, xi, e_old, has_tau, tau_i, sh_m1, sh_m2, sh_cv, sh_ck);
}

}  // namespace

template <typename T, int D>
hipError_t launch_row1(const SweepArgs<T> &a, int threads, bool tail, hipStream_t st) {
#define HAP_LAUNCH(NTG)                                                                                      \
    do {                                                                                                     \
        if (tail)                                                                                            \
            hipLaunchKernelGGL((sweep_row1_kernel<T, NTG, true, D>), dim3(a.rows), dim3(NTG), 0, st, a);     \
        else                                                                                                 \
            hipLaunchKernelGGL((sweep_row1_kernel<T, NTG, false, D>), dim3(a.rows), dim3(NTG), 0, st, a);    \
        return hipGetLastError();                                                                            \
    } while (0)
    if (threads == 64) HAP_LAUNCH(64);
    if (threads == 128) HAP_LAUNCH(128);
    if (threads == 256) HAP_LAUNCH(256);
    if (threads == 512) HAP_LAUNCH(512);
#undef HAP_LAUNCH
    return hipErrorInvalidValue;
}

template hipError_t launch_row1<float, 0>(const SweepArgs<float> &, int, bool, hipStream_t);
template hipError_t launch_row1<float, -1>(const SweepArgs<float> &, int, bool, hipStream_t);
template hipError_t launch_row1<float, 2>(const SweepArgs<float> &, int, bool, hipStream_t);
template hipError_t launch_row1<float, 3>(const SweepArgs<float> &, int, bool, hipStream_t);
template hipError_t launch_row1<double, 0>(const SweepArgs<double> &, int, bool, hipStream_t);
template hipError_t launch_row1<double, -1>(const SweepArgs<double> &, int, bool, hipStream_t);

}  // namespace hap
