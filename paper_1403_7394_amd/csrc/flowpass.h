// Row pass with several rows of a workgroup in flight.
//
// A workgroup of RG groups of NTG threads works on RG of its rows at a time, group g on its row slots
// g, g + RG, ...; no workgroup barrier separates the rows.  The waves of a group exchange their
// reductions through LDS and wait for one another on a counter there.  The column sums live in LDS, and
// a row's contribution is added by the wave that holds the columns once the row before it has been
// added (a turn per wave position), so every column is summed in row order, with the bits of one
// group running all rows.  While one group reduces or waits, the loads and the arithmetic of the others
// go on.  Every wait is for waves of the same workgroup that work on the same or an earlier row, so
// the lowest row in flight always proceeds and every wait ends.
//
// The arithmetic gives the values of sweep_rows with fewer instructions:
//   - the column that a row's maximum excludes is found by value: max_{k != j} is M2 exactly where
//     alpha + s equals M1 (with the maximum attained twice, M2 = M1 and either reading is the same),
//     so no index is carried for it;
//   - min(tau, -M) has two values per row, formed once;
//   - the diagonal and the ragged end are handled in the chunks of a wave that hold them (a
//     wave-uniform branch), and chunks past n are left out.
#pragma once

#include "rowpass.h"

namespace hap {

// Cache policy (AUX) of a row's loads and stores.  Every word is touched once a pass, so non-temporal, except
// rows of 256 threads (FP32 up to 4096 columns): there matrices stay in the 256 MB Infinity Cache from pass to
// pass, and the accesses are cached where they pay (us a level, non-temporal and cached):
//   - S and the messages of every level fit it together: 3000 points, two levels, 12 rows 41.2, 37.6, three
//     rows 50.7, 48.2;
//   - or they do not, and a workgroup has more than four rows: 4000 points, two levels (320 MB), 16 rows 66.6,
//     62.9, but three rows 77.7, 83.3;
//   - the all-level pass goes through every level's matrices at once, so their sum decides: 3800 points, two
//     levels (289 MB) 53.1, 48.9, 4096 (336 MB) 59.9, 58.2, but three levels of 3500 (343 MB) 44.2, 45.0 and of
//     4000 (448 MB) 56.7, 61.3.
// Longer rows lose (6000 points 136 -> 152 us) and so do shorter ones (2000 points 20.6 -> 22.2 us).

template <typename T, int NTG, int NCH, int RG, int D>
struct FlowLds {
    static constexpr int NWG = NTG / 64;
    typename Vec<T>::type q[NCH][NTG];                  // column sums
    T x[D > 0 ? D : 1][D > 0 ? NCH * NTG * Vec<T>::N : 1];   // points mode: the columns' coordinates
    T m1[2][RG][NWG], m2[2][RG][NWG], cv[2][RG][NWG];
    int ck[2][RG][NWG];
    int arrived[RG];                                    // waves of the group that published, in total
    int turn[NWG];                                      // row slot whose contribution is added next
    T p[kWin], tau[kWin], d[kWin], xi[kWin][D > 0 ? D : 1];  // per-row scalars
    int e[kWin], has[kWin];
};
// One row per group: nothing staged, and a slab of contributions per group instead of turns.
template <typename T, int NTG, int NCH, int RG>
struct FlowOneLds {
    static constexpr int NWG = NTG / 64;
    typename Vec<T>::type q[RG][NCH][NTG];
    T m1[RG][NWG], m2[RG][NWG], cv[RG][NWG];
    int ck[RG][NWG];
    int arrived[RG];
};

// This wave's LDS accesses are done and stay on their side of this point (global accesses in flight are
// not waited for).
__device__ __forceinline__ void lds_settle() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void lds_wait(const int *p, int at_least) {
    while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < at_least)
        __builtin_amdgcn_s_sleep(1);
    asm volatile("" ::: "memory");
}

// Second maximum after y joins (m1 the maximum before): a y that compares with nothing (NaN) is ignored.
// v_med3_f32 does so (with a NaN among its operands it gives the least of the others, m2), but the compiler folds a
// median with a constant -inf into a minimum, which would give m1: m1 and m2 start opaque (flow_phase1).
// y > m1 ? m1 : fmax(m2, y) needs an instruction more (2000 points 20.2 -> 20.6 us a level, others the same).
__device__ __forceinline__ float second_max(float m1, float m2, float y) { return __builtin_amdgcn_fmed3f(m1, m2, y); }
__device__ __forceinline__ double second_max(double m1, double m2, double y) { return y > m1 ? m1 : fmax(m2, y); }

// Two (max, second max) pairs: the smaller maximum competes for second place.
template <typename T>
__device__ __forceinline__ void pair_merge(T &m1, T &m2, T om1, T om2) {
    const T lo = fmin(m1, om1);
    m1 = fmax(m1, om1);
    m2 = fmax(fmax(m2, om2), lo);
}

template <typename T, bool WITH_C, int CTRL, int ROW_MASK>
__device__ __forceinline__ void flow_step(T &m1, T &m2, T &cv, int &ck) {
    const T ninf = neg_inf<T>();
    const T om1 = dpp_val<CTRL, ROW_MASK>(ninf, m1);
    const T om2 = dpp_val<CTRL, ROW_MASK>(ninf, m2);
    pair_merge(m1, m2, om1, om2);
    if constexpr (WITH_C) {
        const T ocv = dpp_val<CTRL, ROW_MASK>(ninf, cv);
        const int ock = dpp_i32<CTRL, ROW_MASK>(INT_MAX, ck);
        argmax_merge(cv, ck, ocv, ock);
    }
}

// Wave-wide (max, second max) and (max, lowest argmax): the tree of wave_reduce; the result is valid in
// lane 63 only.
template <typename T, bool WITH_C>
__device__ __forceinline__ void flow_reduce(T &m1, T &m2, T &cv, int &ck) {
    flow_step<T, WITH_C, 0xb1, 0xf>(m1, m2, cv, ck);    // quad_perm [1,0,3,2]
    flow_step<T, WITH_C, 0x4e, 0xf>(m1, m2, cv, ck);    // quad_perm [2,3,0,1]
    flow_step<T, WITH_C, 0x141, 0xf>(m1, m2, cv, ck);   // row_half_mirror
    flow_step<T, WITH_C, 0x140, 0xf>(m1, m2, cv, ck);   // row_mirror
    flow_step<T, WITH_C, 0x142, 0xa>(m1, m2, cv, ck);   // row_bcast:15 into rows 1, 3
    flow_step<T, WITH_C, 0x143, 0xc>(m1, m2, cv, ck);   // row_bcast:31 into rows 2, 3
}
__device__ __forceinline__ float lane63(float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); }
__device__ __forceinline__ double lane63(double v) {
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(x & 0xffffffffll), 63);
    const int hi = __builtin_amdgcn_readlane((int)(x >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// One row of one level, as a group of NTG threads holds it: s and rho of the row, and in `a` alpha
// (before) or alpha + s (after phase 1) of this thread's columns.
template <typename T, int NTG, int NCH>
struct FlowRow {
    typename Vec<T>::type s[NCH], r[NCH], a[NCH];
};

// Phase 1 of row i: finish alpha^{t-1} (stored through rA), reduce (M1, M2) of alpha + s and
// (c, e) of alpha + rho over this thread's columns.  make_s(c): s of chunk c in points mode.
template <typename T, int NTG, int NCH, bool FIRST, bool TAIL, bool OFFSET, int AUX, typename MakeS, typename BaseOf>
__device__ __forceinline__ void flow_phase1(FlowRow<T, NTG, NCH> &x, int i, int n, int wid, int base, T lam, T oml,
                                            T p_i, T d_i, const __amdgpu_buffer_rsrc_t rA, int voff, T &m1, T &m2,
                                            T &cv, int &ck, MakeS make_s, BaseOf base_of) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N;
    constexpr int CB = NTG * VW * (int)sizeof(T);
    const T zero = T(0), ninf = neg_inf<T>();
    m1 = m2 = cv = ninf;
    ck = INT_MAX;   // offset from base
    asm("" : "+v"(m1), "+v"(m2));   // not known to be -inf: see second_max
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        asm volatile("" ::: "memory");
        // the wave's columns of this chunk
        const int lo = c * NTG * VW + wid * 64 * VW;
        if (TAIL && lo >= n) continue;
        make_s(c, x.s[c]);
        V ah;
        if constexpr (!FIRST) {
            const V bv = base_of(c);
#pragma unroll
            for (int v = 0; v < VW; ++v) ah[v] = fmin(zero, bv[v] - fmax(zero, x.r[c][v]));
            if ((unsigned)(i - lo) < (unsigned)(64 * VW)) {
#pragma unroll
                for (int v = 0; v < VW; ++v)
                    if (c * NTG * VW + base + v == i) ah[v] = bv[v] - x.r[c][v];
            }
        }
        if constexpr (OFFSET) x.s[c] = x.s[c] + d_i;
        if ((unsigned)(i - lo) < (unsigned)(64 * VW)) {
#pragma unroll
            for (int v = 0; v < VW; ++v)
                if (c * NTG * VW + base + v == i) x.s[c][v] = p_i;
        }
        // whole vectors past n were not loaded; inside the last one the padding columns of alpha hold -inf or
        // NaN, which no comparison takes
        if (TAIL && lo + 64 * VW > n) {
            if (c * NTG * VW + base >= n) x.a[c] = (V)(ninf);
        }
        V y;
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            const int j = c * NTG * VW + v;
            const T rj = x.r[c][v];
            T al = x.a[c][v];
            if constexpr (!FIRST) {
                al = lam * al + oml * ah[v];
                x.a[c][v] = al;
                const T cx = al + rj;
                const bool g = cx > cv;
                cv = g ? cx : cv;
                ck = g ? j : ck;
            }
            y[v] = al + x.s[c][v];
            m2 = second_max(m1, m2, y[v]);
            m1 = y[v] > m1 ? y[v] : m1;
        }
        if constexpr (!FIRST) buf_store<V, AUX>(x.a[c], rA, voff, c * CB);
        x.a[c] = y;
    }
}

// Phase 2 of row i: rho^t (stored through rR); s becomes the row's contribution to the column sums.
// u1, u2: min(tau_i, -M1) and min(tau_i, -M2).
template <typename T, int NTG, int NCH, bool TAIL, int AUX>
__device__ __forceinline__ void flow_phase2(FlowRow<T, NTG, NCH> &x, int i, int n, int wid, int base, T lam, T oml, T m1,
                                            T u1, T u2, const __amdgpu_buffer_rsrc_t rR, int voff) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N;
    constexpr int CB = NTG * VW * (int)sizeof(T);
    const T zero = T(0);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        asm volatile("" ::: "memory");
        const int lo = c * NTG * VW + wid * 64 * VW;
        if (TAIL && lo >= n) continue;
        V out;
#pragma unroll
        for (int v = 0; v < VW; ++v) {
            const T rh = x.s[c][v] + (x.a[c][v] == m1 ? u2 : u1);
            const T rn = lam * x.r[c][v] + oml * rh;
            out[v] = rn;
            x.s[c][v] = fmax(zero, rn);
        }
        if ((unsigned)(i - lo) < (unsigned)(64 * VW)) {
#pragma unroll
            for (int v = 0; v < VW; ++v)
                if (c * NTG * VW + base + v == i) x.s[c][v] = out[v];
        }
        buf_store<V, AUX>(out, rR, voff, c * CB);
    }
}

template <typename T, int NTG, int NCH, int RG, bool FIRST, bool TAIL, int D, int AUX>
__device__ __forceinline__ void flow_rows(const SweepArgs<T> &a, const int t, const int row0, const int row1,
                                          const typename Vec<T>::type (&Bv)[NCH],
                                          FlowLds<T, NTG, NCH, RG, D> &L) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N;
    constexpr int NWG = NTG / 64;
    constexpr int CB = NTG * VW * (int)sizeof(T);   // bytes per chunk
    const int grp = RG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NTG) : 0;
    const int ltid = threadIdx.x % NTG, lane = ltid & 63, wid = __builtin_amdgcn_readfirstlane(ltid >> 6);
    const int n = a.n;
    const int64_t ldw = a.ldw;
    const int base = ltid * VW, voff = ltid * 16;
    // a row's whole 16-byte vectors: loads past them return 0, stores past them are dropped
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * (int)sizeof(T);
    int chg = 0, step = 0;
    for (int ii = row0 + grp; ii < row1; ii += RG, ++step) {
        const int i = slot_row(ii, row0, a.rb, a.row_stride);
        const int r = ii - row0;
        const int buf = step & 1;
        const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * ldw, row_bytes);
        const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * ldw, row_bytes);
        FlowRow<T, NTG, NCH> x;
        {
            const __amdgpu_buffer_rsrc_t rS = row_rsrc(a.S + (int64_t)i * a.lds, row_bytes);
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if constexpr (D <= 0) x.s[c] = buf_load<V, AUX>(rS, voff, c * CB);
                x.r[c] = buf_load<V, AUX>(rR, voff, c * CB);
                x.a[c] = buf_load<V, AUX>(rA, voff, c * CB);
            }
        }
        T m1, m2, cv;
        int ck;
        flow_phase1<T, NTG, NCH, FIRST, TAIL, (D < 0), AUX>(
            x, i, n, wid, base, a.lam, a.oml, L.p[r], L.d[r], rA, voff, m1, m2, cv, ck,
            [&](int c, V &s) {
                if constexpr (D > 0) {
                    // s_ij from the coordinates, with the direct build's arithmetic
                    V xj[D];
#pragma unroll
                    for (int d = 0; d < D; ++d) xj[d] = *(const V *)&L.x[d][c * NTG * VW + base];
#pragma unroll
                    for (int v = 0; v < VW; ++v) {
                        double acc = 0.0;
#pragma unroll
                        for (int d = 0; d < D; ++d) {
                            const double df = (double)L.xi[r][d] - (double)xj[d][v];
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
                L.m1[buf][grp][wid] = m1;
                L.m2[buf][grp][wid] = m2;
                if constexpr (!FIRST) {
                    L.cv[buf][grp][wid] = cv;
                    L.ck[buf][grp][wid] = ck;
                }
            }
            lds_settle();
            if (lane == 0) __hip_atomic_fetch_add(&L.arrived[grp], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            lds_wait(&L.arrived[grp], (step + 1) * NWG);
            m1 = L.m1[buf][grp][0];
            m2 = L.m2[buf][grp][0];
#pragma unroll
            for (int w = 1; w < NWG; ++w) pair_merge(m1, m2, L.m1[buf][grp][w], L.m2[buf][grp][w]);
        } else {
            m1 = lane63(m1);
            m2 = lane63(m2);
        }
        const T tau_i = L.tau[r];
        const bool has_tau = L.has[r] != 0;
        if (ltid == 63) {
            if constexpr (!FIRST) {
                if constexpr (NWG > 1) {
                    cv = L.cv[buf][grp][0];
                    ck = L.ck[buf][grp][0];
                    for (int w = 1; w < NWG; ++w) argmax_merge(cv, ck, L.cv[buf][grp][w], L.ck[buf][grp][w]);
                }
                a.C[i] = cv;
                a.E[i] = ck;
                chg |= (t >= 3 && L.e[r] != ck) ? 1 : 0;
            }
            if (a.phi_down && (!FIRST || a.mrhap)) a.phi_down[i] = m1;
            if (a.tau_store) a.tau_store[i] = has_tau ? tau_i : pos_inf<T>();
        }
        flow_phase2<T, NTG, NCH, TAIL, AUX>(x, i, n, wid, base, a.lam, a.oml, m1, has_tau ? fmin(tau_i, -m1) : -m1,
                                       has_tau ? fmin(tau_i, -m2) : -m2, rR, voff);
        if constexpr (RG > 1) lds_wait(&L.turn[wid], r);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (TAIL && c * NTG * VW + wid * 64 * VW >= n) continue;
            V q = L.q[c][ltid];
#pragma unroll
            for (int v = 0; v < VW; ++v) q[v] += x.s[c][v];
            L.q[c][ltid] = q;
        }
        if constexpr (RG > 1) {
            lds_settle();
            if (lane == 0) __hip_atomic_store(&L.turn[wid], r + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    if (chg) atomicOr(&a.ds->changed, 1);
}

template <typename T, int NTG, int NCH, int RG, bool TAIL, int D, int AUX = kNT>
__global__ __launch_bounds__(NTG *RG) void sweep_flow_kernel(SweepArgs<T> a) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N;
    constexpr int NT = NTG * RG;
    __shared__ __attribute__((aligned(16))) FlowLds<T, NTG, NCH, RG, D> L;
    const int tid = threadIdx.x, ltid = tid % NTG;
    const int n = a.n;
    const int row0 = blockIdx.x * a.rb;
    const int row1 = slots_end(a.rows, a.rb, row0, a.row_stride);
    const DevState *ds = a.ds;
    V Bv[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j0 = c * NTG * VW + ltid * VW;
        Bv[c] = (!TAIL || j0 < n) ? *(const V *)(a.B + j0) : (V)(T(0));
    }
    if (ds->done) return;
    const int t = ds->t + 1;
    if (tid < kWin && row0 + tid < row1) {
        const int k = slot_row(row0 + tid, row0, a.rb, a.row_stride);
        L.p[tid] = a.pref[k];
        T tv = T(0);
        L.has[tid] = row_tau(a, k, t, tv) ? 1 : 0;
        L.tau[tid] = tv;
        L.d[tid] = (D < 0) ? a.delta[k] : T(0);
        L.e[tid] = a.E[k];
        if constexpr (D > 0) {
#pragma unroll
            for (int d = 0; d < D; ++d) L.xi[tid][d] = a.X[(int64_t)k * a.ldx + d];
        }
    }
    if (tid < RG) L.arrived[tid] = 0;
    if (tid < NTG / 64) L.turn[tid] = 0;
    for (int e = tid; e < NCH * NTG; e += NT) L.q[e / NTG][e % NTG] = (V)(T(0));
    if constexpr (D > 0) {
        for (int j = tid; j < NCH * NTG * VW; j += NT)
#pragma unroll
            for (int d = 0; d < D; ++d) L.x[d][j] = j < n ? a.X[(int64_t)j * a.ldx + d] : T(0);
    }
    __syncthreads();
    if (t == 1)
        flow_rows<T, NTG, NCH, RG, true, TAIL, D, AUX>(a, t, row0, row1, Bv, L);
    else
        flow_rows<T, NTG, NCH, RG, false, TAIL, D, AUX>(a, t, row0, row1, Bv, L);
    __syncthreads();
    T *qrow = a.Qpart + (int64_t)blockIdx.x * a.ldw;
    for (int e = tid; e < NCH * NTG; e += NT) {
        const int c = e / NTG, lt = e % NTG;
        const int j0 = c * NTG * VW + lt * VW;
        if (!TAIL || j0 < n) *(V *)(qrow + j0) = L.q[c][lt];
    }
}

// At most one row per group (the default up to 2048 points): a chain of latencies, so every load goes out
// before the first is waited for, the row's scalars come straight from memory, and the contributions are
// added in row order from a slab per group after one barrier.  788 points: 7.9 us a launch with staged
// scalars and turns, 6.0 us here.  Reads S: in points mode the columns' coordinates are better staged in
// LDS (2000 points, with column sums, 19.1 us a level against 29.7 with every lane gathering its own).
template <typename T, int NTG, int NCH, int RG, bool FIRST, bool TAIL, int D>
__device__ __forceinline__ void flow_one(const SweepArgs<T> &a, const int t, const int i, FlowRow<T, NTG, NCH> &x,
                                         const typename Vec<T>::type (&Bv)[NCH], const T p_i, const T d_i,
                                         const int e_old, const bool has_tau, const T tau_i,
                                         FlowOneLds<T, NTG, NCH, RG> &L) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N, NWG = NTG / 64;
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / NTG);
    const int ltid = threadIdx.x % NTG, lane = ltid & 63, wid = __builtin_amdgcn_readfirstlane(ltid >> 6);
    const int n = a.n;
    const int base = ltid * VW, voff = ltid * 16;
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * a.ldw, row_bytes);
    const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * a.ldw, row_bytes);
    T m1, m2, cv;
    int ck;
    flow_phase1<T, NTG, NCH, FIRST, TAIL, (D < 0), kNT>(
        x, i, n, wid, base, a.lam, a.oml, p_i, d_i, rA, voff, m1, m2, cv, ck,
        [&](int, V &) {}, [&](int c) { return Bv[c]; });
    ck = (ck == INT_MAX) ? INT_MAX : ck + base;
    flow_reduce<T, !FIRST>(m1, m2, cv, ck);
    if constexpr (NWG > 1) {
        if (lane == 63) {
            L.m1[grp][wid] = m1;
            L.m2[grp][wid] = m2;
            L.cv[grp][wid] = cv;
            L.ck[grp][wid] = ck;
        }
        lds_settle();
        if (lane == 0) __hip_atomic_fetch_add(&L.arrived[grp], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        lds_wait(&L.arrived[grp], NWG);
        m1 = L.m1[grp][0];
        m2 = L.m2[grp][0];
#pragma unroll
        for (int w = 1; w < NWG; ++w) pair_merge(m1, m2, L.m1[grp][w], L.m2[grp][w]);
    } else {
        m1 = lane63(m1);
        m2 = lane63(m2);
    }
    flow_phase2<T, NTG, NCH, TAIL, kNT>(x, i, n, wid, base, a.lam, a.oml, m1, has_tau ? fmin(tau_i, -m1) : -m1,
                                   has_tau ? fmin(tau_i, -m2) : -m2, rR, voff);
#pragma unroll
    for (int c = 0; c < NCH; ++c) L.q[grp][c][ltid] = x.s[c];
    if (ltid == 63) {
        if constexpr (!FIRST) {
            if constexpr (NWG > 1) {
                cv = L.cv[grp][0];
                ck = L.ck[grp][0];
                for (int w = 1; w < NWG; ++w) argmax_merge(cv, ck, L.cv[grp][w], L.ck[grp][w]);
            }
            a.C[i] = cv;
            a.E[i] = ck;
            if (t >= 3 && e_old != ck) atomicOr(&a.ds->changed, 1);
        }
        if (a.phi_down && (!FIRST || a.mrhap)) a.phi_down[i] = m1;
        if (a.tau_store) a.tau_store[i] = has_tau ? tau_i : pos_inf<T>();
    }
}

template <typename T, int NTG, int NCH, int RG, bool TAIL, int D>
__global__ __launch_bounds__(NTG *RG) void sweep_flow_one_kernel(SweepArgs<T> a) {
#pragma clang fp contract(off)
    using V = typename Vec<T>::type;
    constexpr int VW = Vec<T>::N, NT = NTG * RG;
    constexpr int CB = NTG * VW * (int)sizeof(T);
    static_assert(D <= 0, "reads S");
    __shared__ __attribute__((aligned(16))) FlowOneLds<T, NTG, NCH, RG> L;
    const int tid = threadIdx.x, ltid = tid % NTG;
    const int grp = __builtin_amdgcn_readfirstlane(tid / NTG);
    const int n = a.n;
    const int row0 = blockIdx.x * a.rb;
    const int row1 = slots_end(a.rows, a.rb, row0, a.row_stride);
    const DevState *ds = a.ds;
    const int done = ds->done, t = ds->t + 1;
    const bool mine = row0 + grp < row1;   // this group has a row
    const int i = slot_row(mine ? row0 + grp : row0, row0, a.rb, a.row_stride);
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * (int)sizeof(T);
    FlowRow<T, NTG, NCH> x;
    V Bv[NCH];
    T p_i = T(0), d_i = T(0), tau_i = T(0);
    int e_old = 0;
    const bool mr = a.tau_c != nullptr;
    if (mine) {
        const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * a.ldw, row_bytes);
        const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * a.ldw, row_bytes);
        const __amdgpu_buffer_rsrc_t rS = row_rsrc(a.S + (int64_t)i * a.lds, row_bytes);
        const __amdgpu_buffer_rsrc_t rB = row_rsrc(a.B, row_bytes);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            x.s[c] = buf_load<V, kNT>(rS, ltid * 16, c * CB);
            x.r[c] = buf_load<V, kNT>(rR, ltid * 16, c * CB);
            x.a[c] = buf_load<V, kNT>(rA, ltid * 16, c * CB);
            Bv[c] = buf_load<V, 0>(rB, ltid * 16, c * CB);
        }
        p_i = a.pref[i];
        if constexpr (D < 0) d_i = a.delta[i];
        e_old = a.E[i];
        // the upward message (row_tau), loaded whether or not this iteration clips with it
        if (mr)
            tau_i = a.tau_c[i] + a.tau_q[i];
        else if (a.tau != nullptr)
            tau_i = a.tau[i];
    }
    if (done) return;
    if constexpr (NTG > 64) {
        if (tid < RG) L.arrived[tid] = 0;
        lds_settle();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    const bool has_tau = mr ? t >= 2 : a.tau != nullptr;
    if (mine) {
        if (t == 1)
            flow_one<T, NTG, NCH, RG, true, TAIL, D>(a, t, i, x, Bv, p_i, d_i, e_old, has_tau, tau_i, L);
        else
            flow_one<T, NTG, NCH, RG, false, TAIL, D>(a, t, i, x, Bv, p_i, d_i, e_old, has_tau, tau_i, L);
    }
    lds_settle();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    T *qrow = a.Qpart + (int64_t)blockIdx.x * a.ldw;
    const int groups = row1 - row0;
    for (int e = tid; e < NCH * NTG; e += NT) {
        const int c = e / NTG, lt = e % NTG;
        const int j0 = c * NTG * VW + lt * VW;
        if (TAIL && j0 >= n) continue;
        V q = (V)(T(0));
#pragma unroll
        for (int g = 0; g < RG; ++g)
            if (g < groups) q += L.q[g][c][lt];
        *(V *)(qrow + j0) = q;
    }
}

template <typename T, int D>
hipError_t launch_flow(const SweepArgs<T> &a, int threads, int nb, bool tail, bool fits, hipStream_t st) {
#define HAP_LAUNCH_FLOW(KERNEL, NTG, RG, ...)                                                            \
    do {                                                                                                 \
        if (tail)                                                                                        \
            hipLaunchKernelGGL((KERNEL<T, NTG, 4, RG, true, D __VA_OPT__(, ) __VA_ARGS__>), dim3(nb), dim3(NTG * RG), 0, st, a);  \
        else                                                                                             \
            hipLaunchKernelGGL((KERNEL<T, NTG, 4, RG, false, D __VA_OPT__(, ) __VA_ARGS__>), dim3(nb), dim3(NTG * RG), 0, st, a); \
        return hipGetLastError();                                                                        \
    } while (0)
    // 1024 threads (128 registers each), as many rows in flight as fit them; rows of one wave: four, the
    // most a workgroup has at these lengths by default.  Workgroups with fewer rows take fewer groups: idle
    // ones hold waves back (2000 points with two rows 32.4 us a level with eight groups, 26.9 with two, 29.2
    // one row at a time; in points mode 37.8, 30.4 and 33.8).
    if constexpr (D <= 0) {
        if (threads == 64 && a.rb <= 4) HAP_LAUNCH_FLOW(sweep_flow_one_kernel, 64, 4);
        if (threads == 128 && a.rb <= 2) HAP_LAUNCH_FLOW(sweep_flow_one_kernel, 128, 2);
        if (threads == 128 && a.rb <= 4) HAP_LAUNCH_FLOW(sweep_flow_one_kernel, 128, 4);
        if (threads == 128 && a.rb <= 8) HAP_LAUNCH_FLOW(sweep_flow_one_kernel, 128, 8);
    } else {
        if (threads == 128 && a.rb <= 2) HAP_LAUNCH_FLOW(sweep_flow_kernel, 128, 2);
    }
    if (threads == 64) HAP_LAUNCH_FLOW(sweep_flow_kernel, 64, 4);
    if (threads == 128) HAP_LAUNCH_FLOW(sweep_flow_kernel, 128, 8);
    if (threads == 256 && (fits || a.rb > 4)) HAP_LAUNCH_FLOW(sweep_flow_kernel, 256, 4, 0);
    if (threads == 256) HAP_LAUNCH_FLOW(sweep_flow_kernel, 256, 4);
    if (threads == 512) HAP_LAUNCH_FLOW(sweep_flow_kernel, 512, 2);
#undef HAP_LAUNCH_FLOW
    return hipErrorInvalidValue;
}

}  // namespace hap
