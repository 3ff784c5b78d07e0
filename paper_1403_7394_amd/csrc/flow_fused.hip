// The fused all-level row pass of the MapReduce schedule (see fused.hip) with several rows of a
// workgroup in flight (see flowpass.h): rows of up to 4096 FP32 columns, one to 64 rows per workgroup.
// A group keeps its row of S in registers over the levels; the levels' availability bases and column
// sums live in LDS (2 x 4 levels x 16 KB at most).  The one-row pass has four waves per CU at 3000
// points and waits out every (row, level) item's loads and barrier: 147 us a sweep of three levels
// against 78 us here (468 MB, much of it from the Infinity Cache, 6.0 TB/s).
#include "flowpass.h"

namespace hap {

namespace {

template <int NTG, int NCH, int RG>
struct FusedLds {
    static constexpr int NWG = NTG / 64;
    Vec<float>::type q[kMaxFused][NCH][NTG], b[kMaxFused][NCH][NTG];
    float m1[2][RG][NWG], m2[2][RG][NWG], cv[2][RG][NWG];
    int ck[2][RG][NWG];
    int arrived[RG];
    int turn[kMaxFused][NWG];
    float p[kMaxFused][kWin], below[kMaxFused][kWin];   // preference; column sum Q^{l-1} of the row's point
    int e[kMaxFused][kWin];
};

template <int NTG, int NCH, int RG, bool FIRST, bool TAIL, int AUX>
__device__ __forceinline__ void fused_flow_rows(const FusedArgs<float> &a, const int t, const int row0, const int row1,
                                                FusedLds<NTG, NCH, RG> &L) {
#pragma clang fp contract(off)
    using T = float;
    using V = Vec<float>::type;
    constexpr int VW = 4;
    constexpr int NWG = NTG / 64;
    constexpr int CB = NTG * 16;
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / NTG);
    const int ltid = threadIdx.x % NTG, lane = ltid & 63, wid = __builtin_amdgcn_readfirstlane(ltid >> 6);
    const int n = a.n;
    const int base = ltid * VW, voff = ltid * 16;
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * 4;
    int chg = 0, item = 0;
    for (int ii = row0 + grp; ii < row1; ii += RG) {
        const int i = slot_row(ii, row0, a.rb, a.row_stride);
        const int r = ii - row0;
        const __amdgpu_buffer_rsrc_t rS = row_rsrc(a.S + (int64_t)i * a.lds, row_bytes);
        V sx[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) sx[c] = buf_load<V, AUX>(rS, voff, c * CB);
        T c_below = 0.f;   // c^{l-1}_i of this iteration
        for (int l = 0; l < a.L; ++l, ++item) {
            const int buf = item & 1;
            const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R[l] + (int64_t)i * a.ldw, row_bytes);
            const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A[l] + (int64_t)i * a.ldw, row_bytes);
            FlowRow<T, NTG, NCH> x;
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                x.r[c] = buf_load<V, AUX>(rR, voff, c * CB);
                x.a[c] = buf_load<V, AUX>(rA, voff, c * CB);
            }
            T m1, m2, cv;
            int ck;
            flow_phase1<T, NTG, NCH, FIRST, TAIL, false, AUX>(
                x, i, n, wid, base, a.lam, a.oml, L.p[l][r], 0.f, rA, voff, m1, m2, cv, ck,
                [&](int c, V &s) { s = sx[c]; }, [&](int c) { return L.b[l][c][ltid]; });
            ck = (ck == INT_MAX) ? INT_MAX : ck + base;
            flow_reduce<T, !FIRST>(m1, m2, cv, ck);
            if constexpr (NWG > 1) {
                if (lane == 63) {
                    L.m1[buf][grp][wid] = m1;
                    L.m2[buf][grp][wid] = m2;
                    L.cv[buf][grp][wid] = cv;
                    L.ck[buf][grp][wid] = ck;
                }
                lds_settle();
                if (lane == 0)
                    __hip_atomic_fetch_add(&L.arrived[grp], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                lds_wait(&L.arrived[grp], (item + 1) * NWG);
                m1 = L.m1[buf][grp][0];
                m2 = L.m2[buf][grp][0];
                cv = L.cv[buf][grp][0];
                ck = L.ck[buf][grp][0];
#pragma unroll
                for (int w = 1; w < NWG; ++w) {
                    pair_merge(m1, m2, L.m1[buf][grp][w], L.m2[buf][grp][w]);
                    argmax_merge(cv, ck, L.cv[buf][grp][w], L.ck[buf][grp][w]);
                }
            } else {
                m1 = lane63(m1);
                m2 = lane63(m2);
                cv = lane63(cv);
                ck = __builtin_amdgcn_readlane(ck, 63);
            }
            // tau^l_i = c^{l-1}_i (this iteration) + Q^{l-1}_i (previous iteration); no clip at l = 0 or in
            // iteration 1
            const bool has_tau = l > 0 && t >= 2;
            const T tau_i = c_below + L.below[l][r];
            if (ltid == 0) {
                if constexpr (!FIRST) {
                    a.C[l][i] = cv;
                    a.E[l][i] = ck;
                    chg |= (t >= 3 && L.e[l][r] != ck) ? 1 : 0;
                }
                if (l > 0) {
                    a.phi[l - 1][i] = m1;
                    a.tau[l][i] = has_tau ? tau_i : pos_inf<T>();
                }
            }
            c_below = cv;
            flow_phase2<T, NTG, NCH, TAIL, AUX>(x, i, n, wid, base, a.lam, a.oml, m1, has_tau ? fmin(tau_i, -m1) : -m1,
                                           has_tau ? fmin(tau_i, -m2) : -m2, rR, voff);
            lds_wait(&L.turn[l][wid], r);
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                if (TAIL && c * NTG * VW + wid * 64 * VW >= n) continue;
                V q = L.q[l][c][ltid];
#pragma unroll
                for (int v = 0; v < VW; ++v) q[v] += x.s[c][v];
                L.q[l][c][ltid] = q;
            }
            lds_settle();
            if (lane == 0)
                __hip_atomic_store(&L.turn[l][wid], r + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    if (chg) atomicOr(&a.ds->changed, 1);
}

template <int NTG, int RG, bool TAIL, int AUX = kNT>
__global__ __launch_bounds__(NTG *RG) void sweep_fused_flow_kernel(FusedArgs<float> a) {
#pragma clang fp contract(off)
    using V = Vec<float>::type;
    constexpr int VW = 4, NCH = 4, NT = NTG * RG;
    __shared__ __attribute__((aligned(16))) FusedLds<NTG, NCH, RG> L;
    const int tid = threadIdx.x, n = a.n;
    const int row0 = blockIdx.x * a.rb;
    const int row1 = slots_end(a.rows, a.rb, row0, a.row_stride);
    const DevState *ds = a.ds;
    if (ds->done) return;
    const int t = ds->t + 1;
    for (int l = 0; l < a.L; ++l) {
        if (tid < kWin && row0 + tid < row1) {
            const int k = slot_row(row0 + tid, row0, a.rb, a.row_stride);
            L.p[l][tid] = a.pref[l][k];
            L.e[l][tid] = a.E[l][k];
            L.below[l][tid] = l > 0 ? a.Q[l - 1][k] : 0.f;
        }
        if (tid < NTG / 64) L.turn[l][tid] = 0;
        for (int e = tid; e < NCH * NTG; e += NT) {
            const int c = e / NTG, lt = e % NTG, j0 = c * NTG * VW + lt * VW;
            L.q[l][c][lt] = (V)(0.f);
            L.b[l][c][lt] = (t > 1 && (!TAIL || j0 < n)) ? *(const V *)(a.B[l] + j0) : (V)(0.f);
        }
    }
    if (tid < RG) L.arrived[tid] = 0;
    __syncthreads();
    if (t == 1)
        fused_flow_rows<NTG, NCH, RG, true, TAIL, AUX>(a, t, row0, row1, L);
    else
        fused_flow_rows<NTG, NCH, RG, false, TAIL, AUX>(a, t, row0, row1, L);
    __syncthreads();
    for (int l = 0; l < a.L; ++l) {
        float *qrow = a.Qpart[l] + (int64_t)blockIdx.x * a.ldw;
        for (int e = tid; e < NCH * NTG; e += NT) {
            const int c = e / NTG, lt = e % NTG, j0 = c * NTG * VW + lt * VW;
            if (!TAIL || j0 < n) *(V *)(qrow + j0) = L.q[l][c][lt];
        }
    }
}

}  // namespace

hipError_t launch_fused_flow(const FusedArgs<float> &a, int threads, int nb, bool tail, hipStream_t st) {
#define HAP_LAUNCH(NTG, RG, ...)                                                                                \
    do {                                                                                                        \
        if (tail)                                                                                               \
            hipLaunchKernelGGL((sweep_fused_flow_kernel<NTG, RG, true __VA_OPT__(, ) __VA_ARGS__>), dim3(nb),   \
                               dim3(NTG * RG), 0, st, a);                                                       \
        else                                                                                                    \
            hipLaunchKernelGGL((sweep_fused_flow_kernel<NTG, RG, false __VA_OPT__(, ) __VA_ARGS__>), dim3(nb),  \
                               dim3(NTG * RG), 0, st, a);                                                       \
        return hipGetLastError();                                                                               \
    } while (0)
    if (threads == 64) HAP_LAUNCH(64, 4);
    // workgroups with fewer rows than groups leave waves idle that others could use (2000 points with two rows,
    // three levels: 26.4 us a level with eight groups, 21.5 with two, 25.0 one row at a time)
    if (threads == 128 && a.rb <= 2) HAP_LAUNCH(128, 2);
    if (threads == 128 && a.rb <= 4) HAP_LAUNCH(128, 4);
    if (threads == 128) HAP_LAUNCH(128, 8);
    if (threads == 256 && a.cached) HAP_LAUNCH(256, 4, 0);
    if (threads == 256) HAP_LAUNCH(256, 4);
#undef HAP_LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace hap
