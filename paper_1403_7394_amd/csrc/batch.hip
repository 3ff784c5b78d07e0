// Batched HAP: many independent instances of up to 2048 points in ONE persistent launch.
//
// Workgroups pull work items from an atomic queue.  An item is either a whole instance, which
// one workgroup runs from start to end (the similarity build (FP64-accumulated, as
// HAP_BUILD_DIRECT), the median preference (radix select in LDS), the Algorithm 1 initial
// state, the sweeps over all rows, whose column partials are then complete column sums in row
// order, the labels of the final iteration (Eq. 2.8) and the FP64 net similarity), or one
// member of a gang: the K workgroups that share a large instance, member m owning a block of
// consecutive rows.  Members build their rows of S, compute the median themselves, sweep their
// rows and meet once per level at a barrier of the gang, where every member adds the members'
// column partials in member order (the order of the single-problem column sums with the same
// rows per workgroup) and forms the same column vectors.  The host orders the queue largest
// instance first with a gang's members consecutive, so only the gang being handed out can be
// incomplete while every earlier item runs to its end; the barrier's wait is bounded and gives
// up (raising an error flag and reporting the instance's iteration count as -1) rather than
// spin forever.
#include <algorithm>

#include "flowpass.h"

namespace hap {

struct BatchArgs {
    const float *X;
    int64_t d;
    const BatchDesc *desc;
    const BatchItem *items; // queue order
    int n_items;
    int count;
    int levels;
    float lam, oml;
    int max_iters, stable_iters;
    float *wsf;             // float workspace
    int32_t *wsi;           // int workspace
    int32_t *queue;         // [0]: next item handed out, [1]: a gang's wait gave up
    int32_t *labels;        // output labels
    double *ns;             // [count][levels + 1]
    int32_t *iters;         // [count]
    uint64_t wait_ticks;    // limit of one gang barrier wait, in wall-clock ticks
};

namespace {

typedef Vec<float>::type float4v;
constexpr int kBins = 2048;

__device__ __forceinline__ unsigned int fkey(float f) {
    const unsigned int u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float fval(unsigned int k) {
    return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

template <int NT>
__device__ void build_instance(const float *__restrict__ X, int64_t d, int n, int ld, float *__restrict__ S,
                               double *xs /* LDS [64 * d] */, int r0, int r1) {
#pragma clang fp contract(off)
    // rows [r0, r1) of S; thread t computes column j = t + NT*c, the rows come through LDS in
    // blocks of 64
    for (int j0 = 0; j0 < n; j0 += NT) {
        const int j = j0 + threadIdx.x;
        for (int i0 = r0; i0 < r1; i0 += 64) {
            const int rows = min(64, r1 - i0);
            __syncthreads();
            for (int e = threadIdx.x; e < rows * d; e += NT) xs[e] = (double)X[(int64_t)(i0 + e / d) * d + e % d];
            __syncthreads();
            if (j < n) {
                // eight rows at a time, so that a coordinate of the column is loaded once for eight of them
                const float *xj = X + (int64_t)j * d;
                for (int r = 0; r < rows; r += 8) {
                    double acc[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc[u] = 0.0;
                    for (int k = 0; k < d; ++k) {
                        const double xk = (double)xj[k];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const double df = xs[min(r + u, rows - 1) * d + k] - xk;
                            const double sq = df * df;
                            acc[u] = acc[u] + sq;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int i = i0 + r + u;
                        if (r + u < rows) S[(int64_t)i * ld + j] = (i == j) ? 0.f : (float)(-acc[u]);
                    }
                }
            }
        }
    }
    __syncthreads();
}

// Barrier of the K workgroups of a gang.  Every member arrives once per barrier, so barrier k
// of an instance completes when its counter reaches k*K.  Thread 0 publishes the workgroup's
// writes (agent-scope fence), arrives, and waits with a bounded spin: it gives up once another
// gang has given up or after `limit` wall-clock ticks, raising the batch's flag.  Returns
// whether the gang met (the same answer for every thread of the workgroup).
__device__ __forceinline__ bool gang_barrier(int32_t *ctr, int32_t target, int32_t *flag, uint64_t limit,
                                             int *sh_ok) {
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int ok = 1;
        const uint64_t t0 = wall_clock64();
        while (__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                ok = 0;
                break;
            }
            if ((uint64_t)wall_clock64() - t0 > limit) {
                __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        __threadfence();
        *sh_ok = ok;
    }
    __syncthreads();
    return *sh_ok != 0;
}

// Median of the off-diagonal entries: mean of the two middle order statistics (FP64),
// rounded to FP32.  Radix select on order-preserving keys with an LDS histogram.
template <int NT>
__device__ float median_instance(const float *__restrict__ S, int n, int ld, unsigned int *hist, int *sh) {
    const long long M = (long long)n * (n - 1);
    long long krem = M / 2 - 1;
    unsigned int prefix = 0, mask = 0;
    long long eqcount = 0;
    int hi = 32;
    while (hi > 0) {
        const int width = hi >= 11 ? 11 : hi;
        const int shift = hi - width;
        for (int b = threadIdx.x; b < kBins; b += NT) hist[b] = 0u;
        __syncthreads();
        // a wave per row
        for (int i = threadIdx.x >> 6; i < n; i += NT / 64)
#pragma unroll 4
            for (int j = threadIdx.x & 63; j < n; j += 64) {
                const unsigned int k = fkey(S[(int64_t)i * ld + j]);
                if (i != j && (k & mask) == prefix) atomicAdd(&hist[(k >> shift) & ((1u << width) - 1u)], 1u);
            }
        __syncthreads();
        if (threadIdx.x == 0) {
            long long cum = 0;
            for (int b = 0; b < (1 << width); ++b) {
                const long long c = hist[b];
                if (krem < cum + c) {
                    sh[0] = b;
                    sh[1] = (int)(krem - cum);
                    sh[2] = (int)c;
                    break;
                }
                cum += c;
            }
        }
        __syncthreads();
        prefix |= ((unsigned int)sh[0]) << shift;
        mask |= ((1u << width) - 1u) << shift;
        krem = sh[1];
        eqcount = sh[2];
        __syncthreads();
        hi = shift;
    }
    const float lo = fval(prefix);
    float hi_v = lo;
    if (krem + 1 >= eqcount) {
        // smallest key above the selected one
        if (threadIdx.x == 0) hist[0] = 0xFFFFFFFFu;
        __syncthreads();
        unsigned int best = 0xFFFFFFFFu;
        for (int i = threadIdx.x >> 6; i < n; i += NT / 64)
#pragma unroll 4
            for (int j = threadIdx.x & 63; j < n; j += 64) {
                const unsigned int k = fkey(S[(int64_t)i * ld + j]);
                if (i != j && k > prefix && k < best) best = k;
            }
        atomicMin(&hist[0], best);
        __syncthreads();
        hi_v = fval(hist[0]);
        __syncthreads();
    }
    return (float)(((double)lo + (double)hi_v) / 2.0);
}


// The rows of one instance (or of one member's block) in G decoupled row groups of NTG threads, as in
// flowpass.h: group g takes rows row0 + g, row0 + g + G, ...; the column sums are added in row order
// through LDS, so they are the sequential column sums whatever the shape.
// Measured at the default shape (512 threads, four groups) against groups that meet at a workgroup barrier
// per step: 512 problems of 64..2048 points, 20 iterations, 280 -> 235 ms; 200 problems of 32..500
// points, 40 iterations, 65 -> 22 ms; 256 of 32..200 points 17.0 -> 5.2 ms.
// Loads and stores are non-temporal: the problems in flight are past every cache together (512 problems, 50
// iterations with 1024 threads and four groups 566 ms with cached stores, 521 without).
// Its LDS is indexed by column vector and by wave, so it is the same for every cut into groups.
constexpr int kBatchVecs = 512;     // column vectors of the longest row (2048 points)
template <int NT>
struct BatchLds {
    Vec<float>::type q[kBatchVecs];   // column sums
    float m1[2][NT / 64], m2[2][NT / 64], cv[2][NT / 64];
    int ck[2][NT / 64];
    int arrived[NT / 64];             // per group
    int turn[NT / 64];                // per wave of a group
};

template <int NTG, int NCH, int G, bool FIRST>
__device__ __forceinline__ void batch_rows(const SweepArgs<float> &a, const int t, const int row0, const int row1,
                                           const Vec<float>::type (&Bv)[NCH], const float p, BatchLds<NTG * G> &L,
                                           int32_t *changed) {
#pragma clang fp contract(off)
    using V = Vec<float>::type;
    constexpr int VW = 4, NWG = NTG / 64, CB = NTG * 16;
    const int grp = G > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NTG) : 0;
    const int ltid = threadIdx.x % NTG, lane = ltid & 63, wid = __builtin_amdgcn_readfirstlane(ltid >> 6);
    const int n = a.n;
    const int64_t ldw = a.ldw;
    const int base = ltid * VW, voff = ltid * 16;
    const bool has_tau = a.tau != nullptr;
    const int64_t row_bytes = (int64_t)((n + VW - 1) / VW * VW) * 4;
    int chg = 0, step = 0;
    for (int i = row0 + grp; i < row1; i += G, ++step) {
        const int buf = step & 1;
        const __amdgpu_buffer_rsrc_t rS = row_rsrc(a.S + (int64_t)i * a.lds, row_bytes);
        const __amdgpu_buffer_rsrc_t rR = row_rsrc(a.R + (int64_t)i * ldw, row_bytes);
        const __amdgpu_buffer_rsrc_t rA = row_rsrc(a.A + (int64_t)i * ldw, row_bytes);
        FlowRow<float, NTG, NCH> x;
        // the row's scalars go out before the row, so that waiting for them is not waiting for it
        const float tau_i = has_tau ? a.tau[i] : 0.f;
        const int e_old = FIRST ? 0 : a.E[i];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            x.s[c] = buf_load<V, kNT>(rS, voff, c * CB);
            x.r[c] = buf_load<V, kNT>(rR, voff, c * CB);
            x.a[c] = buf_load<V, kNT>(rA, voff, c * CB);
        }
        float m1, m2, cv;
        int ck;
        flow_phase1<float, NTG, NCH, FIRST, true, false, kNT>(
            x, i, n, wid, base, a.lam, a.oml, p, 0.f, rA, voff, m1, m2, cv, ck, [&](int, V &) {},
            [&](int c) { return Bv[c]; });
        ck = (ck == INT_MAX) ? INT_MAX : ck + base;
        flow_reduce<float, !FIRST>(m1, m2, cv, ck);
        const int w0 = grp * NWG;   // the group's first wave
        if constexpr (NWG > 1) {
            if (lane == 63) {
                L.m1[buf][w0 + wid] = m1;
                L.m2[buf][w0 + wid] = m2;
                L.cv[buf][w0 + wid] = cv;
                L.ck[buf][w0 + wid] = ck;
            }
            lds_settle();
            if (lane == 0) __hip_atomic_fetch_add(&L.arrived[grp], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            lds_wait(&L.arrived[grp], (step + 1) * NWG);
            m1 = L.m1[buf][w0];
            m2 = L.m2[buf][w0];
#pragma unroll
            for (int w = 1; w < NWG; ++w) pair_merge(m1, m2, L.m1[buf][w0 + w], L.m2[buf][w0 + w]);
        } else {
            m1 = lane63(m1);
            m2 = lane63(m2);
        }
        if (ltid == 63) {
            if constexpr (!FIRST) {
                if constexpr (NWG > 1) {
                    cv = L.cv[buf][w0];
                    ck = L.ck[buf][w0];
                    for (int w = 1; w < NWG; ++w) argmax_merge(cv, ck, L.cv[buf][w0 + w], L.ck[buf][w0 + w]);
                }
                a.C[i] = cv;
                if (a.phi_down) a.phi_down[i] = m1;
                a.E[i] = ck;
                chg |= (t >= 3 && e_old != ck) ? 1 : 0;
            }
        }
        flow_phase2<float, NTG, NCH, true, kNT>(x, i, n, wid, base, a.lam, a.oml, m1, has_tau ? fminf(tau_i, -m1) : -m1,
                                           has_tau ? fminf(tau_i, -m2) : -m2, rR, voff);
        if constexpr (G > 1) lds_wait(&L.turn[wid], i - row0);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c * NTG * VW + wid * 64 * VW >= n) continue;
            V q = L.q[c * NTG + ltid];
#pragma unroll
            for (int v = 0; v < VW; ++v) q[v] += x.s[c][v];
            L.q[c * NTG + ltid] = q;
        }
        if constexpr (G > 1) {
            lds_settle();
            if (lane == 0)
                __hip_atomic_store(&L.turn[wid], i - row0 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    if (chg) atomicOr(changed, 1);
}

// One level's rows: the bases, the rows, the column sums in L.q.
template <int NTG, int NCH, int G>
__device__ __forceinline__ void batch_level(const SweepArgs<float> &a, const int t, const int row0, const int row1,
                                            const float p, BatchLds<NTG * G> &L, int32_t *changed) {
    using V = Vec<float>::type;
    constexpr int NT = NTG * G;
    const int tid = threadIdx.x, ltid = tid % NTG;
    V Bv[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j0 = (c * NTG + ltid) * 4;
        Bv[c] = (t > 1 && j0 < a.n) ? *(const V *)(a.B + j0) : (V)(0.f);
    }
    for (int v = tid; v < kBatchVecs; v += NT) L.q[v] = (V)(0.f);
    if (tid < NT / 64) L.arrived[tid] = L.turn[tid] = 0;
    __syncthreads();
    if (t == 1)
        batch_rows<NTG, NCH, G, true>(a, t, row0, row1, Bv, p, L, changed);
    else
        batch_rows<NTG, NCH, G, false>(a, t, row0, row1, Bv, p, L, changed);
    __syncthreads();   // c^l, phi^{l-1}, labels of this workgroup's rows are written
}

template <int NT, int G, int CH>
__global__ __launch_bounds__(NT) void batch_kernel(BatchArgs g) {
#pragma clang fp contract(off)
    using V = Vec<float>::type;
    constexpr int VW = 4;
    constexpr int NW = NT / 64;
    constexpr int NTG = NT / G;          // threads per row group
    __shared__ __attribute__((aligned(16))) BatchLds<NT> L;
    __shared__ unsigned int hist[kBins];
    __shared__ double xs[64 * 32];
    __shared__ int sh[4];
    __shared__ int sh_ok;
    __shared__ double shd[NW];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int levels = g.levels;
    for (;;) {
        if (tid == 0) sh[3] = atomicAdd(&g.queue[0], 1);
        __syncthreads();
        const int q = sh[3];
        __syncthreads();
        if (q >= g.n_items) break;
        const BatchItem item = g.items[q];
        const int b = item.b, m = item.m;
        const BatchDesc D = g.desc[b];
        const int n = D.n, ld = D.ld, K = D.K;
        // member m's rows (the whole instance when one workgroup runs it)
        const int r0 = (K > 1) ? m * D.rbm : 0;
        const int r1 = (K > 1) ? min(n, r0 + D.rbm) : n;
        float *S = g.wsf + D.w_off;
        float *RA = S + (int64_t)n * ld;                       // per level: R then A
        float *vec = RA + (int64_t)2 * levels * n * ld;             // per level: pref, Q, phi, tau, C, B
        int32_t *E = g.wsi + D.i_off;
        DevState *ds = (DevState *)(E + (int64_t)levels * ld);
        int32_t *sync = (K > 1) ? g.wsi + D.s_off : nullptr;   // [0] barrier counter, [4 + 2m + p] flags
        float *P = (K > 1) ? g.wsf + D.g_off : nullptr;        // column partials [2][K][ld]
        auto R = [&](int l) { return RA + (int64_t)(2 * l) * n * ld; };
        auto A = [&](int l) { return RA + (int64_t)(2 * l + 1) * n * ld; };
        auto vp = [&](int l, int k) { return vec + (int64_t)(6 * l + k) * ld; };
        int met = 0;   // gang barriers passed
        auto gang_sync = [&]() -> bool {
            if (K == 1) {
                __syncthreads();
                return true;
            }
            ++met;
            return gang_barrier(sync, met * K, &g.queue[1], g.wait_ticks, &sh_ok);
        };

        // 1. similarity rows, then the preference (every member computes the same median)
        build_instance<NT>(g.X + D.x_off * g.d, g.d, n, ld, S, xs, r0, r1);
        if (!gang_sync()) goto gave_up;
        {
            const float p = median_instance<NT>(S, n, ld, hist, sh);
            // 2. Algorithm 1 initial state (alpha = rho = 0, phi = c = 0; tau^1 is never read and
            //    tau^l is written before it is read); padding columns of alpha hold -inf.  Each
            //    member clears its own rows; member 0 the vectors and labels.
            for (int l = 0; l < levels; ++l) {
                float *Rl = R(l), *Al = A(l);
                for (int64_t e = (int64_t)r0 * ld + tid; e < (int64_t)r1 * ld; e += NT) {
                    Rl[e] = 0.f;
                    Al[e] = ((int)(e % ld) < n) ? 0.f : neg_inf<float>();
                }
                if (m == 0) {
                    for (int j = tid; j < ld; j += NT) {
                        vp(l, 0)[j] = (j < n) ? p : 0.f;
                        for (int k = 1; k < 6; ++k) vp(l, k)[j] = 0.f;
                        E[(int64_t)l * ld + j] = 0;
                    }
                }
            }
            if (tid == 0) {
                ds->t = ds->stable = ds->done = ds->stop_iter = ds->changed = ds->final_changed = 0;
                if (K > 1) sync[4 + 2 * m] = sync[5 + 2 * m] = 0;
            }
            if (!gang_sync()) goto gave_up;
            // 3. sweeps
            int t = 0, stable = 0, stop_iter = -1, par = 0;
            for (int it = 0; it < g.max_iters; ++it) {
                t += 1;
                int32_t *chg_flag = (K > 1) ? &sync[4 + 2 * m + (t & 1)] : &ds->changed;
                for (int l = 0; l < levels; ++l) {
                    SweepArgs<float> a;
                    a.S = S;
                    a.lds = ld;
                    a.R = R(l);
                    a.A = A(l);
                    a.ldw = ld;
                    a.pref = vp(l, 0);
                    a.C = vp(l, 4);
                    a.phi_down = l > 0 ? vp(l - 1, 2) : nullptr;
                    a.B = vp(l, 5);
                    a.tau = l > 0 ? vp(l, 3) : nullptr;
                    a.E = E + (int64_t)l * ld;
                    a.Qpart = nullptr;
                    a.X = nullptr;
                    a.ldx = 0;
                    a.tau_c = nullptr;
                    a.tau_q = nullptr;
                    a.tau_store = nullptr;
                    a.mrhap = 0;
                    a.delta = nullptr;
                    a.row_stride = 0;
                    a.n = n;
                    a.rb = n;
                    a.rows = n;
                    a.lam = g.lam;
                    a.oml = g.oml;
                    a.ds = ds;
                    // four row groups: rows that one wave holds take a wave each, twice the groups or more
                    if (G == 4 && n <= 1024)
                        batch_level<64, 4, NT / 64>(a, t, r0, r1, p, L, chg_flag);
                    else
                        batch_level<NTG, CH, G>(a, t, r0, r1, p, L, chg_flag);
                    if (K > 1) {
                        // publish this member's column partials, then meet the gang
                        for (int j0 = tid * VW; j0 < n; j0 += NT * VW)
                            *(V *)(P + ((int64_t)par * K + m) * ld + j0) = L.q[j0 / VW];
                        if (!gang_sync()) goto gave_up;
                    }
                    // column sums (this workgroup's own, in row order, or the members' partials added in
                    // member order), tau^{l+1}, B^{l-1} and B^l at the top
                    for (int j0 = tid * VW; j0 < n; j0 += NT * VW) {
                        V tot = L.q[j0 / VW];
                        if (K > 1) {
                            tot = *(const V *)(P + ((int64_t)par * K) * ld + j0);
                            for (int k = 1; k < K; ++k) tot += *(const V *)(P + ((int64_t)par * K + k) * ld + j0);
                        }
                        *(V *)(vp(l, 1) + j0) = tot;
                        if (l + 1 < levels) *(V *)(vp(l + 1, 3) + j0) = *(const V *)(vp(l, 4) + j0) + tot;
                        if (l == levels - 1) *(V *)(vp(l, 5) + j0) = tot;
                        if (l > 0)
                            *(V *)(vp(l - 1, 5) + j0) =
                                (*(const V *)(vp(l - 1, 4) + j0) + *(const V *)(vp(l - 1, 2) + j0)) +
                                *(const V *)(vp(l - 1, 1) + j0);
                    }
                    par ^= 1;
                    __syncthreads();
                }
                // With two levels no gang barrier separates the column sums of level 1 (which read
                // c^0 of every row) from the next iteration's level-0 pass (which rewrites c^0 of its
                // rows); with more levels one does.
                if (K > 1 && levels == 2 && !gang_sync()) goto gave_up;
                // stop rule: the row passes of iteration t compared the labels of iteration t-1
                int changed_any;
                if (K > 1) {
                    changed_any = 0;
                    for (int k = 0; k < K; ++k)
                        changed_any |= __hip_atomic_load(&sync[4 + 2 * k + (t & 1)], __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    changed_any = ds->changed;
                }
                if (t >= 2) {
                    const int lit = t - 1;
                    stable = (lit >= 2 && !changed_any) ? stable + 1 : 0;
                }
                __syncthreads();
                // this member's flag for the next iteration (every member has read it for iteration
                // t - 1 before the first barrier of iteration t)
                if (tid == 0) {
                    if (K > 1)
                        __hip_atomic_store(&sync[4 + 2 * m + ((t + 1) & 1)], 0, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    else
                        ds->changed = 0;
                }
                if (g.stable_iters > 0 && stable >= g.stable_iters) {
                    stop_iter = t - 1;
                    break;
                }
                __syncthreads();
            }
            __syncthreads();
            // 4. labels of this workgroup's rows: those recorded by the last row pass after an early
            //    stop, otherwise the labels of iteration t from alpha^t finished on the fly
            int32_t *out = g.labels + D.out_off;
            for (int l = 0; l < levels; ++l) {
                if (stop_iter >= 0) {
                    for (int i = r0 + tid; i < r1; i += NT) out[(int64_t)l * n + i] = E[(int64_t)l * ld + i];
                    continue;
                }
                const float *Rl = R(l), *Al = A(l), *Bl = vp(l, 5);
                // a wave per row
                for (int i = r0 + wid; i < r1; i += NW) {
                    float cv = neg_inf<float>();
                    int ck = INT_MAX;
#pragma unroll 4
                    for (int j = lane; j < n; j += 64) {
                        const float rj = Rl[(int64_t)i * ld + j];
                        float al = Al[(int64_t)i * ld + j];
                        if (t >= 1) {
                            const float ah = (j == i) ? Bl[j] - rj : fminf(0.f, Bl[j] - fmaxf(0.f, rj));
                            al = g.lam * al + g.oml * ah;
                        }
                        const float x = al + rj;
                        if (x > cv) {
                            cv = x;
                            ck = j;
                        }
                    }
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) {
                        const float ocv = __shfl_xor(cv, off, 64);
                        const int ock = __shfl_xor(ck, off, 64);
                        argmax_merge(cv, ck, ocv, ock);
                    }
                    if (lane == 0) out[(int64_t)l * n + i] = ck;
                }
            }
            __syncthreads();
            if (!gang_sync()) goto gave_up;
            // 5. net similarity per level and total, FP64, fixed-order reduction (member 0)
            if (m == 0) {
                double total = 0.0;
                for (int l = 0; l < levels; ++l) {
                    double acc = 0.0;
                    for (int i = tid; i < n; i += NT) {
                        const int e = out[(int64_t)l * n + i];
                        if (e < 0 || e >= n)
                            acc += __builtin_nan("");   // no valid exemplar (non-finite messages)
                        else
                            acc += (e == i) ? (double)p : (double)S[(int64_t)i * ld + e];
                    }
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
                    if (lane == 0) shd[wid] = acc;
                    __syncthreads();
                    if (tid == 0) {
                        double s2 = 0.0;
                        for (int w = 0; w < NW; ++w) s2 += shd[w];
                        g.ns[(int64_t)b * (levels + 1) + l] = s2;
                        total += s2;
                    }
                    __syncthreads();
                }
                if (tid == 0) {
                    g.ns[(int64_t)b * (levels + 1) + levels] = total;
                    g.iters[b] = stop_iter >= 0 ? stop_iter : t;
                }
            }
            __syncthreads();
            continue;
        }
    gave_up:
        // the gang did not meet within the wait limit: the instance's results are not valid
        if (tid == 0) g.iters[b] = -1;
        __syncthreads();
    }
}

// Start of a run: the queue, the flag and every gang's barrier counter back to 0.
__global__ void batch_reset(int32_t *queue, const BatchDesc *desc, int count, int32_t *wsi) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k == 0) {
        queue[0] = 0;
        queue[1] = 0;
    }
    if (k < count && desc[k].K > 1) wsi[desc[k].s_off] = 0;
}



}  // namespace

namespace {

// Workgroups of one batch kernel instance that fit the device at once (all of them run from the
// start, so every gang's members are handed out to running workgroups).
template <int NT, int G, int CH>
int resident_workgroups() {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, batch_kernel<NT, G, CH>, NT, 0) != hipSuccess) return 0;
    return per_cu * cus;
}

template <int NT, int G, int CH>
hipError_t launch_shape(const BatchArgs &g, int workgroups, bool gangs, hipStream_t st) {
    int grid = workgroups;
    if (gangs) {
        const int res = resident_workgroups<NT, G, CH>();
        if (res < kMaxGang) return hipErrorInvalidConfiguration;
        grid = std::min(grid, res);
    }
    hipLaunchKernelGGL((batch_kernel<NT, G, CH>), dim3(grid), dim3(NT), 0, st, g);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_batch(const float *X, int64_t d, const BatchDesc *desc, const BatchItem *items, int n_items,
                        int count, int levels, double lam, int max_iters, int stable_iters, float *wsf, int32_t *wsi,
                        int32_t *queue, int32_t *labels, double *ns, int32_t *iters, int threads, int workgroups,
                        int groups, bool gangs, hipStream_t st) {
    BatchArgs g;
    g.X = X;
    g.d = d;
    g.desc = desc;
    g.items = items;
    g.n_items = n_items;
    g.count = count;
    g.levels = levels;
    g.lam = (float)lam;
    g.oml = (float)(1.0 - lam);
    g.max_iters = max_iters;
    g.stable_iters = stable_iters;
    g.wsf = wsf;
    g.wsi = wsi;
    g.queue = queue;
    g.labels = labels;
    g.ns = ns;
    g.iters = iters;
    // a gang waits at most 60 s per barrier, longer for very long runs (a member may wait for
    // the other members to be handed out, which can take as long as one whole instance)
    int dev = 0, khz = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess) return e;
    const double seconds = 60.0 * std::max(1.0, max_iters / 200.0);
    g.wait_ticks = (uint64_t)(seconds * 1000.0 * (double)(khz > 0 ? khz : 100000));
    hipLaunchKernelGGL(batch_reset, dim3((count + 255) / 256), dim3(256), 0, st, queue, desc, count, wsi);
    // threads x row groups: every row group covers 2048 columns
    if (threads == 256 && groups == 1) return launch_shape<256, 1, 2>(g, workgroups, gangs, st);
    if (threads == 512 && groups == 1) return launch_shape<512, 1, 1>(g, workgroups, gangs, st);
    if (threads == 512 && groups == 2) return launch_shape<512, 2, 2>(g, workgroups, gangs, st);
    if (threads == 512 && groups == 4) return launch_shape<512, 4, 4>(g, workgroups, gangs, st);
    if (threads == 1024 && groups == 4) return launch_shape<1024, 4, 2>(g, workgroups, gangs, st);
    return hipErrorInvalidValue;
}

}  // namespace hap
