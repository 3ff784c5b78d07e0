// Small kernels around the sweep: preference fill, distinct-exemplar count and the
// FP64 net similarity.
#include "hap_internal.h"

namespace hap {

namespace {

template <typename T>
__global__ void fill_pref_kernel(T *pref, int64_t ldw, int n, int levels, const double *value) {
    const T v = (T)(*value);
    const int64_t total = (int64_t)levels * ldw;
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(k % ldw);
        if (j < n) pref[k] = v;
    }
}

// Number of distinct values in [0, n) among labels[0, rows), and (copy != nullptr) labels[0, n) copied.
// One workgroup with a bit per point in LDS: a launch, where clearing, marking and summing an array of
// marks took three and the copy another.
constexpr int kMaxLabels = 65536;   // the most points a context holds
__global__ __launch_bounds__(1024) void count_labels_kernel(const int32_t *__restrict__ labels, int rows, int n,
                                                            int32_t *__restrict__ copy, int32_t *__restrict__ out) {
    __shared__ unsigned int bits[kMaxLabels / 32];
    __shared__ int part[16];
    const int tid = threadIdx.x;
    for (int w = tid; w < (n + 31) / 32; w += 1024) bits[w] = 0u;
    __syncthreads();
#pragma unroll 8
    for (int k = tid; k < n; k += 1024) {
        const int e = labels[k];
        if (copy) copy[k] = e;
        if (k < rows && e >= 0 && e < n) atomicOr(&bits[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    int acc = 0;
    for (int w = tid; w < (n + 31) / 32; w += 1024) acc += __popc(bits[w]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) part[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        int s = 0;
        for (int w = 0; w < 16; ++w) s += part[w];
        *out = s;
    }
}

// NS^l = sum_i s^l_{i,e_i}, s^l_ii = p^l_i, in FP64; out[l] per level and out[levels] the total.
// One workgroup; every thread accumulates a fixed subset of points, then a fixed-order tree,
// so the result does not depend on scheduling.
template <typename T, typename TX>
__global__ __launch_bounds__(1024) void net_similarity_kernel(const T *__restrict__ S, int64_t lds,
                                                              const T *__restrict__ pref, int64_t ldw,
                                                              const int32_t *__restrict__ E, int n, int levels,
                                                              const TX *__restrict__ X, int64_t d, int64_t ldx,
                                                              double *out) {
    __shared__ double part[1024];
    double total = 0.0;
    for (int l = 0; l < levels; ++l) {
        const int32_t *e = E + (int64_t)l * ldw;
        const T *p = pref + (int64_t)l * ldw;
        double acc = 0.0;
        for (int i = threadIdx.x; i < n; i += 1024) {
            const int k = e[i];
            double v;
            if (k < 0 || k >= n) {
                v = __builtin_nan("");   // no valid exemplar (non-finite messages)
            } else if (k == i) {
                v = (double)p[i];
            } else if (X != nullptr) {
                double s2 = 0.0;
                for (int64_t q = 0; q < d; ++q) {
                    const double df = (double)X[(int64_t)i * ldx + q] - (double)X[(int64_t)k * ldx + q];
                    s2 += df * df;
                }
                v = -s2;
            } else {
                v = (double)S[(int64_t)i * lds + k];
            }
            acc += v;
        }
        part[threadIdx.x] = acc;
        __syncthreads();
        for (int off = 512; off > 0; off >>= 1) {
            if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            out[l] = part[0];
            total += part[0];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) out[levels] = total;
}

// Points-mode check: every sampled off-diagonal pair (i, j) has s_ij recomputed from the FP32
// points with the direct build's arithmetic (FP64 squared differences summed in coordinate
// order, negated and rounded once) and compared bit for bit with S.  One wave, one pair per
// lane; bad[0] receives the number of pairs that differ.
__global__ __launch_bounds__(64) void points_check_kernel(const float *__restrict__ S, int64_t lds,
                                                          const float *__restrict__ X, int64_t ldx, int d,
                                                          PairSample ps, int32_t *bad) {
#pragma clang fp contract(off)
    const int k = threadIdx.x;
    int diff = 0;
    if (k < ps.count) {
        const int i = ps.i[k], j = ps.j[k];
        double acc = 0.0;
        for (int q = 0; q < d; ++q) {
            const double df = (double)X[(int64_t)i * ldx + q] - (double)X[(int64_t)j * ldx + q];
            const double sq = df * df;
            acc = acc + sq;
        }
        const float want = (float)(-acc);
        diff = __float_as_uint(want) != __float_as_uint(S[(int64_t)i * lds + j]) ? 1 : 0;
    }
    const unsigned long long m = __ballot(diff);
    if (k == 0) bad[0] = __popcll(m);
}

// Bandwidth probe with the row pass's access pattern: of G workgroups of 512 threads,
// workgroup g takes rows g, g + G, g + 2G, ... (BLOCKS: the rows_per_block rows from
// g * rows_per_block); a thread owns fixed 16-byte column chunks.  Per element it reads R arrays
// and writes W arrays, every access non-temporal as in the row pass (CACHED: the inputs after
// the first with cached loads); every output is the sum of the inputs, so no read can be
// dropped.
template <int R, int W, bool CACHED, bool BLOCKS>
__global__ __launch_bounds__(512) void probe_kernel(ProbeArgs a) {
    typedef float V __attribute__((ext_vector_type(4)));
    constexpr int NCH = 4;   // 16-byte chunks per thread and row: rows of up to 8192 columns
    const int64_t first = BLOCKS ? (int64_t)blockIdx.x * a.rows_per_block : blockIdx.x;
    const int64_t end = BLOCKS ? (first + a.rows_per_block < a.rows ? first + a.rows_per_block : a.rows) : a.rows;
    const int64_t step = BLOCKS ? 1 : gridDim.x;
    for (int64_t i = first; i < end; i += step) {
        V acc[NCH];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t j = (int64_t)c * 2048 + threadIdx.x * 4;
            if (j < a.cols) {
                const int64_t o = i * a.ld + j;
                if constexpr (R == 0) {
                    acc[c] = (V)((float)i);   // write only: the row index
                } else {
                    acc[c] = __builtin_nontemporal_load((const V *)(a.in[0] + o));
#pragma unroll
                    for (int r = 1; r < R; ++r)
                        acc[c] += CACHED ? *(const V *)(a.in[r] + o) : __builtin_nontemporal_load((const V *)(a.in[r] + o));
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int64_t j = (int64_t)c * 2048 + threadIdx.x * 4;
            if (j < a.cols) {
                const int64_t o = i * a.ld + j;
#pragma unroll
                for (int w = 0; w < W; ++w) __builtin_nontemporal_store(acc[c], (V *)(a.out[w] + o));
                if constexpr (W == 0) {
                    // keep the loads: a value that is never the row's own is never stored
                    if (acc[c][0] == 1.2345e-38f && acc[c][1] == -1.2345e-38f) a.out[0][0] = acc[c][2];
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_probe(int reads, int writes, bool cached, bool blocks, const ProbeArgs &a, hipStream_t st) {
    const int grid = (int)((a.rows + a.rows_per_block - 1) / a.rows_per_block);
#define HAP_PROBE_1(RR, WW, CC, BB)                                                               \
    if (reads == RR && writes == WW && cached == CC && blocks == BB) {                            \
        hipLaunchKernelGGL((probe_kernel<RR, WW, CC, BB>), dim3(grid), dim3(512), 0, st, a);      \
        return hipGetLastError();                                                                 \
    }
#define HAP_PROBE(RR, WW)             \
    HAP_PROBE_1(RR, WW, false, false) \
    HAP_PROBE_1(RR, WW, false, true)  \
    HAP_PROBE_1(RR, WW, true, false)  \
    HAP_PROBE_1(RR, WW, true, true)
    HAP_PROBE(0, 1)
    HAP_PROBE(1, 0)
    HAP_PROBE(1, 1)
    HAP_PROBE(2, 2)
    HAP_PROBE(3, 2)
#undef HAP_PROBE
#undef HAP_PROBE_1
    return hipErrorInvalidValue;
}

hipError_t launch_points_check(const float *S, int64_t lds, const float *X, int64_t ldx, int d, const PairSample &ps,
                               int32_t *bad, hipStream_t st) {
    hipLaunchKernelGGL(points_check_kernel, dim3(1), dim3(64), 0, st, S, lds, X, ldx, d, ps, bad);
    return hipGetLastError();
}

hipError_t launch_fill_pref(void *pref_base, int64_t ldw, int n, int levels, int dtype, const double *value_dev,
                            hipStream_t st) {
    const int64_t total = (int64_t)levels * ldw;
    const int grid = (int)((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
    if (dtype == HAP_F32)
        hipLaunchKernelGGL((fill_pref_kernel<float>), dim3(grid), dim3(256), 0, st, (float *)pref_base, ldw, n,
                           levels, value_dev);
    else
        hipLaunchKernelGGL((fill_pref_kernel<double>), dim3(grid), dim3(256), 0, st, (double *)pref_base, ldw, n,
                           levels, value_dev);
    return hipGetLastError();
}

hipError_t launch_count_distinct(const int32_t *labels, int rows, int n, int32_t *copy, int32_t *out, hipStream_t st) {
    if (n > kMaxLabels) return hipErrorInvalidValue;
    hipLaunchKernelGGL(count_labels_kernel, dim3(1), dim3(1024), 0, st, labels, rows, n, copy, out);
    return hipGetLastError();
}

hipError_t launch_net_similarity(const void *S, int64_t lds, int dtype, const void *pref_base, int64_t ldw,
                                 const int32_t *Efinal_base, int n, int levels, const void *X, int64_t d,
                                 int64_t ldx, int x_dtype, double *out, hipStream_t st) {
#define HAP_NS(T, TX)                                                                                   \
    hipLaunchKernelGGL((net_similarity_kernel<T, TX>), dim3(1), dim3(1024), 0, st, (const T *)S, lds,  \
                       (const T *)pref_base, ldw, Efinal_base, n, levels, (const TX *)X, d, ldx, out)
    if (dtype == HAP_F32) {
        if (x_dtype == HAP_F64) HAP_NS(float, double); else HAP_NS(float, float);
    } else {
        if (x_dtype == HAP_F64) HAP_NS(double, double); else HAP_NS(double, float);
    }
#undef HAP_NS
    return hipGetLastError();
}

}  // namespace hap
