// The warm start's perceptron: n_in -> hidden -> hidden -> n_out with ReLU after both hidden
// layers, mean-squared-error loss, backpropagation and Adam.  Every product is one GEMM
// kernel on the matrix cores (FP32 operands on the 16x16x4 FP32 MFMA, or BF16 operands on the
// 16x16x32 BF16 MFMA, FP32 accumulation in both); bias, ReLU and the ReLU mask of the backward
// pass are fused into its epilogue.  Parameters are one flat FP32 vector (the master copy):
// W1 (n_in x hidden, row-major), b1, W2 (hidden x hidden), b2, W3 (hidden x n_out), b3.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "hap_internal.h"

namespace hap {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// float -> bf16, round to nearest even (finite inputs)
__device__ __forceinline__ __bf16 rne_bf16(float x) {
    unsigned int u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __builtin_bit_cast(__bf16, (unsigned short)(u >> 16));
}

enum { EPI_STORE = 0, EPI_BIAS = 1, EPI_BIAS_RELU = 2, EPI_MASK = 3 };

// C(m, n) = epilogue(sum_k A(m, k) B(k, n)) with A(m, k) = A[m*sam + k*sak] and
// B(k, n) = B[k*sbk + n*sbn], so transposed operands are plain stride choices.
struct GemmArgs {
    const float *A;
    int64_t sam, sak;
    const float *B;
    int64_t sbk, sbn;
    float *C;
    int64_t ldc;
    const float *bias;   // [N] (EPI_BIAS, EPI_BIAS_RELU)
    const float *mask;   // C(m, n) is kept where mask[m*ldm + n] > 0 (EPI_MASK)
    int64_t ldm;
    int M, N, K;
    int epi;
};

constexpr int TM = 64, TN = 64, TK = 32, LDT = TK + 4;

// 64 x 64 output tile per workgroup; four waves of 32 x 32, each 2 x 2 MFMA blocks of 16 x 16
// (lane l, register r of a block holds row 4*(l/16) + r, column l%16).  Tiles of A and of B^T
// are staged in LDS as FP32 with zero fill past M, N and K; the fragment of lane l is row
// l%16 of the A tile and row l%16 of the B^T tile at the same k slots.
template <bool BF16>
__global__ __launch_bounds__(256) void mlp_gemm_kernel(GemmArgs g) {
    __shared__ float As[TM][LDT];
    __shared__ float Bs[TN][LDT];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    const int wm = (wid >> 1) * 32, wn = (wid & 1) * 32;
    const int r16 = lane & 15, kg = lane >> 4;
    const bool a_kfast = g.sak == 1, b_nfast = g.sbn == 1;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};

    for (int k0 = 0; k0 < g.K; k0 += TK) {
        for (int e = tid; e < TM * TK; e += 256) {
            const int m = a_kfast ? e / TK : e % TM;
            const int k = a_kfast ? e % TK : e / TM;
            const int gm = m0 + m, gk = k0 + k;
            As[m][k] = (gm < g.M && gk < g.K) ? g.A[(int64_t)gm * g.sam + (int64_t)gk * g.sak] : 0.f;
        }
        for (int e = tid; e < TN * TK; e += 256) {
            const int nn = b_nfast ? e % TN : e / TK;
            const int k = b_nfast ? e / TN : e % TK;
            const int gn = n0 + nn, gk = k0 + k;
            Bs[nn][k] = (gn < g.N && gk < g.K) ? g.B[(int64_t)gk * g.sbk + (int64_t)gn * g.sbn] : 0.f;
        }
        __syncthreads();
        if constexpr (BF16) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float *pa = &As[wm + 16 * i + r16][8 * kg];
                const float *pb = &Bs[wn + 16 * i + r16][8 * kg];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    fa[i][e] = rne_bf16(pa[e]);
                    fb[i][e] = rne_bf16(pb[e]);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int kk = 0; kk < TK; kk += 4) {
                float fa[2], fb[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    fa[i] = As[wm + 16 * i + r16][kk + kg];
                    fb[i] = Bs[wn + 16 * i + r16][kk + kg];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + 4 * kg + r;
                const int n = n0 + wn + 16 * j + r16;
                if (m >= g.M || n >= g.N) continue;
                float v = acc[i][j][r];
                if (g.epi == EPI_BIAS || g.epi == EPI_BIAS_RELU) v = v + g.bias[n];
                if (g.epi == EPI_BIAS_RELU) v = v > 0.f ? v : 0.f;
                if (g.epi == EPI_MASK) v = g.mask[(int64_t)m * g.ldm + n] > 0.f ? v : 0.f;
                g.C[(int64_t)m * g.ldc + n] = v;
            }
}

// dY = 2 (Y - T) / (rows * n_out) and loss = sum (Y - T)^2 / (rows * n_out); one workgroup,
// FP64 accumulation in a fixed order.
__global__ __launch_bounds__(1024) void mse_kernel(const float *__restrict__ Y, int64_t ldy, const float *__restrict__ T,
                                                   int64_t ldt, int rows, int nout, float *__restrict__ dY,
                                                   double *__restrict__ loss) {
    __shared__ double part[16];
    const int tid = threadIdx.x;
    const int64_t cnt = (int64_t)rows * nout;
    const float scale = (float)(2.0 / (double)cnt);
    double acc = 0.0;
    for (int64_t e = tid; e < cnt; e += 1024) {
        const int64_t r = e / nout, o = e % nout;
        const float d = Y[r * ldy + o] - T[r * ldt + o];
        dY[e] = scale * d;
        acc += (double)d * (double)d;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) part[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += part[w];
        *loss = s / (double)cnt;
    }
}

// out[n] = sum over rows of X[r*ldx + n]; one workgroup per column, fixed order.
__global__ __launch_bounds__(256) void colsum_rows_kernel(const float *__restrict__ X, int64_t ldx, int rows,
                                                          float *__restrict__ out) {
    __shared__ float part[4];
    const int n = blockIdx.x, tid = threadIdx.x;
    float acc = 0.f;
    for (int r = tid; r < rows; r += 256) acc += X[(int64_t)r * ldx + n];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) part[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) out[n] = (part[0] + part[1]) + (part[2] + part[3]);
}

// Adam (Kingma and Ba, 2015): m and v are the first and second moment estimates, bc1 and bc2
// the bias corrections 1 - beta^step.
struct AdamArgs {
    float b1, omb1, b2, omb2, lr, eps, bc1, bc2;
};
__device__ __forceinline__ void adam_update(float &p, float &mv, float &vv, float g, const AdamArgs &ad) {
#pragma clang fp contract(off)
    const float m = ad.b1 * mv + ad.omb1 * g;
    const float v = ad.b2 * vv + ad.omb2 * (g * g);
    mv = m;
    vv = v;
    p = p - ad.lr * (m / ad.bc1) / (sqrtf(v / ad.bc2) + ad.eps);
}
__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ P, const float *__restrict__ G,
                                                   float *__restrict__ Mv, float *__restrict__ Vv, int64_t count,
                                                   AdamArgs ad) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
        adam_update(P[i], Mv[i], Vv[i], G[i], ad);
}

// ---------------------------------------------------------------------------
// The whole perceptron in one or two launches (n_in <= 32, hidden <= 256, n_out <= 16; the warm
// start's is 32 -> 128 -> 128 -> L).
//
// mlp_tile_kernel: a workgroup takes tiles of 32 rows; wave w owns hidden columns
// [32 w, 32 w + 32) of both hidden layers, so everything between two layers passes through LDS
// and only X and Y touch memory.  TRAIN: the backward pass of the tile too, and what the
// parameter gradients contract over the rows goes to memory once, in the order in which the MFMA
// of the gradient reads it (one 16 x 32-row fragment is 64 consecutive lane vectors).
// mlp_grad_kernel: a wave per 16 x 16 tile of a weight gradient runs one chain of MFMAs over all
// rows and applies the Adam step to its parameters.
//
// Every product is the one mlp_gemm_kernel forms (the same MFMA, k ascending from a zero
// accumulator, the same epilogue) and the bias gradients add in colsum_rows_kernel's order, so outputs,
// gradients and parameters are those of the layer-by-layer path bit for bit; the loss adds the same FP64
// squares tile by tile, another order.  That path spends a step of
// 32 -> 128 -> 128 -> 3 at 4096 rows (1.96 ms) in its weight gradients: a 128 x 128 product over
// 4096 rows is four 64 x 64 tiles, four workgroups that each wait for 128 loads in turn.  The
// chain itself (128 MFMAs of 8 passes) takes 2 us; both kernels here are bound by latency.  Measured
// in BF16: that step 1.96 ms -> 28 us (tiles 17 us, 26 while every workgroup gathered and rounded the FP32
// weights; gradients and Adam 11 us, 14 with fewer loads in flight), the prediction of 65536
// rows 99 -> 13 us (layer by layer H1 and H2 travel through memory, 134 MB).
// ---------------------------------------------------------------------------
constexpr int kTile = 32;   // rows of a tile: one k step of the BF16 MFMA

template <bool BF16> struct Mx;
template <> struct Mx<true> {
    typedef __bf16 E;
    typedef bf16x8 F;
    static constexpr int KS = 32, PAD = 8;
    static __device__ __forceinline__ E cvt(float x) { return rne_bf16(x); }
    static __device__ __forceinline__ F ld(const E *row, int k0, int kg) { return *(const F *)(row + k0 + 8 * kg); }
    static __device__ __forceinline__ f32x4 mma(F a, F b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    // elements k of p[k * stride], zero from K >= 1 on and where !ok (loads from valid addresses and
    // selects: a branch per element costs more than the load)
    static __device__ __forceinline__ F global(const float *p, int stride, int k0, int kg, int K, bool ok) {
        float v[8];
        F f;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = p[min(k0 + 8 * kg + e, K - 1) * stride];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = rne_bf16(ok && k0 + 8 * kg + e < K ? v[e] : 0.f);
        return f;
    }
    // rows 16 rb + 4 kg + r (r = 0..3) of unit u = lane % 16 into the tile's fragment, in which
    // lane 16 (row / 8) + u holds rows 8 (row / 8) .. + 7
    static __device__ __forceinline__ void put(E *frag, int rb, int kg, int u, f32x4 v) {
        typedef E E4 __attribute__((ext_vector_type(4)));
        E4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = rne_bf16(v[r]);
        *(E4 *)(frag + ((2 * rb + (kg >> 1)) * 16 + u) * 8 + 4 * (kg & 1)) = o;
    }
    static __device__ __forceinline__ void put1(E *frag, int row, int u, float v) {
        frag[((row >> 3) * 16 + u) * 8 + (row & 7)] = rne_bf16(v);
    }
};
template <> struct Mx<false> {
    typedef float E;
    typedef float F;
    static constexpr int KS = 4, PAD = 4;
    static __device__ __forceinline__ E cvt(float x) { return x; }
    static __device__ __forceinline__ F ld(const E *row, int k0, int kg) { return row[k0 + kg]; }
    static __device__ __forceinline__ f32x4 mma(F a, F b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ F global(const float *p, int stride, int k0, int kg, int K, bool ok) {
        const int k = k0 + kg;
        return ok && k < K ? p[k * stride] : 0.f;
    }
    // fragment of k step q (rows 4 q .. 4 q + 3): lane 16 (row % 4) + u holds row 4 q + row % 4
    static __device__ __forceinline__ void put(E *frag, int rb, int kg, int u, f32x4 v) {
#pragma unroll
        for (int r = 0; r < 4; ++r) frag[(4 * rb + kg) * 64 + r * 16 + u] = v[r];
    }
    static __device__ __forceinline__ void put1(E *frag, int row, int u, float v) {
        frag[(row >> 2) * 64 + (row & 3) * 16 + u] = v;
    }
};

constexpr int kFuseIn = 32, kFuseOut = 16, kFuseHidden = 256;
constexpr int kFrag = 16 * kTile;   // elements of one block of 16 units over one tile

// Where the training kernels keep a batch's operands in the workspace (bytes).  Fragments:
// [block of 16 units][tile][kFrag] of X, H1, H2, dY, dH1, dH2; in BF16 the unrounded dH1, dH2 and dY for the
// bias gradients too: [unit][row] (FP32 fragments hold them unrounded, a block as [row][16 units]; with a second
// copy a batch of 65536 rows over 128 units took 215 MB instead of the 148 here, layer by layer 146); one
// squared-error sum per tile.
struct FuseLayout {
    int tiles, bh;         // tiles of rows; blocks of hidden units
    int64_t rows;          // tiles * kTile
    size_t X, H1, H2, dY, d1, d2, f1, f2, fy, loss, bytes;
    // BF16 only: W1, W2 and W2^T rounded and in fragment order for the tile kernel, which the gradient
    // kernel keeps up to date over the steps of one training call
    size_t p1, p2, p2t, bytes_packed;
};
// hidden units as the tile kernel is built for them
inline int padded_hidden(int hidden) { return hidden <= 64 ? 64 : hidden <= 128 ? 128 : 256; }
// element (k, col) of an operand of nk k steps of 32, in fragment order
__host__ __device__ inline int frag_at(int col, int k, int nk) {
    return ((col >> 4) * nk + (k >> 5)) * 512 + (((k & 31) >> 3) * 16 + (col & 15)) * 8 + (k & 7);
}
FuseLayout fuse_layout(int hidden, int n_out, int64_t rows, bool bf16) {
    FuseLayout f{};
    f.tiles = (int)((rows + kTile - 1) / kTile);
    f.rows = (int64_t)f.tiles * kTile;
    f.bh = (hidden + 15) / 16;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const size_t frag = (size_t)f.tiles * kFrag * (bf16 ? 2 : 4);
    f.X = take(frag * (kFuseIn / 16));
    f.H1 = take(frag * f.bh);
    f.H2 = take(frag * f.bh);
    f.dY = take(frag);
    f.d1 = take(frag * f.bh);
    f.d2 = take(frag * f.bh);
    if (bf16) {
        f.f1 = take((size_t)f.rows * hidden * 4);
        f.f2 = take((size_t)f.rows * hidden * 4);
        f.fy = take((size_t)f.rows * n_out * 4);
    }
    f.loss = take((size_t)f.tiles * 8);
    f.bytes = off;
    const int hp = padded_hidden(hidden);
    f.p1 = take((size_t)hp * kFuseIn * 2);
    f.p2 = take((size_t)hp * hp * 2);
    f.p2t = take((size_t)hp * hp * 2);
    f.bytes_packed = bf16 ? off : f.bytes;
    return f;
}

struct FuseArgs {
    const float *P;          // parameters
    MlpLayout lo;
    int n_in, H, n_out;
    const float *X;
    int64_t ldx;
    const int32_t *idx;      // rows of X and T to take (nullptr: 0, 1, ...); outside [0, x_rows): NaN
    int x_rows;
    int rows, tiles;
    float *Y;                // forward
    int64_t ldy;
    const float *T;          // TRAIN
    int64_t ldt;
    float scale;             // 2 / (rows n_out)
    FuseLayout fl;
    char *ws;
};

template <bool BF16, int HP, bool TRAIN, bool PACKED>
__global__ __launch_bounds__(2 * HP) void mlp_tile_kernel(FuseArgs g) {
    using M = Mx<BF16>;
    using E = typename M::E;
    using F = typename M::F;
    constexpr int RT = kTile, RB = RT / 16, NT = 2 * HP;
    constexpr int KS = M::KS, PAD = M::PAD;
    constexpr int NKH = HP / KS, NKI = kFuseIn / KS;              // k steps over hidden units, inputs
    constexpr int KO = BF16 ? 32 : 16, NKO = KO / KS;             // over outputs (zero past 16)
    __shared__ __attribute__((aligned(16))) E Xs[RT][kFuseIn + PAD];
    __shared__ __attribute__((aligned(16))) E H1s[RT][HP + PAD];
    __shared__ __attribute__((aligned(16))) E H2s[RT][HP + PAD];  // TRAIN: then dH2
    __shared__ __attribute__((aligned(16))) E dYs[TRAIN ? RT : 1][TRAIN ? KO + PAD : 1];
    __shared__ double redl[RB];

    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int r16 = lane & 15, kg = lane >> 4;
    const int H = g.H, n_in = g.n_in, n_out = g.n_out;
    const float *W1 = g.P + g.lo.oW1, *W2 = g.P + g.lo.oW2, *W3 = g.P + g.lo.oW3;
    // this lane's column of each of the wave's two blocks of hidden units (clamped for addresses)
    int col[2], colc[2];
    float bias1[2], bias2[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        col[c] = wid * 32 + 16 * c + r16;
        colc[c] = col[c] < H ? col[c] : H - 1;
        bias1[c] = col[c] < H ? g.P[g.lo.ob1 + col[c]] : 0.f;
        bias2[c] = col[c] < H ? g.P[g.lo.ob2 + col[c]] : 0.f;
    }
    const float bias3 = r16 < n_out ? g.P[g.lo.ob3 + r16] : 0.f;
    const int outc = r16 < n_out ? r16 : n_out - 1;
    // Weight fragments: in registers over the tiles (they are the same for every tile), except
    // where they do not fit (training at 256 units), which reads them where they are used.
    constexpr bool KEEP = HP <= 128 || !TRAIN;
    auto packed = [&](size_t region, int k, int c, int nk) {
        return *(const F *)((const E *)(g.ws + region) + (((wid * 2 + c) * nk + k) * 64 + lane) * 8);
    };
    auto read_w1 = [&](int k, int c) {
        if constexpr (PACKED)
            return packed(g.fl.p1, k, c, NKI);
        else
            return M::global(W1 + colc[c], H, k * KS, kg, n_in, col[c] < H);
    };
    auto read_w2 = [&](int k, int c) {
        if constexpr (PACKED)
            return packed(g.fl.p2, k, c, NKH);
        else
            return M::global(W2 + colc[c], H, k * KS, kg, H, col[c] < H);
    };
    auto read_w2t = [&](int k, int c) {
        if constexpr (PACKED)
            return packed(g.fl.p2t, k, c, NKH);
        else
            return M::global(W2 + colc[c] * H, 1, k * KS, kg, H, col[c] < H);
    };
    auto read_w3 = [&](int k) { return M::global(W3 + outc, n_out, k * KS, kg, H, r16 < n_out); };
    F w1[NKI][2], w2[KEEP ? NKH : 1][2], w3[KEEP ? NKH : 1];
    F w2t[TRAIN && KEEP ? NKH : 1][2], w3t[TRAIN ? NKO : 1][2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int k = 0; k < NKI; ++k) w1[k][c] = read_w1(k, c);
    if constexpr (KEEP) {
#pragma unroll
        for (int k = 0; k < NKH; ++k) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                w2[k][c] = read_w2(k, c);
                if constexpr (TRAIN) w2t[k][c] = read_w2t(k, c);
            }
            if (wid < RB) w3[k] = read_w3(k);
        }
    }
    if constexpr (TRAIN) {
#pragma unroll
        for (int k = 0; k < NKO; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                w3t[k][c] = M::global(W3 + colc[c] * n_out, 1, k * KS, kg, n_out, col[c] < H);
        // outputs 16.. of the dY tile stay zero
        if constexpr (KO > kFuseOut)
            for (int e = tid; e < RT * (KO - kFuseOut); e += NT)
                dYs[e / (KO - kFuseOut)][kFuseOut + e % (KO - kFuseOut)] = M::cvt(0.f);
    }
    const f32x4 z4 = (f32x4){0.f, 0.f, 0.f, 0.f};

    for (int tile = blockIdx.x; tile < g.tiles; tile += gridDim.x) {
        const int64_t row0 = (int64_t)tile * RT;
        // a tile's fragment of block b of an operand
        auto frag = [&](size_t region, int b) { return (E *)(g.ws + region) + ((int64_t)b * g.tiles + tile) * kFrag; };
        for (int e = tid; e < RT * kFuseIn; e += NT) {
            const int r = e / kFuseIn, k = e % kFuseIn;
            const int64_t row = row0 + r;
            float v = 0.f;
            if (row < g.rows && k < n_in) {
                const int64_t src = g.idx ? g.idx[row] : row;
                v = (src >= 0 && src < g.x_rows) ? g.X[src * g.ldx + k] : __builtin_nanf("");
            }
            Xs[r][k] = M::cvt(v);
            if constexpr (TRAIN) M::put1(frag(g.fl.X, k >> 4), r, k & 15, v);
        }
        __syncthreads();
        // hidden layers; rows past the end hold zero from layer 1 on, so they add nothing below
        unsigned on1 = 0, on2 = 0;   // bit 8 rb + 4 c + r: unit active at that row
        f32x4 acc[RB][2];
        auto clear = [&]() {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[rb][c] = z4;
        };
        auto activate = [&](E(*hs)[HP + PAD], size_t region, const float(&bias)[2], unsigned &on) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    f32x4 h;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int m = 16 * rb + 4 * kg + r;
                        float v = acc[rb][c][r] + bias[c];
                        v = v > 0.f ? v : 0.f;
                        if (row0 + m >= g.rows) v = 0.f;
                        on |= (v > 0.f ? 1u : 0u) << (8 * rb + 4 * c + r);
                        h[r] = v;
                        hs[m][col[c]] = M::cvt(v);
                    }
                    if constexpr (TRAIN) {
                        if (wid * 2 + c < g.fl.bh) M::put(frag(region, wid * 2 + c), rb, kg, r16, h);
                    }
                }
        };
        // acc += hs x (the wave's columns of a hidden x hidden weight), k ascending
        auto over_hidden = [&](const E(*hs)[HP + PAD], const F(*kept)[2], auto &&read) {
            auto step = [&](int k, const F(&b)[2]) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const F a = M::ld(hs[16 * rb + r16], k * KS, kg);
#pragma unroll
                    for (int c = 0; c < 2; ++c) acc[rb][c] = M::mma(a, b[c], acc[rb][c]);
                }
            };
            if constexpr (KEEP) {
#pragma unroll
                for (int k = 0; k < NKH; ++k) step(k, kept[k]);
            } else {
#pragma unroll(BF16 && !PACKED ? 1 : 8)
                for (int k = 0; k < NKH; ++k) {
                    const F b[2] = {read(k, 0), read(k, 1)};
                    step(k, b);
                }
            }
        };
        clear();
#pragma unroll
        for (int k = 0; k < NKI; ++k)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[rb][c] = M::mma(M::ld(Xs[16 * rb + r16], k * KS, kg), w1[k][c], acc[rb][c]);
        activate(H1s, g.fl.H1, bias1, on1);
        __syncthreads();
        clear();
        over_hidden(H1s, w2, read_w2);
        activate(H2s, g.fl.H2, bias2, on2);
        __syncthreads();
        // outputs: wave w < RB holds rows 16 w .. 16 w + 15
        if (wid < RB) {
            f32x4 y = z4;
            if constexpr (KEEP) {
#pragma unroll
                for (int k = 0; k < NKH; ++k) y = M::mma(M::ld(H2s[16 * wid + r16], k * KS, kg), w3[k], y);
            } else {
#pragma unroll(BF16 ? 1 : 8)
                for (int k = 0; k < NKH; ++k) y = M::mma(M::ld(H2s[16 * wid + r16], k * KS, kg), read_w3(k), y);
            }
            f32x4 dy = z4;
            double lsum = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 16 * wid + 4 * kg + r;
                const int64_t row = row0 + m;
                const float v = y[r] + bias3;
                const bool in = row < g.rows && r16 < n_out;
                if constexpr (!TRAIN) {
                    if (in) g.Y[row * g.ldy + r16] = v;
                } else {
                    if (in) {
                        const int64_t src = g.idx ? g.idx[row] : row;
                        const float t = (src >= 0 && src < g.x_rows) ? g.T[src * g.ldt + r16] : __builtin_nanf("");
                        const float d = v - t;
                        dy[r] = g.scale * d;
                        lsum += (double)d * (double)d;
                    }
                    dYs[m][r16] = M::cvt(dy[r]);
                }
            }
            if constexpr (TRAIN) {
                M::put(frag(g.fl.dY, 0), wid, kg, r16, dy);
                if (BF16 && r16 < n_out)
                    *(f32x4 *)((float *)(g.ws + g.fl.fy) + r16 * g.fl.rows + row0 + 16 * wid + 4 * kg) = dy;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
                if (lane == 0) redl[wid] = lsum;
            }
        }
        if constexpr (TRAIN) {
            __syncthreads();
            if (tid == 0) ((double *)(g.ws + g.fl.loss))[tile] = redl[0] + redl[1];
            // masks acc where the unit was off and hands it on
            auto masked = [&](unsigned on, size_t region, size_t plain, bool keep) {
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        f32x4 v;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            v[r] = (on >> (8 * rb + 4 * c + r)) & 1u ? acc[rb][c][r] : 0.f;
                            if (keep) H2s[16 * rb + 4 * kg + r][col[c]] = M::cvt(v[r]);
                        }
                        if (wid * 2 + c < g.fl.bh) M::put(frag(region, wid * 2 + c), rb, kg, r16, v);
                        if (BF16 && col[c] < H)
                            *(f32x4 *)((float *)(g.ws + plain) + col[c] * g.fl.rows + row0 + 16 * rb + 4 * kg) = v;
                    }
            };
            // dH2 = (dY W3^T) where H2 > 0, dH1 = (dH2 W2^T) where H1 > 0
            clear();
#pragma unroll
            for (int k = 0; k < NKO; ++k)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[rb][c] = M::mma(M::ld(dYs[16 * rb + r16], k * KS, kg), w3t[k][c], acc[rb][c]);
            masked(on2, g.fl.d2, g.fl.f2, true);
            __syncthreads();
            clear();
            over_hidden(H2s, w2t, read_w2t);
            masked(on1, g.fl.d1, g.fl.f1, false);
        }
        __syncthreads();
    }
}

// W1, W2 and W2^T rounded to BF16 in fragment order, zero past their ends.
__global__ __launch_bounds__(256) void mlp_pack_kernel(const float *P, MlpLayout lo, FuseLayout fl, int n_in, int H,
                                                       int hp, char *ws) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= hp * hp) return;
    const int k = e / hp, c = e % hp, nk = hp / 32;
    const float *W1 = P + lo.oW1, *W2 = P + lo.oW2;
    const bool in = k < H && c < H;
    const __bf16 v = rne_bf16(in ? W2[(int64_t)k * H + c] : 0.f);
    ((__bf16 *)(ws + fl.p2))[frag_at(c, k, nk)] = v;
    ((__bf16 *)(ws + fl.p2t))[frag_at(k, c, nk)] = v;
    if (k < kFuseIn) ((__bf16 *)(ws + fl.p1))[frag_at(c, k, 1)] = rne_bf16(k < n_in && c < H ? W1[(int64_t)k * H + c] : 0.f);
}

struct GradArgs {
    MlpLayout lo;
    FuseLayout fl;
    const char *ws;
    int n_in, H, n_out, rows;
    double *loss;             // or nullptr
    float *G;                 // gradient (no ADAM)
    float *P, *Mv, *Vv;       // ADAM
    AdamArgs ad;
    char *pack;               // the workspace where the packed weights are to follow, or nullptr
    int hp;
};

// Parameter gradients from a batch's operands.  Workgroups, in order: one per 16 x 16 tile of
// gW2, gW1, gW3 (one wave, one accumulator, rows ascending; the loads of 24 tiles of rows in BF16, of 4 in
// FP32, are in flight together), one per bias (256 threads, colsum_rows_kernel's sum; FP32: one per four of them, a
// quarter of a fragment's row per thread), one for the loss.
template <bool BF16, bool ADAM>
__global__ __launch_bounds__(256) void mlp_grad_kernel(GradArgs g) {
    using M = Mx<BF16>;
    using E = typename M::E;
    using F = typename M::F;
    constexpr int PER = BF16 ? 1 : 8;        // MFMA steps per tile of rows
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int bh = g.fl.bh, bi = (g.n_in + 15) / 16;
    auto emit = [&](int64_t i, float v) {
        if constexpr (ADAM)
            adam_update(g.P[i], g.Mv[i], g.Vv[i], v, g.ad);
        else
            g.G[i] = v;
    };
    int b = blockIdx.x;
    const int n2 = bh * bh, n1 = bi * bh, n3 = bh;
    if (b < n2 + n1 + n3) {
        if (wid > 0) return;
        size_t ra, rb;
        int ba, bb, M_, N_;
        int64_t out;
        if (b < n2) {
            ra = g.fl.H1, rb = g.fl.d2, ba = b / bh, bb = b % bh, M_ = g.H, N_ = g.H, out = g.lo.oW2;
        } else if (b < n2 + n1) {
            b -= n2;
            ra = g.fl.X, rb = g.fl.d1, ba = b / bh, bb = b % bh, M_ = g.n_in, N_ = g.H, out = g.lo.oW1;
        } else {
            ra = g.fl.H2, rb = g.fl.dY, ba = b - n2 - n1, bb = 0, M_ = g.H, N_ = g.n_out, out = g.lo.oW3;
        }
        const F *A = (const F *)((const E *)(g.ws + ra) + (int64_t)ba * g.fl.tiles * kFrag) + lane;
        const F *B = (const F *)((const E *)(g.ws + rb) + (int64_t)bb * g.fl.tiles * kFrag) + lane;
        f32x4 acc = (f32x4){0.f, 0.f, 0.f, 0.f};
        constexpr int UN = BF16 ? 24 : 4;    // tiles of rows in flight
        int t = 0;
        for (; t + UN <= g.fl.tiles; t += UN) {
            F fa[UN * PER], fb[UN * PER];
#pragma unroll
            for (int k = 0; k < UN * PER; ++k) {
                fa[k] = A[((int64_t)t * PER + k) * 64];
                fb[k] = B[((int64_t)t * PER + k) * 64];
            }
            __builtin_amdgcn_sched_barrier(0);   // every load before the first product
#pragma unroll
            for (int k = 0; k < UN * PER; ++k) acc = M::mma(fa[k], fb[k], acc);
        }
        for (; t < g.fl.tiles; ++t)
#pragma unroll
            for (int k = 0; k < PER; ++k)
                acc = M::mma(A[((int64_t)t * PER + k) * 64], B[((int64_t)t * PER + k) * 64], acc);
        const int n = 16 * bb + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * ba + 4 * (lane >> 4) + r;
            if (m < M_ && n < N_) {
                const int64_t i = out + (int64_t)m * N_ + n;
                emit(i, acc[r]);
                if constexpr (BF16 && ADAM) {
                    if (g.pack && rb != g.fl.dY) {
                        const __bf16 w = rne_bf16(g.P[i]);
                        if (rb == g.fl.d2) {
                            ((__bf16 *)(g.pack + g.fl.p2))[frag_at(n, m, g.hp / 32)] = w;
                            ((__bf16 *)(g.pack + g.fl.p2t))[frag_at(m, n, g.hp / 32)] = w;
                        } else {
                            ((__bf16 *)(g.pack + g.fl.p1))[frag_at(n, m, 1)] = w;
                        }
                    }
                }
            }
        }
        return;
    }
    b -= n2 + n1 + n3;
    const int biases = BF16 ? 2 * g.H + g.n_out : 4 * (2 * bh + 1);   // workgroups
    if constexpr (!BF16) {
        if (b < biases) {
            // bias gradients: the sums of four columns of a block of dH1, dH2 or dY
            __shared__ f32x4 part[4];
            const int four = b & 3;
            b >>= 2;
            const size_t region = b < bh ? g.fl.d1 : b < 2 * bh ? g.fl.d2 : g.fl.dY;
            const int blk = b < bh ? b : b < 2 * bh ? b - bh : 0;
            const f32x4 *x = (const f32x4 *)((const float *)(g.ws + region) + (int64_t)blk * g.fl.rows * 16) + four;
            f32x4 acc = (f32x4)(0.f);
#pragma unroll 8
            for (int r = tid; r < g.rows; r += 256) acc += x[(int64_t)r * 4];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
            if (lane == 0) part[wid] = acc;
            __syncthreads();
            const int u = blk * 16 + four * 4 + tid;
            if (tid < 4 && u < (b < 2 * bh ? g.H : g.n_out))
                emit((b < bh ? g.lo.ob1 : b < 2 * bh ? g.lo.ob2 : g.lo.ob3) + u,
                     (part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
            return;
        }
    } else if (b < biases) {
        // bias gradient: the sum of one unit's row of f1, f2 or fy
        __shared__ float part[4];
        const size_t region = b < g.H ? g.fl.f1 : b < 2 * g.H ? g.fl.f2 : g.fl.fy;
        const int u = b < g.H ? b : b < 2 * g.H ? b - g.H : b - 2 * g.H;
        const float *x = (const float *)(g.ws + region) + u * g.fl.rows;
        float acc = 0.f;
#pragma unroll 8
        for (int r = tid; r < g.rows; r += 256) acc += x[r];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (lane == 0) part[wid] = acc;
        __syncthreads();
        if (tid == 0)
            emit((b < g.H ? g.lo.ob1 : b < 2 * g.H ? g.lo.ob2 : g.lo.ob3) + u,
                 (part[0] + part[1]) + (part[2] + part[3]));
        return;
    }
    // loss: the tiles' squared errors, in a fixed order
    __shared__ double lp[4];
    double s = 0.0;
    for (int t = tid; t < g.fl.tiles; t += 256) s += ((const double *)(g.ws + g.fl.loss))[t];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) lp[wid] = s;
    __syncthreads();
    if (tid == 0 && g.loss) *g.loss = ((lp[0] + lp[1]) + (lp[2] + lp[3])) / ((double)g.rows * g.n_out);
}

// Rows idx[0..rows) of X (width w, row stride ldx, x_rows rows) into a packed buffer; an
// index outside [0, x_rows) yields NaN instead of a read.
__global__ __launch_bounds__(256) void gather_rows_kernel(const float *__restrict__ X, int64_t ldx, int w,
                                                          const int32_t *__restrict__ idx, int rows, int x_rows,
                                                          float *__restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)rows * w) return;
    const int64_t r = e / w, c = e % w;
    const int32_t src = idx[r];
    out[e] = (src >= 0 && src < x_rows) ? X[(int64_t)src * ldx + c] : __builtin_nanf("");
}

hipError_t gemm(bool bf16, const GemmArgs &g, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0) return hipSuccess;
    const dim3 grid((g.N + TN - 1) / TN, (g.M + TM - 1) / TM);
    if (bf16)
        hipLaunchKernelGGL(mlp_gemm_kernel<true>, grid, dim3(256), 0, st, g);
    else
        hipLaunchKernelGGL(mlp_gemm_kernel<false>, grid, dim3(256), 0, st, g);
    return hipGetLastError();
}

GemmArgs make_gemm(const float *A, int64_t sam, int64_t sak, const float *B, int64_t sbk, int64_t sbn, float *C,
                   int64_t ldc, int M, int N, int K, int epi, const float *bias = nullptr,
                   const float *mask = nullptr, int64_t ldm = 0) {
    GemmArgs g;
    g.A = A;
    g.sam = sam;
    g.sak = sak;
    g.B = B;
    g.sbk = sbk;
    g.sbn = sbn;
    g.C = C;
    g.ldc = ldc;
    g.bias = bias;
    g.mask = mask;
    g.ldm = ldm;
    g.M = M;
    g.N = N;
    g.K = K;
    g.epi = epi;
    return g;
}

#define MLP_TRY(expr)                        \
    do {                                     \
        hipError_t _e = (expr);              \
        if (_e != hipSuccess) return _e;     \
    } while (0)

bool overlap(const float *a, int64_t na, const float *b, int64_t nb) {
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + (uintptr_t)nb * 4 && pb < pa + (uintptr_t)na * 4;
}

// Rows of Y that touch no row of X but their own: columns of one matrix, either apart or of the same row.
bool own_rows(const float *X, int64_t ldx, int n_in, const float *Y, int64_t ldy, int n_out) {
    const int64_t bytes = (intptr_t)Y - (intptr_t)X, off = bytes / 4;
    if (ldx != ldy || bytes % 4 != 0) return false;
    const int64_t col = (off % ldx + ldx) % ldx;
    return col + n_out <= ldx && (col >= n_in || off == col);
}

// Networks small enough for the fused kernels (register and LDS budgets set the limits).
bool fuse_ok(int n_in, int hidden, int n_out) {
    return n_in <= kFuseIn && hidden <= kFuseHidden && n_out <= kFuseOut;
}

// As many workgroups as the 256 CUs hold at once (by the registers of each instance): past that a
// workgroup takes several tiles and reads the weights once for all of them.  Forward passes of 65536
// rows in BF16 with 128 units: 13.7 us with these 768, 16.3 with 512, 19.6 with 1024 (a second, nearly
// empty wave); 256 units: 28.3 with 256, 51.2 with 1024.
template <bool BF16, int HP, bool TRAIN>
constexpr int tile_workgroups() {
    const int waves = TRAIN ? ((BF16 || HP != 128) ? 2 : 1) : HP == 256 ? 2 : BF16 ? 3 : HP == 64 ? 4 : 2;   // per SIMD
    return 256 * (waves * 4 * 32 / HP);
}

template <bool BF16, int HP, bool TRAIN>
hipError_t launch_tile(const FuseArgs &g, bool packed, hipStream_t st) {
    constexpr int most = tile_workgroups<BF16, HP, TRAIN>();
    const int grid = g.tiles < most ? g.tiles : most;
    if constexpr (BF16 && TRAIN) {
        if (packed) {
            hipLaunchKernelGGL((mlp_tile_kernel<BF16, HP, TRAIN, true>), dim3(grid), dim3(2 * HP), 0, st, g);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((mlp_tile_kernel<BF16, HP, TRAIN, false>), dim3(grid), dim3(2 * HP), 0, st, g);
    return hipGetLastError();
}

template <bool TRAIN>
hipError_t run_tiles(bool bf16, const FuseArgs &g, bool packed, hipStream_t st) {
    const int hp = padded_hidden(g.H);
    if (hp == 64) return bf16 ? launch_tile<true, 64, TRAIN>(g, packed, st) : launch_tile<false, 64, TRAIN>(g, false, st);
    if (hp == 128)
        return bf16 ? launch_tile<true, 128, TRAIN>(g, packed, st) : launch_tile<false, 128, TRAIN>(g, false, st);
    return bf16 ? launch_tile<true, 256, TRAIN>(g, packed, st) : launch_tile<false, 256, TRAIN>(g, false, st);
}

FuseArgs fuse_args(const MlpLayout &lo, int n_in, int hidden, int n_out, const float *P, const float *X, int64_t ldx,
                   int rows) {
    FuseArgs g{};
    g.P = P;
    g.lo = lo;
    g.n_in = n_in;
    g.H = hidden;
    g.n_out = n_out;
    g.X = X;
    g.ldx = ldx;
    g.x_rows = rows;
    g.rows = rows;
    g.tiles = (int)(((int64_t)rows + kTile - 1) / kTile);
    return g;
}

// Loss and gradient (G), or loss and Adam step (P, Mv, Vv) of `rows` rows, idx[r] of X and T if idx.
// packed: the tile kernel reads the packed weights, which this call makes anew (fresh) or finds as the
// last call's Adam step left them.
template <bool ADAM>
hipError_t run_train(const MlpLayout &lo, int n_in, int hidden, int n_out, bool bf16, const float *P, const float *X,
                     int64_t ldx, const float *T, int64_t ldt, const int32_t *idx, int rows, int x_rows, double *loss,
                     float *G, float *Pw, float *Mv, float *Vv, const AdamArgs &ad, bool packed, bool fresh, char *ws,
                     hipStream_t st) {
    FuseArgs g = fuse_args(lo, n_in, hidden, n_out, P, X, ldx, rows);
    g.idx = idx;
    g.x_rows = x_rows;
    g.T = T;
    g.ldt = ldt;
    g.scale = (float)(2.0 / ((double)rows * n_out));
    g.fl = fuse_layout(hidden, n_out, rows, bf16);
    g.ws = ws;
    const int hp = padded_hidden(hidden);
    if (packed && fresh) {
        hipLaunchKernelGGL(mlp_pack_kernel, dim3((hp * hp + 255) / 256), dim3(256), 0, st, P, lo, g.fl, n_in, hidden, hp, ws);
        MLP_TRY(hipGetLastError());
    }
    MLP_TRY(run_tiles<true>(bf16, g, packed, st));
    GradArgs a{};
    a.lo = lo;
    a.fl = g.fl;
    a.ws = ws;
    a.n_in = n_in;
    a.H = hidden;
    a.n_out = n_out;
    a.rows = rows;
    a.loss = loss;
    a.G = G;
    a.P = Pw;
    a.Mv = Mv;
    a.Vv = Vv;
    a.ad = ad;
    a.pack = packed ? ws : nullptr;
    a.hp = hp;
    const int bh = g.fl.bh;
    const int grid = bh * bh + (n_in + 15) / 16 * bh + bh + (bf16 ? 2 * hidden + n_out : 4 * (2 * bh + 1)) + 1;
    if (bf16)
        hipLaunchKernelGGL((mlp_grad_kernel<true, ADAM>), dim3(grid), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((mlp_grad_kernel<false, ADAM>), dim3(grid), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace

MlpLayout mlp_layout(int n_in, int hidden, int n_out, int64_t rows) {
    MlpLayout lo{};
    const int64_t H = hidden;
    lo.oW1 = 0;
    lo.ob1 = lo.oW1 + (int64_t)n_in * H;
    lo.oW2 = lo.ob1 + H;
    lo.ob2 = lo.oW2 + H * H;
    lo.oW3 = lo.ob2 + H;
    lo.ob3 = lo.oW3 + H * n_out;
    lo.count = lo.ob3 + n_out;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    lo.Xb = take((size_t)rows * n_in * 4);
    lo.Tb = take((size_t)rows * n_out * 4);
    lo.H1 = take((size_t)rows * H * 4);
    lo.H2 = take((size_t)rows * H * 4);
    lo.Y = take((size_t)rows * n_out * 4);
    lo.dY = take((size_t)rows * n_out * 4);
    lo.dH2 = take((size_t)rows * H * 4);
    lo.dH1 = take((size_t)rows * H * 4);
    lo.G = take((size_t)lo.count * 4);
    lo.loss = take(64);
    lo.bytes = off;
    return lo;
}

size_t mlp_workspace_bytes(int n_in, int hidden, int n_out, int64_t rows) {
    size_t b = mlp_layout(n_in, hidden, n_out, rows).bytes;
    if (fuse_ok(n_in, hidden, n_out))
        for (const bool bf16 : {false, true}) b = std::max(b, fuse_layout(hidden, n_out, rows, bf16).bytes_packed);
    return b;
}

namespace {

// Layer by layer; leaves H1 and H2 in the workspace for the backward pass.
hipError_t layered_forward(const MlpLayout &lo, int n_in, int hidden, int n_out, bool bf16, const float *P,
                           const float *X, int64_t ldx, int rows, float *Y, int64_t ldy, char *ws, hipStream_t st) {
    float *H1 = (float *)(ws + lo.H1), *H2 = (float *)(ws + lo.H2);
    const int H = hidden;
    MLP_TRY(gemm(bf16, make_gemm(X, ldx, 1, P + lo.oW1, H, 1, H1, H, rows, H, n_in, EPI_BIAS_RELU, P + lo.ob1), st));
    MLP_TRY(gemm(bf16, make_gemm(H1, H, 1, P + lo.oW2, H, 1, H2, H, rows, H, H, EPI_BIAS_RELU, P + lo.ob2), st));
    MLP_TRY(gemm(bf16, make_gemm(H2, H, 1, P + lo.oW3, n_out, 1, Y, ldy, rows, n_out, H, EPI_BIAS, P + lo.ob3), st));
    return hipSuccess;
}

}  // namespace

hipError_t mlp_forward(const MlpLayout &lo, int n_in, int hidden, int n_out, bool bf16, const float *P,
                       const float *X, int64_t ldx, int rows, float *Y, int64_t ldy, char *ws, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    // The fused kernel writes outputs while other rows are still to be read; layer by layer, X has been read
    // before Y is written, so that they may share memory (and the parameters of the first two layers).
    const int64_t y_len = (int64_t)(rows - 1) * ldy + n_out;
    const bool shared = (overlap(Y, y_len, X, (int64_t)(rows - 1) * ldx + n_in) &&
                         !own_rows(X, ldx, n_in, Y, ldy, n_out)) ||
                        overlap(Y, y_len, P, lo.count);
    if (!fuse_ok(n_in, hidden, n_out) || shared)
        return layered_forward(lo, n_in, hidden, n_out, bf16, P, X, ldx, rows, Y, ldy, ws, st);
    FuseArgs g = fuse_args(lo, n_in, hidden, n_out, P, X, ldx, rows);
    g.Y = Y;
    g.ldy = ldy;
    return run_tiles<false>(bf16, g, false, st);
}

namespace {

AdamArgs adam_args(int64_t step, double lr, double b1, double b2, double eps) {
    const double bc1 = 1.0 - std::pow(b1, (double)step), bc2 = 1.0 - std::pow(b2, (double)step);
    return {(float)b1, (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)lr, (float)eps, (float)bc1, (float)bc2};
}

}  // namespace

hipError_t mlp_loss_grad(const MlpLayout &lo, int n_in, int hidden, int n_out, bool bf16, const float *P,
                         const float *X, int64_t ldx, const float *T, int64_t ldt, int rows, float *G, double *loss,
                         char *ws, size_t ws_bytes, hipStream_t st) {
    const int H = hidden;
    if (fuse_ok(n_in, hidden, n_out) && ws_bytes >= fuse_layout(hidden, n_out, rows, bf16).bytes)
        return run_train<false>(lo, n_in, hidden, n_out, bf16, P, X, ldx, T, ldt, nullptr, rows, rows, loss, G, nullptr,
                                nullptr, nullptr, AdamArgs{}, false, false, ws, st);
    float *H1 = (float *)(ws + lo.H1), *H2 = (float *)(ws + lo.H2), *Y = (float *)(ws + lo.Y);
    float *dY = (float *)(ws + lo.dY), *dH2 = (float *)(ws + lo.dH2), *dH1 = (float *)(ws + lo.dH1);
    MLP_TRY(layered_forward(lo, n_in, hidden, n_out, bf16, P, X, ldx, rows, Y, n_out, ws, st));
    hipLaunchKernelGGL(mse_kernel, dim3(1), dim3(1024), 0, st, Y, (int64_t)n_out, T, ldt, rows, n_out, dY, loss);
    MLP_TRY(hipGetLastError());
    // layer 3: gW3 = H2^T dY, gb3 = column sums of dY, dH2 = (dY W3^T) masked by H2 > 0
    MLP_TRY(gemm(bf16, make_gemm(H2, 1, H, dY, n_out, 1, G + lo.oW3, n_out, H, n_out, rows, EPI_STORE), st));
    hipLaunchKernelGGL(colsum_rows_kernel, dim3(n_out), dim3(256), 0, st, dY, (int64_t)n_out, rows, G + lo.ob3);
    MLP_TRY(hipGetLastError());
    MLP_TRY(gemm(bf16, make_gemm(dY, n_out, 1, P + lo.oW3, 1, n_out, dH2, H, rows, H, n_out, EPI_MASK, nullptr, H2, H),
                 st));
    // layer 2
    MLP_TRY(gemm(bf16, make_gemm(H1, 1, H, dH2, H, 1, G + lo.oW2, H, H, H, rows, EPI_STORE), st));
    hipLaunchKernelGGL(colsum_rows_kernel, dim3(H), dim3(256), 0, st, dH2, (int64_t)H, rows, G + lo.ob2);
    MLP_TRY(hipGetLastError());
    MLP_TRY(gemm(bf16, make_gemm(dH2, H, 1, P + lo.oW2, 1, H, dH1, H, rows, H, H, EPI_MASK, nullptr, H1, H), st));
    // layer 1
    MLP_TRY(gemm(bf16, make_gemm(X, 1, ldx, dH1, H, 1, G + lo.oW1, H, n_in, H, rows, EPI_STORE), st));
    hipLaunchKernelGGL(colsum_rows_kernel, dim3(H), dim3(256), 0, st, dH1, (int64_t)H, rows, G + lo.ob1);
    return hipGetLastError();
}

hipError_t mlp_adam(float *P, const float *G, float *M, float *V, int64_t count, int64_t step, double lr, double b1,
                    double b2, double eps, hipStream_t st) {
    const int64_t blocks = (count + 255) / 256;
    const int grid = (int)(blocks < 4096 ? blocks : 4096);
    hipLaunchKernelGGL(adam_kernel, dim3(grid), dim3(256), 0, st, P, G, M, V, count, adam_args(step, lr, b1, b2, eps));
    return hipGetLastError();
}

namespace {

hipError_t mlp_gather(const float *X, int64_t ldx, int w, const int32_t *idx, int rows, int x_rows, float *out,
                      hipStream_t st) {
    const int64_t total = (int64_t)rows * w;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, ldx, w, idx,
                       rows, x_rows, out);
    return hipGetLastError();
}

}  // namespace

hipError_t mlp_train_step(const MlpLayout &lo, int n_in, int hidden, int n_out, bool bf16, float *P, float *M, float *V,
                          int64_t step, const float *X, int64_t ldx, const float *T, int64_t ldt, int rows,
                          const int32_t *idx, int batch, double lr, double *loss, bool first, char *ws, size_t ws_bytes,
                          hipStream_t st) {
    float *G = (float *)(ws + lo.G);
    const FuseLayout fl = fuse_layout(hidden, n_out, batch, bf16);
    if (fuse_ok(n_in, hidden, n_out) && ws_bytes >= fl.bytes)
        return run_train<true>(lo, n_in, hidden, n_out, bf16, P, X, ldx, T, ldt, idx, batch, rows, loss, nullptr, P, M, V,
                               adam_args(step, lr, 0.9, 0.999, 1e-8), bf16 && ws_bytes >= fl.bytes_packed, first, ws, st);
    float *Xb = (float *)(ws + lo.Xb), *Tb = (float *)(ws + lo.Tb);
    MLP_TRY(mlp_gather(X, ldx, n_in, idx, batch, rows, Xb, st));
    MLP_TRY(mlp_gather(T, ldt, n_out, idx, batch, rows, Tb, st));
    MLP_TRY(mlp_loss_grad(lo, n_in, hidden, n_out, bf16, P, Xb, n_in, Tb, n_out, batch, G,
                          loss ? loss : (double *)(ws + lo.loss), ws, 0, st));
    return mlp_adam(P, G, M, V, lo.count, step, lr, 0.9, 0.999, 1e-8, st);
}

}  // namespace hap
