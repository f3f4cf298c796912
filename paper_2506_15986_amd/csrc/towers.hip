// Two-tower entry model (two-tower score of the preliminaries; projection
// network of the high-tier graph section): forward, backward, contrastive
// loss and Adam, all deterministic (no floating-point atomics; every
// reduction runs in a fixed order).
//
// tower(x) = normalise(W2 . relu(W1 . x + b1) + b2), FP32 master weights with
// BF16 working copies.  Each matrix product takes BF16 operands (rounded to
// nearest even) and accumulates in FP32 on the matrix cores
// (v_mfma_f32_16x16x32_bf16): the tower input, the weights, the hidden
// activation after ReLU and, backwards, the pre-activation gradients entering
// the weight and input products.  Bias, ReLU, normalisation, logits and
// softmax stay in FP32.
//
// Loss (Eq. 2 / Eq. 4 read query-anchored over all hubs, the positive inside
// the denominator): L = mean_i [logsumexp_h(s_ih) - s_i,y_i],
// s_ih = <e_q_i, e_h> / tau.
#include "common.h"
#include "internal.h"

namespace ann {
namespace {

typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ inline uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);   // inf / nan
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ---------------------------------------------------------------- BF16 GEMM
// C[m][n] = sum_k A(m,k) * B(n,k) with A(m,k) = A[m*sam + k*sak] and
// B(n,k) = B[n*sbn + k*sbk] (bf16).  Epilogue: + bias[n]; optional ReLU;
// optional multiply by (mask[m*ldc+n] > 0); FP32 result to C and/or BF16 to Cb.
struct GemmArgs {
    const uint16_t *A;
    int64_t sam, sak;
    const uint16_t *B;
    int64_t sbn, sbk;
    int M, N, K;
    const float *bias;
    int relu;
    const float *mask;
    float *C;
    uint16_t *Cb;
    int ldc;
};

constexpr int GT = 64;   // tile
constexpr int GK = 32;   // k step: one 16x16x32 product per block

__global__ void __launch_bounds__(256) gemm_bf16_kernel(GemmArgs g)
{
    __shared__ uint16_t As[GT][GK + 4];
    __shared__ uint16_t Bs[GT][GK + 4];
    const int t = threadIdx.x;
    const int w = t >> 6, lane = t & 63;
    const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
    v4f acc[4];
    for (int b = 0; b < 4; ++b) acc[b] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < g.K; k0 += GK) {
        for (int e = t; e < GT * GK; e += 256) {
            int r = e / GK, kk = e % GK;
            int m = m0 + r, n = n0 + r, k = k0 + kk;
            As[r][kk] = (m < g.M && k < g.K) ? g.A[(int64_t)m * g.sam + (int64_t)k * g.sak] : 0;
            Bs[r][kk] = (n < g.N && k < g.K) ? g.B[(int64_t)n * g.sbn + (int64_t)k * g.sbk] : 0;
        }
        __syncthreads();
        // each lane: eight consecutive k of its row (A) and column (B); the
        // same k for both operands, so the products are those of the sum
        v8s a;
        const int ar = 16 * w + (lane & 15), kq = 8 * (lane >> 4);
        for (int q = 0; q < 8; ++q) a[q] = (short)As[ar][kq + q];
        for (int b = 0; b < 4; ++b) {
            v8s bv;
            const int bc = 16 * b + (lane & 15);
            for (int q = 0; q < 8; ++q) bv[q] = (short)Bs[bc][kq + q];
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                             __builtin_bit_cast(v8bf, bv), acc[b],
                                                             0, 0, 0);
        }
        __syncthreads();
    }
    for (int b = 0; b < 4; ++b) {
        const int n = n0 + 16 * b + (lane & 15);
        for (int i = 0; i < 4; ++i) {
            const int m = m0 + 16 * w + 4 * (lane >> 4) + i;
            if (m >= g.M || n >= g.N) continue;
            float v = acc[b][i];
            if (g.bias) v += g.bias[n];
            if (g.relu) v = v > 0.f ? v : 0.f;
            const int64_t o = (int64_t)m * g.ldc + n;
            if (g.mask && !(g.mask[o] > 0.f)) v = 0.f;
            if (g.C) g.C[o] = v;
            if (g.Cb) g.Cb[o] = f2bf(v);
        }
    }
}

// ---------------------------------------------------------------- FP32 GEMM
// C[m][n] = alpha * sum_k A(m,k) * B(n,k), one chain of fused multiply-adds
// per element in k order (the training's bits depend on it).  A and B are
// contiguous along k or along m / n.
//
// The chain cannot be split, so what shortens it is many small tiles (8 x 64:
// a wavefront takes two rows, a lane one column) and wide LDS reads: both
// operands lie there along k, four of a column's values come in one read, four
// of a row's in one read that all lanes share, and the next 64 k are on their
// way while the staged ones are added.  The three products of a step (1,024
// queries, 1,024 hubs, 64 dimensions): 367 us with 64 x 64 tiles (16 workgroups
// on 256 CUs for the gradients), 43 us now, the two gradients in one launch.
// Scalar loads for the rows (52 us a launch) and 128 k at a time (29 us)
// measured slower.
struct GemmF {
    const float *A;
    int64_t sam, sak;
    const float *B;
    int64_t sbn, sbk;
    int M, N, K;
    float alpha;
    float *C;
    int ldc;
};

constexpr int FR = 2, FM = 4 * FR, FN = 64, FK = 64, FS = FK + 4;

// Rows [r0, r0 + R) x k [k0, k0 + FK) of X into registers, in the order that
// X is contiguous in, and from there to LDS as [row][k].
template <int R>
struct FStage {
    static constexpr int U = R * FK / 256;
    float v[U];
    __device__ void load(const float *X, int64_t sr, int64_t sk, int r0, int rows, int k0, int K)
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = (int)threadIdx.x + 256 * u;
            const int r = sk == 1 ? e / FK : e % R, k = sk == 1 ? e % FK : e / R;
            v[u] = r0 + r < rows && k0 + k < K
                       ? X[(int64_t)(r0 + r) * sr + (int64_t)(k0 + k) * sk]
                       : 0.f;
        }
    }
    __device__ void store(float *s, int64_t sk) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = (int)threadIdx.x + 256 * u;
            const int r = sk == 1 ? e / FK : e % R, k = sk == 1 ? e % FK : e / R;
            s[r * FS + k] = v[u];
        }
    }
};

// Two products in one launch: the lowest bit of blockIdx.z picks.  A launch
// holds 65,535 workgroups in y; TALL: further rows follow in z.
template <bool TALL>
__global__ void __launch_bounds__(256) gemm_f32_kernel(GemmF g0, GemmF g1)
{
    const GemmF &g = blockIdx.z & 1u ? g1 : g0;
    const int n0 = (int)blockIdx.x * FN;
    int m0 = (int)blockIdx.y * FM;
    if (TALL) {
        const int64_t row = ((int64_t)(blockIdx.z >> 1) * gridDim.y + blockIdx.y) * FM;
        if (row >= g.M) return;
        m0 = (int)row;
    }
    if (m0 >= g.M || n0 >= g.N) return;
    __shared__ __align__(16) float As[FM * FS], Bs[FN * FS];
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    FStage<FM> a;
    FStage<FN> b;
    a.load(g.A, g.sam, g.sak, m0, g.M, 0, g.K);
    b.load(g.B, g.sbn, g.sbk, n0, g.N, 0, g.K);
    float acc[FR] = {};
    for (int k0 = 0; k0 < g.K; k0 += FK) {
        __syncthreads();
        a.store(As, g.sak);
        b.store(Bs, g.sbk);
        __syncthreads();
        if (k0 + FK < g.K) {
            a.load(g.A, g.sam, g.sak, m0, g.M, k0 + FK, g.K);
            b.load(g.B, g.sbn, g.sbk, n0, g.N, k0 + FK, g.K);
        }
#pragma unroll
        for (int k = 0; k < FK; k += 4) {
            const float4 y = *reinterpret_cast<const float4 *>(Bs + lane * FS + k);
            float4 x[FR];
#pragma unroll
            for (int r = 0; r < FR; ++r)
                x[r] = *reinterpret_cast<const float4 *>(As + (FR * w + r) * FS + k);
#pragma unroll
            for (int r = 0; r < FR; ++r) {
                acc[r] += x[r].x * y.x;
                acc[r] += x[r].y * y.y;
                acc[r] += x[r].z * y.z;
                acc[r] += x[r].w * y.w;
            }
        }
    }
#pragma unroll
    for (int r = 0; r < FR; ++r) {
        const int m = m0 + FR * w + r;
        if (m < g.M && n0 + lane < g.N) g.C[(int64_t)m * g.ldc + n0 + lane] = g.alpha * acc[r];
    }
}

// ---------------------------------------------------------------- elementwise
__global__ void to_bf16_kernel(const float *x, int64_t count, uint16_t *out)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = f2bf(x[i]);
}

// rows idx[i] of x (ld cols), times `scale`, -> bf16 rows i; idx NULL = identity
__global__ void gather_bf16_kernel(const float *x, int cols, const int32_t *idx, int rows,
                                   float scale, uint16_t *out)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)rows * cols;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t r = e / cols, c = e % cols;
        int64_t src = idx ? idx[r] : r;
        out[e] = f2bf(x[src * cols + c] * scale);
    }
}

// hub tower input [x_hub * vec_scale | features]: rows of base (hub ids) then the features
__global__ void hub_input_kernel(const float *base, int dim, const int32_t *hub_ids,
                                 const float *feat, int nfeat, int nh, float vec_scale,
                                 float *out32, uint16_t *outb)
{
    const int cols = dim + nfeat;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < (int64_t)nh * cols;
         e += (int64_t)gridDim.x * blockDim.x) {
        int64_t r = e / cols, c = e % cols;
        float v = c < dim ? base[(int64_t)hub_ids[r] * dim + c] * vec_scale
                          : feat[r * nfeat + (c - dim)];
        if (out32) out32[e] = v;
        if (outb) outb[e] = f2bf(v);
    }
}

// ------------------------------------------------------- fused tower kernels
// The forward and the row-wise half of the backward of a tower, 16 rows to a
// workgroup whose four wavefronts share the 16-wide column blocks of each
// product.  Every step is the arithmetic of the generic kernels in the same
// order (operand rounding, lane layout and sequence of 32-deep MFMA steps per
// output element, the normalisation's sums and shuffles), so the results are
// the same bits.
//
// They are latency chains (a row block's products are a few hundred MFMA), so
// what counts is how few launches and dependent loads there are: rows are
// staged in LDS once, both towers of a training step share a launch, and four
// wavefronts to 16 rows shorten the chain of column blocks (10,000 rows of
// 128 -> 128 -> 64: 22 us with one wavefront per 16 rows, 11.6 us with four; one
// row 10.5 and 5.4 us).
struct TowerArgs {
    const float *x;
    const int32_t *idx;   // row i of the input is x row idx[i] (NULL: row i)
    int rows, din, hidden, dout;
    float scale;
    const uint16_t *W1b, *W2b;
    const float *b1, *b2;
    float *e;             // rows x dout, unit rows
    // training: kept for the backward
    uint16_t *xb, *a1b;
    float *z1, *nrm;
    const float *de;
    float *dz2, *dz1;
    uint16_t *dz2b, *dz1b;
};

struct TowerPair {
    TowerArgs t[2];
    int blocks0;          // workgroups of t[0]
};

// LDS of the fused kernels: input, hidden and output rows
__host__ __device__ inline size_t fused_lds(int din, int hidden, int dout)
{
    return (size_t)16 * 2 * (din + 8) + (size_t)16 * 2 * (hidden + 8) + (size_t)16 * 4 * (dout + 1);
}

__device__ inline v4f mfma_bf16(v8s a, v8s b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

template <bool TRAIN>
__global__ void __launch_bounds__(256) tower_fwd_kernel(TowerPair p)
{
    const bool second = (int)blockIdx.x >= p.blocks0;
    const TowerArgs &a = p.t[second ? 1 : 0];
    extern __shared__ __align__(16) unsigned char tw_lds[];
    uint16_t *X = reinterpret_cast<uint16_t *>(tw_lds);            // 16 x (din + 8)
    const int xs = a.din + 8, hs = a.hidden + 8, zs = a.dout + 1;
    uint16_t *H = X + 16 * xs;                                     // 16 x (hidden + 8)
    float *Z = reinterpret_cast<float *>(H + 16 * hs);             // 16 x (dout + 1)
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int rl = lane & 15, kq = 8 * (lane >> 4), rq = 4 * (lane >> 4);
    const int r0 = ((int)blockIdx.x - (second ? p.blocks0 : 0)) * 16;
    const v8s zero = {0, 0, 0, 0, 0, 0, 0, 0};
    const int q4 = a.din >> 2;
    for (int e = t; e < 16 * q4; e += 256) {
        const int r = e / q4, j = 4 * (e - r * q4);
        ushort4 v = make_ushort4(0, 0, 0, 0);
        if (r0 + r < a.rows) {
            const int64_t src = a.idx ? a.idx[r0 + r] : r0 + r;
            const float4 f = *reinterpret_cast<const float4 *>(a.x + src * a.din + j);
            v = make_ushort4(f2bf(f.x * a.scale), f2bf(f.y * a.scale), f2bf(f.z * a.scale),
                             f2bf(f.w * a.scale));
            if (TRAIN) *reinterpret_cast<ushort4 *>(a.xb + (int64_t)(r0 + r) * a.din + j) = v;
        }
        *reinterpret_cast<ushort4 *>(X + r * xs + j) = v;
    }
    __syncthreads();
    for (int b = w; b < (a.hidden >> 4); b += 4) {
        const int n = 16 * b + rl;
        const uint16_t *wr = a.W1b + (size_t)n * a.din;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < a.din; k0 += 32) {
            const int k = k0 + kq;
            const bool in = k < a.din;
            const v8s bv = in ? *reinterpret_cast<const v8s *>(wr + k) : zero;
            const v8s av = in ? *reinterpret_cast<const v8s *>(X + rl * xs + k) : zero;
            acc = mfma_bf16(av, bv, acc);
        }
        const float bias = a.b1[n];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = acc[i] + bias;
            v = v > 0.f ? v : 0.f;
            const uint16_t h = f2bf(v);
            H[(rq + i) * hs + n] = h;
            if (TRAIN && r0 + rq + i < a.rows) {
                const int64_t o = (int64_t)(r0 + rq + i) * a.hidden + n;
                a.z1[o] = v;
                a.a1b[o] = h;
            }
        }
    }
    __syncthreads();
    for (int b = w; b < (a.dout >> 4); b += 4) {
        const int n = 16 * b + rl;
        const uint16_t *wr = a.W2b + (size_t)n * a.hidden;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < a.hidden; k0 += 32) {
            const int k = k0 + kq;
            const bool in = k < a.hidden;
            const v8s bv = in ? *reinterpret_cast<const v8s *>(wr + k) : zero;
            const v8s av = in ? *reinterpret_cast<const v8s *>(H + rl * hs + k) : zero;
            acc = mfma_bf16(av, bv, acc);
        }
        const float bias = a.b2[n];
#pragma unroll
        for (int i = 0; i < 4; ++i) Z[(rq + i) * zs + n] = acc[i] + bias;
    }
    __syncthreads();
    // normalise_kernel's arithmetic, a row at a time
    for (int r = w; r < 16 && r0 + r < a.rows; r += 4) {
        float s = 0.f;
        for (int c = lane; c < a.dout; c += 64) s += Z[r * zs + c] * Z[r * zs + c];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        const float n = sqrtf(s);
        for (int c = lane; c < a.dout; c += 64) a.e[(int64_t)(r0 + r) * a.dout + c] = Z[r * zs + c] / n;
        if (TRAIN && lane == 0) a.nrm[r0 + r] = n;
    }
}

// dz2 = (de - e <e, de>) / |z|, its BF16 rounding, and dz1 = (dz2b . W2b) where
// the hidden activation is positive
__global__ void __launch_bounds__(256) tower_bwd_rows_kernel(TowerPair p)
{
    const bool second = (int)blockIdx.x >= p.blocks0;
    const TowerArgs &a = p.t[second ? 1 : 0];
    extern __shared__ __align__(16) unsigned char tw_lds[];
    uint16_t *D = reinterpret_cast<uint16_t *>(tw_lds);            // 16 x (dout + 8)
    const int ds = a.dout + 8;
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int rl = lane & 15, kq = 8 * (lane >> 4), rq = 4 * (lane >> 4);
    const int r0 = ((int)blockIdx.x - (second ? p.blocks0 : 0)) * 16;
    for (int r = w; r < 16; r += 4) {
        if (r0 + r >= a.rows) {
            for (int c = lane; c < a.dout; c += 64) D[r * ds + c] = 0;
            continue;
        }
        const int64_t at = (int64_t)(r0 + r) * a.dout;
        float s = 0.f;
        for (int c = lane; c < a.dout; c += 64) s += a.e[at + c] * a.de[at + c];
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
        for (int c = lane; c < a.dout; c += 64) {
            const float v = (a.de[at + c] - a.e[at + c] * s) / a.nrm[r0 + r];
            const uint16_t h = f2bf(v);
            a.dz2[at + c] = v;
            a.dz2b[at + c] = h;
            D[r * ds + c] = h;
        }
    }
    __syncthreads();
    const v8s zero = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = w; b < (a.hidden >> 4); b += 4) {
        const int n = 16 * b + rl;
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < a.dout; k0 += 32) {
            const int k = k0 + kq;
            const bool in = k < a.dout;
            v8s bv = zero;
            if (in)
#pragma unroll
                for (int q = 0; q < 8; ++q) bv[q] = (short)a.W2b[(size_t)(k + q) * a.hidden + n];
            const v8s av = in ? *reinterpret_cast<const v8s *>(D + rl * ds + k) : zero;
            acc = mfma_bf16(av, bv, acc);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (r0 + rq + i >= a.rows) continue;
            const int64_t o = (int64_t)(r0 + rq + i) * a.hidden + n;
            const float v = a.z1[o] > 0.f ? acc[i] : 0.f;
            a.dz1[o] = v;
            a.dz1b[o] = f2bf(v);
        }
    }
}

// one wavefront per row: e = z / |z|, keeps |z|
__global__ void normalise_kernel(const float *z, int rows, int cols, float *e, float *nrm)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    float s = 0.f;
    for (int c = lane; c < cols; c += 64) s += z[r * cols + c] * z[r * cols + c];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    const float n = sqrtf(s);
    for (int c = lane; c < cols; c += 64) e[r * cols + c] = z[r * cols + c] / n;
    if (lane == 0 && nrm) nrm[r] = n;
}

// dz = (de - e <e, de>) / |z|; also BF16 copy
__global__ void normalise_bwd_kernel(const float *e, const float *de, const float *nrm, int rows,
                                     int cols, float *dz, uint16_t *dzb)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    float s = 0.f;
    for (int c = lane; c < cols; c += 64) s += e[r * cols + c] * de[r * cols + c];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    for (int c = lane; c < cols; c += 64) {
        float v = (de[r * cols + c] - e[r * cols + c] * s) / nrm[r];
        dz[r * cols + c] = v;
        dzb[r * cols + c] = f2bf(v);
    }
}

constexpr int CE_W = 16;   // logits of a row that a lane can hold

// one wavefront per query row of logits: loss_i and ds = (softmax - onehot)/B
__global__ void softmax_ce_kernel(const float *s, int rows, int cols, const int32_t *labels,
                                  const int32_t *idx, float inv_b, float *ds, float *loss_rows)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const float *row = s + r * cols;
    if (cols <= 64 * CE_W) {
        // the lane's values of the row in registers: one pass over memory
        // instead of three, the sums in the same order
        float v[CE_W];
#pragma unroll
        for (int k = 0; k < CE_W; ++k)
            v[k] = lane + 64 * k < cols ? row[lane + 64 * k] : -__int_as_float(0x7f800000);
        const int y = labels[idx ? idx[r] : r];
        const float ry = row[y];
        float mx = -__int_as_float(0x7f800000);
#pragma unroll
        for (int k = 0; k < CE_W; ++k)
            if (lane + 64 * k < cols) mx = fmaxf(mx, v[k]);
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
        float se = 0.f;
#pragma unroll
        for (int k = 0; k < CE_W; ++k)
            if (lane + 64 * k < cols) {
                v[k] = expf(v[k] - mx);
                se += v[k];
            }
        for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
#pragma unroll
        for (int k = 0; k < CE_W; ++k) {
            const int c = lane + 64 * k;
            if (c < cols) {
                const float p = v[k] / se;
                ds[r * cols + c] = (p - (c == y ? 1.f : 0.f)) * inv_b;
            }
        }
        if (lane == 0) loss_rows[r] = logf(se) + mx - ry;
        return;
    }
    float mx = -__int_as_float(0x7f800000);
    for (int c = lane; c < cols; c += 64) mx = fmaxf(mx, row[c]);
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float se = 0.f;
    for (int c = lane; c < cols; c += 64) se += expf(row[c] - mx);
    for (int o = 32; o > 0; o >>= 1) se += __shfl_xor(se, o);
    const int y = labels[idx ? idx[r] : r];
    for (int c = lane; c < cols; c += 64) {
        float p = expf(row[c] - mx) / se;
        ds[r * cols + c] = (p - (c == y ? 1.f : 0.f)) * inv_b;
    }
    if (lane == 0) loss_rows[r] = logf(se) + mx - row[y];
}

// Eq. 4 read hub-anchored: row i of s (Bh rows of `cols` scores) owns the
// block of W = P + N columns starting at i * W, its P positives then its N
// negatives.  One wavefront per hub row: loss_i = P * LSE_i - sum_pos s and
// ds = (P * softmax - [positive]) * inv_b inside the block, 0 elsewhere.
__global__ void hub_ce_kernel(const float *s, int rows, int cols, int P, int N, float inv_b,
                              float *ds, float *loss_rows)
{
    const int64_t r = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const int W = P + N;
    const float *row = s + r * cols + r * W;
    float mx = -__int_as_float(0x7f800000);
    for (int c = lane; c < W; c += 64) mx = fmaxf(mx, row[c]);
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    float se = 0.f, sp = 0.f;
    for (int c = lane; c < W; c += 64) {
        se += expf(row[c] - mx);
        if (c < P) sp += row[c];
    }
    for (int o = 32; o > 0; o >>= 1) {
        se += __shfl_xor(se, o);
        sp += __shfl_xor(sp, o);
    }
    float *drow = ds + r * cols;
    for (int c = lane; c < cols; c += 64) {
        const int j = c - (int)(r * W);
        float g = 0.f;
        if (j >= 0 && j < W) g = ((float)P * expf(row[j] - mx) / se - (j < P ? 1.f : 0.f)) * inv_b;
        drow[c] = g;
    }
    if (lane == 0) loss_rows[r] = (float)P * (logf(se) + mx) - sp;
}

// Column sums of x [rows x cols], each summed row by row in order (the
// training's bits depend on it); the loads of 16 rows are issued together
// before their adds, so the chain waits on memory once per 16 rows.
__global__ void bias_grad_kernel(const float *x, int rows, int cols, float *out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= cols) return;
    float s = 0.f;
    int r = 0;
    for (; r + 16 <= rows; r += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = x[(int64_t)(r + u) * cols + c];
#pragma unroll
        for (int u = 0; u < 16; ++u) s += v[u];
    }
    for (; r < rows; ++r) s += x[(int64_t)r * cols + c];
    out[c] = s;
}

struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};

// The fused multiply-adds are written out: left to the compiler, which of two
// products is fused differs from one caller to the next, and with it the bits
// of the training.
__device__ inline void adam_update(const AdamStep &s, float gi, float *p, float *m, float *v,
                                   uint16_t *pb)
{
    const float mi = __builtin_fmaf(1.f - s.b1, gi, s.b1 * *m);
    const float vi = __builtin_fmaf(gi, (1.f - s.b2) * gi, s.b2 * *v);
    *m = mi;
    *v = vi;
    const float mh = mi / s.c1, vh = vi / s.c2;
    const float pi = *p - s.lr * mh / (sqrtf(vh) + s.eps);
    *p = pi;
    if (pb) *pb = f2bf(pi);
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int64_t count, AdamStep s,
                            uint16_t *pb)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        adam_update(s, g[i], p + i, m + i, v + i, pb ? pb + i : nullptr);
}

// ---- the other half of the backward: weight and bias gradients of both
// towers, each updated by Adam where it is made, and the mean loss, in one
// launch.  A wavefront takes a 16 x 16 tile of a weight gradient, one chain of
// 32-deep MFMA steps over all rows (as gemm_bf16_kernel's, so the same bits);
// a workgroup takes 64 columns of a bias gradient, whose rows are added in
// order (bias_grad_kernel's sum) from LDS.  21 us for both towers at the
// default configuration, where six products, four sums and eight updates in
// launches of their own took 350 us; the whole step 939 -> 86 us.
struct GradArgs {
    int rows, din, hidden, dout;
    const uint16_t *xb, *a1b, *dz2b, *dz1b;
    const float *dz2, *dz1;
    float *g[4];                 // gW1, gb1, gW2, gb2
    float *p[4], *m[4], *v[4];   // the same order; NULL when step is 0
    uint16_t *W1b, *W2b;
    int w2_tiles, tiles;         // tiles of gW2, of gW2 and gW1
    int tile_blocks, bias2_blocks, blocks;
};

struct GradPair {
    GradArgs t[2];
    AdamStep adam;
    int step;
    const float *loss_rows;
    int loss_count;
    float *loss;
};

constexpr int BG_ROWS = 128;     // rows of a bias gradient staged at a time

__device__ inline void mean_of(const float *x, int count, float *out, float *sh)
{
    float s = 0.f;
    for (int i = threadIdx.x; i < count; i += 256) s += x[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = sh[0] / (float)count;
}

__global__ void __launch_bounds__(256) tower_grad_kernel(GradPair p)
{
    __shared__ float stage[BG_ROWS][64];
    int blk = blockIdx.x;
    if (blk == p.t[0].blocks + p.t[1].blocks) return mean_of(p.loss_rows, p.loss_count, p.loss, &stage[0][0]);
    const bool second = blk >= p.t[0].blocks;
    const GradArgs &a = p.t[second ? 1 : 0];
    if (second) blk -= p.t[0].blocks;
    const int t = threadIdx.x, lane = t & 63;
    if (blk < a.tile_blocks) {
        int tile = 4 * blk + (t >> 6);
        if (tile >= a.tiles) return;
        const bool w2 = tile < a.w2_tiles;
        if (!w2) tile -= a.w2_tiles;
        // C[m][n] = sum over rows k of A[k][m] B[k][n]
        const uint16_t *A = w2 ? a.dz2b : a.dz1b, *B = w2 ? a.a1b : a.xb;
        const int M = w2 ? a.dout : a.hidden, N = w2 ? a.hidden : a.din;
        const int nt = (N + 15) / 16;
        const int m0 = tile / nt * 16, n0 = tile % nt * 16;
        const int rl = lane & 15, kq = 8 * (lane >> 4), rq = 4 * (lane >> 4);
        const int m = m0 + rl, n = n0 + rl;
        const int nc = n < N ? n : N - 1;      // a column past the end is not stored
        v4f acc = {0.f, 0.f, 0.f, 0.f};
        int k0 = 0;
        for (; k0 + 128 <= a.rows; k0 += 128) {
            v8s av[4], bv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int64_t k = k0 + 32 * u + kq + q;
                    av[u][q] = (short)A[k * M + m];
                    bv[u][q] = (short)B[k * N + nc];
                }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = mfma_bf16(av[u], bv[u], acc);
        }
        for (; k0 < a.rows; k0 += 32) {
            v8s av, bv;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t k = k0 + kq + q;
                av[q] = k < a.rows ? (short)A[k * M + m] : (short)0;
                bv[q] = k < a.rows ? (short)B[k * N + nc] : (short)0;
            }
            acc = mfma_bf16(av, bv, acc);
        }
        if (n >= N) return;
        const int j = w2 ? 2 : 0;
        uint16_t *pb = w2 ? a.W2b : a.W1b;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t o = (int64_t)(m0 + rq + i) * N + n;
            a.g[j][o] = acc[i];
            if (p.step > 0) adam_update(p.adam, acc[i], a.p[j] + o, a.m[j] + o, a.v[j] + o, pb + o);
        }
        return;
    }
    // 64 columns of a bias gradient
    blk -= a.tile_blocks;
    const bool second_bias = blk < a.bias2_blocks;
    if (!second_bias) blk -= a.bias2_blocks;
    const float *x = second_bias ? a.dz2 : a.dz1;
    const int cols = second_bias ? a.dout : a.hidden;
    const int c = 64 * blk + lane;
    float s = 0.f;
    for (int r0 = 0; r0 < a.rows; r0 += BG_ROWS) {
        const int m = a.rows - r0 < BG_ROWS ? a.rows - r0 : BG_ROWS;
        float v[BG_ROWS / 4];
#pragma unroll
        for (int u = 0; u < BG_ROWS / 4; ++u) {
            const int r = (t >> 6) + 4 * u;
            v[u] = r < m && c < cols ? x[(int64_t)(r0 + r) * cols + c] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < BG_ROWS / 4; ++u) stage[(t >> 6) + 4 * u][lane] = v[u];
        __syncthreads();
        if (t < 64) {
            int r = 0;
            for (; r + 16 <= m; r += 16) {
                float y[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) y[u] = stage[r + u][lane];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += y[u];
            }
            for (; r < m; ++r) s += stage[r][lane];
        }
    }
    if (t >= 64 || c >= cols) return;
    const int j = second_bias ? 3 : 1;
    a.g[j][c] = s;
    if (p.step > 0) adam_update(p.adam, s, a.p[j] + c, a.m[j] + c, a.v[j] + c, nullptr);
}

__global__ void scale_kernel(float *x, int64_t count, float a)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        x[i] *= a;
}

__global__ void __launch_bounds__(256) mean_kernel(const float *x, int count, float *out)
{
    __shared__ float sh[256];
    mean_of(x, count, out, sh);
}

inline dim3 grid2(int M, int N) { return dim3((N + GT - 1) / GT, (M + GT - 1) / GT); }
inline int gridn(int64_t n) { return (int)((n + 255) / 256 > 4096 ? 4096 : (n + 255) / 256); }

ann_status gemm_bf16(const GemmArgs &g, hipStream_t st)
{
    hipLaunchKernelGGL(gemm_bf16_kernel, grid2(g.M, g.N), dim3(256), 0, st, g);
    ANN_LAUNCHED();
    return ANN_OK;
}

ann_status gemm_f32(const GemmF &g, const GemmF *h, hipStream_t st)
{
    const GemmF &g1 = h ? *h : g;
    const int M = g.M > g1.M ? g.M : g1.M, N = g.N > g1.N ? g.N : g1.N;
    const unsigned nx = (unsigned)((N + FN - 1) / FN), my = ((unsigned)M + FM - 1) / FM;
    if (my <= 65535u)
        hipLaunchKernelGGL(gemm_f32_kernel<false>, dim3(nx, my, h ? 2 : 1), dim3(256), 0, st, g, g1);
    else    // (one product: the second of each pair of layers, an empty one)
        hipLaunchKernelGGL(gemm_f32_kernel<true>, dim3(nx, 65535u, 2 * ((my + 65534u) / 65535u)), dim3(256), 0,
                           st, g, h ? g1 : GemmF{});
    ANN_LAUNCHED();
    return ANN_OK;
}

#define TRY(x)                              \
    do {                                    \
        ann_status s_ = (x);                \
        if (s_ != ANN_OK) return s_;        \
    } while (0)

// scratch of one tower pass over `rows` rows
struct TowerBufs {
    uint16_t *xb;    // rows x din
    float *z1;       // rows x hidden
    uint16_t *a1b;   // rows x hidden
    float *z2;       // rows x dout
    float *e;        // rows x dout
    float *nrm;      // rows
    float *de;       // rows x dout
    float *dz2;      // rows x dout
    uint16_t *dz2b;
    float *dz1;      // rows x hidden
    uint16_t *dz1b;
};

size_t tower_bufs_bytes(int rows, int din, int hidden, int dout)
{
    size_t b = 0;
    b += round_up((size_t)rows * din * 2, 256);
    b += round_up((size_t)rows * hidden * 4, 256) + round_up((size_t)rows * hidden * 2, 256);
    b += round_up((size_t)rows * dout * 4, 256) * 2 + round_up((size_t)rows * 4, 256);
    b += round_up((size_t)rows * dout * 4, 256) * 2 + round_up((size_t)rows * dout * 2, 256);
    b += round_up((size_t)rows * hidden * 4, 256) + round_up((size_t)rows * hidden * 2, 256);
    return b;
}

TowerBufs carve_tower(Carve &cv, int rows, int din, int hidden, int dout)
{
    TowerBufs t;
    t.xb = cv.take<uint16_t>((size_t)rows * din);
    t.z1 = cv.take<float>((size_t)rows * hidden);
    t.a1b = cv.take<uint16_t>((size_t)rows * hidden);
    t.z2 = cv.take<float>((size_t)rows * dout);
    t.e = cv.take<float>((size_t)rows * dout);
    t.nrm = cv.take<float>((size_t)rows);
    t.de = cv.take<float>((size_t)rows * dout);
    t.dz2 = cv.take<float>((size_t)rows * dout);
    t.dz2b = cv.take<uint16_t>((size_t)rows * dout);
    t.dz1 = cv.take<float>((size_t)rows * hidden);
    t.dz1b = cv.take<uint16_t>((size_t)rows * hidden);
    return t;
}

// forward from xb (already BF16) to e
ann_status tower_fwd(const ann_tower &w, const TowerBufs &b, int rows, hipStream_t st)
{
    GemmArgs g{};
    g.A = b.xb;
    g.sam = w.din;
    g.sak = 1;
    g.B = w.W1b;
    g.sbn = w.din;
    g.sbk = 1;
    g.M = rows;
    g.N = w.hidden;
    g.K = w.din;
    g.bias = w.b1;
    g.relu = 1;
    g.C = b.z1;   // post-ReLU activation (its sign is the ReLU mask)
    g.Cb = b.a1b;
    g.ldc = w.hidden;
    TRY(gemm_bf16(g, st));
    GemmArgs h{};
    h.A = b.a1b;
    h.sam = w.hidden;
    h.sak = 1;
    h.B = w.W2b;
    h.sbn = w.hidden;
    h.sbk = 1;
    h.M = rows;
    h.N = w.dout;
    h.K = w.hidden;
    h.bias = w.b2;
    h.C = b.z2;
    h.ldc = w.dout;
    TRY(gemm_bf16(h, st));
    hipLaunchKernelGGL(normalise_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, b.z2, rows, w.dout,
                       b.e, b.nrm);
    ANN_LAUNCHED();
    return ANN_OK;
}

// backward from b.de; writes gradients into gr
ann_status tower_bwd(const ann_tower &w, const ann_tower_grads &gr, const TowerBufs &b, int rows,
                     hipStream_t st)
{
    hipLaunchKernelGGL(normalise_bwd_kernel, dim3((rows + 3) / 4), dim3(256), 0, st, b.e, b.de,
                       b.nrm, rows, w.dout, b.dz2, b.dz2b);
    ANN_LAUNCHED();
    // dW2 [dout x hidden] = dz2b^T . a1b
    GemmArgs g{};
    g.A = b.dz2b;
    g.sam = 1;
    g.sak = w.dout;
    g.B = b.a1b;
    g.sbn = 1;
    g.sbk = w.hidden;
    g.M = w.dout;
    g.N = w.hidden;
    g.K = rows;
    g.C = gr.gW2;
    g.ldc = w.hidden;
    TRY(gemm_bf16(g, st));
    hipLaunchKernelGGL(bias_grad_kernel, dim3((w.dout + 255) / 256), dim3(256), 0, st, b.dz2, rows,
                       w.dout, gr.gb2);
    ANN_LAUNCHED();
    // dz1 [rows x hidden] = (dz2b . W2b) * (z1 > 0)
    GemmArgs h{};
    h.A = b.dz2b;
    h.sam = w.dout;
    h.sak = 1;
    h.B = w.W2b;
    h.sbn = 1;
    h.sbk = w.hidden;
    h.M = rows;
    h.N = w.hidden;
    h.K = w.dout;
    h.mask = b.z1;
    h.C = b.dz1;
    h.Cb = b.dz1b;
    h.ldc = w.hidden;
    TRY(gemm_bf16(h, st));
    hipLaunchKernelGGL(bias_grad_kernel, dim3((w.hidden + 255) / 256), dim3(256), 0, st, b.dz1, rows,
                       w.hidden, gr.gb1);
    ANN_LAUNCHED();
    // dW1 [hidden x din] = dz1b^T . xb
    GemmArgs k{};
    k.A = b.dz1b;
    k.sam = 1;
    k.sak = w.hidden;
    k.B = b.xb;
    k.sbn = 1;
    k.sbk = w.din;
    k.M = w.hidden;
    k.N = w.din;
    k.K = rows;
    k.C = gr.gW1;
    k.ldc = w.din;
    TRY(gemm_bf16(k, st));
    return ANN_OK;
}

AdamStep adam_step(int step, float lr)
{
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    return AdamStep{lr, b1, b2, eps, 1.f - powf(b1, (float)step), 1.f - powf(b2, (float)step)};
}

ann_status adam(ann_tower &w, const ann_tower_grads &gr, const ann_adam_state &a, int step,
                float lr, hipStream_t st)
{
    const AdamStep s = adam_step(step, lr);
    const int64_t n1 = (int64_t)w.hidden * w.din, n2 = (int64_t)w.dout * w.hidden;
    hipLaunchKernelGGL(adam_kernel, dim3(gridn(n1)), dim3(256), 0, st, w.W1, gr.gW1, a.mW1, a.vW1, n1,
                       s, w.W1b);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(adam_kernel, dim3(gridn(w.hidden)), dim3(256), 0, st, w.b1, gr.gb1, a.mb1,
                       a.vb1, (int64_t)w.hidden, s, (uint16_t *)nullptr);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(adam_kernel, dim3(gridn(n2)), dim3(256), 0, st, w.W2, gr.gW2, a.mW2, a.vW2, n2,
                       s, w.W2b);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(adam_kernel, dim3(gridn(w.dout)), dim3(256), 0, st, w.b2, gr.gb2, a.mb2,
                       a.vb2, (int64_t)w.dout, s, (uint16_t *)nullptr);
    ANN_LAUNCHED();
    return ANN_OK;
}

// The fused kernels take whole 16-wide column blocks and 16-byte groups of an
// input row; other shapes and alignments go through the generic kernels.  More
// than 64 KB of staged rows would leave a CU one workgroup.
bool fused_ok(const ann_tower &w, const float *x)
{
    return w.din >= 8 && w.din % 8 == 0 && w.hidden % 16 == 0 && w.dout % 16 == 0 && aligned(x, 16) &&
           aligned(w.W1b, 16) && aligned(w.W2b, 16) && fused_lds(w.din, w.hidden, w.dout) <= 65536;
}

TowerArgs tower_args(const ann_tower &w, const TowerBufs &b, const float *x, const int32_t *idx, int rows)
{
    TowerArgs a{};
    a.x = x;
    a.idx = idx;
    a.rows = rows;
    a.din = w.din;
    a.hidden = w.hidden;
    a.dout = w.dout;
    a.scale = w.in_scale;
    a.W1b = w.W1b;
    a.W2b = w.W2b;
    a.b1 = w.b1;
    a.b2 = w.b2;
    a.e = b.e;
    a.xb = b.xb;
    a.a1b = b.a1b;
    a.z1 = b.z1;
    a.nrm = b.nrm;
    a.de = b.de;
    a.dz2 = b.dz2;
    a.dz1 = b.dz1;
    a.dz2b = b.dz2b;
    a.dz1b = b.dz1b;
    return a;
}

GradArgs grad_args(const ann_tower &w, const ann_tower_grads &gr, const ann_adam_state *ad, const TowerBufs &b,
                   int rows)
{
    GradArgs a{};
    a.rows = rows;
    a.din = w.din;
    a.hidden = w.hidden;
    a.dout = w.dout;
    a.xb = b.xb;
    a.a1b = b.a1b;
    a.dz2b = b.dz2b;
    a.dz1b = b.dz1b;
    a.dz2 = b.dz2;
    a.dz1 = b.dz1;
    float *g[4] = {gr.gW1, gr.gb1, gr.gW2, gr.gb2}, *p[4] = {w.W1, w.b1, w.W2, w.b2};
    for (int i = 0; i < 4; ++i) {
        a.g[i] = g[i];
        a.p[i] = p[i];
    }
    if (ad) {
        float *m[4] = {ad->mW1, ad->mb1, ad->mW2, ad->mb2}, *v[4] = {ad->vW1, ad->vb1, ad->vW2, ad->vb2};
        for (int i = 0; i < 4; ++i) {
            a.m[i] = m[i];
            a.v[i] = v[i];
        }
    }
    a.W1b = w.W1b;
    a.W2b = w.W2b;
    a.w2_tiles = (w.dout / 16) * (w.hidden / 16);
    a.tiles = a.w2_tiles + (w.hidden / 16) * ((w.din + 15) / 16);
    a.tile_blocks = (a.tiles + 3) / 4;
    a.bias2_blocks = (w.dout + 63) / 64;
    a.blocks = a.tile_blocks + a.bias2_blocks + (w.hidden + 63) / 64;
    return a;
}

inline int row_blocks(int rows) { return (rows + 15) / 16; }

// Both towers' gradients and updates are written in one launch, so what one
// tower writes must be apart from what the other writes; towers that share
// parameters, gradients or moments are updated one after the other, in the
// generic step.
bool written_apart(const GradArgs &a, const GradArgs &b, int step)
{
    struct Range {
        uintptr_t begin, end;
    };
    auto ranges = [&](const GradArgs &x, Range *r) {
        const size_t n[4] = {(size_t)x.hidden * x.din, (size_t)x.hidden, (size_t)x.dout * x.hidden, (size_t)x.dout};
        int c = 0;
        auto add = [&](const void *p, size_t bytes) {
            r[c++] = Range{reinterpret_cast<uintptr_t>(p), reinterpret_cast<uintptr_t>(p) + bytes};
        };
        for (int i = 0; i < 4; ++i) {
            add(x.g[i], n[i] * 4);
            if (step < 1) continue;
            add(x.p[i], n[i] * 4);
            add(x.m[i], n[i] * 4);
            add(x.v[i], n[i] * 4);
        }
        if (step > 0) {
            add(x.W1b, n[0] * 2);
            add(x.W2b, n[2] * 2);
        }
        return c;
    };
    Range ra[18], rb[18];
    const int na = ranges(a, ra), nb = ranges(b, rb);
    for (int i = 0; i < na; ++i)
        for (int j = 0; j < nb; ++j)
            if (ra[i].begin < rb[j].end && rb[j].begin < ra[i].end) return false;
    return true;
}

// One training step around a loss: both towers' forward, `loss` (which
// enqueues the logits, the loss rows and the embeddings' gradients b.de), both
// backwards, `inputs` (work that needs the old weights), Adam when step >= 1
// and the mean of the loss rows.
template <class Loss, class Inputs>
ann_status train_towers(ann_tower &qt, ann_tower &ht, const ann_tower_grads &qg, const ann_tower_grads &hg,
                        const ann_adam_state *qa, const ann_adam_state *ha, const TowerBufs &bq,
                        const TowerBufs &bh, const float *xq, const int32_t *iq, int rq, const float *xh,
                        const int32_t *ih, int rh, float lr, int step, const float *loss_rows, int loss_count,
                        float *mean_loss, Loss loss, Inputs inputs, hipStream_t st)
{
    GradPair g{{grad_args(qt, qg, qa, bq, rq), grad_args(ht, hg, ha, bh, rh)},
               step > 0 ? adam_step(step, lr) : AdamStep{}, step, loss_rows, loss_count, mean_loss};
    if (fused_ok(qt, xq) && fused_ok(ht, xh) && written_apart(g.t[0], g.t[1], step)) {
        TowerPair p{{tower_args(qt, bq, xq, iq, rq), tower_args(ht, bh, xh, ih, rh)}, row_blocks(rq)};
        const dim3 grid((unsigned)(p.blocks0 + row_blocks(rh)));
        const int din = qt.din > ht.din ? qt.din : ht.din;
        const size_t lds = fused_lds(din, qt.hidden, qt.dout);
        hipLaunchKernelGGL(tower_fwd_kernel<true>, grid, dim3(256), lds, st, p);
        ANN_LAUNCHED();
        TRY(loss());
        hipLaunchKernelGGL(tower_bwd_rows_kernel, grid, dim3(256), (size_t)32 * (qt.dout + 8), st, p);
        ANN_LAUNCHED();
        TRY(inputs());
        hipLaunchKernelGGL(tower_grad_kernel, dim3((unsigned)(g.t[0].blocks + g.t[1].blocks + 1)), dim3(256),
                           0, st, g);
        ANN_LAUNCHED();
        return ANN_OK;
    }
    hipLaunchKernelGGL(gather_bf16_kernel, dim3(gridn((int64_t)rq * qt.din)), dim3(256), 0, st, xq, qt.din, iq,
                       rq, qt.in_scale, bq.xb);
    ANN_LAUNCHED();
    TRY(tower_fwd(qt, bq, rq, st));
    hipLaunchKernelGGL(gather_bf16_kernel, dim3(gridn((int64_t)rh * ht.din)), dim3(256), 0, st, xh, ht.din, ih,
                       rh, ht.in_scale, bh.xb);
    ANN_LAUNCHED();
    TRY(tower_fwd(ht, bh, rh, st));
    TRY(loss());
    hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, st, loss_rows, loss_count, mean_loss);
    ANN_LAUNCHED();
    TRY(tower_bwd(qt, qg, bq, rq, st));
    TRY(tower_bwd(ht, hg, bh, rh, st));
    TRY(inputs());
    if (step > 0) {
        TRY(adam(qt, qg, *qa, step, lr, st));
        TRY(adam(ht, hg, *ha, step, lr, st));
    }
    return ANN_OK;
}

ann_status check_tower(const ann_tower *w, const char *name)
{
    ANN_REQUIRE(w != nullptr, "%s tower is NULL", name);
    ANN_REQUIRE(w->W1 && w->b1 && w->W2 && w->b2 && w->W1b && w->W2b, "%s tower has a NULL pointer",
                name);
    ANN_REQUIRE(w->din >= 1 && w->hidden >= 1 && w->dout >= 1, "%s tower has a bad shape", name);
    ANN_REQUIRE(w->in_scale > 0.f, "%s tower in_scale must be > 0", name);
    ANN_SUPPORTED(w->dout <= 1024 && w->hidden <= 4096 && w->din <= 4096, "%s tower too large",
                  name);
    return ANN_OK;
}

}  // namespace

size_t tower_forward_ws(int rows, const ann_tower *w)
{
    return tower_bufs_bytes(rows, w->din, w->hidden, w->dout) + 256;
}

size_t train_step_ws(int batch, int nh, int din_q, int din_h, int hidden, int dout)
{
    size_t b = tower_bufs_bytes(batch, din_q, hidden, dout) + tower_bufs_bytes(nh, din_h, hidden, dout);
    b += round_up((size_t)batch * nh * 4, 256) * 2;    // logits, dlogits
    b += round_up((size_t)batch * 4, 256) + 1024;
    return b;
}

size_t train_hub_ws(int bh, int P, int N, int din_q, int din_h, int hidden, int dout)
{
    const int rows = bh * (P + N);
    size_t b = tower_bufs_bytes(rows, din_q, hidden, dout) + tower_bufs_bytes(bh, din_h, hidden, dout);
    b += round_up((size_t)bh * rows * 4, 256) * 2;     // scores, their gradient
    b += round_up((size_t)bh * 4, 256) + 1024;
    return b;
}

// forward of one tower over rows of x (FP32, rows x din) -> unit embeddings
ann_status tower_forward_run(const ann_tower &w, const float *x, const int32_t *idx, int rows,
                             float *out, void *ws, hipStream_t st)
{
    Carve cv{static_cast<unsigned char *>(ws)};
    TowerBufs b = carve_tower(cv, rows, w.din, w.hidden, w.dout);
    b.e = out;
    if (rows > 0 && fused_ok(w, x)) {
        const TowerArgs a = tower_args(w, b, x, idx, rows);
        const TowerPair p{{a, a}, row_blocks(rows)};
        hipLaunchKernelGGL(tower_fwd_kernel<false>, dim3((unsigned)row_blocks(rows)), dim3(256),
                           fused_lds(w.din, w.hidden, w.dout), st, p);
        ANN_LAUNCHED();
        return ANN_OK;
    }
    hipLaunchKernelGGL(gather_bf16_kernel, dim3(gridn((int64_t)rows * w.din)), dim3(256), 0, st, x,
                       w.din, idx, rows, w.in_scale, b.xb);
    ANN_LAUNCHED();
    return tower_fwd(w, b, rows, st);
}

ann_status refresh_bf16(const ann_tower &w, hipStream_t st)
{
    const int64_t n1 = (int64_t)w.hidden * w.din, n2 = (int64_t)w.dout * w.hidden;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(gridn(n1)), dim3(256), 0, st, w.W1, n1, w.W1b);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(to_bf16_kernel, dim3(gridn(n2)), dim3(256), 0, st, w.W2, n2, w.W2b);
    ANN_LAUNCHED();
    return ANN_OK;
}

}  // namespace ann

using namespace ann;

extern "C" ann_status ann_hub_input(const float *base, int64_t n, int32_t dim, const int32_t *hub_ids,
                                    int32_t n_hubs, const float *features, int32_t n_feat,
                                    float vec_scale, float *out, void *stream)
{
    ANN_REQUIRE(base && hub_ids && out, "a required pointer is NULL");
    ANN_REQUIRE(n_feat == 0 || features, "features is NULL");
    ANN_REQUIRE(n >= 1 && dim >= 1 && n_hubs >= 1 && n_feat >= 0, "bad sizes");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t count = (int64_t)n_hubs * (dim + n_feat);
    hipLaunchKernelGGL(hub_input_kernel, dim3(gridn(count)), dim3(256), 0, st, base, dim, hub_ids,
                       features, n_feat, n_hubs, vec_scale, out, (uint16_t *)nullptr);
    ANN_LAUNCHED();
    return ANN_OK;
}

extern "C" size_t ann_tower_workspace_size(const ann_tower *tower, int32_t rows)
{
    return tower ? tower_forward_ws(rows, tower) : 0;
}

extern "C" size_t ann_train_workspace_size(int32_t batch, int32_t n_hubs, int32_t din_q,
                                           int32_t din_h, int32_t hidden, int32_t dout)
{
    return train_step_ws(batch, n_hubs, din_q, din_h, hidden, dout);
}

extern "C" ann_status ann_tower_sync(const ann_tower *tower, void *stream)
{
    ann_status s = check_tower(tower, "the");
    if (s != ANN_OK) return s;
    return refresh_bf16(*tower, static_cast<hipStream_t>(stream));
}

extern "C" ann_status ann_tower_forward(const ann_tower *tower, const float *x, int32_t rows,
                                        float *out, void *workspace, size_t ws_bytes, void *stream)
{
    ann_status s = check_tower(tower, "the");
    if (s != ANN_OK) return s;
    ANN_REQUIRE(rows >= 0, "rows must be >= 0");
    ANN_REQUIRE(rows == 0 || (x && out && workspace), "a required pointer is NULL");
    ANN_REQUIRE(ws_bytes >= tower_forward_ws(rows, tower), "workspace too small");
    if (rows == 0) return ANN_OK;
    return tower_forward_run(*tower, x, nullptr, rows, out, workspace,
                             static_cast<hipStream_t>(stream));
}

extern "C" ann_status ann_train_step(ann_tower *qt, ann_tower *ht, const ann_tower_grads *qg,
                                     const ann_tower_grads *hg, const ann_adam_state *qa,
                                     const ann_adam_state *ha, const float *train_q,
                                     const int32_t *batch_idx, int32_t batch,
                                     const int32_t *labels, const float *hub_in, int32_t n_hubs,
                                     float tau, float lr, int32_t step, float *loss,
                                     float *q_emb, float *h_emb, float *hub_in_grad,
                                     void *workspace, size_t ws_bytes, void *stream)
{
    ann_status s = check_tower(qt, "query");
    if (s != ANN_OK) return s;
    s = check_tower(ht, "hub");
    if (s != ANN_OK) return s;
    ANN_REQUIRE(qg && hg, "gradient buffers are NULL");
    ANN_REQUIRE(qg->gW1 && qg->gb1 && qg->gW2 && qg->gb2 && hg->gW1 && hg->gb1 && hg->gW2 && hg->gb2,
                "a gradient pointer is NULL");
    ANN_REQUIRE(train_q && labels && hub_in && loss && workspace, "a required pointer is NULL");
    ANN_REQUIRE(batch >= 1 && n_hubs >= 1, "batch and n_hubs must be >= 1");
    ANN_REQUIRE(qt->dout == ht->dout && qt->hidden == ht->hidden,
                "towers must share hidden and output sizes");
    ANN_REQUIRE(tau > 0.f, "tau must be > 0");
    ANN_REQUIRE(step >= 0, "step must be >= 0");
    ANN_REQUIRE(step == 0 || (qa && ha), "Adam state needed when step > 0");
    ANN_REQUIRE(ws_bytes >= train_step_ws(batch, n_hubs, qt->din, ht->din, qt->hidden, qt->dout),
                "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    TowerBufs bq = carve_tower(cv, batch, qt->din, qt->hidden, qt->dout);
    TowerBufs bh = carve_tower(cv, n_hubs, ht->din, ht->hidden, ht->dout);
    float *logits = cv.take<float>((size_t)batch * n_hubs);
    float *dlog = cv.take<float>((size_t)batch * n_hubs);
    float *lrow = cv.take<float>((size_t)batch);
    if (q_emb) bq.e = q_emb;
    if (h_emb) bh.e = h_emb;

    const int e = qt->dout;
    auto contrast = [&]() -> ann_status {
        GemmF lg{bq.e, e, 1, bh.e, e, 1, batch, n_hubs, e, 1.f / tau, logits, n_hubs};
        TRY(gemm_f32(lg, nullptr, st));
        hipLaunchKernelGGL(softmax_ce_kernel, dim3((batch + 3) / 4), dim3(256), 0, st, logits, batch,
                           n_hubs, labels, batch_idx, 1.f / (float)batch, dlog, lrow);
        ANN_LAUNCHED();
        // dEq [batch x e] = dlog . Eh / tau ; dEh [nh x e] = dlog^T . Eq / tau
        GemmF gq{dlog, n_hubs, 1, bh.e, 1, e, batch, e, n_hubs, 1.f / tau, bq.de, e};
        GemmF gh{dlog, 1, n_hubs, bq.e, 1, e, n_hubs, e, batch, 1.f / tau, bh.de, e};
        return gemm_f32(gq, &gh, st);
    };
    auto inputs = [&]() -> ann_status {
        if (!hub_in_grad) return ANN_OK;
        // dL/d hub_in [n_hubs x din_h] = in_scale * (dz1b . W1b)
        GemmArgs g{};
        g.A = bh.dz1b;
        g.sam = ht->hidden;
        g.sak = 1;
        g.B = ht->W1b;
        g.sbn = 1;
        g.sbk = ht->din;
        g.M = n_hubs;
        g.N = ht->din;
        g.K = ht->hidden;
        g.C = hub_in_grad;
        g.ldc = ht->din;
        TRY(gemm_bf16(g, st));
        if (ht->in_scale != 1.f) {
            const int64_t cnt = (int64_t)n_hubs * ht->din;
            hipLaunchKernelGGL(scale_kernel, dim3(gridn(cnt)), dim3(256), 0, st, hub_in_grad, cnt,
                               ht->in_scale);
            ANN_LAUNCHED();
        }
        return ANN_OK;
    };
    return train_towers(*qt, *ht, *qg, *hg, qa, ha, bq, bh, train_q, batch_idx, batch, hub_in, nullptr, n_hubs,
                        lr, step, lrow, batch, loss, contrast, inputs, st);
}

extern "C" size_t ann_train_hub_workspace_size(int32_t hubs, int32_t P, int32_t N, int32_t din_q,
                                               int32_t din_h, int32_t hidden, int32_t dout)
{
    if (hubs < 1 || P < 1 || N < 0) return 0;
    return train_hub_ws(hubs, P, N, din_q, din_h, hidden, dout);
}

extern "C" ann_status ann_train_step_hub(ann_tower *qt, ann_tower *ht, const ann_tower_grads *qg,
                                         const ann_tower_grads *hg, const ann_adam_state *qa,
                                         const ann_adam_state *ha, const float *train_q,
                                         const int32_t *q_idx, const int32_t *hub_idx,
                                         int32_t hubs, int32_t P, int32_t N, const float *hub_in,
                                         float tau, float lr, int32_t step, float *loss,
                                         float *q_emb, float *h_emb, void *workspace,
                                         size_t ws_bytes, void *stream)
{
    ann_status s = check_tower(qt, "query");
    if (s != ANN_OK) return s;
    s = check_tower(ht, "hub");
    if (s != ANN_OK) return s;
    ANN_REQUIRE(qg && hg, "gradient buffers are NULL");
    ANN_REQUIRE(qg->gW1 && qg->gb1 && qg->gW2 && qg->gb2 && hg->gW1 && hg->gb1 && hg->gW2 && hg->gb2,
                "a gradient pointer is NULL");
    ANN_REQUIRE(train_q && q_idx && hub_idx && hub_in && loss && workspace,
                "a required pointer is NULL");
    ANN_REQUIRE(hubs >= 1 && P >= 1 && N >= 0, "need hubs >= 1, P >= 1, N >= 0");
    ANN_REQUIRE(qt->dout == ht->dout && qt->hidden == ht->hidden,
                "towers must share hidden and output sizes");
    ANN_REQUIRE(tau > 0.f, "tau must be > 0");
    ANN_REQUIRE(step >= 0, "step must be >= 0");
    ANN_REQUIRE(step == 0 || (qa && ha), "Adam state needed when step > 0");
    ANN_REQUIRE(ws_bytes >= train_hub_ws(hubs, P, N, qt->din, ht->din, qt->hidden, qt->dout),
                "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int rows = hubs * (P + N);
    Carve cv{static_cast<unsigned char *>(workspace)};
    TowerBufs bq = carve_tower(cv, rows, qt->din, qt->hidden, qt->dout);
    TowerBufs bh = carve_tower(cv, hubs, ht->din, ht->hidden, ht->dout);
    float *sc = cv.take<float>((size_t)hubs * rows);
    float *dsc = cv.take<float>((size_t)hubs * rows);
    float *lrow = cv.take<float>((size_t)hubs);
    if (q_emb) bq.e = q_emb;
    if (h_emb) bh.e = h_emb;

    const int e = qt->dout;
    auto contrast = [&]() -> ann_status {
        // scores [hubs x rows] = Eh . Eq^T / tau (only each hub's own block is used)
        GemmF lg{bh.e, e, 1, bq.e, e, 1, hubs, rows, e, 1.f / tau, sc, rows};
        TRY(gemm_f32(lg, nullptr, st));
        hipLaunchKernelGGL(hub_ce_kernel, dim3((hubs + 3) / 4), dim3(256), 0, st, sc, hubs, rows, P, N,
                           1.f / (float)hubs, dsc, lrow);
        ANN_LAUNCHED();
        // dEh [hubs x e] = dS . Eq / tau ; dEq [rows x e] = dS^T . Eh / tau
        GemmF gh{dsc, rows, 1, bq.e, 1, e, hubs, e, rows, 1.f / tau, bh.de, e};
        GemmF gq{dsc, 1, rows, bh.e, 1, e, rows, e, hubs, 1.f / tau, bq.de, e};
        return gemm_f32(gh, &gq, st);
    };
    return train_towers(*qt, *ht, *qg, *hg, qa, ha, bq, bh, train_q, q_idx, rows, hub_in, hub_idx,
                        hubs, lr, step, lrow, hubs, loss, contrast, []() -> ann_status { return ANN_OK; }, st);
}
