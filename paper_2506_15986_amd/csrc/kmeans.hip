// Hub nodes (Definition 3) on Lloyd k-means clusters.
//
// Assignment: each point goes to argmin_c (d2(x, mu_c), c) where d2 is the
// FP64 sum over dimensions in order, each term (x_j - mu_cj)^2 rounded
// separately (no fused multiply-add) -- the same arithmetic as a plain
// sequential loop, so every decision is reproducible bit for bit.  The matrix
// cores find, with a certified bound, the few centroids that can be the
// argmin, and FP64 decides among them.
// Update: per-cluster FP64 sums over the points sorted by cluster, pieces added
// by atomics (exact when the data sit on a dyadic grid whose partial sums fit
// in 53 bits, so order does not matter), mean = sum / count; an empty cluster
// keeps its centroid.  The loop stops after an assignment step that changes
// nothing, or after `iters` steps.
// Hub of a cluster: the member nearest its mean by (d2, id); an empty
// cluster takes the nearest point that is not yet a hub (cluster order).
#include <cmath>
#include <unordered_set>
#include <vector>

#include "common.h"
#include "internal.h"

namespace ann {
namespace {

constexpr int KP = 64;    // points per block
constexpr int KC = 32;    // centroids per LDS chunk
constexpr int KD = 128;   // dims per LDS stage

__device__ inline double term(float x, double m)
{
#pragma clang fp contract(off)
    double t = (double)x - m;
    return t * t;
}

// vec4: both rows are whole and 16-byte aligned, and x's are read in float4s
// (a lane walks its own row, so the loads, not the sums, are the cost)
__device__ inline double d2_to(const float *x, const double *m, int dim, bool vec4)
{
#pragma clang fp contract(off)
    double s = 0.0;
    if (vec4) {
#pragma unroll 8
        for (int j = 0; j < dim; j += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(x + j);
            const double2 a = *reinterpret_cast<const double2 *>(m + j);
            const double2 b = *reinterpret_cast<const double2 *>(m + j + 2);
            s = s + term(v.x, a.x);
            s = s + term(v.y, a.y);
            s = s + term(v.z, b.x);
            s = s + term(v.w, b.y);
        }
    } else {
        for (int j = 0; j < dim; ++j) s = s + term(x[j], m[j]);
    }
    return s;
}

__global__ void __launch_bounds__(256) assign_kernel(const float *base, int64_t n, int dim,
                                                     const double *mu, int nh, int32_t *assign,
                                                     int32_t *changed)
{
#pragma clang fp contract(off)
    __shared__ float xs[KP][KD + 1];
    __shared__ double ms[KC][KD];
    __shared__ double bestv[4][KP];
    __shared__ int bestc[4][KP];
    const int t = threadIdx.x;
    const int p = t & 63;          // point within the block
    const int g = t >> 6;          // wave: centroids 8g..8g+7 of each chunk
    const int64_t i = (int64_t)blockIdx.x * KP + p;
    double bv = __longlong_as_double(0x7ff0000000000000ll);
    int bc = 0x7fffffff;
    for (int c0 = 0; c0 < nh; c0 += KC) {
        double acc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = 0.0;
        for (int d0 = 0; d0 < dim; d0 += KD) {
            const int dd = dim - d0 < KD ? dim - d0 : KD;
            __syncthreads();
            for (int e = t; e < KP * KD; e += 256) {
                int r = e / KD, j = e % KD;
                int64_t g2 = (int64_t)blockIdx.x * KP + r;
                xs[r][j] = (g2 < n && j < dd) ? base[g2 * dim + d0 + j] : 0.f;
            }
            for (int e = t; e < KC * KD; e += 256) {
                int r = e / KD, j = e % KD;
                ms[r][j] = (c0 + r < nh && j < dd) ? mu[(int64_t)(c0 + r) * dim + d0 + j] : 0.0;
            }
            __syncthreads();
            for (int j = 0; j < dd; ++j) {
                const float xv = xs[p][j];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[u] = acc[u] + term(xv, ms[8 * g + u][j]);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            int c = c0 + 8 * g + u;
            if (c < nh && (acc[u] < bv || (acc[u] == bv && c < bc))) {
                bv = acc[u];
                bc = c;
            }
        }
    }
    bestv[g][p] = bv;
    bestc[g][p] = bc;
    __syncthreads();
    if (g == 0 && i < n) {
        for (int q = 1; q < 4; ++q) {
            double v = bestv[q][p];
            int c = bestc[q][p];
            if (v < bv || (v == bv && c < bc)) {
                bv = v;
                bc = c;
            }
        }
        if (bc == 0x7fffffff) bc = 0;   // no distance is a number
        if (assign[i] != bc) {
            assign[i] = bc;
            *changed = 1;
        }
    }
}

// ---- assignment on the matrix cores in FP32, with a certified shortlist: for
// the points that the FP16 products below leave open, for small calls, and for
// more centroids or dimensions than those take.
//
// The matrix cores compute the dot products x . mu~ in FP32
// (v_mfma_f32_16x16x4_f32; mu~ = the FP32 rounding of the FP64 centroid) and
// each pair gets the estimate s = (|x|^2 + |mu|^2) - 2 x . mu~ in FP32 with a
// rigorous bound E on its distance from the FP64 distance of the plain
// step (coefficients ea, eb from the host: FP32 rounding of the norms, of mu~,
// of the dot product's accumulation over dim terms and of s itself).  Every
// centroid whose lower bound s - E does not exceed the smallest upper bound
// s + E of the point is kept on a shortlist (the plain step's argmin is
// always on it); the point then takes its only candidate, or the plain
// step's FP64 argmin over its few candidates, or -- when more than MLIST
// centroids tie that closely (repeated centroids) -- over all centroids.
// The result is the plain step's assignment bit for bit.
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int MP = 64;     // points per block (16 per wavefront)
constexpr int MC = 64;     // centroids per pass (four 16-wide MFMA tiles)
constexpr int MK = 32;     // dimensions per LDS stage
constexpr int MLIST = 8;   // shortlist capacity per point

struct ShortArgs {
    const float *base;
    int64_t n;
    int dim;
    const double *mu;      // nh x dim FP64 centroids
    const float *mu32;     // their FP32 rounding
    const float *cn2;      // |mu|^2 per centroid (FP64 sum, rounded to FP32)
    const float *cn;       // |mu|
    const float *xn2;      // |x|^2 per point
    const float *xn;       // |x|
    int nh;
    float ea, eb;          // E = ea (|x|^2 + |mu|^2) + eb |x| |mu|
    int32_t *assign;
    int32_t *changed;
    const int2 *list;      // NULL, or the points to assign,
    const int32_t *count;  // how many they are,
    int few;               // and up to how many are left alone
    bool vec4;             // mu's rows are aligned too
};

__global__ void point_norms_kernel(const float *base, int64_t n, int dim, float *xn2, float *xn)
{
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
#pragma unroll 8
    for (int j = 0; j < dim; j += 4) {
        const float4 v = *reinterpret_cast<const float4 *>(base + i * dim + j);
        s = s + (double)v.x * v.x;
        s = s + (double)v.y * v.y;
        s = s + (double)v.z * v.z;
        s = s + (double)v.w * v.w;
    }
    xn2[i] = (float)s;
    xn[i] = (float)sqrt(s);
}

__global__ void __launch_bounds__(256) assign_mfma_kernel(ShortArgs a)
{
#pragma clang fp contract(off)
    __shared__ float xs[MP][MK + 1];
    __shared__ float ms[MC][MK + 1];
    __shared__ float U[MP];
    __shared__ int cnt[MP];
    __shared__ int64_t pid[MP];   // the block's points, -1 past the last
    __shared__ int lc[MP][MLIST];
    __shared__ float ll[MP][MLIST];
    const float inf = __builtin_inff();
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const int64_t total = a.list ? *a.count : a.n;
    if (a.list && total <= a.few) return;
    for (int64_t p0 = (int64_t)blockIdx.x * MP; p0 < total; p0 += (int64_t)gridDim.x * MP) {
    __syncthreads();
    if (t < MP) {
        U[t] = inf;
        cnt[t] = 0;
        pid[t] = p0 + t >= total ? -1 : a.list ? a.list[p0 + t].x : p0 + t;
    }
    __syncthreads();
    // this lane's rows of the 16 x 16 output tiles: points 16w + 4 (lane >> 4) + i
    float X[4], XN[4];
    bool live[4];
    for (int i = 0; i < 4; ++i) {
        const int64_t pi = pid[16 * w + 4 * (lane >> 4) + i];
        live[i] = pi >= 0;
        X[i] = live[i] ? a.xn2[pi] : 0.f;
        XN[i] = live[i] ? a.xn[pi] : 0.f;
    }
    for (int c0 = 0; c0 < a.nh; c0 += MC) {
        v4f acc[4];
        for (int b = 0; b < 4; ++b) acc[b] = v4f{0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < a.dim; k0 += MK) {
            __syncthreads();
            for (int e = t; e < MP * (MK / 4); e += 256) {
                const int r = e / (MK / 4), j = 4 * (e % (MK / 4));
                const int64_t gi = pid[r];
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (gi >= 0 && k0 + j < a.dim)
                    v = *reinterpret_cast<const float4 *>(a.base + gi * a.dim + k0 + j);
                xs[r][j] = v.x;
                xs[r][j + 1] = v.y;
                xs[r][j + 2] = v.z;
                xs[r][j + 3] = v.w;
                const int c = c0 + r;
                float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
                if (c < a.nh && k0 + j < a.dim)
                    m = *reinterpret_cast<const float4 *>(a.mu32 + (int64_t)c * a.dim + k0 + j);
                ms[r][j] = m.x;
                ms[r][j + 1] = m.y;
                ms[r][j + 2] = m.z;
                ms[r][j + 3] = m.w;
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < MK / 4; ++q) {
                const float av = xs[16 * w + (lane & 15)][4 * q + (lane >> 4)];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const float bv = ms[16 * b + (lane & 15)][4 * q + (lane >> 4)];
                    acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[b], 0, 0, 0);
                }
            }
        }
        // bounds of this pass's pairs; the smallest upper bound per point
        float lo[4][4], hmin[4];
        for (int i = 0; i < 4; ++i) {
            hmin[i] = inf;
            for (int b = 0; b < 4; ++b) {
                const int c = c0 + 16 * b + (lane & 15);
                lo[i][b] = inf;
                if (!live[i] || c >= a.nh) continue;
                const float C = a.cn2[c];
                const float s1 = X[i] + C;
                const float sv = s1 - 2.f * acc[b][i];
                const float e1 = a.ea * s1;
                const float e2 = a.eb * (XN[i] * a.cn[c]);
                const float E = e1 + e2;
                lo[i][b] = sv - E;
                const float hv = sv + E;
                hmin[i] = hv < hmin[i] ? hv : hmin[i];
            }
            for (int o = 1; o < 16; o <<= 1) {
                const float h2 = __shfl_xor(hmin[i], o);
                hmin[i] = h2 < hmin[i] ? h2 : hmin[i];
            }
        }
        __syncthreads();
        if ((lane & 15) == 0)
            for (int i = 0; i < 4; ++i) {
                const int P = 16 * w + 4 * (lane >> 4) + i;
                if (hmin[i] < U[P]) U[P] = hmin[i];
            }
        __syncthreads();
        // drop candidates whose lower bound now exceeds the point's bound
        if (t < MP && cnt[t] <= MLIST) {
            int m = 0;
            for (int r = 0; r < cnt[t]; ++r)
                if (ll[t][r] <= U[t]) {
                    lc[t][m] = lc[t][r];
                    ll[t][m] = ll[t][r];
                    ++m;
                }
            cnt[t] = m;
        }
        __syncthreads();
        for (int i = 0; i < 4; ++i) {
            const int P = 16 * w + 4 * (lane >> 4) + i;
            const float u = U[P];
            for (int b = 0; b < 4; ++b)
                if (lo[i][b] <= u && lo[i][b] < inf) {
                    const int slot = atomicAdd(&cnt[P], 1);
                    if (slot < MLIST) {
                        lc[P][slot] = c0 + 16 * b + (lane & 15);
                        ll[P][slot] = lo[i][b];
                    }
                }
        }
    }
    __syncthreads();
    if (t >= MP || pid[t] < 0) continue;
    const int64_t i = pid[t];
    const float *x = a.base + i * a.dim;
    int bc;
    if (cnt[t] == 1) {
        bc = lc[t][0];
    } else {
        // the plain step's FP64 argmin, over the shortlist or (when it
        // overflowed) over every centroid
        const bool all = cnt[t] > MLIST || cnt[t] == 0;
        const int m = all ? a.nh : cnt[t];
        double bv = __longlong_as_double(0x7ff0000000000000ll);
        bc = 0x7fffffff;
        for (int r = 0; r < m; ++r) {
            const int c = all ? r : lc[t][r];
            const double v = d2_to(x, a.mu + (int64_t)c * a.dim, a.dim, a.vec4);
            if (v < bv || (v == bv && c < bc)) {
                bv = v;
                bc = c;
            }
        }
    }
    if (bc == 0x7fffffff) bc = 0;   // no distance is a number
    if (a.assign[i] != bc) {
        a.assign[i] = bc;
        *a.changed = 1;
    }
    }
}

// ---- assignment on the FP16 matrix cores.
//
// Points and centroids are moved by a fixed vector c0 and scaled by a power of
// two: y = (x - c0) s, m = (mu - c0) s, with FP16 roundings yh, mh.  The
// matrix cores give V~ = yh . mh - (|m|^2 / 2 - m . (m - mh)) (the sum starts
// at the part in brackets, negated); |y - m|^2 = |y|^2 - 2 V with V = y . m -
// |m|^2 / 2, so the nearest centroid has the largest V.  With em = m - mh and
// d = |y - m|,
//   V~ - V = (m - yh) . em - (y - yh) . m, so
//   |V~ - V| <= d EM + |y - yh| (M + EM) + rounding =: d EM + F,
// M and EM the largest |m| and |em| of a step, rounding that of the FP32
// accumulation and of the low mantissa bits given up below.  Let t have the
// largest V~ and b be the plain step's argmin: V_b >= V_t and d_b <= d_t, so
// V~_b >= V~_t - 2 (d_t EM + F), where d_t^2 = |y|^2 - 2 V_t <= |y|^2 - 2 V~_t
// + 2 (d_t EM + F) bounds d_t.  (The part m . em of the centroid's rounding
// error is known and taken out: without it the bound had |y| where d is now,
// and 35 % of the points of a mixture in 128 dimensions stayed open, 0.15 ms a
// step for them against 0.04.)  F also holds the FP64 rounding of the plain step, and FP16
// denormals taken as zeros.
//
// A lane sees the centroids c = lane & 15 modulo 16 of its points and keeps
// the largest and the second largest V~ of each, the tile number written into
// the low mantissa bits: three vector instructions a pair.  A point whose only
// value in the band is a lane's largest is done; one with up to four lanes'
// largest goes to the FP64 decision among them; the others (a second value of
// one lane in the band, more than four, or a band that is no number) have the
// classes modulo 16 of those lanes searched in FP64 if they are few, and go to
// the FP32 kernel above if they are many.
//
// Bound by those three instructions and the matrix instructions, about even at
// 128 dimensions.  The centroids' fragments pass through LDS in the order in
// which the lanes read them, 16 KB at a time, shared by four wavefronts; the
// points' fragments stay in registers.  1,000,000 x 128 against 1,024 centroids:
// 0.36 ms a step (742 TFLOP/s), and 0.13 for the points left open, against 4.1
// with the FP32 products alone.
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int HB_MAX_NH = 16384;   // tile numbers of at most 10 bits
constexpr int HB_MAX_DIM = 1024;   // 32 fragments of 32 dimensions

// fragments (32 dimensions) of a row, tiles of 16 points per wavefront and
// tiles of 16 centroids in LDS
inline __host__ __device__ constexpr int row_tiles(int KS) { return KS <= 4 ? 4 : KS <= 16 ? 2 : 1; }
inline __host__ __device__ constexpr int lds_tiles(int KS) { return KS == 3 ? 4 : KS >= 16 ? 1 : 16 / KS; }
inline int frags_of(int dim)
{
    const int k = (dim + 31) / 32;
    return k <= 4 ? k : k <= 8 ? 8 : k <= 16 ? 16 : 32;
}

// The state of a step on the device.  changed, M and EM are kept for two steps
// in turn, so that the next step's can be cleared while this one's are read.
struct StepState {
    int32_t changed[2];
    int32_t n_open, n_left;      // lengths of the two lists
    float M[2], EM[2];
};

struct OpenPoint {               // up to four centroids, 0xffff for none
    int32_t point;
    uint16_t c[4];
    uint32_t pad;
};

struct HalfArgs {
    const float *base;
    int64_t n;
    int dim;
    const float *c0;
    const float *scale;
    const v4u *mh;               // fragments: tile x KS x 64 lanes x 8 halves
    const float *cv;             // |m|^2 / 2 - m . em per centroid, 1e30 past the last
    int tiles;                   // a multiple of lds_tiles(KS)
    int bits;                    // of a tile number
    float g, gb;                 // relative rounding: accumulation, tile number's bits
    StepState *state;
    int parity;
    int32_t *assign;
    OpenPoint *open;
    int2 *left;                  // point, the classes modulo 16 that hold its argmin
};

template <int KS>
__global__ void __launch_bounds__(256, KS <= 8 ? 3 : 1) assign_half_kernel(HalfArgs a)
{
    constexpr int RT = row_tiles(KS), TC = lds_tiles(KS);
    constexpr int PW = 16 * RT, PB = 4 * PW;          // points of a wavefront, of a block
    constexpr int UNITS = TC * KS * 64;               // 16-byte units of a chunk
    constexpr int PER = UNITS / 256;
    __shared__ v4u sb[2][UNITS];
    __shared__ float sc[2][TC * 16];
    __shared__ float s_f[PB], s_y2[PB];   // F and |y|^2 of the points
    __shared__ int s_n[2], s_at[2];
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int64_t p0 = (int64_t)blockIdx.x * PB + w * PW;
    const float scale = *a.scale;
    const int chunks = a.tiles / TC;
    static_assert(UNITS % 256 == 0, "a chunk is whole rounds of the block");
    v4u stage[PER];
    float stage_c = 0.f;
    auto fetch = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PER; ++u) stage[u] = a.mh[(size_t)ch * UNITS + u * 256 + t];
        if (t < TC * 16) stage_c = a.cv[ch * TC * 16 + t];
    };
    auto put = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PER; ++u) sb[buf][u * 256 + t] = stage[u];
        if (t < TC * 16) sc[buf][t] = stage_c;
    };
    fetch(0);
    if (t < 2) s_n[t] = 0;

    // this lane's fragments: row lane & 15 of each tile, dimensions
    // 32 k + 8 (lane >> 4) ... + 8
    v8h A[RT][KS];
    const float M = a.state->M[a.parity], EM = a.state->EM[a.parity];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int64_t p = p0 + 16 * r + (lane & 15);
        float h2 = 0.f, e2 = 0.f, y2 = 0.f;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int d = 32 * k + 8 * (lane >> 4) + 4 * q;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f), c = v;
                if (p < a.n && d < a.dim) {
                    v = *reinterpret_cast<const float4 *>(a.base + p * a.dim + d);
                    c = *reinterpret_cast<const float4 *>(a.c0 + d);
                }
                const float y[4] = {(v.x - c.x) * scale, (v.y - c.y) * scale, (v.z - c.z) * scale,
                                    (v.w - c.w) * scale};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const _Float16 h = (_Float16)y[j];
                    const float hf = (float)h, e = y[j] - hf;
                    A[r][k][4 * q + j] = h;
                    h2 += hf * hf;
                    e2 += e * e;
                    y2 += y[j] * y[j];
                }
            }
        }
        for (int o = 16; o < 64; o <<= 1) {
            h2 += __shfl_xor(h2, o);
            e2 += __shfl_xor(e2, o);
            y2 += __shfl_xor(y2, o);
        }
        const float yn = sqrtf(h2), tiny = 6.2e-5f * sqrtf((float)a.dim);
        const float en = sqrtf(e2) + 1.2e-7f * sqrtf(y2) + tiny;
        if (lane < 16) {
            s_f[w * PW + 16 * r + lane] =
                1.01f * (en * (M + EM) + a.g * M * (yn + 0.5f * M + EM) + 1e-12f * y2);
            s_y2[w * PW + 16 * r + lane] = 1.0002f * y2;
        }
    }
    float m1[RT][4], m2[RT][4];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) m1[r][i] = m2[r][i] = -3e38f;
    put(0);
    __syncthreads();
    // opaque, so that a value's tile number goes in with one instruction (a
    // vector mask and a scalar number)
    uint32_t keep = ~((1u << a.bits) - 1u), tile = 0u;
    asm volatile("" : "+v"(keep));
    for (int ch = 0; ch < chunks; ++ch) {
        const int buf = ch & 1;
        if (ch + 1 < chunks) fetch(ch + 1);
#pragma unroll 1
        for (int ti = 0; ti < TC; ++ti) {
            const float c = -sc[buf][16 * ti + (lane & 15)];
            v4f acc[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = v4f{c, c, c, c};
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const v8h B = *reinterpret_cast<const v8h *>(&sb[buf][(ti * KS + k) * 64 + lane]);
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[r][k], B, acc[r], 0, 0, 0);
            }
            asm volatile("" : "+s"(tile));
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = __uint_as_float((__float_as_uint(acc[r][i]) & keep) | tile);
                    m2[r][i] = __builtin_amdgcn_fmed3f(v, m1[r][i], m2[r][i]);
                    asm("v_max_f32 %0, %1, %2" : "=v"(m1[r][i]) : "v"(m1[r][i]), "v"(v));
                }
            ++tile;
        }
        if (ch + 1 < chunks) put(buf ^ 1);
        __syncthreads();
    }

    // the points: row 4 (lane >> 4) + i of each tile, its 16 lanes side by side
    OpenPoint *s_open = reinterpret_cast<OpenPoint *>(sb);                 // PB of them
    int2 *s_left = reinterpret_cast<int2 *>(s_open + PB);                  // PB
    static_assert(sizeof(sb) >= PB * (sizeof(OpenPoint) + 8), "lists fit");
    bool changed = false;
    const int g16 = lane & 48;
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * (lane >> 4) + i;
            const int64_t p = p0 + 16 * r + row;
            float top = m1[r][i];
            for (int o = 1; o < 16; o <<= 1) top = fmaxf(top, __shfl_xor(top, o));
            const float f = s_f[w * PW + 16 * r + row] + a.gb * fabsf(top);
            const float d2 = fmaxf(s_y2[w * PW + 16 * r + row] - 2.f * top + 4.f * f, 0.f);
            const float d = 1.001f * (2.f * EM + sqrtf(d2));
            const float thr = top - 2.02f * (d * EM + f);
            const bool cand = m1[r][i] >= thr;
            const bool clear = m2[r][i] < thr;
            const uint32_t cb = (uint32_t)(__ballot(cand) >> g16) & 0xffffu;
            const uint32_t nb = (uint32_t)(__ballot(clear) >> g16) & 0xffffu;
            const int m = __popc(cb);
            const uint32_t c = 16u * (__float_as_uint(m1[r][i]) & ~keep) + (uint32_t)(lane & 15);
            if (p >= a.n) continue;
            if (nb == 0xffffu && m == 1) {
                if (cand && a.assign[p] != (int32_t)c) {
                    a.assign[p] = (int32_t)c;
                    changed = true;
                }
            } else if (nb == 0xffffu && m >= 2 && m <= 4) {
                int at = 0;
                if ((lane & 15) == 0) at = atomicAdd(&s_n[0], 1);
                at = __shfl(at, g16);
                if ((lane & 15) == 0) s_open[at].point = (int32_t)p;
                // places 0 .. m - 1 and m .. 3: each written once
                if (cand) s_open[at].c[__popc(cb & ((1u << (lane & 15)) - 1u))] = (uint16_t)c;
                if ((lane & 15) >= m && (lane & 15) < 4) s_open[at].c[lane & 15] = 0xffff;
            } else if ((lane & 15) == 0) {
                s_left[atomicAdd(&s_n[1], 1)] = make_int2((int)p, (int)(cb | (~nb & 0xffffu)));
            }
        }
    if (__any(changed) && lane == 0) a.state->changed[a.parity] = 1;
    __syncthreads();
    if (t < 2 && s_n[t]) s_at[t] = atomicAdd(t ? &a.state->n_left : &a.state->n_open, s_n[t]);
    __syncthreads();
    for (int e = t; e < s_n[0]; e += 256) a.open[s_at[0] + e] = s_open[e];
    for (int e = t; e < s_n[1]; e += 256) a.left[s_at[1] + e] = s_left[e];
}

// the plain step's FP64 argmin among a point's open centroids: four lanes each
__global__ void __launch_bounds__(256) open_kernel(const float *base, int dim, bool vec4,
                                                   const double *mu, const OpenPoint *open,
                                                   const int32_t *count, int32_t *assign,
                                                   int32_t *changed)
{
    const int64_t total = 4 * (int64_t)*count;     // more than 2^31 from 2^29 points on
    const int sub = threadIdx.x & 3;
    // every lane of a group of four takes part in the exchange below
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const OpenPoint &o = open[e >> 2];
        int c = o.c[sub];
        double v = __longlong_as_double(0x7ff0000000000000ll);
        if (c != 0xffff) v = d2_to(base + (int64_t)o.point * dim, mu + (int64_t)c * dim, dim, vec4);
        for (int x = 1; x < 4; x <<= 1) {
            const double ov = __shfl_xor(v, x);
            const int oc = __shfl_xor(c, x);
            if (ov < v || (ov == v && oc < c)) {
                v = ov;
                c = oc;
            }
        }
        if (sub == 0 && assign[o.point] != c) {
            assign[o.point] = c;
            *changed = 1;
        }
    }
}

// the plain step's FP64 argmin in the classes of the points left, one wavefront
// a point and one centroid a lane, when they are at most `few`.  The FP32
// kernel takes 0.2 ms for any number up to some thousands (a block goes through
// all centroids for its 64 points), this one 0.07 to 0.09 for about 5,000.
constexpr int LEFT_FEW = 16384;

__global__ void __launch_bounds__(256) left_kernel(const float *base, int dim, bool vec4,
                                                   const double *mu, int nh, const int2 *left,
                                                   const int32_t *count, int few, int32_t *assign,
                                                   int32_t *changed)
{
    const int total = *count;
    if (total > few) return;
    const int lane = threadIdx.x & 63;
    for (int e = blockIdx.x * 4 + (int)(threadIdx.x >> 6); e < total; e += gridDim.x * 4) {
        const int2 l = left[e];
        double v = __longlong_as_double(0x7ff0000000000000ll);
        int c = 0x7fffffff;
        for (int mask = l.y; mask; mask &= mask - 1) {
            for (int q = __ffs(mask) - 1 + 16 * lane; q < nh; q += 1024) {
                const double d = d2_to(base + (int64_t)l.x * dim, mu + (int64_t)q * dim, dim, vec4);
                if (d < v || (d == v && q < c)) {
                    v = d;
                    c = q;
                }
            }
        }
        for (int o = 1; o < 64; o <<= 1) {
            const double ov = __shfl_xor(v, o);
            const int oc = __shfl_xor(c, o);
            if (ov < v || (ov == v && oc < c)) {
                v = ov;
                c = oc;
            }
        }
        if (c == 0x7fffffff) c = 0;   // no distance is a number
        if (lane == 0 && assign[l.x] != c) {
            assign[l.x] = c;
            *changed = 1;
        }
    }
}

// c0: the mean of up to 256 of the initial centroids, on a grid of 2^-8 of
// their spread (so whole numbers stay whole numbers); scale: takes the spread
// to about 64.  Any vector and scale would do; they only set how wide E is.
__global__ void __launch_bounds__(1024) frame_kernel(const double *mu, int nh, int dim, float *c0,
                                                     float *scale)
{
    __shared__ float part[1024];
    const int t = threadIdx.x;
    const int groups = 1024 / dim, rows = nh < 256 ? nh : 256;   // dim <= 1024
    const int j = t % dim, gr = t / dim;
    float s = 0.f;
    if (gr < groups)
        for (int r = gr; r < rows; r += groups) s += (float)mu[(int64_t)r * nh / rows * dim + j];
    part[t] = s;
    __syncthreads();
    float mean = 0.f;
    for (int q = 0; q < groups; ++q) mean += part[q * dim + j];
    mean /= (float)rows;
    float far = 0.f;
    if (gr < groups)
        for (int r = gr; r < rows; r += groups)
            far = fmaxf(far, fabsf((float)mu[(int64_t)r * nh / rows * dim + j] - mean));
    __syncthreads();
    part[t] = far;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (t < o) part[t] = fmaxf(part[t], part[t + o]);
        __syncthreads();
    }
    far = part[0];
    int e = 0;
    if (far > 1e-30f && far < 1e30f) frexpf(far, &e);   // far < 2^e
    if (t < dim) c0[t] = ldexpf(rintf(ldexpf(mean, 8 - e)), e - 8);
    if (t == 0) *scale = ldexpf(1.f, 6 - e);
}

// A wavefront per centroid.  Takes the step's mean (count > 0), clears the sums
// and the count for the next one, and lays down what the next assignment reads:
// the FP32 rounding and norms, and for the FP16 products the fragments,
// where the sums start and the largest |m| and |em|.  Wavefronts past the last
// centroid lay down the padding.
struct CentroidArgs {
    double *mu, *sums;
    int64_t *count;
    int nh, dim;
    bool update;           // false before the first step
    float *mu32, *cn2, *cn;   // NULL: not wanted
    _Float16 *mh;             // NULL: not wanted
    float *cv;
    int padded, KS;
    const float *c0, *scale;
    StepState *state;
    int parity;            // of the next step
};

constexpr int CENTROID_WAVES = 16;

__global__ void __launch_bounds__(64 * CENTROID_WAVES) centroid_kernel(CentroidArgs a)
{
    // >= 0 (or not a number, which compares above): bit order = value order
    __shared__ int s_max[2];
    const int c = blockIdx.x * CENTROID_WAVES + (int)(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 2) s_max[threadIdx.x] = 0;
    __syncthreads();
    const bool real = c < a.nh;
    const double members = real ? (double)a.count[c] : 0.0;
    double s2 = 0.0, h2 = 0.0, e2 = 0.0, me = 0.0;
    const int width = c >= a.padded ? 0 : a.mh ? 32 * a.KS : a.dim;
    for (int j = lane; j < width; j += 64) {
        const int64_t at = (int64_t)c * a.dim + j;
        double v = 0.0;
        const bool in = real && j < a.dim;
        if (in) {
            v = a.mu[at];
            if (a.update) {
                if (members > 0.0) {
                    v = a.sums[at] / members;
                    a.mu[at] = v;
                }
                a.sums[at] = 0.0;
            }
            if (a.mu32) a.mu32[at] = (float)v;
            s2 += v * v;
        }
        if (a.mh) {
            const double m = in ? (v - (double)a.c0[j]) * (double)*a.scale : 0.0;
            const _Float16 h = (_Float16)(float)m;
            const double e = m - (double)(float)h;
            h2 += m * m;
            e2 += e * e;
            me += m * e;
            const int k = j >> 5, q = (j & 31) >> 3;
            a.mh[(((int64_t)(c >> 4) * a.KS + k) * 64 + 16 * q + (c & 15)) * 8 + (j & 7)] = h;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        s2 += __shfl_xor(s2, o);
        h2 += __shfl_xor(h2, o);
        e2 += __shfl_xor(e2, o);
        me += __shfl_xor(me, o);
    }
    if (lane == 0 && c < a.padded) {
        if (a.update && real) a.count[c] = 0;
        if (a.mu32 && real) {
            a.cn2[c] = (float)s2;
            a.cn[c] = (float)sqrt(s2);
        }
        if (a.mh) a.cv[c] = real ? (float)(0.5 * h2 - me) : 1e30f;
        if (a.mh && real) {
            const float em = 1.001f * (float)sqrt(e2) + 6.2e-5f * sqrtf((float)a.dim);
            const float mm = 1.001f * (float)sqrt(h2) + em;
            atomicMax(&s_max[0], __float_as_int(fabsf(mm)));
            atomicMax(&s_max[1], __float_as_int(fabsf(em)));
        }
    }
    __syncthreads();
    if (a.mh && threadIdx.x == 0) {
        atomicMax(reinterpret_cast<int *>(&a.state->M[a.parity]), s_max[0]);
        atomicMax(reinterpret_cast<int *>(&a.state->EM[a.parity]), s_max[1]);
    }
}

// ---- sums per cluster over the points sorted by cluster.
//
// One atomic per point and dimension on the clusters' sums took 0.95 ms at
// 1,000,000 x 128 (135 GB/s of additions).  A counting sort of the points (8
// bytes a point) lets a group of threads add a run of one cluster's rows in
// registers, so that the atomics are one per run: 0.14 ms, of which 0.115 are
// the rows' gather (4.4 TB/s).
constexpr int SORT_POINTS = 4096;    // points of a block of the sort
constexpr int SORT_MAX_NH = 16384;   // counters of a block in LDS

__global__ void __launch_bounds__(256) cluster_count_kernel(const int32_t *assign, int64_t n, int nh,
                                                            int64_t *count)
{
    extern __shared__ int32_t lh[];
    for (int c = threadIdx.x; c < nh; c += 256) lh[c] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * SORT_POINTS;
#pragma unroll
    for (int u = 0; u < SORT_POINTS / 256; ++u) {
        const int64_t i = b0 + u * 256 + threadIdx.x;
        if (i < n) atomicAdd(&lh[assign[i]], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < nh; c += 256)
        if (lh[c]) atomicAdd((unsigned long long *)&count[c], (unsigned long long)lh[c]);
}

// first place of every cluster; also clears the state of the next step
__global__ void __launch_bounds__(1024) cluster_scan_kernel(const int64_t *count, int nh,
                                                            int32_t *cursor, StepState *state,
                                                            int next)
{
    __shared__ int32_t part[1024];
    const int t = threadIdx.x;
    const int per = (nh + 1023) / 1024;
    int32_t sum = 0;
    for (int q = 0; q < per; ++q)
        if (t * per + q < nh) sum += (int32_t)count[t * per + q];
    part[t] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int32_t v = t >= o ? part[t - o] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int32_t at = t ? part[t - 1] : 0;
    for (int q = 0; q < per; ++q)
        if (t * per + q < nh) {
            cursor[t * per + q] = at;
            at += (int32_t)count[t * per + q];
        }
    if (t == 0) {
        state->changed[next] = 0;
        state->n_open = state->n_left = 0;
        state->M[next] = state->EM[next] = 0.f;
    }
}

__global__ void __launch_bounds__(256) cluster_sort_kernel(const int32_t *assign, int64_t n, int nh,
                                                           int32_t *cursor, int2 *sorted)
{
    extern __shared__ int32_t lh[];
    for (int c = threadIdx.x; c < nh; c += 256) lh[c] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * SORT_POINTS;
    int cl[SORT_POINTS / 256], rank[SORT_POINTS / 256];
#pragma unroll
    for (int u = 0; u < SORT_POINTS / 256; ++u) {
        const int64_t i = b0 + u * 256 + threadIdx.x;
        cl[u] = i < n ? assign[i] : -1;
        rank[u] = cl[u] >= 0 ? atomicAdd(&lh[cl[u]], 1) : 0;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < nh; c += 256)
        if (lh[c]) lh[c] = atomicAdd(&cursor[c], lh[c]);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < SORT_POINTS / 256; ++u)
        if (cl[u] >= 0)
            sorted[lh[cl[u]] + rank[u]] = make_int2((int)(b0 + u * 256 + threadIdx.x), cl[u]);
}

// A group of `wide` threads (a row's columns, four or one to a thread) adds
// `len` sorted points.
template <int VEC>
__global__ void __launch_bounds__(256) cluster_sum_kernel(const float *base, int64_t n, int dim,
                                                          const int2 *sorted, int wide, int len,
                                                          double *sums)
{
    const int groups = 256 / wide;
    const int gr = threadIdx.x / wide;
    const int j = ((int)blockIdx.y * wide + threadIdx.x % wide) * VEC;
    const int64_t s0 = ((int64_t)blockIdx.x * groups + gr) * len;
    if (gr >= groups || j >= dim || s0 >= n) return;
    const int64_t s1 = s0 + len < n ? s0 + len : n;
    double acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
    int cur = sorted[s0].y;
    auto flush = [&]() {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            atomicAdd(&sums[(int64_t)cur * dim + j + v], acc[v]);
            acc[v] = 0.0;
        }
    };
    constexpr int U = 8;
    for (int64_t s = s0; s < s1; s += U) {
        float x[U][VEC];
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int2 e = sorted[s + u < s1 ? s + u : s1 - 1];
            c[u] = e.y;
            const float *row = base + (int64_t)e.x * dim + j;
            if (VEC == 4) {
                const float4 v = *reinterpret_cast<const float4 *>(row);
                x[u][0] = v.x;
                x[u][VEC == 4 ? 1 : 0] = v.y;
                x[u][VEC == 4 ? 2 : 0] = v.z;
                x[u][VEC == 4 ? 3 : 0] = v.w;
            } else {
                x[u][0] = *row;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + u >= s1) break;
            if (c[u] != cur) {
                flush();
                cur = c[u];
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] += (double)x[u][v];
        }
    }
    flush();
}

// one wavefront per point, one atomic per dimension: for clusters too many for
// the sort's counters in LDS, and for few values
__global__ void accumulate_kernel(const float *base, int64_t n, int dim, const int32_t *assign,
                                  double *sums, int64_t *count)
{
    const int64_t i = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    if (i >= n) return;
    const int lane = threadIdx.x & 63;
    const int c = assign[i];
    for (int j = lane; j < dim; j += 64)
        atomicAdd(&sums[(int64_t)c * dim + j], (double)base[i * dim + j]);
    if (lane == 0) atomicAdd((unsigned long long *)&count[c], 1ull);
}

__global__ void update_kernel(const double *sums, const int64_t *count, int nh, int dim, double *mu)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)nh * dim) return;
    const int64_t c = e / dim;
    if (count[c] > 0) mu[e] = sums[e] / (double)count[c];
}

__global__ void hub_min_kernel(const float *base, int64_t n, int dim, bool vec4, const double *mu,
                               const int32_t *assign, const int2 *order, unsigned long long *best_bits)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t i = order ? order[p].x : p;
    const int c = assign[i];
    const double v = d2_to(base + i * dim, mu + (int64_t)c * dim, dim, vec4);
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    // a whole wavefront in one cluster (sorted points): one atomic
    if (__ballot(c == __builtin_amdgcn_readfirstlane(c)) == ~0ull) {
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long other = __shfl_xor(b, o);
            b = other < b ? other : b;
        }
        if (__lane_id()) return;
    }
    atomicMin(&best_bits[c], b);
}

__global__ void hub_id_kernel(const float *base, int64_t n, int dim, bool vec4, const double *mu,
                              const int32_t *assign, const int2 *order, const unsigned long long *best_bits,
                              int32_t *hub)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int64_t i = order ? order[p].x : p;
    const int c = assign[i];
    double v = d2_to(base + i * dim, mu + (int64_t)c * dim, dim, vec4);
    if ((unsigned long long)__double_as_longlong(v) == best_bits[c]) atomicMin(&hub[c], (int32_t)i);
}

__global__ void init_mu_kernel(const float *base, int dim, const int32_t *init_ids, int nh,
                               double *mu)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (int64_t)nh * dim) return;
    const int64_t c = e / dim, j = e % dim;
    mu[e] = (double)base[(int64_t)init_ids[c] * dim + j];
}

__global__ void fill_i32(int32_t *p, int64_t n, int32_t v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void fill_u64(unsigned long long *p, int64_t n, unsigned long long v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void fill_f64(double *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// nearest point to each of up to EMPTY_BATCH centroids that is not flagged in
// `taken`; (d2, id) order.  One pass over the points for all of them (one pass
// per centroid, a lane's loads one float at a time, took 0.6 to 0.8 ms each at
// 1,000,000 x 128, eight centroids take 0.19 now).
constexpr int EMPTY_BATCH = 8;
constexpr int EMPTY_BLOCKS = 512;

struct Best {
    double v;
    int64_t id;
};

struct EmptyList {
    int32_t c[EMPTY_BATCH];   // places past the last hold it again
    int m;
};

__global__ void __launch_bounds__(256) empty_scan_kernel(const float *base, int64_t n, int dim,
                                                         bool vec4, const double *mu, EmptyList l,
                                                         const int32_t *taken, Best *partial)
{
#pragma clang fp contract(off)
    __shared__ Best sh[256];
    Best b[EMPTY_BATCH];
#pragma unroll
    for (int q = 0; q < EMPTY_BATCH; ++q)
        b[q] = Best{__longlong_as_double(0x7ff0000000000000ll), 0x7fffffffffffffffll};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (taken[i]) continue;
        const float *x = base + i * dim;
        double v[EMPTY_BATCH];
#pragma unroll
        for (int q = 0; q < EMPTY_BATCH; ++q) v[q] = 0.0;
        if (vec4) {
            for (int j0 = 0; j0 < dim; j0 += 32) {
                float4 xv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (j0 + 4 * u < dim) xv[u] = *reinterpret_cast<const float4 *>(x + j0 + 4 * u);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int j = j0 + 4 * u;
                    if (j >= dim) break;
#pragma unroll
                    for (int q = 0; q < EMPTY_BATCH; ++q) {
                        const double *m = mu + (int64_t)l.c[q] * dim + j;
                        v[q] = v[q] + term(xv[u].x, m[0]);
                        v[q] = v[q] + term(xv[u].y, m[1]);
                        v[q] = v[q] + term(xv[u].z, m[2]);
                        v[q] = v[q] + term(xv[u].w, m[3]);
                    }
                }
            }
        } else {
            for (int j = 0; j < dim; ++j)
#pragma unroll
                for (int q = 0; q < EMPTY_BATCH; ++q)
                    v[q] = v[q] + term(x[j], mu[(int64_t)l.c[q] * dim + j]);
        }
#pragma unroll
        for (int q = 0; q < EMPTY_BATCH; ++q)
            if (v[q] < b[q].v || (v[q] == b[q].v && i < b[q].id)) b[q] = Best{v[q], i};
    }
#pragma unroll
    for (int q = 0; q < EMPTY_BATCH; ++q) {
        if (q >= l.m) break;
        __syncthreads();
        sh[threadIdx.x] = b[q];
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if (threadIdx.x < s) {
                Best o = sh[threadIdx.x + s];
                if (o.v < sh[threadIdx.x].v ||
                    (o.v == sh[threadIdx.x].v && o.id < sh[threadIdx.x].id))
                    sh[threadIdx.x] = o;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) partial[q * gridDim.x + blockIdx.x] = sh[0];
    }
}

struct TakenList {
    int32_t id[EMPTY_BATCH];
    int m;
};

__global__ void mark_points_kernel(TakenList l, int32_t *taken)
{
    if ((int)threadIdx.x < l.m) taken[l.id[threadIdx.x]] = 1;
}

__global__ void mark_taken_kernel(const int32_t *hub, int nh, int32_t *taken)
{
    int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < nh && hub[c] >= 0) taken[hub[c]] = 1;
}

inline int grid_for(int64_t n, int per = 256, int cap = 8192)
{
    int64_t b = (n + per - 1) / per;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

// ---------------------------------------------------------------- HBKM
// distance of every point to the k children of its cluster (the same FP64
// arithmetic as the assignment above)
__global__ void child_dist_kernel(const float *base, int64_t n, int dim, bool vec4,
                                  const int32_t *parent,
                                  const double *mu, int k, double *D)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * k) return;
    const int64_t i = e / k;
    const int j = (int)(e - i * k);
    D[e] = d2_to(base + i * dim, mu + ((int64_t)parent[i] * k + j) * dim, dim, vec4);
}

// Child j of cluster c starts at point init_ids[c * k + j], or at the
// parent's centroid when the parent has no member (init id -1).
__global__ void init_children_kernel(const float *base, int dim, const int32_t *init_ids, int64_t nc,
                                     int k, const double *parent_mu, double *mu)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nc * dim) return;
    const int64_t c = e / dim, j = e % dim;
    const int32_t id = init_ids[c];
    mu[e] = id >= 0 ? (double)base[(int64_t)id * dim + j] : parent_mu[(c / k) * dim + j];
}

// One wavefront per parent cluster: its members (id order) join children in
// turn, each the child j of smallest d2(x, mu_j) + lambda * (2 (s_j - m/k) + 1)
// with s_j child j's size so far (ties to the smaller j).  Lane j keeps s_j;
// the distances of 64 members at a time are staged in LDS, so the sequential
// chain only waits on LDS and shuffles.
constexpr int HB_CHUNK = 64;

__global__ void __launch_bounds__(64) balanced_pass_kernel(const int32_t *members,
                                                           const int64_t *start, int64_t np,
                                                           const double *D, int k, double lambda,
                                                           int32_t *child)
{
#pragma clang fp contract(off)
    extern __shared__ __align__(16) unsigned char hb_lds[];
    double *ds = reinterpret_cast<double *>(hb_lds);                  // HB_CHUNK x k
    int32_t *ms = reinterpret_cast<int32_t *>(ds + HB_CHUNK * k);     // HB_CHUNK
    const int64_t p = blockIdx.x;
    if (p >= np) return;
    const int lane = threadIdx.x;
    const int64_t s0 = start[p];
    const int64_t m = start[p + 1] - s0;
    const double target = (double)m / (double)k;
    const double inf = __longlong_as_double(0x7ff0000000000000ll);
    int64_t s = 0;
    for (int64_t r0 = 0; r0 < m; r0 += HB_CHUNK) {
        const int cnt = (int)(m - r0 < HB_CHUNK ? m - r0 : HB_CHUNK);
        if (lane < cnt) ms[lane] = members[s0 + r0 + lane];
        __syncthreads();
        for (int e = lane; e < cnt * k; e += 64) {
            const int q = e / k, j = e - q * k;
            ds[e] = D[(int64_t)ms[q] * k + j];
        }
        __syncthreads();
        for (int q = 0; q < cnt; ++q) {
            double v = inf;
            int idx = lane;
            if (lane < k) {
                const double dev = (double)s - target;
                const double pen = lambda * (2.0 * dev + 1.0);
                v = ds[q * k + lane] + pen;
            }
            for (int o = 32; o > 0; o >>= 1) {
                const double ov = __shfl_xor(v, o);
                const int oi = __shfl_xor(idx, o);
                if (ov < v || (ov == v && oi < idx)) {
                    v = ov;
                    idx = oi;
                }
            }
            if (lane == idx) ++s;
            if (lane == 0) child[ms[q]] = (int32_t)(p * k + idx);
        }
        __syncthreads();
    }
}

}  // namespace

namespace {

// Definition 3 hubs of given clusters: the member nearest the cluster's
// mean by (d2, id); an empty cluster takes the nearest point that is not yet
// a hub (clusters in index order).
// order: NULL, or the points sorted by cluster (the lanes then share a mean).
ann_status hubs_of_clusters(const float *base, int64_t n, int dim, int nh, const double *mu,
                            const int32_t *assign, const int2 *order, int32_t *hub_ids, unsigned long long *bits,
                            int32_t *taken, Best *partial, hipStream_t st)
{
    const bool vec4 = dim % 4 == 0 && aligned(base, 16) && aligned(mu, 16);
    hipLaunchKernelGGL(fill_u64, dim3(grid_for(nh)), dim3(256), 0, st, bits, (int64_t)nh,
                       0xFFFFFFFFFFFFFFFFull);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(fill_i32, dim3(grid_for(nh)), dim3(256), 0, st, hub_ids, (int64_t)nh,
                       0x7fffffff);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(hub_min_kernel, dim3(grid_for(n, 256, 1 << 22)), dim3(256), 0, st, base, n, dim,
                       vec4, mu, assign, order, bits);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(hub_id_kernel, dim3(grid_for(n, 256, 1 << 22)), dim3(256), 0, st, base, n, dim,
                       vec4, mu, assign, order, bits, hub_ids);
    ANN_LAUNCHED();
    // empty clusters (no member): nearest point that is not yet a hub
    std::vector<int32_t> hh((size_t)nh);
    ANN_HIP(hipMemcpyAsync(hh.data(), hub_ids, sizeof(int32_t) * nh, hipMemcpyDeviceToHost, st));
    ANN_HIP(hipStreamSynchronize(st));
    bool any_empty = false;
    for (int c = 0; c < nh; ++c) any_empty |= (hh[c] == 0x7fffffff);
    if (any_empty) {
        hipLaunchKernelGGL(fill_i32, dim3(grid_for(n)), dim3(256), 0, st, taken, n, 0);
        ANN_LAUNCHED();
        // flag the hubs of non-empty clusters
        for (int c = 0; c < nh; ++c)
            if (hh[c] == 0x7fffffff) hh[c] = -1;
        ANN_HIP(hipMemcpyAsync(hub_ids, hh.data(), sizeof(int32_t) * nh, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(mark_taken_kernel, dim3(grid_for(nh)), dim3(256), 0, st, hub_ids, nh, taken);
        ANN_LAUNCHED();
        const int blocks = grid_for(n, 256, EMPTY_BLOCKS);
        std::vector<int> empty;
        for (int c = 0; c < nh; ++c)
            if (hh[c] < 0) empty.push_back(c);
        std::vector<Best> pb((size_t)blocks * EMPTY_BATCH);
        for (size_t e0 = 0; e0 < empty.size();) {
            EmptyList l{};
            l.m = (int)(empty.size() - e0 < EMPTY_BATCH ? empty.size() - e0 : EMPTY_BATCH);
            for (int q = 0; q < EMPTY_BATCH; ++q) l.c[q] = empty[e0 + (size_t)(q < l.m ? q : l.m - 1)];
            hipLaunchKernelGGL(empty_scan_kernel, dim3(blocks), dim3(256), 0, st, base, n, dim, vec4,
                               mu, l, taken, partial);
            ANN_LAUNCHED();
            ANN_HIP(hipMemcpyAsync(pb.data(), partial, sizeof(Best) * (size_t)blocks * l.m,
                                   hipMemcpyDeviceToHost, st));
            ANN_HIP(hipStreamSynchronize(st));
            // clusters in order, up to the first whose nearest point an
            // earlier one of this pass has taken: that one needs a new pass
            TakenList tl{};
            for (int q = 0; q < l.m; ++q) {
                Best b = pb[(size_t)q * blocks];
                for (int r = 1; r < blocks; ++r) {
                    const Best o = pb[(size_t)q * blocks + r];
                    if (o.v < b.v || (o.v == b.v && o.id < b.id)) b = o;
                }
                bool clash = false;
                for (int r = 0; r < q; ++r) clash |= tl.id[r] == (int32_t)b.id;
                if (clash) break;
                if (b.id < 0 || b.id >= n)
                    return fail(ANN_EINVAL, "no point is left for an empty cluster (base not finite?)");
                hh[(size_t)l.c[q]] = (int32_t)b.id;
                tl.id[tl.m++] = (int32_t)b.id;
            }
            hipLaunchKernelGGL(mark_points_kernel, dim3(1), dim3(64), 0, st, tl, taken);
            ANN_LAUNCHED();
            e0 += (size_t)tl.m;
        }
        ANN_HIP(hipMemcpyAsync(hub_ids, hh.data(), sizeof(int32_t) * nh, hipMemcpyHostToDevice, st));
        ANN_HIP(hipStreamSynchronize(st));
    }
    return ANN_OK;
}

}  // namespace

namespace {

// centroids padded to whole chunks of the FP16 assignment, 0 where it is not
// taken
int half_padded(int dim, int nh)
{
    if (dim < 4 || dim % 4 || dim > HB_MAX_DIM || nh > HB_MAX_NH) return 0;
    const int per = 16 * lds_tiles(frags_of(dim));
    return (nh + per - 1) / per * per;
}

template <int KS>
ann_status launch_half(const HalfArgs &a, hipStream_t st)
{
    constexpr int PB = 64 * row_tiles(KS);
    hipLaunchKernelGGL(assign_half_kernel<KS>, dim3((unsigned)((a.n + PB - 1) / PB)), dim3(256), 0, st,
                       a);
    ANN_LAUNCHED();
    return ANN_OK;
}

ann_status assign_half(const HalfArgs &a, int KS, hipStream_t st)
{
    switch (KS) {
    case 1: return launch_half<1>(a, st);
    case 2: return launch_half<2>(a, st);
    case 3: return launch_half<3>(a, st);
    case 4: return launch_half<4>(a, st);
    case 8: return launch_half<8>(a, st);
    case 16: return launch_half<16>(a, st);
    default: return launch_half<32>(a, st);
    }
}

}  // namespace

size_t select_hubs_ws(int64_t n, int dim, int nh)
{
    size_t b = round_up((size_t)nh * dim * 8, 256) * 2;       // mu, sums
    b += round_up((size_t)nh * 8, 256) * 2;                   // count, best bits
    b += round_up((size_t)n * 4, 256) * 2;                    // assign, taken
    b += round_up(EMPTY_BATCH * EMPTY_BLOCKS * sizeof(Best), 256) + 1024;
    b += round_up((size_t)nh * dim * 4, 256);                 // FP32 centroids
    b += round_up((size_t)nh * 4, 256) * 3;                   // their norms, first places
    b += round_up((size_t)n * 4, 256) * 2;                    // point norms
    b += round_up((size_t)n * sizeof(OpenPoint), 256);        // open points; sorted points
    if (const int padded = half_padded(dim, nh)) {
        b += round_up((size_t)n * sizeof(int2), 256);         // points left
        b += round_up((size_t)padded * 64 * frags_of(dim), 256);   // FP16 centroids
        b += round_up((size_t)padded * 4, 256) + round_up((size_t)dim * 4, 256);
    }
    return b;
}

ann_status select_hubs_run(const float *base, int64_t n, int dim, int nh, int iters,
                           const int32_t *init_ids, int32_t *hub_ids, double *centroids_out,
                           int32_t *assign_out, int32_t *steps_out, void *ws, hipStream_t st)
{
    Carve cv{static_cast<unsigned char *>(ws)};
    double *mu = centroids_out ? centroids_out : cv.take<double>((size_t)nh * dim);
    if (centroids_out) cv.take<double>((size_t)nh * dim);
    double *sums = cv.take<double>((size_t)nh * dim);
    int64_t *count = cv.take<int64_t>((size_t)nh);
    unsigned long long *bits = cv.take<unsigned long long>((size_t)nh);
    int32_t *assign = assign_out ? assign_out : cv.take<int32_t>((size_t)n);
    if (assign_out) cv.take<int32_t>((size_t)n);
    int32_t *taken = cv.take<int32_t>((size_t)n);
    Best *partial = cv.take<Best>(EMPTY_BATCH * EMPTY_BLOCKS);
    StepState *state = cv.take<StepState>(1);
    float *scale = cv.take<float>(1);
    float *mu32 = cv.take<float>((size_t)nh * dim);
    float *cn2 = cv.take<float>((size_t)nh);
    float *cn = cv.take<float>((size_t)nh);
    int32_t *cursor = cv.take<int32_t>((size_t)nh);
    float *xn2 = cv.take<float>((size_t)n);
    float *xn = cv.take<float>((size_t)n);
    // the open points are decided before the points are sorted
    OpenPoint *open = cv.take<OpenPoint>((size_t)n);
    int2 *sorted = reinterpret_cast<int2 *>(open);
    // the matrix-core assignments need whole float4 rows
    const bool mfma = dim % 4 == 0 && aligned(base, 16);
    const bool vec4 = mfma && aligned(mu, 16);
    // few products, of short rows with few centroids (which a workgroup of the
    // FP32 kernel goes through one after the other): one launch of that instead
    // of the four that the FP16 products and what they leave open take.  us a step,
    // FP32 / FP16: 1,000 points x 64 centroids x 16 dimensions 51 / 79, 16,384 x
    // 128 x 128 96 / 113; but 16,384 x 512 x 32 103 / 94, 4,096 x 500 x 128 151 / 106,
    // and beyond 2^28 products FP16 is ahead with any number.
    const bool few = dim <= 128 && nh <= 256 && nh * dim <= (1 << 14) &&
                     n * nh * (int64_t)dim <= (1 << 28);
    const int padded = mfma && !few ? half_padded(dim, nh) : 0;
    // few values, and few of them on one address: the atomics cost less than the
    // two launches more that the sort takes (us a step at 256 clusters: 2,000 x
    // 16 78 / 86, 1,000 x 64 93 / 99; with more than 64 points on an address the sort
    // is ahead: 1,000 x 15, 8 clusters 60 / 56)
    const bool sort = nh <= SORT_MAX_NH && ((int64_t)n * dim > (1 << 18) || n > 64 * (int64_t)nh);
    ShortArgs sa{};
    HalfArgs ha{};
    CentroidArgs ca{};
    ca.mu = mu;
    ca.sums = sums;
    ca.count = count;
    ca.nh = nh;
    ca.dim = dim;
    ca.padded = padded ? padded : nh;
    ca.state = state;
    if (mfma) {
        hipLaunchKernelGGL(point_norms_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                           base, n, dim, xn2, xn);
        ANN_LAUNCHED();
        // bound coefficients (unit roundoff u = 2^-24): the norms and mu~ are
        // FP32 roundings, the dot product accumulates dim FP32 terms (gamma),
        // s and the bounds themselves add a few roundings; margins of >= 30 %
        const double u = std::ldexp(1.0, -24);
        const double K = (double)dim + 2.0;
        const double gam = K * u / (1.0 - K * u);
        const double gp = gam * (1.0 + u) + u;
        sa = ShortArgs{base, n, dim, mu, mu32, cn2, cn, xn2, xn, nh,
                       (float)(8.0 * u), (float)(2.1 * gp + 12.0 * u), assign, nullptr, nullptr, nullptr,
                       LEFT_FEW, vec4};
        ca.mu32 = mu32;
        ca.cn2 = cn2;
        ca.cn = cn;
    }

    const int64_t md = (int64_t)nh * dim;
    hipLaunchKernelGGL(init_mu_kernel, dim3(grid_for(md, 256, 1 << 20)), dim3(256), 0, st, base, dim,
                       init_ids, nh, mu);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(fill_i32, dim3(grid_for(n)), dim3(256), 0, st, assign, n, -1);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, st, reinterpret_cast<int32_t *>(state),
                       (int64_t)(sizeof(StepState) / 4), 0);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(fill_f64, dim3(grid_for(md)), dim3(256), 0, st, sums, md);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(fill_u64, dim3(grid_for(nh)), dim3(256), 0, st, (unsigned long long *)count,
                       (int64_t)nh, 0ull);
    ANN_LAUNCHED();
    if (padded) {
        const int KS = frags_of(dim);
        ha.left = cv.take<int2>((size_t)n);
        ca.mh = cv.take<_Float16>((size_t)padded * 32 * KS);
        ca.cv = cv.take<float>((size_t)padded);
        float *c0 = cv.take<float>((size_t)dim);
        hipLaunchKernelGGL(frame_kernel, dim3(1), dim3(1024), 0, st, mu, nh, dim, c0, scale);
        ANN_LAUNCHED();
        ca.KS = KS;
        ca.c0 = c0;
        ca.scale = scale;
        ha.base = base;
        ha.n = n;
        ha.dim = dim;
        ha.c0 = c0;
        ha.scale = scale;
        ha.mh = reinterpret_cast<const v4u *>(ca.mh);
        ha.cv = ca.cv;
        ha.tiles = padded / 16;
        while ((1 << ha.bits) < ha.tiles) ++ha.bits;
        // FP32 accumulation of the products and of |m|^2 / 2 (an addition may
        // lose a unit in the last place), and the bits given to the tile number
        ha.g = (float)((32.0 * KS + 8.0) * std::ldexp(1.0, -23));
        ha.gb = (float)std::ldexp(1.0, ha.bits - 22);
        ha.state = state;
        ha.assign = assign;
        ha.open = open;
        sa.list = ha.left;
        sa.count = &state->n_left;
    }
    const dim3 cgrid((unsigned)((ca.padded + CENTROID_WAVES - 1) / CENTROID_WAVES));
    hipLaunchKernelGGL(centroid_kernel, cgrid, dim3(64 * CENTROID_WAVES), 0, st, ca);
    ANN_LAUNCHED();
    ca.update = true;
    const unsigned sblocks = (unsigned)((n + SORT_POINTS - 1) / SORT_POINTS);
    const size_t slds = (size_t)nh * 4;
    // columns of a row per thread, threads of a row, rows of a run: enough
    // threads for the chip (2^18), then runs of up to 64 rows
    const int vec = mfma ? 4 : 1;
    const int cols = (dim + vec - 1) / vec;
    const int wide = cols < 256 ? cols : 256;
    int64_t len = n * cols >> 18;
    len = len < 8 ? 8 : len > 64 ? 64 : len;
    const int64_t per_block = len * (256 / wide);
    const dim3 agrid((unsigned)((n + per_block - 1) / per_block), (unsigned)((cols + wide - 1) / wide));
    int steps = 0;
    for (int t = 0; t < iters; ++t) {
        const int parity = t & 1;
        int32_t *changed = &state->changed[parity];
        sa.changed = changed;
        if (padded) {
            ha.parity = parity;
            ann_status hs = assign_half(ha, ca.KS, st);
            if (hs != ANN_OK) return hs;
            hipLaunchKernelGGL(open_kernel, dim3(grid_for(4 * n, 256, 2048)), dim3(256), 0, st, base,
                               dim, vec4, mu, open, &state->n_open, assign, changed);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(left_kernel, dim3(grid_for(n, 4, LEFT_FEW / 4)), dim3(256), 0, st, base,
                               dim, vec4, mu, nh, ha.left, &state->n_left, LEFT_FEW, assign, changed);
            ANN_LAUNCHED();
        }
        if (mfma)
            hipLaunchKernelGGL(assign_mfma_kernel, dim3(grid_for(n, MP, padded ? 2048 : 1 << 26)),
                               dim3(256), 0, st, sa);
        else
            hipLaunchKernelGGL(assign_kernel, dim3((unsigned)((n + KP - 1) / KP)), dim3(256), 0, st,
                               base, n, dim, mu, nh, assign, changed);
        ANN_LAUNCHED();
        ++steps;
        if (sort) {
            hipLaunchKernelGGL(cluster_count_kernel, dim3(sblocks), dim3(256), slds, st, assign, n, nh,
                               count);
            ANN_LAUNCHED();
        } else {
            hipLaunchKernelGGL(accumulate_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, base,
                               n, dim, assign, sums, count);
            ANN_LAUNCHED();
        }
        hipLaunchKernelGGL(cluster_scan_kernel, dim3(1), dim3(1024), 0, st, count, nh, cursor, state,
                           parity ^ 1);
        ANN_LAUNCHED();
        if (sort) {
            hipLaunchKernelGGL(cluster_sort_kernel, dim3(sblocks), dim3(256), slds, st, assign, n, nh,
                               cursor, sorted);
            ANN_LAUNCHED();
            if (vec == 4)
                hipLaunchKernelGGL(cluster_sum_kernel<4>, agrid, dim3(256), 0, st, base, n, dim, sorted,
                                   wide, (int)len, sums);
            else
                hipLaunchKernelGGL(cluster_sum_kernel<1>, agrid, dim3(256), 0, st, base, n, dim, sorted,
                                   wide, (int)len, sums);
            ANN_LAUNCHED();
        }
        ca.parity = parity ^ 1;
        hipLaunchKernelGGL(centroid_kernel, cgrid, dim3(64 * CENTROID_WAVES), 0, st, ca);
        ANN_LAUNCHED();
        int32_t h = 0;
        ANN_HIP(hipMemcpyAsync(&h, changed, 4, hipMemcpyDeviceToHost, st));
        ANN_HIP(hipStreamSynchronize(st));
        if (!h) break;
    }
    ann_status hs = hubs_of_clusters(base, n, dim, nh, mu, assign, sort ? sorted : nullptr, hub_ids,
                                     bits, taken, partial, st);
    if (hs != ANN_OK) return hs;
    if (steps_out) *steps_out = steps;
    return ANN_OK;
}

}  // namespace ann

using namespace ann;

namespace ann {
namespace {

int64_t ipow(int64_t b, int e)
{
    int64_t r = 1;
    for (int i = 0; i < e; ++i) r *= b;
    return r;
}

size_t hbkm_ws(int64_t n, int dim, int k, int levels)
{
    const int64_t nc = ipow(k, levels), np = ipow(k, levels - 1);
    size_t b = round_up((size_t)n * k * 8, 256);                 // distances to the children
    b += round_up((size_t)n * 4, 256) * 4;                        // parent, child, members, taken
    b += round_up((size_t)(np + 1) * 8, 256);                     // member offsets
    b += round_up((size_t)nc * 4, 256);                           // initial members
    b += round_up((size_t)nc * dim * 8, 256) * 3;                 // mu, parent mu, sums
    b += round_up((size_t)nc * 8, 256) * 2;                       // count, best bits
    b += round_up(EMPTY_BATCH * EMPTY_BLOCKS * sizeof(Best), 256);
    return b + 1024;
}

ann_status hbkm_run(const float *base, int64_t n, int dim, int k, int levels, double lambda,
                    int iters, int32_t *hub_ids, double *centroids_out, int32_t *assign_out,
                    void *ws, hipStream_t st)
{
    const int64_t nc_max = ipow(k, levels), np_max = ipow(k, levels - 1);
    Carve cv{static_cast<unsigned char *>(ws)};
    double *D = cv.take<double>((size_t)n * k);
    int32_t *cur = cv.take<int32_t>((size_t)n);
    int32_t *nxt = cv.take<int32_t>((size_t)n);
    int32_t *mem_d = cv.take<int32_t>((size_t)n);
    int32_t *taken = cv.take<int32_t>((size_t)n);
    int64_t *start_d = cv.take<int64_t>((size_t)np_max + 1);
    int32_t *init_d = cv.take<int32_t>((size_t)nc_max);
    double *mu = cv.take<double>((size_t)nc_max * dim);
    double *pmu = cv.take<double>((size_t)nc_max * dim);
    double *sums = cv.take<double>((size_t)nc_max * dim);
    int64_t *count = cv.take<int64_t>((size_t)nc_max);
    unsigned long long *bits = cv.take<unsigned long long>((size_t)nc_max);
    Best *partial = cv.take<Best>(EMPTY_BATCH * EMPTY_BLOCKS);
    // (mu and pmu change places: both start on 256 bytes)
    const bool vec4 = dim % 4 == 0 && aligned(base, 16);

    hipLaunchKernelGGL(fill_i32, dim3(grid_for(n)), dim3(256), 0, st, cur, n, 0);
    ANN_LAUNCHED();
    std::vector<int32_t> lab((size_t)n), members((size_t)n), init;
    std::vector<int64_t> start;
    const size_t pass_lds = (size_t)HB_CHUNK * k * 8 + HB_CHUNK * 4;
    int64_t np = 1;
    for (int l = 1; l <= levels; ++l) {
        const int64_t nc = np * k;
        // members of every parent in id order, and each child's first member
        ANN_HIP(hipMemcpyAsync(lab.data(), cur, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost, st));
        ANN_HIP(hipStreamSynchronize(st));
        start.assign((size_t)np + 1, 0);
        for (int64_t i = 0; i < n; ++i) start[(size_t)lab[(size_t)i] + 1]++;
        for (int64_t p = 0; p < np; ++p) start[(size_t)p + 1] += start[(size_t)p];
        {
            std::vector<int64_t> fill(start.begin(), start.end() - 1);
            for (int64_t i = 0; i < n; ++i) members[(size_t)fill[(size_t)lab[(size_t)i]]++] = (int32_t)i;
        }
        init.assign((size_t)nc, -1);
        for (int64_t p = 0; p < np; ++p) {
            const int64_t m = start[(size_t)p + 1] - start[(size_t)p];
            if (m == 0) continue;
            for (int j = 0; j < k; ++j)
                init[(size_t)(p * k + j)] = members[(size_t)(start[(size_t)p] + (2 * j + 1) * m / (2 * k))];
        }
        ANN_HIP(hipMemcpyAsync(mem_d, members.data(), sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, st));
        ANN_HIP(hipMemcpyAsync(start_d, start.data(), sizeof(int64_t) * (size_t)(np + 1),
                               hipMemcpyHostToDevice, st));
        ANN_HIP(hipMemcpyAsync(init_d, init.data(), sizeof(int32_t) * (size_t)nc, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(init_children_kernel, dim3((unsigned)((nc * dim + 255) / 256)), dim3(256), 0,
                           st, base, dim, init_d, nc, k, pmu, mu);
        ANN_LAUNCHED();
        const int64_t md = nc * dim;
        for (int t = 0; t < iters; ++t) {
            hipLaunchKernelGGL(child_dist_kernel, dim3((unsigned)((n * k + 255) / 256)), dim3(256), 0, st,
                               base, n, dim, vec4, cur, mu, k, D);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(balanced_pass_kernel, dim3((unsigned)np), dim3(64), pass_lds, st, mem_d,
                               start_d, np, D, k, lambda, nxt);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(fill_f64, dim3(grid_for(md)), dim3(256), 0, st, sums, md);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(fill_u64, dim3(grid_for(nc)), dim3(256), 0, st,
                               (unsigned long long *)count, nc, 0ull);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(accumulate_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, st, base,
                               n, dim, nxt, sums, count);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(update_kernel, dim3((unsigned)((md + 255) / 256)), dim3(256), 0, st, sums,
                               count, (int)nc, dim, mu);
            ANN_LAUNCHED();
        }
        std::swap(cur, nxt);
        std::swap(mu, pmu);
        np = nc;
    }
    // cur: final clusters, pmu: their centroids
    ANN_HIP(hipMemcpyAsync(assign_out, cur, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, st));
    if (centroids_out)
        ANN_HIP(hipMemcpyAsync(centroids_out, pmu, sizeof(double) * (size_t)np * dim,
                               hipMemcpyDeviceToDevice, st));
    ann_status hs = hubs_of_clusters(base, n, dim, (int)np, pmu, cur, nullptr, hub_ids, bits, taken, partial, st);
    if (hs != ANN_OK) return hs;
    ANN_HIP(hipStreamSynchronize(st));
    return ANN_OK;
}

bool hbkm_shape_ok(int64_t n, int32_t k, int32_t levels)
{
    if (k < 2 || k > 64 || levels < 1 || levels > 20) return false;
    int64_t nc = 1;
    for (int l = 0; l < levels; ++l) {
        nc *= k;
        if (nc > n || nc > (1 << 20)) return false;
    }
    return true;
}

}  // namespace
}  // namespace ann

extern "C" size_t ann_select_hubs_hbkm_workspace_size(int64_t n, int32_t dim, int32_t k,
                                                      int32_t levels)
{
    if (n < 1 || dim < 1 || !hbkm_shape_ok(n, k, levels)) return 0;
    return hbkm_ws(n, dim, k, levels);
}

extern "C" ann_status ann_select_hubs_hbkm(const float *base, int64_t n, int32_t dim, int32_t k,
                                           int32_t levels, double lambda, int32_t iters,
                                           int32_t *hub_ids, double *centroids, int32_t *assign,
                                           void *workspace, size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && hub_ids && assign && workspace, "a required pointer is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF, "n must be in [1, 2^31)");
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");
    ANN_REQUIRE(hbkm_shape_ok(n, k, levels),
                "need 2 <= k <= 64, levels >= 1 and k^levels <= min(n, 2^20)");
    ANN_REQUIRE(lambda >= 0.0 && lambda < 1e300, "lambda must be finite and >= 0");
    ANN_REQUIRE(iters >= 1, "iters must be >= 1");
    ANN_REQUIRE(ws_bytes >= hbkm_ws(n, dim, k, levels), "workspace too small");
    return no_throw([&] {
        return hbkm_run(base, n, dim, k, levels, lambda, iters, hub_ids, centroids, assign, workspace,
                        static_cast<hipStream_t>(stream));
    });
}

extern "C" ann_status ann_select_hubs(const float *base, int64_t n, int32_t dim, int32_t n_hubs,
                                      int32_t iters, const int32_t *init_ids, int32_t *hub_ids,
                                      double *centroids, int32_t *assign, int32_t *steps,
                                      void *workspace, size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && init_ids && hub_ids && workspace, "a required pointer is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF, "n must be in [1, 2^31)");
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");
    ANN_REQUIRE(n_hubs >= 1 && n_hubs <= n, "n_hubs must be in [1, n]");
    ANN_REQUIRE(iters >= 1, "iters must be >= 1");
    ANN_REQUIRE(ws_bytes >= ann_workspace_size(ANN_OP_SELECT_HUBS, n, dim, n_hubs, 0),
                "workspace too small");
    return no_throw([&] {
        return select_hubs_run(base, n, dim, n_hubs, iters, init_ids, hub_ids, centroids, assign, steps,
                               workspace, static_cast<hipStream_t>(stream));
    });
}

// Seeded k-means start.  The generator is SplitMix64 (Steele, Lea and Flood,
// OOPSLA 2014): the state advances by the golden-ratio increment and each
// output is the state through the generator's finaliser.  The i-th output x
// picks t in [0, j] as the high word of x * (j + 1) (Lemire's multiply-shift,
// 2019, no rejection), and Floyd's sampling (Bentley and Floyd, CACM 1987)
// takes t, or j when t is already taken, for j = n - n_hubs .. n - 1.
extern "C" ann_status ann_hub_init_ids(int64_t n, int32_t n_hubs, uint64_t seed, int32_t *ids)
{
    ANN_REQUIRE(ids != nullptr, "ids is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF, "n must be in [1, 2^31)");
    ANN_REQUIRE(n_hubs >= 1 && n_hubs <= n, "n_hubs must be in [1, n]");
    return no_throw([&]() -> ann_status {
        std::unordered_set<int64_t> taken;
        taken.reserve((size_t)n_hubs * 2);
        uint64_t state = seed;
        int32_t i = 0;
        for (int64_t j = n - n_hubs; j < n; ++j) {
            state += 0x9E3779B97F4A7C15ull;
            uint64_t z = state;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            const int64_t t = (int64_t)(((unsigned __int128)z * (uint64_t)(j + 1)) >> 64);
            const int64_t v = taken.count(t) ? j : t;
            taken.insert(v);
            ids[i++] = (int32_t)v;
        }
        return ANN_OK;
    });
}
