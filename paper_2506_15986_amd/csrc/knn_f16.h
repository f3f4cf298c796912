// Exact kNN of real-valued data: a shortlist on the FP16 matrix cores, the
// distances of the shortlist in FP64.
//
// With c a vector near the data's mean and s a power of two, every vector
// becomes h = fp16(s (x - c)) (and, for the second level, l = fp16 of what h
// leaves).  With V = |s (x - c)|^2 the matrix cores give
//     p(x, y) = V_x + V_y - 2 h_x . h_y,
// which differs from the scaled squared distance by at most E_x + E_y, with
// E = eV * V + eS * sqrt(V) + e0 from the rounding of the operands, of the
// accumulation and of the test itself (coef() below).  So with t the K-th
// smallest p + E_x + E_y of a row, every true neighbour has
// p - E_x - E_y <= t.  A row collects the columns that pass this test under
// its current t, and t falls as it collects; what is left at the end gets the
// FP64 distance of the plain engine, in the same order of operations, and is
// sorted by (distance, id).  The result is the plain engine's, bit for bit.
//
// (One level of FP16 reaches 1.1 PFLOP/s on this card where FP64 vector
// arithmetic, 3 operations per coordinate, gave 22 TFLOP/s.)
//
// A row whose list cannot be cut down to its buffer (more columns near the
// K-th neighbour than the bound can tell apart) is done again with h and l
// (three products, a bound some hundred times smaller), and one that fails
// there too by the plain FP64 engine, as is everything when a value is not
// finite.
#pragma once

#include "knn_core.h"

namespace ann {
namespace f16 {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kRowsWG = 256;     // rows per workgroup, 64 per wavefront
constexpr int kCols = 128;       // columns per tile
constexpr int kDk = 64;          // dimensions per LDS stage
constexpr int kMaxMerged = 4096; // shortlist entries of a row over all slices
constexpr int kMaxSample = 4096; // columns the first thresholds are taken from
constexpr int kRing = 512;       // candidates a wavefront holds back in LDS before writing them out
constexpr int kRsrcWord3 = 0x00020000;  // buffer resource word 3 (raw, 32-bit data)
constexpr int kWaitVmcnt0 = 0x0F70;   // s_waitcnt vmcnt(0), the other counters left alone
constexpr uint32_t kNotFinite = 0x7f800000u;   // a spread from here on: infinities, NaN, FP32 overflow

// order-preserving image of a float
__device__ inline uint32_t ord(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u >> 31) ? ~u : (u | 0x80000000u);
}

__device__ inline float unord(uint32_t k)
{
    return __uint_as_float((k >> 31) ? (k & 0x7fffffffu) : ~k);
}

struct Coef {
    float eV, eS, e0;
};

// Bound coefficients for `dim` dimensions.  Each operand element is off by at
// most a |x| + b: level 1 keeps 11 bits (a = 2^-11), level 2 keeps 22 (a =
// 2^-21 also covers the rounding of x - c and the product of the two l's); b
// covers values that fall below the normal range of FP16, kept or flushed
// (2^-14 for each part).  By Cauchy-Schwarz the dot product is then off by
// (2a + a^2) |x||y| + b sqrt(dim) (1 + a)(|x| + |y|) + b^2 dim; its FP32
// accumulation adds one truncation of 2^-23 of the partial sum per product;
// twice that, |x||y| <= (V_x + V_y) / 2, and 32 units of 2^-24 for V, the
// test and the bound themselves.  5 % on top for the coefficients' own
// rounding.
inline Coef coef(int dim, bool level2)
{
    const double a = level2 ? 1.0 / (1 << 21) : 1.0 / (1 << 11) + 1.0 / (1 << 22);
    const double b = (level2 ? 2.0 : 1.0) / (1 << 14);
    const double adds = (double)dim * (level2 ? 3.0 : 1.0) + 64.0;
    const double gam = adds / (double)(1 << 23);
    Coef c;
    c.eV = (float)(1.05 * (2.0 * a + a * a + gam * (1.0 + a) * (1.0 + a) + 32.0 / (1 << 24)));
    c.eS = (float)(1.05 * 2.0 * b * std::sqrt((double)dim) * (1.0 + 2.0 * a + gam));
    c.e0 = (float)(1.05 * b * b * dim * (1.0 + gam));
    return c;
}

// centre: the mean of up to 1,024 evenly spaced rows (any vector would do)
__global__ void __launch_bounds__(1024) centre_kernel(const float *x, int64_t n, int dim, float *c)
{
    __shared__ float part[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane;
    const int m = n < 1024 ? (int)n : 1024;
    float s = 0.f;
    if (j < dim)
        for (int i = w; i < m; i += 16) s += x[((int64_t)i * n / m) * dim + j];
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && j < dim) {
        for (int q = 1; q < 16; ++q) s += part[q][lane];
        c[j] = s / (float)m;
    }
}

// *bits = max over the data of |x - c| as FP32 bits (infinities and NaN last).
// A workgroup reports once: with a report of every wavefront, 22,000 x 96 took
// 36 to 55 us, most of it at the one address; 19 now.
__global__ void __launch_bounds__(256) spread_kernel(const float *x, int64_t n, int dim,
                                                     const float *c, uint32_t *bits)
{
    const int lane = threadIdx.x & 63;
    uint32_t mx = 0u;
    for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4)
        for (int j = lane; j < dim; j += 64) {
            const uint32_t b = __float_as_uint(fabsf(x[r * dim + j] - c[j]));
            mx = b > mx ? b : mx;
        }
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t other = __shfl_xor(mx, o);
        mx = other > mx ? other : mx;
    }
    __shared__ uint32_t top[4];
    if (lane == 0) top[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x) return;
    for (int w = 1; w < 4; ++w) mx = top[w] > mx ? top[w] : mx;
    if (mx > *bits) atomicMax(bits, mx);
}

// the power of two that takes the largest |x - c| into [2^14, 2^15)
__device__ inline float scale_of(uint32_t bits)
{
    int e = (int)(bits >> 23) - 127;
    if (bits == 0u) e = 14;
    int k = 14 - e;
    k = k > 126 ? 126 : k;
    return __uint_as_float((uint32_t)(k + 127) << 23);
}

// One wavefront per row: h (and l, for the second level), V and E.  Row i of
// the result is row rows[i], or with `of` > 0 the i-th of n evenly spaced rows
// among `of`, or row i.  hi NULL: V and E alone.
template <bool LO>
__global__ void __launch_bounds__(256) convert_kernel(const float *x, int64_t n, int dim, int dpad,
                                                      const float *c, const uint32_t *bits,
                                                      const int32_t *rows, int64_t of, Coef co,
                                                      _Float16 *hi, _Float16 *lo, float *V, float *E)
{
    const int lane = threadIdx.x & 63;
    const float s = scale_of(*bits);
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < n; i += (int64_t)gridDim.x * 4) {
        const int64_t r = rows ? (int64_t)rows[i] : of ? i * of / n : i;
        double v = 0.0;
        for (int j = lane; j < dpad; j += 64) {
            float y = 0.f;
            if (j < dim) {
                const float xv = x[r * dim + j], cv = c[j];
                const double d = ((double)xv - (double)cv) * (double)s;
                v += d * d;
                y = (xv - cv) * s;
            }
            if (!hi) continue;
            const _Float16 h = (_Float16)y;
            hi[i * dpad + j] = h;
            if (LO) lo[i * dpad + j] = (_Float16)(y - (float)h);
        }
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) {
            const float vf = (float)v;
            V[i] = vf;
            E[i] = co.eV * vf + co.eS * sqrtf(vf) + co.e0;
        }
    }
}

// ---- cluster order for all-pairs passes, as the int8 engine's: rows grouped
// by their nearest of up to kGroups sample rows (about 1,024 rows to a
// group), each workgroup taking its first thresholds from its own group's
// columns and visiting them first.  Only the visiting order changes.
constexpr int kGroups = 256;
constexpr int64_t kGroupedMinN = 16384;
constexpr int64_t kGroupedMaxN = 1 << 28;    // of a launch with a wavefront per 16 rows

inline int groups_of(int64_t n)
{
    return n >= 1024 * kGroups ? kGroups : (int)(n / 1024);
}

// the sample rows (every (n / G)-th of blockIdx.x < G; the others are as far
// as can be from every row) and their V
__global__ void sample_kernel(const _Float16 *h, const float *V, int64_t n, int G, int dpad,
                              _Float16 *sh, float *sV)
{
    const int c = blockIdx.x;
    const int64_t r = c < G ? (int64_t)c * n / G : 0;
    for (int j = threadIdx.x; j < dpad; j += blockDim.x) sh[(size_t)c * dpad + j] = h[r * dpad + j];
    if (threadIdx.x == 0) sV[c] = c < G ? V[r] : __builtin_inff();
}

// one wavefront per 16 rows: the nearest sample row of each (by the FP16
// products; any choice will do), and the groups' sizes
__global__ void __launch_bounds__(256) nearest_sample_kernel(const _Float16 *h, int64_t n, int dpad,
                                                             const _Float16 *sh, const float *sV,
                                                             int32_t *group, int32_t *hist)
{
    const int lane = threadIdx.x & 63, rl = lane & 15, kq = lane >> 4;
    const int64_t r0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (r0 >= n) return;
    const int64_t row = r0 + rl < n ? r0 + rl : n - 1;
    v4f acc[kGroups / 16];
#pragma unroll
    for (int j = 0; j < kGroups / 16; ++j) acc[j] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < dpad; k += 32) {
        const v8h av = *reinterpret_cast<const v8h *>(h + row * dpad + k + 8 * kq);
#pragma unroll
        for (int j = 0; j < kGroups / 16; ++j) {
            const v8h bv = *reinterpret_cast<const v8h *>(sh + (size_t)(16 * j + rl) * dpad + k + 8 * kq);
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc[j], 0, 0, 0);
        }
    }
    float best[4];
    int who[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        best[e] = __builtin_inff();
        who[e] = 0;
    }
#pragma unroll
    for (int j = 0; j < kGroups / 16; ++j) {
        const float v = sV[16 * j + rl];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d = v - 2.f * acc[j][e];
            if (d < best[e]) {
                best[e] = d;
                who[e] = 16 * j + rl;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        for (int o = 1; o < 16; o <<= 1) {
            const float ob = __shfl_xor(best[e], o);
            const int ow = __shfl_xor(who[e], o);
            if (ob < best[e] || (ob == best[e] && ow < who[e])) {
                best[e] = ob;
                who[e] = ow;
            }
        }
        const int64_t r = r0 + 4 * kq + e;
        if (rl == 0 && r < n) {
            group[r] = who[e];
            atomicAdd(&hist[who[e]], 1);
        }
    }
}

// each workgroup's first column: the start of the group of its first row
__global__ void start_kernel(const int32_t *group, const int32_t *perm, const int32_t *start,
                             int64_t blocks, int32_t *start_col)
{
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b < blocks) start_col[b] = start[group[perm[b * kRowsWG]]];
}

struct Args {
    const _Float16 *bh, *bl;   // columns, n x dpad (second level: of the estimates only)
    const _Float16 *qh, *ql;   // rows, rows x dpad
    const float *base, *c;     // second level: the columns' vectors, split as they are staged
    int dim;
    int vec4;                  // ... whole, aligned groups of four floats
    const float *bV, *bE, *qV, *qE;
    const uint32_t *bits;      // the data's spread
    int64_t n, rows;
    int dpad;
    int K;                     // neighbours that a row's threshold guards
    int keep;                  // most entries a (row, slice) may leave behind
    int slices;
    int64_t slice_len;         // multiple of kCols
    const int32_t *start;      // per workgroup: the column its pass starts at (NULL: the slice's first)
    const float *first;        // the rows' first t (NULL: every column passes until a list fills)
    float *est;                // first thresholds: rows x S estimates
    int S;
    uint64_t *buf;             // rows x slices x cap words (ord(V_x + lower part) << 32 | column)
    int32_t *cnt;              // rows x slices; -1: the row's list did not fit
};

// For RB sets of 64 W values over a wavefront (up, ord() words, 0xffffffff for
// none): a T with at least K values <= T, the K-th smallest or a little
// above it.  Bisection between the extremes, stopped once at most K / 16
// further values come along.
template <int W, int RB>
__device__ inline void kth(const uint32_t (&up)[RB][W], int K, uint32_t (&T)[RB])
{
    uint32_t lo[RB];
    bool open = false;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            mn = up[b][k] < mn ? up[b][k] : mn;
            mx = up[b][k] != 0xffffffffu && up[b][k] > mx ? up[b][k] : mx;
        }
        for (int o = 32; o > 0; o >>= 1) {
            const uint32_t a = __shfl_xor(mn, o), c = __shfl_xor(mx, o);
            mn = a < mn ? a : mn;
            mx = c > mx ? c : mx;
        }
        lo[b] = __builtin_amdgcn_readfirstlane(mn);
        T[b] = __builtin_amdgcn_readfirstlane(mx);
        open |= lo[b] < T[b];
    }
    while (open) {
        open = false;
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            if (lo[b] >= T[b]) continue;
            const uint32_t mid = lo[b] + ((T[b] - lo[b]) >> 1);
            int n = 0;
#pragma unroll
            for (int k = 0; k < W; ++k) n += __popcll(__builtin_amdgcn_ballot_w64(up[b][k] <= mid));
            if (n < K) lo[b] = mid + 1;
            else {
                T[b] = mid;
                if (n <= K + (K >> 4)) lo[b] = mid;
            }
            open |= lo[b] < T[b];
        }
    }
}

// A wavefront cuts RB rows' lists at once, each of c >= K words, down to
// those that can still be among the K nearest: the K-th smallest upper bound
// gives t, and words whose lower bound exceeds it go.  The rows' loads are in
// flight together: one row at a time, a cut is three waits on memory.
// c[b] = 0: no row b.  Writes the kept counts to c and t, in the lower
// bounds' terms, to th.
template <int W, int RB>
__device__ inline void cut(uint64_t *const (&g)[RB], int (&c)[RB], int K, const float (&twoE)[RB],
                           const float *bE, float (&th)[RB])
{
    const int lane = __lane_id();
    uint64_t w[RB][W];
    uint32_t up[RB][W], T[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int k = 0; k < W; ++k) w[b][k] = lane + 64 * k < c[b] ? g[b][lane + 64 * k] : ~0ull;
#pragma unroll
    for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int k = 0; k < W; ++k)
            up[b][k] = lane + 64 * k < c[b]
                           ? ord(unord((uint32_t)(w[b][k] >> 32)) + 2.f * bE[(uint32_t)w[b][k]])
                           : 0xffffffffu;
    kth<W, RB>(up, K, T);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        th[b] = unord(T[b]) + twoE[b];
        const uint32_t to = ord(th[b]);
        int kept = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const bool in = lane + 64 * k < c[b] && (uint32_t)(w[b][k] >> 32) <= to;
            const uint64_t m = __builtin_amdgcn_ballot_w64(in);
            if (in)
                g[b][kept + (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                    w[b][k];
            kept += __popcll(m);
        }
        c[b] = kept;
    }
}

// First thresholds: one wavefront per row, the K-th smallest upper bound of
// the row's S = 64 W sample columns (est: V_x + V_y + E_y - 2 dot), as the
// t that the row's tests start with.
template <int W>
__global__ void __launch_bounds__(256) threshold_kernel(const float *est, int64_t rows, int K,
                                                        const float *qE, float *first)
{
    const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= rows) return;
    const int lane = threadIdx.x & 63;
    uint32_t up[1][W], T[1];
#pragma unroll
    for (int k = 0; k < W; ++k) up[0][k] = ord(est[g * (64 * W) + lane + 64 * k]);
    kth<W, 1>(up, K, T);
    if (lane == 0) first[g] = unord(T[0]) + 2.f * qE[g];
}

// the sample columns of a first-level pass without groups: S evenly spaced ones
__global__ void __launch_bounds__(64) pick_columns_kernel(const _Float16 *h, const float *V, const float *E,
                                                          int64_t n, int S, int dpad, _Float16 *oh,
                                                          float *oV, float *oE)
{
    const int s = blockIdx.x;
    const int64_t c = (int64_t)s * n / S;
    for (int j = 8 * (int)threadIdx.x; j < dpad; j += 512)
        *reinterpret_cast<v8h *>(oh + (size_t)s * dpad + j) =
            *reinterpret_cast<const v8h *>(h + c * dpad + j);
    if (threadIdx.x == 0) {
        oV[s] = V[c];
        oE[s] = E[c];
    }
}

// LDS of a workgroup: the staged operands and the per-row state
template <bool LO>
constexpr size_t tile_lds()
{
    return (size_t)(kRowsWG + kCols) * kDk * 2 * (LO ? 2 : 1) + kRowsWG * 12 + kCols * 4 +
           4 * (size_t)kRing * 12;
}

// CAPW: words of a row's buffer per lane (its capacity is 64 CAPW).
//
// What bounds it: the matrix cores while a tile has many dimensions, the
// test of the 128 products per lane (one multiply-add and half a max3 each)
// when it has few.  A workgroup takes 256 rows, a wavefront 64 of them
// against all 128 columns of a tile, so that a wavefront owns its rows'
// thresholds and lists without any block-wide step, and each operand
// fragment read from LDS feeds 4 or 8 products.  Two workgroups share a CU:
// one's loads and barriers run behind the other's products.
//
// CAPW = 0: instead of lists, the estimates of the workgroup's rows against
// the columns [start, start + S) (blockIdx.y = 128 of them), for the first
// thresholds.  Without those a row's list fills with strangers first (the
// first two tiles alone were 64 KB of stores per wavefront) and is cut several
// times: 50,001 x 96, K = 64 10.5 ms against 2.3 ms.
//
// Data whose spread is not finite ends here at once (the host learns of it with
// the pass's results and takes the plain engine): its products may be
// infinite, and the lists' bounds hold for finite values only.  The bound of a
// row that takes no columns, past the last or given up, is NaN: no value
// passes it, an infinite one neither.
//
// The second level's columns come from the vectors themselves and are split
// into h and l on the way to LDS (as many bytes as the two halves would have;
// few rows get here, and the halves of all columns were most of the memory).
//
// Measured against the plain FP64 engine: the candidates of 50,001 x 96 (K = 64)
// 109 ms, this kernel 2.15 (ann_build_graph 4.9 ms, 114 with the plain engine);
// the 10 nearest of 1,000 queries among 150,000 x 960 526 -> 1.13 ms (this kernel
// 0.57 ms = 0.51 PFLOP/s; without any passing column it takes 0.46 ms).
template <int CAPW, bool LO>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LO ? 1 : 2)))
tile_kernel(Args a)
{
    constexpr bool EST = CAPW == 0;
    constexpr int CAP = 64 * CAPW;
    if (*a.bits >= kNotFinite) return;
    constexpr int RB = CAPW <= 4 ? 4 : CAPW <= 8 ? 2 : 1;         // rows cut together
    constexpr bool SPLIT = LO && !EST;
    constexpr int AS = kRowsWG * 8 / 256, BS = kCols * 8 / 256;   // 16-byte slots per thread
    extern __shared__ __align__(16) unsigned char dyn[];
    v8h *Ah = reinterpret_cast<v8h *>(dyn);
    v8h *Bh = Ah + kRowsWG * 8;
    v8h *Al = Bh + kCols * 8;
    v8h *Bl = Al + (LO ? kRowsWG * 8 : 0);
    float *r_rt = reinterpret_cast<float *>(Bl + (LO ? kCols * 8 : 0));   // 2 dot - lower(column) >= r_rt
    float *r_V = r_rt + kRowsWG;
    int32_t *r_cnt = reinterpret_cast<int32_t *>(r_V + kRowsWG);          // -1: the list did not fit
    float *c_low = reinterpret_cast<float *>(r_cnt + kRowsWG);            // V - E of the tile's columns
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    uint64_t *ring_w = reinterpret_cast<uint64_t *>(c_low + kCols) + w * kRing;
    uint32_t *ring_m = reinterpret_cast<uint32_t *>(c_low + kCols) + 8 * kRing + w * kRing;   // row << 16 | slot
    int ring_n = 0;
    const int rl = lane & 15, kq = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.x * kRowsWG;
    const int slice = blockIdx.y;
    const int64_t c_begin = (int64_t)slice * a.slice_len;
    int64_t c_end = c_begin + a.slice_len;
    if (c_end > a.n) c_end = a.n;
    const int ntiles = EST ? 1 : c_end > c_begin ? (int)((c_end - c_begin + kCols - 1) / kCols) : 0;
    // the slice's tiles are visited cyclically from start0 (the tiles of the
    // workgroup's own group first, when the rows are grouped and it is here)
    int start0 = a.start ? (int)((a.start[blockIdx.x] - c_begin) / kCols) : 0;
    if (start0 < 0 || start0 >= ntiles) start0 = 0;
    int64_t e_begin = 0;
    if (EST) {
        e_begin = a.start ? a.start[blockIdx.x] : 0;
        if (e_begin > a.n - a.S) e_begin = a.n - a.S;
        e_begin += (int64_t)blockIdx.y * kCols;
        c_end = e_begin + kCols;
    }
    auto tile_c0 = [&](int it) {
        if (EST) return e_begin;
        int j = start0 + it;
        if (j >= ntiles) j -= ntiles;
        return c_begin + (int64_t)j * kCols;
    };
    const int nch = (a.dpad + kDk - 1) / kDk;
    const float big = 3.0e38f, inf = __builtin_inff(), none = __builtin_nanf("");
    {
        const int64_t g = row0 + t;
        r_rt[t] = g < a.rows ? (a.first ? a.qV[g] - a.first[g] : -big) : none;
        r_V[t] = g < a.rows ? a.qV[g] : 0.f;
        r_cnt[t] = 0;
    }
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const float scale = SPLIT ? scale_of(*a.bits) : 0.f;
    v4u sa[AS], sb[BS], la[LO ? AS : 1], lb[LO ? BS : 1];
    float s_low = 0.f;
    // Thread t stages 16-byte slot t % 8 of rows t / 8 + 32 e.  Buffer loads
    // through resources based at the workgroup's first row and the tile's
    // first column: one offset per lane for the whole pass, and what lies past
    // the data reads as zero (such rows' and columns' tests never pass).  The
    // half chunk past dpad is read from what follows the row and not used.
    const int rowb = a.dpad * 2;
    const int voff = (t >> 3) * rowb + 16 * (t & 7);
    const int64_t left = a.rows - row0;
    const int abytes = (int)(left < kRowsWG ? left : kRowsWG) * rowb;
    const __amdgpu_buffer_rsrc_t rah = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.qh + row0 * a.dpad), (short)0, abytes, kRsrcWord3);
    const __amdgpu_buffer_rsrc_t ral = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((LO ? a.ql : a.qh) + row0 * a.dpad), (short)0, abytes, kRsrcWord3);
    auto fetch = [&](int it, int ch) {
        const int64_t c0 = tile_c0(it);
        // recomputed here: kept, the twelve offsets cost twelve registers
        int vo = voff;
        asm volatile("" : "+v"(vo));
        const int64_t cl = a.n - c0;
        const int bbytes = (int)(cl < kCols ? cl : kCols) * rowb;
        const __amdgpu_buffer_rsrc_t rbh = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(a.bh + c0 * a.dpad), (short)0, bbytes, kRsrcWord3);
        const __amdgpu_buffer_rsrc_t rbl = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((LO ? a.bl : a.bh) + c0 * a.dpad), (short)0, bbytes, kRsrcWord3);
#pragma unroll
        for (int e = 0; e < AS; ++e) {
            sa[e] = __builtin_amdgcn_raw_buffer_load_b128(rah, vo + 32 * e * rowb, 128 * ch, 0);
            if (LO) la[e] = __builtin_amdgcn_raw_buffer_load_b128(ral, vo + 32 * e * rowb, 128 * ch, 0);
        }
#pragma unroll
        for (int e = 0; e < BS; ++e) {
            if constexpr (SPLIT) {
                // eight floats of a column: sb the first four, lb the others
                const int64_t c = c0 + (t >> 3) + 32 * e;
                const int j = kDk * ch + 8 * (t & 7);
                const float *src = a.base + c * a.dim + j;
                sb[e] = lb[e] = v4u{0u, 0u, 0u, 0u};
                if (c >= a.n) continue;
                if (a.vec4) {
                    if (j < a.dim) sb[e] = *reinterpret_cast<const v4u *>(src);
                    if (j + 4 < a.dim) lb[e] = *reinterpret_cast<const v4u *>(src + 4);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (j + q < a.dim) sb[e][q] = __float_as_uint(src[q]);
                        if (j + 4 + q < a.dim) lb[e][q] = __float_as_uint(src[4 + q]);
                    }
                }
            } else {
                sb[e] = __builtin_amdgcn_raw_buffer_load_b128(rbh, vo + 32 * e * rowb, 128 * ch, 0);
                if (LO) lb[e] = __builtin_amdgcn_raw_buffer_load_b128(rbl, vo + 32 * e * rowb, 128 * ch, 0);
            }
        }
        if (ch == 0 && t < kCols) {
            const int64_t c = c0 + t;
            s_low = c < c_end ? (EST ? a.bV[c] + a.bE[c] : a.bV[c] - a.bE[c]) : inf;
        }
    };
    // A row's eight 16-byte slots are permuted by its number, so that the 16
    // rows a fragment load touches fall on different banks: slot s of row r
    // lies at 8 r + (s ^ (r & 7)), and rows 8, 16, 32 apart share the
    // permutation.
    const int st_at = 8 * (t >> 3) + ((t & 7) ^ ((t >> 3) & 7));
    const int fr_at[2] = {8 * rl + (kq ^ (rl & 7)), 8 * rl + ((4 + kq) ^ (rl & 7))};
    auto store = [&](int ch) {
#pragma unroll
        for (int e = 0; e < AS; ++e) {
            Ah[st_at + 256 * e] = __builtin_bit_cast(v8h, sa[e]);
            if (LO) Al[st_at + 256 * e] = __builtin_bit_cast(v8h, la[e]);
        }
        float cv[8];
        if constexpr (SPLIT) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int j = kDk * ch + 8 * (t & 7) + q;
                cv[q] = j < a.dim ? a.c[j] : 0.f;
            }
        }
#pragma unroll
        for (int e = 0; e < BS; ++e) {
            if constexpr (SPLIT) {
                // convert_kernel's h and l; zero past the row's end
                v8h hi, lo;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float x = __uint_as_float(q < 4 ? sb[e][q & 3] : lb[e][q & 3]);
                    const float y = kDk * ch + 8 * (t & 7) + q < a.dim ? (x - cv[q]) * scale : 0.f;
                    hi[q] = (_Float16)y;
                    lo[q] = (_Float16)(y - (float)hi[q]);
                }
                Bh[st_at + 256 * e] = hi;
                Bl[st_at + 256 * e] = lo;
            } else {
                Bh[st_at + 256 * e] = __builtin_bit_cast(v8h, sb[e]);
                if (LO) Bl[st_at + 256 * e] = __builtin_bit_cast(v8h, lb[e]);
            }
        }
        if (ch == 0 && t < kCols) c_low[t] = s_low;
    };
    // the ring's candidates to their rows' buffers
    auto flush = [&]() {
        const int m = ring_n < kRing ? ring_n : kRing;
        knn::wsync();
        for (int x = lane; x < m; x += 64) {
            const uint32_t tag = ring_m[x];
            a.buf[((row0 + (tag >> 16)) * a.slices + slice) * (int64_t)CAP + (tag & 0xffffu)] = ring_w[x];
        }
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        knn::wsync();
        ring_n = 0;
    };
    // cuts the next RB of the wavefront's rows in `which`; a list that stays
    // above `most` is given up (its row goes to the next level)
    auto cut_rows = [&](uint64_t &which, int most, bool more) {
        uint64_t *g[RB];
        int c[RB], r[RB];
        float twoE[RB], th[RB];
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            r[b] = 64 * w + (which ? (int)__builtin_ctzll(which) : 0);
            c[b] = which ? __builtin_amdgcn_readfirstlane(r_cnt[r[b]]) : 0;
            which &= which - 1;
            const int64_t row = c[b] ? row0 + r[b] : row0;
            g[b] = a.buf + (row * a.slices + slice) * (int64_t)CAP;
            twoE[b] = 2.f * a.qE[row];
        }
        cut<EST ? 1 : CAPW, RB>(g, c, a.K, twoE, a.bE, th);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (lane == 0 && c[b] > 0) {
                const bool fits = c[b] <= most;
                r_cnt[r[b]] = fits ? c[b] : -1;
                if (more) r_rt[r[b]] = fits ? r_V[r[b]] - th[b] : none;
            }
        knn::wsync();
    };
    v4f acc[4][8];
    if (ntiles > 0) fetch(0, 0);
    for (int it = 0; it < ntiles; ++it) {
        const int64_t c0 = tile_c0(it);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
        for (int ch = 0; ch < nch; ++ch) {
            __syncthreads();
            store(ch);
            __syncthreads();
            if (ch + 1 < nch) fetch(it, ch + 1);
            else if (it + 1 < ntiles) fetch(it + 1, 0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if (ch * kDk + 32 * ks >= a.dpad) break;
                v8h av[4], al[LO ? 4 : 1];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    av[i] = Ah[512 * w + 128 * i + fr_at[ks]];
                    if (LO) al[i] = Al[512 * w + 128 * i + fr_at[ks]];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const v8h bv = Bh[128 * j + fr_at[ks]];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[i], bv, acc[i][j], 0, 0, 0);
                    if (LO) {
                        const v8h bl = Bl[128 * j + fr_at[ks]];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[i], bv, acc[i][j], 0, 0, 0);
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[i], bl, acc[i][j], 0, 0, 0);
                        }
                    }
                }
            }
        }
        // the test: v = 2 dot - (V - E)(column) >= r_rt(row).  The largest v
        // of each of the lane's 16 rows first; nearly always none passes.
        float low[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) low[j] = c_low[16 * j + rl];
        if constexpr (EST) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 64 * w + 16 * i + 4 * kq + e;
                    if (row0 + r >= a.rows) continue;
                    float *o = a.est + (row0 + r) * a.S + blockIdx.y * kCols;
                    const float rv = r_V[r];
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        o[16 * j + rl] = rv - __builtin_fmaf(2.f, acc[i][j][e], -low[j]);
                }
            return;
        } else {
        uint64_t some[4][4], any = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v4f rt = *reinterpret_cast<const v4f *>(r_rt + 64 * w + 16 * i + 4 * kq);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float mx = -inf;
#pragma unroll
                for (int j = 0; j < 8; j += 2)
                    mx = fmaxf(mx, fmaxf(__builtin_fmaf(2.f, acc[i][j][e], -low[j]),
                                         __builtin_fmaf(2.f, acc[i][j + 1][e], -low[j + 1])));
                some[i][e] = __builtin_amdgcn_ballot_w64(mx >= rt[e]);
                any |= some[i][e];
            }
        }
        if (any) {
            // Element e of row block i: the 16 lanes of a quarter wavefront
            // hold one row's 16 columns of each block, so ballots give every
            // passing column its place behind the row's count.  It waits in
            // the wavefront's LDS ring: a store to memory here would keep
            // the next tile's operands waiting for it.  The lane number goes
            // through an empty asm, so that what derives from it is computed
            // here and not held (and spilled) over the whole pass.
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int cn = ln & 15, q4 = ln >> 4;
            const uint32_t under = (1u << cn) - 1u;
            const uint32_t col = (uint32_t)c0 + cn;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (!some[i][e]) continue;
                    const int r = 64 * w + 16 * i + 4 * q4 + e;
                    const float rt = r_rt[r], rv = r_V[r];
                    const int at0 = r_cnt[r];
                    int at = at0;
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float v = __builtin_fmaf(2.f, acc[i][j][e], -low[j]);
                        const uint64_t b = __builtin_amdgcn_ballot_w64(v >= rt);
                        if (!b) continue;
                        const uint32_t m = (uint32_t)(b >> (16 * q4)) & 0xffffu;
                        if (v >= rt) {
                            const int slot = at + __popc(m & under);
                            const uint64_t word = ((uint64_t)ord(rv - v) << 32) | (col + 16 * j);
                            const int pos = ring_n + (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                            if (pos < kRing) {
                                ring_w[pos] = word;
                                ring_m[pos] = ((uint32_t)r << 16) | (uint32_t)slot;
                            } else {
                                // ring full (a first tile without thresholds)
                                a.buf[((row0 + r) * a.slices + slice) * (int64_t)CAP + slot] = word;
                            }
                        }
                        at += __popc(m);
                        ring_n += __popcll(b);
                    }
                    if (cn == 0 && at > at0) r_cnt[r] = at;
                }
        }
        // cut the lists that could not take another tile
        knn::wsync();
        uint64_t full = __builtin_amdgcn_ballot_w64(r_cnt[64 * w + lane] > CAP - kCols);
        if (full || ring_n > kRing / 2) flush();
        while (full) cut_rows(full, CAP - kCols, true);
        }
    }
    if constexpr (EST) return;
    else {
    flush();
    uint64_t over = __builtin_amdgcn_ballot_w64(r_cnt[64 * w + lane] > a.keep);
    while (over) cut_rows(over, a.keep, false);
    if (row0 + 64 * w + lane < a.rows)
        a.cnt[(row0 + 64 * w + lane) * a.slices + slice] = r_cnt[64 * w + lane];
    }
}

// bytes of the part of final_kernel's LDS that holds the words, then the
// sorted entries
__host__ __device__ inline size_t final_words(int most, int sort)
{
    const size_t w = (size_t)most * 8, e = (size_t)sort * sizeof(knn::Ent);
    return w > e ? w : e;
}

struct FinalArgs {
    const float *base, *queries;
    int64_t rows;
    int dim;
    int64_t row0;
    const int32_t *row_list;   // query row of list row g (NULL: row0 + g)
    const int32_t *col_id;     // base row of column p (NULL: p)
    const float *qE, *bE;
    const uint32_t *bits;      // the data's spread (level 1: not finite = every row goes on)
    const uint64_t *buf;
    const int32_t *cnt;
    int slices, cap, K, Kp;
    int most, sort;            // words, and sorted entries (a power of two), the LDS arrays hold
    int vec4;                  // rows are whole, aligned groups of four floats
    int exclude;
    const int32_t *self_col;
    int32_t *out_ids;
    float *out_f;
    double *out_d;
    int32_t *todo;             // rows for the next level, and their count
    int32_t *todo_n;
};

// the K-th smallest upper bound of the c <= 64 W words (kth), as an ord() word
template <int W>
__device__ inline uint32_t kth_upper(const uint64_t *word, int c, int K, const float *bE)
{
    const int lane = __lane_id();
    uint32_t up[1][W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        up[0][k] = 0xffffffffu;
        if (lane + 64 * k < c) {
            const uint64_t w = word[lane + 64 * k];
            up[0][k] = ord(unord((uint32_t)(w >> 32)) + 2.f * bE[(uint32_t)w]);
        }
    }
    uint32_t T[1];
    kth<W, 1>(up, K, T);
    return T[0];
}

// One wavefront per row: the slices' lists cut to one shortlist, its FP64
// distances (the plain engine's sum: dimensions in order, fused
// multiply-adds), the sort by (distance, id), the first K written.
__global__ void __launch_bounds__(64) final_kernel(FinalArgs a)
{
    extern __shared__ __align__(16) unsigned char dyn[];
    knn::Ent *ent = reinterpret_cast<knn::Ent *>(dyn);             // `sort`
    uint64_t *word = reinterpret_cast<uint64_t *>(dyn);            // `most`, in the same bytes
    int32_t *pick = reinterpret_cast<int32_t *>(dyn + final_words(a.most, a.sort));   // `sort`
    const int lane = threadIdx.x;
    const int64_t g = blockIdx.x;
    const int64_t q = a.row_list ? (int64_t)a.row_list[g] : a.row0 + g;
    // the slices' counts, one per lane, and their places; then the words,
    // sixteen lanes to a slice, four slices' loads in flight
    const int mine = lane < a.slices ? a.cnt[g * a.slices + lane] : 0;
    bool ok = *a.bits < kNotFinite && !__builtin_amdgcn_ballot_w64(mine < 0);
    int end = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const int other = __shfl_up(end, o);
        if (lane >= o) end += other;
    }
    const int c = __builtin_amdgcn_readlane(end, 63);
    ok = ok && c <= a.most;
    if (!ok) {
        if (lane == 0) a.todo[atomicAdd(a.todo_n, 1)] = (int32_t)q;
        return;
    }
    for (int s0 = 0; s0 < a.slices; s0 += 4) {
        const int s = s0 + (lane >> 4);
        const int m = __shfl(mine, s & 63), at = __shfl(end, s & 63) - m;
        const uint64_t *src = a.buf + (g * a.slices + s) * (int64_t)a.cap;
        for (int t0 = lane & 15; s < a.slices && t0 < m; t0 += 64) {
            uint64_t v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = t0 + 16 * k < m ? src[t0 + 16 * k] : 0ull;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (t0 + 16 * k < m) word[at + t0 + 16 * k] = v[k];
        }
    }
    knn::wsync();
    uint32_t to = 0xffffffffu;
    if (c > a.Kp) {
        uint32_t T;
        if (c <= 512) T = kth_upper<8>(word, c, a.Kp, a.bE);
        else if (c <= 2048) T = kth_upper<32>(word, c, a.Kp, a.bE);
        else T = kth_upper<64>(word, c, a.Kp, a.bE);
        to = ord(unord(T) + 2.f * a.qE[g]);
    }
    const int64_t self = a.exclude ? (a.self_col ? (int64_t)a.self_col[q] : q) : -1;
    int m = 0;
    for (int t0 = 0; t0 < c; t0 += 64) {
        const uint64_t wd = t0 + lane < c ? word[t0 + lane] : 0ull;
        const int32_t id = t0 + lane < c ? (a.col_id ? a.col_id[(uint32_t)wd] : (int32_t)(uint32_t)wd) : 0;
        const bool in = t0 + lane < c && (uint32_t)(wd >> 32) <= to && id != self;
        const uint64_t b = __builtin_amdgcn_ballot_w64(in);
        if (m + __popcll(b) > a.sort) {
            if (lane == 0) a.todo[atomicAdd(a.todo_n, 1)] = (int32_t)q;
            return;
        }
        if (in)
            pick[m + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = id;
        m += __popcll(b);
    }
    knn::wsync();
    int P = 2;
    while (P < m) P <<= 1;
    const float *xq = a.queries + q * a.dim;
    for (int t = lane; t < P; t += 64) {
        knn::Ent e = knn::ent_max();
        if (t < m) {
            const int32_t id = pick[t];
            const float *xb = a.base + (int64_t)id * a.dim;
            double acc = 0.0;
            auto add = [&](float x, float y) {
                const double d = (double)x - (double)y;
                acc += d * d;
            };
            if (a.vec4) {
#pragma unroll 8
                for (int j = 0; j < a.dim; j += 4) {
                    const float4 x = *reinterpret_cast<const float4 *>(xq + j);
                    const float4 y = *reinterpret_cast<const float4 *>(xb + j);
                    add(x.x, y.x);
                    add(x.y, y.y);
                    add(x.z, y.z);
                    add(x.w, y.w);
                }
            } else {
#pragma unroll 8
                for (int j = 0; j < a.dim; ++j) add(xq[j], xb[j]);
            }
            e.k = knn::key_of(acc);
            e.id = (uint32_t)id;
        }
        ent[t] = e;
    }
    knn::wsync();
    for (int size = 2; size <= P; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = lane; t < P / 2; t += 64) {
                const int lo = 2 * t - (t & (stride - 1)), hi = lo + stride;
                const bool up = (lo & size) == 0;
                const knn::Ent x = ent[lo], y = ent[hi];
                if (up ? knn::less(y, x) : knn::less(x, y)) {
                    ent[lo] = y;
                    ent[hi] = x;
                }
            }
            knn::wsync();
        }
    for (int t = lane; t < a.K; t += 64) {
        int32_t id = -1;
        double v = __longlong_as_double(0x7ff0000000000000ll);
        if (t < m) {
            id = (int32_t)ent[t].id;
            v = knn::value_of(ent[t].k);
        }
        a.out_ids[q * a.K + t] = id;
        if (a.out_f) a.out_f[q * a.K + t] = (float)v;
        if (a.out_d) a.out_d[q * a.K + t] = v;
    }
}

struct Plan {
    int Kp, cap, keep, slices, most, sort, S;
    int64_t slice_len;
};

// A row's buffer holds its K neighbours, half as many again and a tile, and
// then what comes in between two cuts.  Column slices fill the GPU when the
// rows alone do not (two workgroups per CU); a slice is at least 2,048
// columns, and all slices' lists of a row fit in kMaxMerged words.  A slice
// leaves twice its K neighbours at most, and the final shortlist holds as
// many: the final kernel's LDS sets how many of its wavefronts run.
// S: the columns the first thresholds are taken from: about a slice's length,
// so that about K columns of a slice pass (150,000 x 960, K = 10, 62 slices:
// the pass takes 0.74 ms after 512 columns and 0.60 ms after 2,048), or about
// a group and a half; the estimates use the row buffers' memory.  0: too few
// columns to gain from it.
// max_slices: 0 = no other limit.  grouped: a group's columns are the sample.
// Empty inputs get a plan too (sizes are asked for before a call refuses them).
inline Plan plan(int64_t n, int64_t rows, int K, int cus, int64_t max_slices, bool grouped)
{
    Plan p{};
    if (n < 1) n = 1;
    if (rows < 1) rows = 1;
    p.Kp = (K > 0 ? K : 0) + 1;     // room for the row's own column
    const int need = 2 * p.Kp + kCols;
    p.cap = need <= 256 ? 256 : need <= 512 ? 512 : p.Kp <= 512 ? 1024 : 2048;
    const int64_t blocks = (rows + kRowsWG - 1) / kRowsWG;
    int64_t s = 2 * (int64_t)cus / blocks;     // at most one round of workgroups
    const int64_t by_len = n / 2048 > 1 ? n / 2048 : 1;
    const int64_t by_merge = kMaxMerged / (p.Kp + p.Kp / 2 + 48);
    if (s > by_len) s = by_len;
    if (s > by_merge) s = by_merge;
    if (s > 64) s = 64;          // the final kernel holds a count per lane
    if (max_slices > 0 && s > max_slices) s = max_slices;
    if (s < 1) s = 1;
    p.slice_len = ((n + s - 1) / s + kCols - 1) / kCols * kCols;
    p.slices = (int)((n + p.slice_len - 1) / p.slice_len);
    p.keep = 2 * p.Kp + 64;
    if (p.keep > kMaxMerged / p.slices) p.keep = kMaxMerged / p.slices;
    if (p.keep > p.cap) p.keep = p.cap;
    p.most = p.slices * p.keep;
    p.sort = 64;
    while (p.sort < 2 * p.Kp + 64) p.sort <<= 1;
    const int64_t want = grouped ? 3 * n / (2 * groups_of(n)) : p.slice_len;
    p.S = 512;
    while (p.S < kMaxSample && (3 * (int64_t)p.S < 2 * want || p.S < 2 * p.Kp) &&
           p.S <= p.slices * p.cap)
        p.S *= 2;
    if (p.S < 2 * p.Kp || 4 * (int64_t)p.S > n) p.S = 0;
    return p;
}

inline int padded(int dim) { return (dim + 31) / 32 * 32; }

// Memory of a pass: the columns' operands, and what a batch of rows takes.  The
// rows go through in batches, so that the lists (4 KB a row at K = 64) stay
// bounded: a size asks for batches of up to kBatchRows, a call takes batches as
// large as its memory allows, whole rounds of workgroups (two per CU, 256 rows
// each): 300,000 x 96 with itself, K = 64, 82 ms in two halves of 1.1 rounds each,
// 62 in one launch of 2.3.
constexpr int64_t kBatchRows = 1 << 18;
constexpr int64_t kLeastRows = 1 << 14;    // no batches smaller than this
constexpr int64_t kMostRows = 1 << 24;     // of a launch with a wavefront per row

inline size_t operand_bytes(int64_t n, int64_t rows, int dim)
{
    const size_t dp = (size_t)padded(dim);
    size_t b = round_up((size_t)n * dp * 2, 256) + round_up((size_t)n * 4, 256) * 2;
    b += round_up((size_t)dim * 4, 256) + round_up((size_t)rows * 4, 256) * 2;
    b += round_up((size_t)kMaxSample * dp * 2, 256) * 2 + round_up((size_t)kMaxSample * 4, 256) * 2;
    if (rows == n) {             // the cluster order
        b += round_up((size_t)n * 4, 256) * 2;
        b += round_up((size_t)(kGroups + 1) * 4, 256) * 2;
        b += round_up((size_t)((n + kRowsWG - 1) / kRowsWG) * 4, 256);
    }
    return b;
}

inline size_t list_bytes(int64_t n, int64_t rows, int K, int cus)
{
    const Plan p = plan(n, rows, K, cus, 0, false);
    return round_up((size_t)rows * p.slices * p.cap * 8, 256) +
           round_up((size_t)rows * p.slices * 4, 256);
}

// besides the lists
inline size_t row_bytes(int64_t rows, int dim)
{
    return round_up((size_t)rows * padded(dim) * 2, 256) * 2 + round_up((size_t)rows * 4, 256) * 3;
}

template <int CAPW, bool LO>
ann_status launch_tile(const Args &a, hipStream_t st)
{
    const size_t lds = tile_lds<LO>();
    ANN_HIP(hipFuncSetAttribute((const void *)tile_kernel<CAPW, LO>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    const dim3 grid((unsigned)((a.rows + kRowsWG - 1) / kRowsWG), (unsigned)a.slices);
    hipLaunchKernelGGL((tile_kernel<CAPW, LO>), grid, dim3(256), lds, st, a);
    ANN_LAUNCHED();
    return ANN_OK;
}

template <bool LO>
ann_status launch_tiles(const Args &a, int cap, hipStream_t st)
{
    switch (cap) {
    case 256: return launch_tile<4, LO>(a, st);
    case 512: return launch_tile<8, LO>(a, st);
    case 1024: return launch_tile<16, LO>(a, st);
    default: return launch_tile<32, LO>(a, st);
    }
}

// the rows' first thresholds from S columns of `a`: its own group's, or the
// sample (sh, sl, sV, sE)
template <bool LO>
ann_status first_thresholds(Args a, int S, float *est, float *first, const _Float16 *sh,
                            const _Float16 *sl, const float *sV, const float *sE, hipStream_t st)
{
    if (!a.start) {
        a.bh = sh;
        a.bl = sl;
        a.bV = sV;
        a.bE = sE;
        a.n = S;
    }
    a.est = est;
    a.S = S;
    a.slices = S / kCols;
    a.first = nullptr;
    ann_status s = launch_tile<0, LO>(a, st);
    if (s != ANN_OK) return s;
    const dim3 grid((unsigned)((a.rows + 3) / 4));
    switch (S) {
#define ANN_THRESHOLD(W)                                                                           \
    case 64 * W:                                                                                   \
        hipLaunchKernelGGL(threshold_kernel<W>, grid, dim3(256), 0, st, est, a.rows, a.K, a.qE, first); \
        break;
        ANN_THRESHOLD(8) ANN_THRESHOLD(16) ANN_THRESHOLD(32) ANN_THRESHOLD(64)
#undef ANN_THRESHOLD
    default: return fail(ANN_ENOTSUP, "kNN sample of %d columns", S);
    }
    ANN_LAUNCHED();
    return ANN_OK;
}

}  // namespace f16
}  // namespace ann
