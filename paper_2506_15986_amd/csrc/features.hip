// Topology features of the hub nodes (feature distillation section).
//
// The paper samples a subgraph around each hub by a guided walk and encodes
// it with a graph-embedding model; here the walk is kept and the encoder is
// replaced by 32 plain statistics of the hub, its neighbourhood and the walk
// subgraph (the list is in include/ann.h).
//
// Guided walk from hub v with max hop h: the subgraph's node list doubles as
// the FIFO.  A dequeued node u (depth < h) samples x = max(2, ceil(MinDeg *
// deg(u) / MaxDeg)) neighbours: the ceil(x/2) nearest and floor(x/2) farthest
// by (d2, id) -- all of them when deg(u) <= x.  Every sampled edge counts; a
// sampled node not yet in the subgraph joins it one hop deeper, while the
// subgraph holds fewer than wcap nodes.
//
// One workgroup per hub.  What a node samples does not depend on the walk, so
// the workgroup's wavefronts take the next nodes of the FIFO side by side, and
// only the joining is in order: the sampled ids of a batch meet in a hash set
// in LDS, where each id keeps its earliest place in the batch.
#include "common.h"
#include "internal.h"

namespace ann {
namespace {

constexpr int FW_MAX = 4096;
constexpr int NU_BLOCKS = 1024;
constexpr int FW_WAVES = 16;     // wavefronts of a walk's workgroup
constexpr uint32_t kNoId = 0xFFFFFFFFu;

// FP64 sum in dimension order.  vec4: whole, aligned groups of four, read as
// such (a lane walks its own row, so the loads, not the sums, are the cost).
__device__ inline double d2_ff(const float *a, const float *b, int dim, bool vec4)
{
    double s = 0.0;
    auto add = [&](float x, float y) {
        const double t = (double)x - (double)y;
        s += t * t;
    };
    if (vec4) {
#pragma unroll 8
        for (int j = 0; j < dim; j += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(a + j);
            const float4 y = *reinterpret_cast<const float4 *>(b + j);
            add(x.x, y.x);
            add(x.y, y.y);
            add(x.z, y.z);
            add(x.w, y.w);
        }
    } else {
#pragma unroll 4
        for (int j = 0; j < dim; ++j) add(a[j], b[j]);
    }
    return s;
}

__device__ inline double d2_fd(const float *a, const double *m, int dim)
{
#pragma clang fp contract(off)
    double s = 0.0;
    for (int j = 0; j < dim; ++j) {
        double t = (double)a[j] - m[j];
        s = s + t * t;
    }
    return s;
}

__device__ inline double wsum(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline double wmin(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}
__device__ inline double wmax(double v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ inline uint64_t dkey(double v)
{
    return (uint64_t)__double_as_longlong(v);   // v >= 0: bit order = value order
}

// ascending bitonic sort of one (key, id) per lane
__device__ inline void wsort(uint64_t &k, uint32_t &id)
{
    const int lane = __lane_id();
    for (int size = 2; size <= 64; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            uint64_t ok = __shfl_xor(k, stride);
            uint32_t oi = __shfl_xor(id, stride);
            bool up = (lane & size) == 0, lower = (lane & stride) == 0;
            bool mine = k < ok || (k == ok && id < oi);
            bool keep = (lower == up) ? mine : !mine;
            if (!keep) {
                k = ok;
                id = oi;
            }
        }
}

// ---- global statistics
// degrees, in-degrees, the least and largest degree of a node with edges, and
// the edge count: one thread per node, the last three gathered per workgroup
// first (an atomic per node on one address each took 0.3 ms at 200,000 nodes)
__global__ void __launch_bounds__(256) degree_kernel(const int32_t *graph, int64_t n, int R, int32_t *deg,
                                                     int32_t *indeg, int32_t *mm,
                                                     unsigned long long *edges)
{
    __shared__ int s_min, s_max;
    __shared__ unsigned long long s_edges;
    if (threadIdx.x == 0) {
        s_min = 0x7fffffff;
        s_max = 0;
        s_edges = 0ull;
    }
    __syncthreads();
    int lo = 0x7fffffff, hi = 0;
    unsigned long long e = 0ull;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        int c = 0;
#pragma unroll 8
        for (int s = 0; s < R; ++s) {
            const int32_t w = graph[v * R + s];
            if (w < 0) continue;
            ++c;
            atomicAdd(&indeg[w], 1);
        }
        deg[v] = c;
        if (c > 0) {
            lo = c < lo ? c : lo;
            hi = c > hi ? c : hi;
        }
        e += (unsigned long long)c;
    }
    atomicMin(&s_min, lo);
    atomicMax(&s_max, hi);
    atomicAdd(&s_edges, e);
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicMin(&mm[0], s_min);
        atomicMax(&mm[1], s_max);
        atomicAdd(edges, s_edges);
    }
}

__global__ void nu_partial_kernel(const float *base, int64_t n, int dim, bool vec4, const int32_t *graph,
                                  int R, double *part, int *cntp)
{
    __shared__ double sh[256];
    __shared__ int shc[256];
    double s = 0.0;
    int c = 0;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x) {
        int32_t first = -1;
        for (int q = 0; q < R && first < 0; ++q) first = graph[v * R + q];
        if (first < 0) continue;
        s += sqrt(d2_ff(base + v * dim, base + (int64_t)first * dim, dim, vec4));
        ++c;
    }
    sh[threadIdx.x] = s;
    shc[threadIdx.x] = c;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            sh[threadIdx.x] += sh[threadIdx.x + o];
            shc[threadIdx.x] += shc[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sh[0];
        cntp[blockIdx.x] = shc[0];
    }
}

// nu: the mean distance of a node to its first neighbour, the partial sums
// added in order
__global__ void __launch_bounds__(256) nu_kernel(const double *part, const int *cntp, int blocks, double *nu)
{
    __shared__ double sp[NU_BLOCKS];
    __shared__ int sc[NU_BLOCKS];
    for (int b = threadIdx.x; b < blocks; b += 256) {
        sp[b] = part[b];
        sc[b] = cntp[b];
    }
    __syncthreads();
    if (threadIdx.x) return;
    double s = 0.0;
    int c = 0;
#pragma unroll 16
    for (int b = 0; b < blocks; ++b) {
        s += sp[b];
        c += sc[b];
    }
    *nu = s / (double)c;
}

__global__ void csize_kernel(const int32_t *assign, int64_t n, int32_t *csize)
{
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n;
         v += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&csize[assign[v]], 1);
}

__global__ void zero_u32(uint32_t *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

struct FeatArgs {
    const float *base;
    int64_t n;
    int dim;
    const int32_t *graph;
    int R;
    int medoid;
    const int32_t *hub_ids;
    int nh;
    const int32_t *assign;
    const double *centroids;
    int h;
    int wcap;
    const int32_t *deg;
    const int32_t *indeg;
    const int32_t *mm;
    const unsigned long long *edges;
    const double *nu;
    const int32_t *csize;
    int hash_log2;
    bool vec4;
    double *raw;          // nh x 32
    int32_t *walk_sizes;  // nh x 6 or null
};

// What bounds it: the chain of batches (graph row, neighbour rows, sort, set)
// of a hub, about 5 us each; sixteen nodes at a time make it as many times
// shorter, and the hubs' chains run side by side.  200,000 x 128, 1,024 hubs:
// 22.7 ms with one wavefront per hub and a bitmap in memory, 4.2 ms now (the whole
// call 24.2 and 4.6).
__global__ void __launch_bounds__(64 * FW_WAVES) walk_kernel(FeatArgs a)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int slots = 1 << a.hash_log2;
    uint32_t *key = reinterpret_cast<uint32_t *>(lds);       // the set's ids
    uint32_t *place = key + slots;                           // their earliest place; 0: from an earlier batch
    double *dist = reinterpret_cast<double *>(lds);          // walk-node distances (after the walk)
    int32_t *S = reinterpret_cast<int32_t *>(place + slots);
    uint8_t *depth = reinterpret_cast<uint8_t *>(S + a.wcap);
    __shared__ int s_fresh[FW_WAVES], s_edges[FW_WAVES];
    __shared__ double s_len[FW_WAVES];
    __shared__ int s_cnt[6], s_maxd, s_other;
    __shared__ unsigned long long s_out, s_in;
    const int c = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const double nu = *a.nu;
    const double mean_in = (double)(*a.edges) / (double)a.n;
    const int mindeg = a.mm[0], maxdeg = a.mm[1];
    const int32_t v = a.hub_ids[c];
    const float *xv = a.base + (int64_t)v * a.dim;

    for (int i = t; i < slots; i += 64 * FW_WAVES) {
        key[i] = kNoId;
        place[i] = kNoId;
    }
    if (t < 6) s_cnt[t] = 0;
    if (t == 0) {
        s_maxd = 0;
        s_other = 0;
        s_out = 0ull;
        s_in = 0ull;
        S[0] = v;
        depth[0] = 0;
    }
    __syncthreads();
    auto slot_of = [&](uint32_t id) { return (int)((id * 2654435761u) >> (32 - a.hash_log2)); };
    if (t == 0) {
        key[slot_of((uint32_t)v)] = (uint32_t)v;
        place[slot_of((uint32_t)v)] = 0u;
    }
    __syncthreads();
    int ns = 1;
    long long wedges = 0;
    double wlen = 0.0;
    for (int head = 0; head < ns;) {
        // depths in the FIFO never fall: past the last hop nothing is left
        if (depth[head] >= a.h) break;
        const int batch = ns - head < FW_WAVES ? ns - head : FW_WAVES;
        const bool mine = wv < batch && depth[head + (wv < batch ? wv : 0)] < a.h;
        uint32_t id = kNoId;
        bool chosen = false;
        int at = -1;
        if (mine) {
            const int32_t u = S[head + wv];
            const int32_t w = lane < a.R ? a.graph[(int64_t)u * a.R + lane] : -1;
            uint64_t k = ~0ull;
            if (w >= 0) {
                k = dkey(d2_ff(a.base + (int64_t)u * a.dim, a.base + (int64_t)w * a.dim, a.dim, a.vec4));
                id = (uint32_t)w;
            }
            const int m = __popcll(__ballot(w >= 0));
            wsort(k, id);
            int x = (int)(((long long)mindeg * m + maxdeg - 1) / maxdeg);
            if (x < 2) x = 2;
            const int lo_n = m <= x ? m : (x + 1) / 2;
            const int hi_n = m <= x ? 0 : x / 2;
            chosen = lane < m && (lane < lo_n || lane >= m - hi_n);
            const double len = wsum(chosen ? sqrt(__longlong_as_double((long long)k)) : 0.0);
            const int ne = __popcll(__ballot(chosen));
            if (lane == 0) {
                s_edges[wv] = ne;
                s_len[wv] = len;
            }
            // into the set, while the subgraph can still grow
            if (chosen && ns < a.wcap) {
                at = slot_of(id);
                for (;;) {
                    const uint32_t old = atomicCAS(&key[at], kNoId, id);
                    if (old == kNoId || old == id) break;
                    at = (at + 1) & (slots - 1);
                }
                atomicMin(&place[at], (uint32_t)(64 * wv + lane + 1));
            }
        } else if (lane == 0) {
            s_edges[wv] = 0;
            s_len[wv] = 0.0;
        }
        __syncthreads();
        const bool fresh = at >= 0 && place[at] == (uint32_t)(64 * wv + lane + 1);
        const uint64_t fb = __ballot(fresh);
        if (lane == 0) s_fresh[wv] = __popcll(fb);
        const int next_depth = mine ? depth[head + wv] + 1 : 0;
        __syncthreads();
        int before = 0, all = 0;
        for (int q = 0; q < FW_WAVES; ++q) {
            before += q < wv ? s_fresh[q] : 0;
            all += s_fresh[q];
            if (q < batch) {
                wedges += s_edges[q];
                wlen += s_len[q];
            }
        }
        if (fresh) {
            place[at] = 0u;
            const int pos = ns + before + __popcll(fb & ((1ull << lane) - 1ull));
            if (pos < a.wcap) {
                S[pos] = (int32_t)id;
                depth[pos] = (uint8_t)next_depth;
            }
        }
        head += batch;
        ns = ns + all < a.wcap ? ns + all : a.wcap;
        __syncthreads();
    }
    // ---- the walk's nodes: counts (whole numbers, any order) and distances
    for (int q = t; q < ns; q += 64 * FW_WAVES) {
        const int dq = depth[q];
        if (dq <= 5) atomicAdd(&s_cnt[dq], 1);
        atomicMax(&s_maxd, dq);
        const int32_t w = S[q];
        if (q > 0 && a.assign[w] != c) atomicAdd(&s_other, 1);
        atomicAdd(&s_out, (unsigned long long)a.deg[w]);
        atomicAdd(&s_in, (unsigned long long)a.indeg[w]);
        if (q > 0) dist[q] = sqrt(d2_ff(xv, a.base + (int64_t)w * a.dim, a.dim, a.vec4)) / nu;
    }
    __syncthreads();
    if (t >= 64) return;
    int cnt_d[6];
    for (int q = 0; q < 6; ++q) cnt_d[q] = s_cnt[q];
    const int maxd = s_maxd, other = s_other;
    const double so = (double)s_out, si = (double)s_in;
    // ---- features
    double f[24];
    for (int q = 0; q < 24; ++q) f[q] = 0.0;
    f[0] = (double)a.deg[v] / a.R;
    f[1] = (double)a.indeg[v] / mean_in;
    for (int q = 1; q <= 5; ++q) f[1 + q] = log2(1.0 + cnt_d[q]);
    f[7] = log2(1.0 + (double)wedges);
    // out-neighbour distances
    {
        int32_t w = lane < a.R ? a.graph[(int64_t)v * a.R + lane] : -1;
        bool ok = w >= 0;
        double dv = ok ? sqrt(d2_ff(xv, a.base + (int64_t)w * a.dim, a.dim, a.vec4)) / nu : 0.0;
        int m = __popcll(__ballot(ok));
        if (m > 0) {
            double mean = wsum(dv) / m;
            double lo = wmin(ok ? dv : 1e300), hi = wmax(ok ? dv : -1e300);
            double q = wsum(ok ? (dv - mean) * (dv - mean) : 0.0);
            f[8] = mean;
            f[9] = lo;
            f[10] = hi;
            f[11] = sqrt(q / m);
        }
    }
    // walk-node distances (two passes)
    if (ns > 1) {
        double s = 0.0, lo = 1e300, hi = -1e300;
        for (int q = 1 + lane; q < ns; q += 64) {
            const double dv = dist[q];
            s += dv;
            lo = fmin(lo, dv);
            hi = fmax(hi, dv);
        }
        const int m = ns - 1;
        const double mean = wsum(s) / m;
        lo = wmin(lo);
        hi = wmax(hi);
        double qq = 0.0;
        for (int q = 1 + lane; q < ns; q += 64) {
            const double dv = dist[q];
            qq += (dv - mean) * (dv - mean);
        }
        qq = wsum(qq);
        f[12] = mean;
        f[13] = lo;
        f[14] = hi;
        f[15] = sqrt(qq / m);
    }
    f[16] = (double)a.csize[c] / ((double)a.n / a.nh);
    f[17] = sqrt(d2_fd(xv, a.centroids + (int64_t)c * a.dim, a.dim)) / nu;
    f[18] = sqrt(d2_ff(xv, a.base + (int64_t)a.medoid * a.dim, a.dim, a.vec4)) / nu;
    f[19] = ns > 1 ? (double)other / (ns - 1) : 0.0;
    f[20] = so / ns / a.R;
    f[21] = si / ns / mean_in;
    f[22] = wedges > 0 ? (wlen / (double)wedges) / nu : 0.0;
    f[23] = (double)maxd / a.h;
    if (lane < 32) a.raw[(int64_t)c * 32 + lane] = lane < 24 ? f[lane < 24 ? lane : 0] : 0.0;
    if (a.walk_sizes && lane < 6) a.walk_sizes[c * 6 + lane] = cnt_d[lane];
}

// Columns to zero mean and unit (population) deviation over the hubs.  The
// sums run over the hubs in order; the rows pass through LDS, 128 at a time.
constexpr int ST_ROWS = 128;

__global__ void __launch_bounds__(1024) standardise_kernel(const double *raw, int nh, int standardise,
                                                           float *out)
{
    __shared__ double row[ST_ROWS][32];
    __shared__ double s_mean[32], s_sd[32];
    const int t = threadIdx.x, col = t & 31;
    double mean = 0.0, sd = 0.0;
    for (int pass = 0; pass < 2 && standardise; ++pass) {
        double s = 0.0;
        for (int c0 = 0; c0 < nh; c0 += ST_ROWS) {
            __syncthreads();
            for (int e = t; e < ST_ROWS * 32; e += 1024) {
                const int c = c0 + e / 32;
                row[e / 32][e % 32] = c < nh ? raw[(int64_t)c * 32 + e % 32] : 0.0;
            }
            __syncthreads();
            const int m = nh - c0 < ST_ROWS ? nh - c0 : ST_ROWS;
            if (t < 32) {
#pragma unroll 16
                for (int c = 0; c < m; ++c) {
                    if (pass == 0) s += row[c][t];
                    else {
                        const double z = row[c][t] - mean;
                        s += z * z;
                    }
                }
            }
        }
        if (t < 32) {
            if (pass == 0) s_mean[t] = s / nh;
            else s_sd[t] = sqrt(s / nh);
        }
        __syncthreads();
        mean = s_mean[col];
        if (pass == 1) sd = s_sd[col];
    }
    for (int64_t e = t; e < (int64_t)nh * 32; e += 1024)
        out[e] = !standardise ? (float)raw[e] : sd > 0 ? (float)((raw[e] - mean) / sd) : 0.f;
}

inline int gridn(int64_t n) { return (int)((n + 255) / 256 > 4096 ? 4096 : (n + 255) / 256); }

// slots of the hash set: at most two thirds full
inline int hash_log2(int wcap)
{
    int l = 8;
    while ((1 << l) * 2 < 3 * (wcap + FW_WAVES * 64)) ++l;
    return l;
}

}  // namespace

size_t hub_features_ws(int64_t n, int nh)
{
    size_t b = round_up((size_t)n * 4, 256) * 2 + round_up(64, 256) * 2;
    b += round_up(NU_BLOCKS * 8, 256) + round_up(NU_BLOCKS * 4, 256) + 256;
    b += round_up((size_t)nh * 4, 256);
    b += round_up((size_t)nh * 32 * 8, 256);
    return b;
}

}  // namespace ann

using namespace ann;

extern "C" ann_status ann_hub_features(const float *base, int64_t n, int32_t dim,
                                       const int32_t *graph, int32_t R, int32_t medoid,
                                       const int32_t *hub_ids, int32_t n_hubs,
                                       const int32_t *assign, const double *centroids, int32_t h,
                                       int32_t wcap, int32_t standardise, float *features,
                                       int32_t *walk_sizes, void *workspace, size_t ws_bytes,
                                       void *stream)
{
    ANN_REQUIRE(base && graph && hub_ids && assign && centroids && features && workspace,
                "a required pointer is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF && dim >= 1, "bad n or dim");
    ANN_REQUIRE(R >= 1 && R <= 64, "R must be in [1, 64]");
    ANN_REQUIRE(medoid >= 0 && medoid < n, "medoid out of range");
    ANN_REQUIRE(n_hubs >= 1 && n_hubs <= n, "n_hubs must be in [1, n]");
    ANN_REQUIRE(h >= 1 && h <= 250, "h must be in [1, 250]");
    ANN_REQUIRE(wcap >= 1 && wcap <= FW_MAX, "wcap must be in [1, 4096]");
    ANN_REQUIRE(ws_bytes >= ann_workspace_size(ANN_OP_HUB_FEATURES, n, dim, n_hubs, R),
                "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    int32_t *deg = cv.take<int32_t>((size_t)n);
    int32_t *indeg = cv.take<int32_t>((size_t)n);
    int32_t *mm = cv.take<int32_t>(16);
    unsigned long long *edges = cv.take<unsigned long long>(8);
    double *nu_part = cv.take<double>(NU_BLOCKS);
    int *nu_cnt = cv.take<int>(NU_BLOCKS);
    double *nu = cv.take<double>(1);
    int32_t *csize = cv.take<int32_t>((size_t)n_hubs);
    double *raw = cv.take<double>((size_t)n_hubs * 32);

    hipLaunchKernelGGL(zero_u32, dim3(gridn(n)), dim3(256), 0, st, (uint32_t *)indeg, n);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(zero_u32, dim3(gridn(n_hubs)), dim3(256), 0, st, (uint32_t *)csize,
                       (int64_t)n_hubs);
    ANN_LAUNCHED();
    const bool vec4 = dim % 4 == 0 && aligned(base, 16);
    int32_t mm_init[2] = {0x7fffffff, 0};
    unsigned long long e0 = 0;
    ANN_HIP(hipMemcpyAsync(mm, mm_init, sizeof(mm_init), hipMemcpyHostToDevice, st));
    ANN_HIP(hipMemcpyAsync(edges, &e0, sizeof(e0), hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(degree_kernel, dim3(gridn(n)), dim3(256), 0, st, graph, n, R, deg, indeg, mm,
                       edges);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(nu_partial_kernel, dim3(NU_BLOCKS), dim3(256), 0, st, base, n, dim, vec4,
                       graph, R, nu_part, nu_cnt);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(nu_kernel, dim3(1), dim3(256), 0, st, nu_part, nu_cnt, NU_BLOCKS, nu);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(csize_kernel, dim3(gridn(n)), dim3(256), 0, st, assign, n, csize);
    ANN_LAUNCHED();
    FeatArgs a{};
    a.base = base;
    a.n = n;
    a.dim = dim;
    a.graph = graph;
    a.R = R;
    a.medoid = medoid;
    a.hub_ids = hub_ids;
    a.nh = n_hubs;
    a.assign = assign;
    a.centroids = centroids;
    a.h = h;
    a.wcap = wcap;
    a.deg = deg;
    a.indeg = indeg;
    a.mm = mm;
    a.edges = edges;
    a.nu = nu;
    a.csize = csize;
    a.hash_log2 = hash_log2(wcap);
    a.vec4 = vec4;
    a.raw = raw;
    a.walk_sizes = walk_sizes;
    // the distances of the walk's nodes take the place of the set's two arrays
    const size_t lds = round_up(((size_t)1 << a.hash_log2) * 8 + (size_t)wcap * 5, 16);
    ANN_HIP(hipFuncSetAttribute((const void *)walk_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds));
    hipLaunchKernelGGL(walk_kernel, dim3(n_hubs), dim3(64 * FW_WAVES), lds, st, a);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(standardise_kernel, dim3(1), dim3(1024), 0, st, raw, n_hubs, standardise,
                       features);
    ANN_LAUNCHED();
    return ANN_OK;
}
