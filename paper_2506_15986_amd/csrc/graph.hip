// Proximity-graph construction on the GPU: exact kNN candidates, alpha-RNG
// pruning (the triangle-inequality pruning NSG applies; alpha = 1 is MRNG),
// the medoid (navigating node), and connectivity repair so that every node
// is reachable from the medoid and can reach it.
//
//  prune   one wavefront per node; candidates in (d2, id) order; candidate c
//          survives unless a kept o has alpha^2 * d2(o,c) <= d2(p,c), with
//          alpha^2 formed in FP64 from the FP32 alpha and FP64 distances;
//          at most R-2 kept, slots R-2 and R-1 left for repair.
//  medoid  point nearest the mean: FP64 column sums / n, then FP64 squared
//          distance to the mean summed in dimension order without FMA,
//          argmin by (d2, id).
//  repair  forward: BFS from the medoid; the smallest unreached id u is
//          linked from the reached node v with slot R-2 free minimising
//          (d2(u,v), v), and the BFS continues from u.  reverse: BFS over
//          reversed edges; the smallest id w that cannot reach the medoid is
//          linked w -> t, t minimising (d2(w,t), t) over nodes that can.
//          The argmin is read off u's exact kNN list when the list holds an
//          eligible node (the first eligible entry is then the global
//          argmin); otherwise a full scan runs.  The bridges are found in
//          parallel (the repair section below).
#include "common.h"
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <vector>
#include "knn.h"

namespace ann {



namespace {

// ---------------------------------------------------------------- prune
constexpr int PG = 8;         // lanes per distance, candidates tested at a time
constexpr int PRUNE_REG = 4;  // float4s of a candidate's row that a lane holds

// One wavefront per node, PG candidates at a time with PG lanes each: all of
// them are tested against one kept node after another (nearest first, until
// none is left), then the first one left is kept and the rest are tested
// against it.  (One candidate at a time against PG kept nodes, the same number
// of distances at once but twice the steps and both rows loaded for each, took
// 14.8 ms on 300,000 x 128 with K = 128; 3.3 now.)
//
// The test a2 * d2 <= dpc is decided in FP32 where it is clear: the terms are
// positive, so the FP32 sum has a relative error of at most `err`, and its
// range is checked.  Otherwise FP64 decides: lane gl of PG sums the dimensions
// gl, gl + PG, ..., the lanes' sums are added pairwise.
// Bound by the kept rows' loads (L2) and their latency.
template <bool VEC>
__global__ void __launch_bounds__(256) prune_kernel(const float *base, int64_t n, int dim,
                                                    const int32_t *cand, const double *cand_d2,
                                                    int K, int R, double a2, double err,
                                                    int32_t *graph)
{
    __shared__ int32_t kept_s[4][64];
    const int w = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * 4 + w;
    if (p >= n) return;
    int32_t *kept = kept_s[w];
    const int gi = lane / PG, gl = lane % PG;
    // chunk i of a row (four dimensions, or one)
    const int chunks = VEC ? dim / 4 : dim;
    auto chunk = [&](const float *row, int i) __attribute__((always_inline)) {
        if (i >= chunks) return make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (VEC) return reinterpret_cast<const float4 *>(row)[i];
        return make_float4(row[i], 0.f, 0.f, 0.f);
    };
    auto add = [](float acc, const float4 &x, const float4 &y) __attribute__((always_inline)) {
        const float a = x.x - y.x;
        acc = __builtin_fmaf(a, a, acc);
        if constexpr (VEC) {
            const float b = x.y - y.y, c = x.z - y.z, d = x.w - y.w;
            acc = __builtin_fmaf(b, b, acc);
            acc = __builtin_fmaf(c, c, acc);
            acc = __builtin_fmaf(d, d, acc);
        }
        return acc;
    };
    int nk = 0;
    bool more = true;
    for (int t0 = 0; t0 < K && nk < R - 2 && more; t0 += PG) {
        const int t = t0 + gi;
        int32_t c = t < K ? cand[p * K + t] : -1;
        // the list ends at its first negative entry
        const uint64_t ends = __ballot(c < 0);
        if (ends) {
            more = false;
            if (gi >= (__ffsll((unsigned long long)ends) - 1) / PG) c = -1;
        }
        const double dpc = c >= 0 ? cand_d2[p * K + t] : 0.0;
        const float *xc = base + (int64_t)(c >= 0 ? c : 0) * dim;
        float4 own[PRUNE_REG];
#pragma unroll
        for (int u = 0; u < PRUNE_REG; ++u) own[u] = chunk(xc, gl + PG * u);
        bool alive = c >= 0;
        // tests the candidates left against kept node o
        auto test = [&](int32_t o) __attribute__((always_inline)) {
            const float *xo = base + (int64_t)o * dim;
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < PRUNE_REG; ++u) acc = add(acc, chunk(xo, gl + PG * u), own[u]);
            for (int i = gl + PG * PRUNE_REG; i < chunks; i += PG)
                acc = add(acc, chunk(xo, i), chunk(xc, i));
            for (int q = PG / 2; q > 0; q >>= 1) acc += __shfl_xor(acc, q);
            const double est = a2 * (double)acc;
            const bool sane = acc > 1e-30f && acc < 1e37f;
            const bool dom = sane && est * (1.0 + err) <= dpc;
            const bool clear = dom || (sane && est * (1.0 - err) > dpc);
            if (__ballot(alive && !clear)) {
                double sum = 0.0;
                for (int j = gl; j < dim; j += PG) {
                    const double df = (double)xo[j] - (double)xc[j];
                    sum = __builtin_fma(df, df, sum);
                }
                for (int q = PG / 2; q > 0; q >>= 1) sum += __shfl_xor(sum, q);
                alive = alive && !(clear ? dom : a2 * sum <= dpc);
            } else {
                alive = alive && !dom;
            }
        };
        uint64_t left = __ballot(alive);
        for (int u = 0; u < nk && left; ++u) {
            test(kept[u]);
            left = __ballot(alive);
        }
        while (left && nk < R - 2) {
            const int first = __ffsll((unsigned long long)left) - 1;
            const int32_t o = __builtin_amdgcn_readlane(c, first);
            if (lane == 0) kept[nk] = o;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            ++nk;
            alive = alive && gi != first / PG;
            left = __ballot(alive);
            if (!left || nk >= R - 2) break;
            test(o);
            left = __ballot(alive);
        }
    }
    for (int s = lane; s < R; s += 64) graph[p * R + s] = s < nk ? kept[s] : -1;
}

// ---------------------------------------------------------------- medoid
constexpr int MED_ROWS = 4096;

__global__ void medoid_colsum_kernel(const float *base, int64_t n, int dim, double *partial)
{
    const int64_t r0 = (int64_t)blockIdx.x * MED_ROWS;
    int64_t r1 = r0 + MED_ROWS;
    if (r1 > n) r1 = n;
    for (int j = threadIdx.x; j < dim; j += blockDim.x) {
        // added one by one, loaded thirty-two at a time (the chain of loads
        // was the cost: 1.1 ms for 300,000 rows, 0.08 now)
        double s = 0.0;
        int64_t r = r0;
        for (; r + 32 <= r1; r += 32) {
            float x[32];
#pragma unroll
            for (int u = 0; u < 32; ++u) x[u] = base[(r + u) * dim + j];
#pragma unroll
            for (int u = 0; u < 32; ++u) s += (double)x[u];
        }
        for (; r < r1; ++r) s += (double)base[r * dim + j];
        partial[(int64_t)blockIdx.x * dim + j] = s;
    }
}

__global__ void medoid_colmean_kernel(const double *partial, int chunks, int dim, int64_t n, double *mu)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= dim) return;
    double s = 0.0;
    for (int c = 0; c < chunks; ++c) s += partial[(int64_t)c * dim + j];
    mu[j] = s / (double)n;
}

struct DKey {
    double v;
    int64_t id;
};

__device__ inline bool dkey_less(const DKey &a, const DKey &b)
{
    return a.v < b.v || (a.v == b.v && a.id < b.id);
}

__device__ double sqdist_to_mean(const float *x, const double *mu, int dim, bool vec4)
{
#pragma clang fp contract(off)
    double s = 0.0;
    auto add = [&](float v, double m) {
        const double t = (double)v - m;
        s = s + t * t;
    };
    if (vec4) {   // whole, aligned rows of float4s
#pragma unroll 8
        for (int j = 0; j < dim; j += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(x + j);
            add(v.x, mu[j]);
            add(v.y, mu[j + 1]);
            add(v.z, mu[j + 2]);
            add(v.w, mu[j + 3]);
        }
        return s;
    }
    for (int j = 0; j < dim; ++j) {
        double t = (double)x[j] - mu[j];
        s = s + t * t;
    }
    return s;
}

__device__ inline DKey block_min(DKey k, DKey *sh)
{
    const int t = threadIdx.x;
    sh[t] = k;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (t < s && dkey_less(sh[t + s], sh[t])) sh[t] = sh[t + s];
        __syncthreads();
    }
    DKey r = sh[0];
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(256) medoid_dist_kernel(const float *base, int64_t n, int dim,
                                                          bool vec4, const double *mu, DKey *partial)
{
    __shared__ DKey sh[256];
    DKey best{__longlong_as_double(0x7ff0000000000000ll), 0x7fffffffffffffffll};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        DKey k{sqdist_to_mean(base + i * dim, mu, dim, vec4), i};
        if (dkey_less(k, best)) best = k;
    }
    DKey r = block_min(best, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = r;
}

__global__ void argmin_final_kernel(const DKey *partial, int count, DKey *out)
{
    __shared__ DKey sh[256];
    DKey best{__longlong_as_double(0x7ff0000000000000ll), 0x7fffffffffffffffll};
    for (int i = threadIdx.x; i < count; i += blockDim.x)
        if (dkey_less(partial[i], best)) best = partial[i];
    DKey r = block_min(best, sh);
    if (threadIdx.x == 0) *out = r;
}

// ---------------------------------------------------------------- repair
// The repair as it is defined takes one bridge after another: the smallest
// unreached id u, a link to it from a reached node, a search from u, the next
// u.  The same bridges come from three parallel steps.
//
//  labels    A link only ever leaves a node that is already reached, so what
//            a search from u reaches is fixed by the pruned graph alone.  Let
//            m(w) be the smallest id that reaches w along its edges (-1 when
//            the medoid does).  The u's are then exactly the nodes with
//            m(u) = u, and w is reached by the search from m(w), so "v is
//            reached when u's turn comes" reads m(v) < u.  m is the fixpoint
//            of m(w) = min m(v) over edges v -> w, shortened by m(w) =
//            min(m(w), m(m(w))) (what reaches m(w) reaches w).  Where distances
//            in the graph are long (points along a line) that would still take
//            a sweep per edge of the way; then the labels of the other
//            direction are kept too, and nodes found to lie on a common cycle
//            are joined: they share both labels.
//  matching  Every u takes the first v of its list with m(v) < u whose slot
//            no smaller u took.  All nodes prefer the smaller u, so this is
//            the one stable matching, and proposals in any order reach it:
//            u proposes down its list, v keeps the smallest proposer, a
//            displaced one goes on down its own list.
//  scans     A u whose list holds no eligible node proposes to its nearest
//            eligible node overall; many such u's share one pass over the
//            base vectors.
// The reverse repair has the same form along reversed edges, without the
// competition for slots (the link leaves w itself).
//
// Bound: the FP64 distances of the scans.  The labels take about eight sweeps
// over the graph rows per phase where distances in the graph are short, and
// about as many again as joining takes rounds where they are long; only a chain
// of one-way edges still takes a sweep per edge.  Measured at 300,000 x 128,
// R = 32 (518 scans): labels 0.65 ms, lists under 0.1 ms, scans 2.2 ms in 4
// passes; one workgroup that followed the definition bridge by bridge, with a
// host round trip and a pass over the base per scan, took 566 ms.  From the
// candidate lists of 100,000 points on a line, R = 16: 1.6 ms with their ids in
// order, 9.9 ms shuffled (838 and 357 ms without joining).
constexpr int32_t kFree = 0x7fffffff;   // a slot nobody holds
constexpr int SCAN_U = 8;               // u's that share one load of a base row
constexpr int SCAN_BATCH = 512;         // u's per scan launch
constexpr int SCAN_BLOCKS = 256;        // workgroups per group of SCAN_U u's
constexpr int SCAN_DK = 128;            // dimensions staged in LDS at a time
constexpr int LONG_SWEEPS = 16;         // sweeps after which joining starts

// atomics are performed in L2; read what they write the same way
__device__ inline int32_t ld_agent(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct RepairCounts {
    int32_t changed;     // a label changed in the last sweep
    int32_t other;       // ... of the other direction (not read)
    int32_t roots;       // u's of this phase
    int32_t left[2];     // u's waiting for a scan (two lists used in turn)
};

__global__ void repair_init_kernel(int32_t *m, int32_t *stamp, int32_t *holder, int64_t n,
                                   int32_t medoid, RepairCounts *c)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        m[i] = i == medoid ? -1 : (int32_t)i;
        stamp[i] = 0;
        holder[i] = kFree;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *c = RepairCounts{0, 0, 0, {0, 0}};
}

__global__ void repair_flag_kernel(int32_t *flag, int32_t v) { *flag = v; }

// Forward labels, one sweep: a node whose label fell in the last sweep (or
// falls now through its label's label) offers it to its out-neighbours.
// 2^lw lanes share a node, lane s its slot s.  A label read here may be older
// than another workgroup's update in the same sweep, hence too large: the
// update's stamp makes the next sweep offer the newer one.
__global__ void __launch_bounds__(256) push_labels_kernel(const int32_t *graph, int64_t n, int R,
                                                          int lw, int32_t *m, int32_t *stamp,
                                                          int round, int32_t *changed)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t v = g >> lw;
    const int s = (int)(g & ((1 << lw) - 1));
    if (v >= n) return;
    int32_t l = m[v];
    bool active = stamp[v] >= round;
    if (l >= 0 && l != v) {
        const int32_t l2 = m[l];
        if (l2 < l) {
            l = l2;
            active = true;
            if (s == 0) atomicMin(&m[v], l);
        }
    }
    if (!active || s >= R) return;
    const int32_t w = graph[v * R + s];
    if (w < 0 || m[w] <= l) return;
    if (atomicMin(&m[w], l) > l) {
        stamp[w] = round + 1;
        *changed = 1;
    }
}

// Reverse labels, one sweep: m(v) = the smallest label among v's own, its
// out-neighbours' and its label's.  Only v's lanes write m[v].
__global__ void __launch_bounds__(256) pull_labels_kernel(const int32_t *graph, int64_t n, int R,
                                                          int lw, int32_t *m, int32_t *changed)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t v = g >> lw;
    const int s = (int)(g & ((1 << lw) - 1));
    int32_t own = -1, l = -1;
    if (v < n) {
        own = m[v];
        l = own;
        if (own >= 0) {
            const int32_t l2 = m[own];
            l = l2 < l ? l2 : l;
            if (s < R) {
                const int32_t w = graph[v * R + s];
                if (w >= 0) {
                    const int32_t lv = m[w];
                    l = lv < l ? lv : l;
                }
            }
        }
    }
    for (int o = (1 << lw) >> 1; o > 0; o >>= 1) {
        const int32_t other = __shfl_xor(l, o);
        l = other < l ? other : l;
    }
    if (v < n && s == 0 && l < own) {
        m[v] = l;
        *changed = 1;
    }
}

// start of joining: the other direction's labels and the joined nodes' roots
__global__ void join_init_kernel(int32_t *other, int32_t *root, int64_t n, int32_t medoid)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) other[i] = root[i] = i == medoid ? -1 : (int32_t)i;
}

// Labels name nodes, -1 the medoid.  A node that is reached by the node it
// reaches (both labels name it) lies on a cycle with it, and so do the roots:
// the larger root gets the smaller one.  Every node and its root then share
// their labels of both directions, so that a label that arrives at one node of
// a joined set is everywhere in it two rounds later.  Whatever the threads see
// of each other's writes, only nodes of one cycle are joined, and labels only
// fall to labels of the same cycle.  m: the phase's labels, pushed: which of the
// two goes by stamps (stamp `next` makes the next sweep offer a label).
__global__ void __launch_bounds__(256) join_kernel(int32_t *m, int32_t *other, int32_t *root, int64_t n,
                                                   int32_t medoid, const int32_t *pushed, int32_t *stamp,
                                                   int next, int32_t *changed)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    auto node = [&](int32_t k) { return k < 0 ? medoid : k; };
    int32_t c = root[v];
    const int32_t a = m[v];
    if (a == other[v] && a != c) {
        const int32_t lo = a < c ? a : c, hi = a < c ? c : a;
        atomicMin(&root[node(hi)], lo);
        c = lo;
    }
    const int32_t up = root[node(c)];
    if (up < c) c = up;
    if (c < root[v]) atomicMin(&root[v], c);
    const int32_t r = node(c);
    if (r == v) return;
    for (int which = 0; which < 2; ++which) {
        int32_t *l = which ? other : m;
        const int32_t lv = l[v], lr = l[r];
        if (lv == lr) continue;
        const int32_t to = lv < lr ? lv : lr;
        const int64_t w = lv < lr ? r : v;
        if (atomicMin(&l[w], to) > to) {
            if (l == pushed) stamp[w] = next;
            if (l == m) *changed = 1;
        }
    }
}

// the u's (m(u) = u), in any order
__global__ void __launch_bounds__(256) collect_roots_kernel(const int32_t *m, int64_t n,
                                                            int32_t *roots, RepairCounts *c)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool is = i < n && m[i] == i;
    const uint64_t b = __ballot(is);
    if (!b) return;
    const int lane = __lane_id();
    int at = 0;
    if (lane == 0) at = atomicAdd(&c->roots, __popcll(b));
    at = __shfl(at, 0);
    if (is) roots[at + __popcll(b & ((1ull << lane) - 1))] = (int32_t)i;
}

// One wavefront: u proposes down its candidate list until a node keeps it; a
// u displaced from there goes on in its place (from the start of its list:
// who refused it holds a smaller one still).  Each turn lowers some holder,
// so this ends.  A u whose list is used up joins the scan list.
__device__ inline void propose(int32_t u, const int32_t *cand, int K, const int32_t *m,
                               int32_t *holder, int32_t *scan_list, int32_t *scan_count)
{
    const int lane = __lane_id();
    for (;;) {
        int32_t displaced = -1;
        bool kept = false;
        for (int q0 = 0; q0 < K && !kept; q0 += 64) {
            const int q = q0 + lane;
            const int32_t v = q < K ? cand[(int64_t)u * K + q] : -1;
            const bool ok = v >= 0 && m[v] < u && ld_agent(&holder[v]) > u;
            for (uint64_t b = __ballot(ok); b; b &= b - 1) {
                const int32_t vb = __shfl(v, (int)__builtin_ctzll(b));
                int32_t old = 0;
                if (lane == 0) old = atomicMin(&holder[vb], u);
                old = __shfl(old, 0);
                if (old > u) {
                    kept = true;
                    displaced = old == kFree ? -1 : old;
                    break;
                }
            }
        }
        if (!kept) {
            if (lane == 0) scan_list[atomicAdd(scan_count, 1)] = u;
            return;
        }
        if (displaced < 0) return;
        u = displaced;
    }
}

__global__ void __launch_bounds__(256) match_kernel(const int32_t *roots, int count,
                                                    const int32_t *cand, int K, const int32_t *m,
                                                    int32_t *holder, int32_t *scan_list,
                                                    int32_t *scan_count)
{
    const int i = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (i >= count) return;
    propose(roots[i], cand, K, m, holder, scan_list, scan_count);
}

// reverse: w links to the first node of its list with m(v) < w
__global__ void __launch_bounds__(256) reverse_link_kernel(const int32_t *roots, int count,
                                                           const int32_t *cand, int K,
                                                           const int32_t *m, int32_t *graph, int R,
                                                           int32_t *scan_list, int32_t *scan_count)
{
    const int i = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (i >= count) return;
    const int lane = __lane_id();
    const int32_t w = roots[i];
    for (int q0 = 0; q0 < K; q0 += 64) {
        const int q = q0 + lane;
        const int32_t v = q < K ? cand[(int64_t)w * K + q] : -1;
        const uint64_t b = __ballot(v >= 0 && m[v] < w);
        if (b) {
            const int32_t t = __shfl(v, (int)__builtin_ctzll(b));
            if (lane == 0) graph[(int64_t)w * R + (R - 1)] = t;
            return;
        }
    }
    if (lane == 0) scan_list[atomicAdd(scan_count, 1)] = w;
}

// Full scan: per u the argmin over eligible v of (d2(u, v), v); eligible =
// m(v) < u and (holder NULL or v's slot not held by a smaller u).  blockIdx.y
// picks SCAN_U u's, one thread takes a base row at a time for all of them (so
// the row is read once per SCAN_U distances).  d2 is the FP64 sum in dimension
// order.  A distance that is no number counts as +inf.  partial: one key per
// (u, workgroup).  VEC: whole, aligned rows of float4s, read as such (a lane
// reads its own row, so the loads were the cost: 500 u's on 300,000 x 128 took
// 11.7 ms one float at a time, 2.2 now).
template <bool VEC>
__global__ void __launch_bounds__(256) scan_batch_kernel(const float *base, int64_t n, int dim,
                                                         const int32_t *m, const int32_t *holder,
                                                         const int32_t *list, int count,
                                                         DKey *partial)
{
    __shared__ double xs[SCAN_U][SCAN_DK];
    __shared__ DKey sh[256];
    __shared__ int32_t us[SCAN_U];
    const int t = threadIdx.x;
    const int u0 = (int)blockIdx.y * SCAN_U;
    if (t < SCAN_U) us[t] = u0 + t < count ? list[u0 + t] : -1;
    __syncthreads();
    const double inf = __longlong_as_double(0x7ff0000000000000ll);
    DKey best[SCAN_U];
#pragma unroll
    for (int k = 0; k < SCAN_U; ++k) best[k] = DKey{inf, 0x7fffffffffffffffll};
    const int64_t tiles = (n + 255) / 256;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t v = tile * 256 + t;
        const float *xv = base + (v < n ? v : 0) * dim;
        double acc[SCAN_U];
#pragma unroll
        for (int k = 0; k < SCAN_U; ++k) acc[k] = 0.0;
        for (int d0 = 0; d0 < dim; d0 += SCAN_DK) {
            const int dd = dim - d0 < SCAN_DK ? dim - d0 : SCAN_DK;
            if (dim > SCAN_DK || tile == (int64_t)blockIdx.x) {
                __syncthreads();
                for (int e = t; e < SCAN_U * dd; e += 256) {
                    const int k = e / dd, j = e - k * dd;
                    xs[k][j] = us[k] >= 0 ? (double)base[(int64_t)us[k] * dim + d0 + j] : 0.0;
                }
                __syncthreads();
            }
            auto add = [&](int j, float v) __attribute__((always_inline)) {
                const double x = (double)v;
#pragma unroll
                for (int k = 0; k < SCAN_U; ++k) {
                    const double d = xs[k][j] - x;
                    acc[k] = __builtin_fma(d, d, acc[k]);
                }
            };
            if constexpr (VEC) {
                for (int j0 = 0; j0 < dd; j0 += 32) {
                    float4 x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (j0 + 4 * u < dd)
                            x[u] = *reinterpret_cast<const float4 *>(xv + d0 + j0 + 4 * u);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int j = j0 + 4 * u;
                        if (j >= dd) break;
                        add(j, x[u].x);
                        add(j + 1, x[u].y);
                        add(j + 2, x[u].z);
                        add(j + 3, x[u].w);
                    }
                }
            } else {
                for (int j = 0; j < dd; ++j) add(j, xv[d0 + j]);
            }
        }
        if (v < n) {
            const int32_t mv = m[v];
            const int32_t hv = holder ? ld_agent(&holder[v]) : kFree;
#pragma unroll
            for (int k = 0; k < SCAN_U; ++k) {
                const int32_t u = us[k];
                if (u < 0 || v == u || mv >= u || hv <= u) continue;
                const DKey key{acc[k] <= inf ? acc[k] : inf, v};
                if (dkey_less(key, best[k])) best[k] = key;
            }
        }
    }
    for (int k = 0; k < SCAN_U; ++k) {
        const DKey r = block_min(best[k], sh);
        if (t == 0 && u0 + k < count) partial[(int64_t)(u0 + k) * gridDim.x + blockIdx.x] = r;
    }
}

// One workgroup per scanned u: its nearest eligible node, then (forward) the
// proposal to it and the way down the list of whoever it displaces, or the
// next scan list when a smaller u got there first; (reverse) the link.
__global__ void __launch_bounds__(256) scan_apply_kernel(const DKey *partial, int blocks,
                                                         const int32_t *list, int64_t n,
                                                         const int32_t *cand, int K,
                                                         const int32_t *m, int32_t *holder,
                                                         int32_t *graph, int R, int32_t *scan_list,
                                                         int32_t *scan_count)
{
    __shared__ DKey sh[256];
    DKey best{__longlong_as_double(0x7ff0000000000000ll), 0x7fffffffffffffffll};
    for (int i = threadIdx.x; i < blocks; i += 256) {
        const DKey k = partial[(int64_t)blockIdx.x * blocks + i];
        if (dkey_less(k, best)) best = k;
    }
    best = block_min(best, sh);
    if (threadIdx.x >= 64 || best.id >= n) return;
    const int lane = __lane_id();
    const int32_t u = list[blockIdx.x], v = (int32_t)best.id;
    if (!holder) {
        if (lane == 0) graph[(int64_t)u * R + (R - 1)] = v;
        return;
    }
    int32_t old = 0;
    if (lane == 0) old = atomicMin(&holder[v], u);
    old = __shfl(old, 0);
    if (old < u) {
        if (lane == 0) scan_list[atomicAdd(scan_count, 1)] = u;
    } else if (old != kFree) {
        propose(old, cand, K, m, holder, scan_list, scan_count);
    }
}

__global__ void forward_link_kernel(const int32_t *holder, int64_t n, int R, int32_t *graph)
{
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v < n && holder[v] != kFree) graph[v * R + (R - 2)] = holder[v];
}

}  // namespace

ann_status medoid_run(const float *base, int64_t n, int dim, double *partial_cols, double *mu,
                      void *partial_keys, void *best_key, int32_t *medoid_host, hipStream_t st)
{
    int chunks = (int)((n + MED_ROWS - 1) / MED_ROWS);
    hipLaunchKernelGGL(medoid_colsum_kernel, dim3(chunks), dim3(128), 0, st, base, n, dim, partial_cols);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(medoid_colmean_kernel, dim3((dim + 127) / 128), dim3(128), 0, st, partial_cols,
                       chunks, dim, n, mu);
    ANN_LAUNCHED();
    int blocks = (int)((n + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    DKey *pk = static_cast<DKey *>(partial_keys);
    DKey *bk = static_cast<DKey *>(best_key);
    const bool vec4 = dim % 4 == 0 && aligned(base, 16);
    hipLaunchKernelGGL(medoid_dist_kernel, dim3(blocks), dim3(256), 0, st, base, n, dim, vec4, mu, pk);
    ANN_LAUNCHED();
    hipLaunchKernelGGL(argmin_final_kernel, dim3(1), dim3(256), 0, st, pk, blocks, bk);
    ANN_LAUNCHED();
    DKey h{};
    ANN_HIP(hipMemcpyAsync(&h, bk, sizeof(DKey), hipMemcpyDeviceToHost, st));
    ANN_HIP(hipStreamSynchronize(st));
    *medoid_host = (int32_t)h.id;
    return ANN_OK;
}

size_t medoid_ws(int64_t n, int dim)
{
    int chunks = (int)((n + MED_ROWS - 1) / MED_ROWS);
    return round_up((size_t)chunks * dim * 8, 256) + round_up((size_t)dim * 8, 256) +
           round_up(2048 * sizeof(DKey), 256) + round_up(sizeof(DKey), 256);
}

}  // namespace ann

using namespace ann;

namespace ann {
namespace {

// Buffers of the steps after the candidate lists: pruning, medoid, repair.
struct TailBufs {
    int32_t *m, *stamp, *holder, *roots;   // n each
    int32_t *list[2];                      // n each: u's waiting for a scan
    RepairCounts *counts;
    double *mu;
    DKey *partial, *best;
    double *med_cols;    // MED_ROWS-chunk column sums for the medoid
};

int scan_blocks(int64_t n)
{
    const int64_t tiles = (n + 255) / 256;
    return (int)(tiles < SCAN_BLOCKS ? tiles : SCAN_BLOCKS);
}

// keys of the medoid's argmin and of a batch of scans
size_t partial_keys(int64_t n)
{
    const size_t scans = (size_t)SCAN_BATCH * scan_blocks(n);
    return scans > 2048 ? scans : 2048;
}

size_t tail_ws(int64_t n, int dim, int R)
{
    (void)R;
    size_t b = round_up((size_t)n * 4, 256) * 6;                                    // labels .. lists
    b += round_up(sizeof(RepairCounts), 256);
    b += round_up((size_t)dim * 8, 256) + round_up(partial_keys(n) * sizeof(DKey), 256);
    b += round_up(sizeof(DKey), 256);
    b += round_up((size_t)((n + MED_ROWS - 1) / MED_ROWS) * dim * 8, 256);
    return b + 1024;
}

TailBufs take_tail(Carve &cv, int64_t n, int dim)
{
    TailBufs t{};
    t.m = cv.take<int32_t>((size_t)n);
    t.stamp = cv.take<int32_t>((size_t)n);
    t.holder = cv.take<int32_t>((size_t)n);
    t.roots = cv.take<int32_t>((size_t)n);
    t.list[0] = cv.take<int32_t>((size_t)n);
    t.list[1] = cv.take<int32_t>((size_t)n);
    t.counts = cv.take<RepairCounts>(1);
    t.mu = cv.take<double>((size_t)dim);
    t.partial = cv.take<DKey>(partial_keys(n));
    t.best = cv.take<DKey>(1);
    t.med_cols = cv.take<double>((size_t)((n + MED_ROWS - 1) / MED_ROWS) * dim);
    return t;
}

ann_status read_counts(const RepairCounts *dev, RepairCounts &h, hipStream_t st)
{
    ANN_HIP(hipMemcpyAsync(&h, dev, sizeof(h), hipMemcpyDeviceToHost, st));
    ANN_HIP(hipStreamSynchronize(st));
    return ANN_OK;
}

// One phase of the repair (0 forward, 1 reverse); *bridges = links added.
ann_status repair_phase(const float *base, int64_t n, int dim, const int32_t *cand, int K, int R,
                        int phase, int32_t medoid, int32_t *graph, int32_t *bridges,
                        const TailBufs &t, hipStream_t st)
{
    int lw = 0;
    while ((1 << lw) < R) ++lw;
    const unsigned sweep = (unsigned)(((n << lw) + 255) / 256);
    const unsigned rows = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(repair_init_kernel, dim3(rows < 4096u ? rows : 4096u), dim3(256), 0, st, t.m,
                       t.stamp, t.holder, n, medoid, t.counts);
    ANN_LAUNCHED();
    // sweeps in fours, so that the host waits for one flag per four
    RepairCounts h{};
    for (int round = 0;;) {
        for (int i = 0; i < 4; ++i, ++round) {
            if (i == 3) {
                hipLaunchKernelGGL(repair_flag_kernel, dim3(1), dim3(1), 0, st, &t.counts->changed, 0);
                ANN_LAUNCHED();
            }
            const bool join = round >= LONG_SWEEPS;
            // the lists for the scans are not in use yet
            int32_t *other = t.list[0], *root = t.list[1], *pushed = phase == 0 ? t.m : other;
            const int turn = phase == 0 ? round : round - LONG_SWEEPS;     // of the pushed labels
            if (round == LONG_SWEEPS) {
                hipLaunchKernelGGL(join_init_kernel, dim3(rows), dim3(256), 0, st, other, root, n, medoid);
                ANN_LAUNCHED();
            }
            if (phase == 0 || join) {
                hipLaunchKernelGGL(push_labels_kernel, dim3(sweep), dim3(256), 0, st, graph, n, R, lw,
                                   pushed, t.stamp, turn,
                                   phase == 0 ? &t.counts->changed : &t.counts->other);
                ANN_LAUNCHED();
            }
            if (phase == 1 || join) {
                hipLaunchKernelGGL(pull_labels_kernel, dim3(sweep), dim3(256), 0, st, graph, n, R, lw,
                                   phase == 1 ? t.m : other,
                                   phase == 1 ? &t.counts->changed : &t.counts->other);
                ANN_LAUNCHED();
            }
            if (join) {
                hipLaunchKernelGGL(join_kernel, dim3(rows), dim3(256), 0, st, t.m, other, root, n, medoid,
                                   pushed, t.stamp, turn + 1, &t.counts->changed);
                ANN_LAUNCHED();
            }
        }
        ann_status s = read_counts(t.counts, h, st);
        if (s != ANN_OK) return s;
        if (!h.changed) break;
    }
    hipLaunchKernelGGL(collect_roots_kernel, dim3(rows), dim3(256), 0, st, t.m, n, t.roots, t.counts);
    ANN_LAUNCHED();
    ann_status s = read_counts(t.counts, h, st);
    if (s != ANN_OK) return s;
    *bridges = h.roots;
    if (h.roots == 0) return ANN_OK;
    const unsigned waves = (unsigned)((h.roots + 3) / 4);
    if (phase == 0)
        hipLaunchKernelGGL(match_kernel, dim3(waves), dim3(256), 0, st, t.roots, h.roots, cand, K, t.m,
                           t.holder, t.list[0], &t.counts->left[0]);
    else
        hipLaunchKernelGGL(reverse_link_kernel, dim3(waves), dim3(256), 0, st, t.roots, h.roots, cand,
                           K, t.m, graph, R, t.list[0], &t.counts->left[0]);
    ANN_LAUNCHED();
    s = read_counts(t.counts, h, st);
    if (s != ANN_OK) return s;
    int sb = scan_blocks(n);
    int32_t *holder = phase == 0 ? t.holder : nullptr;
    int per = SCAN_BATCH;
    std::vector<int32_t> sorted;
    for (int cur = 0, left = h.left[0]; left > 0; cur ^= 1) {
        hipLaunchKernelGGL(repair_flag_kernel, dim3(1), dim3(1), 0, st, &t.counts->left[cur ^ 1], 0);
        ANN_LAUNCHED();
        if (per == 1) {
            // one at a time, smallest first
            sorted.resize((size_t)left);
            ANN_HIP(hipMemcpyAsync(sorted.data(), t.list[cur], sizeof(int32_t) * (size_t)left,
                                   hipMemcpyDeviceToHost, st));
            ANN_HIP(hipStreamSynchronize(st));
            std::sort(sorted.begin(), sorted.end());
            ANN_HIP(hipMemcpyAsync(t.list[cur], sorted.data(), sizeof(int32_t) * (size_t)left,
                                   hipMemcpyHostToDevice, st));
        }
        for (int b0 = 0; b0 < left; b0 += per) {
            const int cnt = left - b0 < per ? left - b0 : per;
            const dim3 sgrid((unsigned)sb, (unsigned)((cnt + SCAN_U - 1) / SCAN_U));
            if (dim % 4 == 0 && aligned(base, 16))
                hipLaunchKernelGGL(scan_batch_kernel<true>, sgrid, dim3(256), 0, st, base, n, dim, t.m,
                                   holder, t.list[cur] + b0, cnt, t.partial);
            else
                hipLaunchKernelGGL(scan_batch_kernel<false>, sgrid, dim3(256), 0, st, base, n, dim, t.m,
                                   holder, t.list[cur] + b0, cnt, t.partial);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(scan_apply_kernel, dim3(cnt), dim3(256), 0, st, t.partial, sb,
                               t.list[cur] + b0, n, cand, K, t.m, holder, graph, R, t.list[cur ^ 1],
                               &t.counts->left[cur ^ 1]);
            ANN_LAUNCHED();
        }
        s = read_counts(t.counts, h, st);
        if (s != ANN_OK) return s;
        // when most of a batch wants the same few nodes (large groups of
        // equal points), each pass settles few of them: then one scan per u
        // in id order costs less
        if (h.left[cur ^ 1] > left - left / 8) {
            per = 1;
            sb = (int)(rows < 2048u ? rows : 2048u);
        }
        left = h.left[cur ^ 1];
    }
    if (phase == 0) {
        hipLaunchKernelGGL(forward_link_kernel, dim3(rows), dim3(256), 0, st, t.holder, n, R, graph);
        ANN_LAUNCHED();
    }
    return ANN_OK;
}

// alpha pruning of the candidate lists, medoid, connectivity repair.  Each
// repair bridge is the first eligible entry of the unreached point's
// candidate list, else the argmin over all eligible points (a full scan);
// for lists of global nearest neighbours the two are the same node.
ann_status graph_tail(const float *base, int64_t n, int dim, const int32_t *cand,
                      const double *cd2, int K, int R, float alpha, int32_t *graph,
                      int32_t *medoid, int32_t *bridges, const TailBufs &t, hipStream_t st)
{
    const double a2 = (double)alpha * (double)alpha;
    // FP32 rounding of a sum of dim squared differences: one unit for each of a
    // lane's terms, a few for the term, and a margin
    const double err = std::ldexp((double)dim + 64.0, -24);
    const dim3 pgrid((unsigned)((n + 3) / 4));
    if (dim % 4 == 0 && aligned(base, 16))
        hipLaunchKernelGGL(prune_kernel<true>, pgrid, dim3(256), 0, st, base, n, dim, cand, cd2, K, R, a2,
                           err, graph);
    else
        hipLaunchKernelGGL(prune_kernel<false>, pgrid, dim3(256), 0, st, base, n, dim, cand, cd2, K, R, a2,
                           err, graph);
    ANN_LAUNCHED();
    int32_t med = -1;
    ann_status s = medoid_run(base, n, dim, t.med_cols, t.mu, t.partial, t.best, &med, st);
    if (s != ANN_OK) return s;
    int32_t nb[2] = {0, 0};
    for (int phase = 0; phase < 2; ++phase) {
        s = repair_phase(base, n, dim, cand, K, R, phase, med, graph, &nb[phase], t, st);
        if (s != ANN_OK) return s;
    }
    // the links of the last phase may still be running
    ANN_HIP(hipStreamSynchronize(st));
    *medoid = med;
    if (bridges) {
        bridges[0] = nb[0];
        bridges[1] = nb[1];
    }
    return ANN_OK;
}

// rows[members[r]] -> out row r
__global__ void gather_rows_kernel(const float *base, int dim, const int32_t *members, int64_t m,
                                   float *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m * dim) return;
    const int64_t r = i / dim;
    out[i] = base[(int64_t)members[r] * dim + (i - r * dim)];
}

// candidate lists of one group's home points (local member indices) -> the
// global lists, -1 / +inf padded
__global__ void scatter_cand_kernel(const int32_t *loc_ids, const double *loc_d2, int Kg,
                                    const int32_t *members, const int32_t *home, int64_t m, int K,
                                    int32_t *cand, double *cd2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m * K) return;
    const int64_t r = i / K;
    const int j = (int)(i - r * K);
    const int64_t dst = (int64_t)home[r] * K + j;
    int32_t id = -1;
    double d = __longlong_as_double(0x7ff0000000000000ll);
    if (j < Kg) {
        const int32_t l = loc_ids[r * Kg + j];
        if (l >= 0) {
            id = members[l];
            d = loc_d2[r * Kg + j];
        }
    }
    cand[dst] = id;
    cd2[dst] = d;
}

}  // namespace

// cand ids, d2 and the steps after them
static size_t build_rest(int64_t n, int dim, int K, int R)
{
    return round_up((size_t)n * K * 4, 256) + round_up((size_t)n * K * 8, 256) + tail_ws(n, dim, R);
}

size_t build_graph_ws(int64_t n, int dim, int K, int R)
{
    return knn_workspace(n, n, dim, K) + build_rest(n, dim, K, R);
}

static size_t group_rest(int dim, int K, int64_t max_mem, int64_t max_home)
{
    size_t b = round_up((size_t)max_mem * dim * 4, 256) + round_up((size_t)max_home * dim * 4, 256);
    b += round_up((size_t)max_mem * 4, 256) + round_up((size_t)max_home * 4, 256) * 2;
    b += round_up((size_t)max_home * K * 4, 256) + round_up((size_t)max_home * K * 8, 256);
    return b + 1024;
}

size_t group_cand_ws(int dim, int K, int64_t max_mem, int64_t max_home)
{
    return knn_workspace(max_mem, max_home, dim, K) + group_rest(dim, K, max_mem, max_home);
}

// what the call is accepted with (knn_accepts)
static size_t group_cand_accepts(int dim, int K, int64_t max_mem, int64_t max_home)
{
    return knn_accepts(max_mem, max_home, dim, K) + group_rest(dim, K, max_mem, max_home);
}

}  // namespace ann

using namespace ann;

extern "C" ann_status ann_build_graph(const float *base, int64_t n, int32_t dim, int32_t knn_k,
                                      int32_t R, float alpha, int32_t *graph, int32_t *medoid,
                                      int32_t *bridges, void *workspace, size_t ws_bytes,
                                      void *stream)
{
    ANN_REQUIRE(base && graph && medoid && workspace, "a required pointer is NULL");
    ANN_REQUIRE(n >= 2 && n <= 0x7FFFFFFF, "n must be in [2, 2^31)");
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");
    ANN_REQUIRE(R >= 3, "R must be >= 3");
    ANN_SUPPORTED(R <= 64, "R must be <= 64");
    ANN_REQUIRE(knn_k >= R - 2 && knn_k <= 1024, "knn_k must be in [R-2, 1024]");
    ANN_REQUIRE(knn_k <= n - 1, "knn_k must be < n");
    ANN_REQUIRE(alpha >= 1.0f, "alpha must be >= 1");
    ANN_REQUIRE(aligned(base, 16), "base must be 16-byte aligned");
    const int K = knn_k;
    ANN_REQUIRE(ws_bytes >= knn_accepts(n, n, dim, K) + build_rest(n, dim, K, R), "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    int32_t *cand = cv.take<int32_t>((size_t)n * K);
    double *cd2 = cv.take<double>((size_t)n * K);
    TailBufs t = take_tail(cv, n, dim);
    void *knn_ws = cv.p;
    const size_t kws = ws_bytes - (size_t)(cv.p - static_cast<unsigned char *>(workspace));
    // exact kNN candidates (self excluded), then pruning, medoid, repair
    ann_status s = knn_run(base, n, dim, base, n, K, true, cand, nullptr, cd2, knn_ws, kws, st, 0);
    if (s != ANN_OK) return s;
    return no_throw([&] { return graph_tail(base, n, dim, cand, cd2, K, R, alpha, graph, medoid, bridges, t, st); });
}

namespace {

// Members and home points of every group, each list in id order.
struct GroupLists {
    std::vector<int64_t> ms, hs;          // offsets (n_groups + 1)
    std::vector<int32_t> members, homes;
    int64_t max_mem = 1, max_home = 1;
};

ann_status group_lists(const int32_t *groups_dev, int64_t n, int32_t n_member, int32_t n_groups,
                       hipStream_t st, GroupLists &L)
{
    const size_t nm = (size_t)n_member;
    std::vector<int32_t> lab((size_t)n * nm);
    ANN_HIP(hipMemcpyAsync(lab.data(), groups_dev, sizeof(int32_t) * lab.size(),
                           hipMemcpyDeviceToHost, st));
    ANN_HIP(hipStreamSynchronize(st));
    auto listed_before = [&](int64_t i, size_t c) {
        for (size_t e = 0; e < c; ++e)
            if (lab[(size_t)i * nm + e] == lab[(size_t)i * nm + c]) return true;
        return false;
    };
    L.ms.assign((size_t)n_groups + 1, 0);
    L.hs.assign((size_t)n_groups + 1, 0);
    for (int64_t i = 0; i < n; ++i) {
        const int32_t h = lab[(size_t)i * nm];
        ANN_REQUIRE(h >= 0 && h < n_groups, "home group of point %lld out of range", (long long)i);
        L.hs[(size_t)h + 1]++;
        for (size_t c = 0; c < nm; ++c) {
            const int32_t g = lab[(size_t)i * nm + c];
            ANN_REQUIRE(g >= -1 && g < n_groups, "group label of point %lld out of range",
                        (long long)i);
            if (g >= 0 && !listed_before(i, c)) L.ms[(size_t)g + 1]++;
        }
    }
    for (int g = 0; g < n_groups; ++g) {
        L.max_mem = std::max<int64_t>(L.max_mem, L.ms[(size_t)g + 1]);
        L.max_home = std::max<int64_t>(L.max_home, L.hs[(size_t)g + 1]);
        L.ms[(size_t)g + 1] += L.ms[(size_t)g];
        L.hs[(size_t)g + 1] += L.hs[(size_t)g];
    }
    L.members.resize((size_t)L.ms[(size_t)n_groups]);
    L.homes.resize((size_t)n);
    std::vector<int64_t> mp(L.ms.begin(), L.ms.end() - 1), hp(L.hs.begin(), L.hs.end() - 1);
    for (int64_t i = 0; i < n; ++i) {
        L.homes[(size_t)hp[(size_t)lab[(size_t)i * nm]]++] = (int32_t)i;
        for (size_t c = 0; c < nm; ++c) {
            const int32_t g = lab[(size_t)i * nm + c];
            if (g >= 0 && !listed_before(i, c)) L.members[(size_t)mp[(size_t)g]++] = (int32_t)i;
        }
    }
    return ANN_OK;
}

// candidate lists of the home points of groups [g0, g1); `bytes` of memory at cv
ann_status group_candidates(const float *base, int dim, int K, const GroupLists &L, int g0, int g1,
                            int32_t *cand, double *cd2, Carve cv, size_t bytes, hipStream_t st)
{
    const unsigned char *begin = cv.p;
    float *mrows = cv.take<float>((size_t)L.max_mem * dim);
    float *hrows = cv.take<float>((size_t)L.max_home * dim);
    int32_t *mem_d = cv.take<int32_t>((size_t)L.max_mem);
    int32_t *home_d = cv.take<int32_t>((size_t)L.max_home);
    int32_t *self_d = cv.take<int32_t>((size_t)L.max_home);
    int32_t *loc_ids = cv.take<int32_t>((size_t)L.max_home * K);
    double *loc_d2 = cv.take<double>((size_t)L.max_home * K);
    void *knn_ws = cv.p;
    const size_t kws = bytes - (size_t)(cv.p - begin);
    std::vector<int32_t> selfc((size_t)L.max_home);
    for (int g = g0; g < g1; ++g) {
        const int64_t m = L.ms[(size_t)g + 1] - L.ms[(size_t)g];
        const int64_t h = L.hs[(size_t)g + 1] - L.hs[(size_t)g];
        if (h == 0) continue;
        const int32_t *mem = L.members.data() + L.ms[(size_t)g];
        const int32_t *hom = L.homes.data() + L.hs[(size_t)g];
        // position of each home point in the member list (both in id order)
        for (int64_t r = 0, e = 0; r < h; ++r) {
            while (mem[e] != hom[r]) ++e;
            selfc[(size_t)r] = (int32_t)e;
        }
        ANN_HIP(hipMemcpyAsync(mem_d, mem, sizeof(int32_t) * (size_t)m, hipMemcpyHostToDevice, st));
        ANN_HIP(hipMemcpyAsync(home_d, hom, sizeof(int32_t) * (size_t)h, hipMemcpyHostToDevice, st));
        ANN_HIP(hipMemcpyAsync(self_d, selfc.data(), sizeof(int32_t) * (size_t)h,
                               hipMemcpyHostToDevice, st));
        const int Kg = (int)std::min<int64_t>(K, m - 1);
        if (Kg >= 1) {
            hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((m * dim + 255) / 256)),
                               dim3(256), 0, st, base, dim, mem_d, m, mrows);
            ANN_LAUNCHED();
            hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((h * dim + 255) / 256)),
                               dim3(256), 0, st, base, dim, home_d, h, hrows);
            ANN_LAUNCHED();
            ann_status s = knn_run(mrows, m, dim, hrows, h, Kg, true, loc_ids, nullptr, loc_d2,
                                   knn_ws, kws, st, 0, self_d);
            if (s != ANN_OK) return s;
        }
        hipLaunchKernelGGL(scatter_cand_kernel, dim3((unsigned)((h * K + 255) / 256)), dim3(256),
                           0, st, loc_ids, loc_d2, Kg, mem_d, home_d, h, K, cand, cd2);
        ANN_LAUNCHED();
        // the staging buffers are rewritten by the next group's copies
        ANN_HIP(hipStreamSynchronize(st));
    }
    return ANN_OK;
}

}  // namespace

#define GROUP_ARGS_OK()                                                                      \
    ANN_REQUIRE(n >= 2 && n <= 0x7FFFFFFF, "n must be in [2, 2^31)");                         \
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");                                                \
    ANN_REQUIRE(knn_k >= 1 && knn_k <= 1024, "knn_k must be in [1, 1024]");                   \
    ANN_REQUIRE(n_member >= 1, "n_member must be >= 1");                                      \
    ANN_REQUIRE(n_groups >= 1, "n_groups must be >= 1");                                      \
    ANN_REQUIRE(aligned(base, 16), "base must be 16-byte aligned")

extern "C" size_t ann_group_candidates_workspace_size(int32_t dim, int32_t knn_k,
                                                      int64_t max_members, int64_t max_home)
{
    if (dim < 1 || knn_k < 1 || max_members < 1 || max_home < 1) return 0;
    return group_cand_ws(dim, knn_k, max_members, max_home);
}

extern "C" ann_status ann_group_candidates(const float *base, int64_t n, int32_t dim, int32_t knn_k,
                                           const int32_t *groups, int32_t n_member,
                                           int32_t n_groups, int32_t g_begin, int32_t g_end,
                                           int32_t *cand, double *cand_d2, void *workspace,
                                           size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && groups && cand && cand_d2 && workspace, "a required pointer is NULL");
    GROUP_ARGS_OK();
    ANN_REQUIRE(g_begin >= 0 && g_begin <= g_end && g_end <= n_groups,
                "group range must satisfy 0 <= g_begin <= g_end <= n_groups");
    hipStream_t st = static_cast<hipStream_t>(stream);
    return no_throw([&]() -> ann_status {
        GroupLists L;
        ann_status s = group_lists(groups, n, n_member, n_groups, st, L);
        if (s != ANN_OK) return s;
        ANN_REQUIRE(ws_bytes >= group_cand_accepts(dim, knn_k, L.max_mem, L.max_home),
                    "workspace too small (largest member set %lld, largest home set %lld)",
                    (long long)L.max_mem, (long long)L.max_home);
        Carve cv{static_cast<unsigned char *>(workspace)};
        return group_candidates(base, dim, knn_k, L, g_begin, g_end, cand, cand_d2, cv, ws_bytes, st);
    });
}

extern "C" size_t ann_graph_from_candidates_workspace_size(int64_t n, int32_t dim, int32_t R)
{
    if (n < 2 || dim < 1 || R < 3) return 0;
    return tail_ws(n, dim, R);
}

extern "C" ann_status ann_graph_from_candidates(const float *base, int64_t n, int32_t dim,
                                                const int32_t *cand, const double *cand_d2,
                                                int32_t knn_k, int32_t R, float alpha,
                                                int32_t *graph, int32_t *medoid,
                                                int32_t *bridges, void *workspace,
                                                size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && cand && cand_d2 && graph && medoid && workspace,
                "a required pointer is NULL");
    ANN_REQUIRE(n >= 2 && n <= 0x7FFFFFFF, "n must be in [2, 2^31)");
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");
    ANN_REQUIRE(R >= 3, "R must be >= 3");
    ANN_SUPPORTED(R <= 64, "R must be <= 64");
    ANN_REQUIRE(knn_k >= R - 2 && knn_k <= 1024, "knn_k must be in [R-2, 1024]");
    ANN_REQUIRE(alpha >= 1.0f, "alpha must be >= 1");
    ANN_REQUIRE(aligned(base, 16), "base must be 16-byte aligned");
    ANN_REQUIRE(ws_bytes >= tail_ws(n, dim, R), "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    TailBufs t = take_tail(cv, n, dim);
    return no_throw([&] { return graph_tail(base, n, dim, cand, cand_d2, knn_k, R, alpha, graph, medoid, bridges, t, st); });
}

extern "C" size_t ann_build_graph_partitioned_workspace_size(int64_t n, int32_t dim,
                                                             int32_t knn_k, int32_t R,
                                                             int64_t max_members, int64_t max_home)
{
    if (n < 2 || dim < 1 || knn_k < 1 || R < 3 || max_members < 1 || max_home < 1) return 0;
    return round_up((size_t)n * knn_k * 4, 256) + round_up((size_t)n * knn_k * 8, 256) +
           std::max(tail_ws(n, dim, R), group_cand_ws(dim, knn_k, max_members, max_home));
}

extern "C" ann_status ann_build_graph_partitioned(const float *base, int64_t n, int32_t dim,
                                                  int32_t knn_k, int32_t R, float alpha,
                                                  const int32_t *groups, int32_t n_member,
                                                  int32_t n_groups, int32_t *graph,
                                                  int32_t *medoid, int32_t *bridges,
                                                  void *workspace, size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && groups && graph && medoid && workspace, "a required pointer is NULL");
    GROUP_ARGS_OK();
    ANN_REQUIRE(R >= 3, "R must be >= 3");
    ANN_SUPPORTED(R <= 64, "R must be <= 64");
    ANN_REQUIRE(knn_k >= R - 2, "knn_k must be >= R-2");
    ANN_REQUIRE(alpha >= 1.0f, "alpha must be >= 1");
    hipStream_t st = static_cast<hipStream_t>(stream);
    return no_throw([&]() -> ann_status {
        GroupLists L;
        ann_status s = group_lists(groups, n, n_member, n_groups, st, L);
        if (s != ANN_OK) return s;
        const size_t lists = round_up((size_t)n * knn_k * 4, 256) + round_up((size_t)n * knn_k * 8, 256);
        ANN_REQUIRE(ws_bytes >= lists + std::max(tail_ws(n, dim, R),
                                                 group_cand_accepts(dim, knn_k, L.max_mem, L.max_home)),
                    "workspace too small (largest member set %lld, largest home set %lld)",
                    (long long)L.max_mem, (long long)L.max_home);
        const int K = knn_k;
        Carve cv{static_cast<unsigned char *>(workspace)};
        int32_t *cand = cv.take<int32_t>((size_t)n * K);
        double *cd2 = cv.take<double>((size_t)n * K);
        // the kNN staging and the tail's buffers share what is left
        s = group_candidates(base, dim, K, L, 0, n_groups, cand, cd2, cv, ws_bytes - lists, st);
        if (s != ANN_OK) return s;
        TailBufs t = take_tail(cv, n, dim);
        return graph_tail(base, n, dim, cand, cd2, K, R, alpha, graph, medoid, bridges, t, st);
    });
}

extern "C" ann_status ann_medoid(const float *base, int64_t n, int32_t dim, int32_t *medoid,
                                 void *workspace, size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && medoid && workspace, "a required pointer is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF, "n must be in [1, 2^31)");
    ANN_REQUIRE(dim >= 1, "dim must be >= 1");
    ANN_REQUIRE(ws_bytes >= medoid_ws(n, dim), "workspace too small");
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    int chunks = (int)((n + MED_ROWS - 1) / MED_ROWS);
    double *pc = cv.take<double>((size_t)chunks * dim);
    double *mu = cv.take<double>((size_t)dim);
    DKey *partial = cv.take<DKey>(2048);
    DKey *best = cv.take<DKey>(1);
    return medoid_run(base, n, dim, pc, mu, partial, best, medoid, st);
}
