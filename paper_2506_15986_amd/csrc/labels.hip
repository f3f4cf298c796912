// Training labels for the entry model: for each historical query, the
// candidate hub from which the plain beam search reaches the target recall
// with the fewest distance computations.
//
// This takes the place of the paper's hop-count queues (Definition 4 and the
// query-aware sample generation, which runs Algorithm 1 from every hub for
// every historical query) with the same intent: which hub serves a query
// best.  For candidate hub m of query q, the cost of (q, m) is the distance
// count of the first width L of an increasing ladder whose beam search from
// that hub (ann_search's) has at least `hits` of the query's true top-kt in
// its top-kt.  The label is the candidate of least cost (ties: smaller hub
// index), or the first candidate when none reaches the target.
//
// One search serves the whole ladder.  A pool of width L holds the L nearest
// nodes seen, and the next node expanded is the nearest one not expanded yet:
// so as long as one of the first L pool entries is unexpanded, the search of
// any larger width does the same steps and its pool begins with the same L
// entries.  The search of width L ends when its L entries are all expanded;
// the widest search passes through exactly that state when its next entry to
// expand lies at place L or later.  There its top-kt and distance count are
// those of width L; if the target is reached the search ends, else it goes on.
// One search per width, restarted each time, took 78 ms for 4,096 queries x 8
// hubs x 10 widths on 150,000 x 128; 5.8 ms now.
#include "beam.h"
#include "common.h"
#include "internal.h"
#include "search_core.h"

namespace ann {
namespace {

constexpr int LB_LOG2_MIN = 11;        // slots of the smallest visited table, log2
constexpr int LB_LOG2 = 13;            // ... of the second
constexpr int LB_LOG2_MAX = 14;        // ... of the largest
constexpr int LB_MAX_WIDTHS = 64;
constexpr int LB_ROWS = 1 << 20;       // (query, candidate) rows searched together

struct LadderArgs {
    const float *base;
    int64_t n;
    int dim;
    const int32_t *graph;
    int R;
    const float *queries;
    const int32_t *truth;
    int kt;
    int hits;
    const int32_t *cand;       // the rows: query row / M, hub cand[row]
    int M;
    int rows;
    const int32_t *hub_ids;
    int n_L;
    int16_t ladder[LB_MAX_WIDTHS];
    const int32_t *list;       // NULL, or the rows to search,
    const int32_t *count;      // and how many they are
    int32_t *again;            // NULL, or the rows whose table overflowed,
    int32_t *n_again;          // and how many they are
    uint32_t *counter;         // work counter, zero at launch
    int32_t *table;
    int32_t *flags;
    int visited_log2;
    beam::FilterShape filter;
    int wave_lds;
};

__global__ void fill_value_kernel(int32_t *p, int64_t count, int32_t v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

// One wavefront per row at a time, persistent grid.  A row whose visited
// table overflowed (its count may hold a node twice) is listed for a search
// with a larger table, or flagged where there is none.
// Bound by the hops' chain (adjacency row, vectors, merge: about 2 us) over as
// many searches as the tables in LDS let run, and by the gather of the vectors:
// 41 million rows of 512 bytes in 5.7 ms are 3.7 TB/s, against 4.8 of a copy.
// A row that is searched again in any case ends where its table overflows
// (7.2 ms when it went on).
template <int G, int CPL>
__global__ void __launch_bounds__(64) ladder_kernel(LadderArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = beam::lane_id();
    const int Lmax = a.ladder[a.n_L - 1];
    Searcher<G, CPL, false, beam::kId32> s;
    s.setup(smem, (Lmax + 15) / 16 * 16, a.visited_log2, a.filter, a.n, a.base, a.dim, a.graph, a.R);
    const int rows = a.list ? *a.count : a.rows;
    for (;;) {
        int slot = 0;
        if (lane == 0) slot = (int)atomicAdd(a.counter, 1u);
        slot = __builtin_amdgcn_readfirstlane(slot);
        if (slot >= rows) break;
        const int row = a.list ? a.list[slot] : slot;
        const int q = row / a.M;
        const int32_t entry = a.hub_ids[a.cand[row]];
        const int32_t want = lane < a.kt ? a.truth[(int64_t)q * a.kt + lane] : -1;
        s.cur = 0;
        s.cnt = 0;
        // true: `hits` of the top-kt are among the true ones
        auto reached = [&]() __attribute__((always_inline)) {
            const int32_t id = s.id_at(lane);
            bool in = false;
            for (int b = 0; b < a.kt; ++b) in |= id == beam::readlane(want, b);
            return __popcll(__ballot(in && lane < a.kt)) >= a.hits;
        };
        int li = 0;
        int32_t cost = -1;
        SearchResult r{0, 0, 0, false};
        if (entry >= 0 && (int64_t)entry < a.n) {
            s.load_query(a.queries + (size_t)q * a.dim);
            r = s.run_until((uint32_t)entry, Lmax, nullptr, 0, [&](int place, const SearchResult &now,
                                                                 bool lost) __attribute__((always_inline)) {
                if (a.again && __any(lost)) return true;
                if (place < a.ladder[li]) return false;
                while (a.ladder[li] <= place) ++li;   // place < Lmax: li stays inside
                if (!reached()) return false;
                cost = now.ndc_exec - now.dups;
                return true;
            });
        }
        // nothing left to expand: the widths not passed yet all end here
        if (cost < 0 && !(r.lost && a.again) && reached()) cost = r.ndc_exec - r.dups;
        if (lane == 0) {
            if (r.lost && a.again) a.again[atomicAdd(a.n_again, 1)] = row;
            else {
                a.table[row] = cost;
                if (r.lost) atomicOr(&a.flags[q], 1);
            }
        }
        beam::wave_sync();
    }
}

__global__ void choose_kernel(const int32_t *table, const int32_t *cand, int nq, int M,
                              int32_t *labels)
{
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    int32_t best = -1, bh = 0x7fffffff;
    for (int m = 0; m < M; ++m) {
        const int32_t v = table[(int64_t)q * M + m];
        const int32_t h = cand[(int64_t)q * M + m];
        if (v < 0) continue;
        if (best < 0 || v < best || (v == best && h < bh)) {
            best = v;
            bh = h;
        }
    }
    labels[q] = best >= 0 ? bh : cand[(int64_t)q * M];
}

inline int blocks_for(int64_t n) { return (int)((n + 255) / 256); }

// log2 of the first visited table's slots: smaller tables let more searches
// run on a CU, and one that proves too small costs its row a second search.
// 4,096 queries x 8 hubs, R = 32, a third to half of the rows going the whole
// ladder, 2^13 / 2^12 / 2^11 / 2^10 slots: to width 256 11.5 / 7.6 / 6.6 /
// 16.2 ms, to 128 6.7 / 3.8 / 3.4 / 5.6, to 32 2.7 / 1.4 / 1.0 / 1.2.  The
// ids seen grow with the width and with the degree.  Up to four rounds of the
// four searches that a CU holds with 2^13 slots, the second searches take
// longer than they save (rows of half the ladder's length: 664 rows 1.0 against
// 2.6 ms, 2,332 rows 1.8 against 2.2, 2,880 rows 1.5 against 2.0).
inline int table_log2(int L, int R, int rows)
{
    if (rows <= 16 * device_cus()) return LB_LOG2;
    int l = LB_LOG2_MIN;
    while (l < LB_LOG2 && (1 << l) < (L + 16) * R * 7 / 32) ++l;
    return l;
}

// queries whose rows are searched together: the lists stay bounded
inline int chunk_queries(int nq, int M)
{
    const int c = M > 1 ? LB_ROWS / M : LB_ROWS;   // M < 1: refused, but its size is asked for
    return nq < 1 ? 0 : nq < c ? nq : c < 1 ? 1 : c;
}

template <int G, int CPL>
ann_status launch_ladder(const LadderArgs &a, hipStream_t st)
{
    auto kern = ladder_kernel<G, CPL>;
    const size_t lds = (size_t)a.wave_lds;
    if (lds > 65536)
        ANN_HIP(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    int per_cu = 0;
    ANN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64, lds));
    if (per_cu < 1) return fail(ANN_ENOTSUP, "label search does not fit on a CU (%zu B LDS)", lds);
    const int blocks = per_cu * device_cus() < a.rows ? per_cu * device_cus() : a.rows;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64), lds, st, a);
    ANN_LAUNCHED();
    return ANN_OK;
}

// the lane groups of ann_search's default plan
ann_status dispatch(const LadderArgs &a, hipStream_t st)
{
    const int chunks = a.dim / 4;
    if (a.dim <= 128) {
        const int cpl = (chunks + 7) / 8;
        if (cpl <= 1) return launch_ladder<8, 1>(a, st);
        if (cpl == 2) return launch_ladder<8, 2>(a, st);
        if (cpl == 3) return launch_ladder<8, 3>(a, st);
        return launch_ladder<8, 4>(a, st);
    }
    const int cpl = (chunks + 15) / 16;
    if (cpl <= 4) return launch_ladder<16, 4>(a, st);
    if (cpl <= 8) return launch_ladder<16, 8>(a, st);
    if (cpl <= 15) return launch_ladder<16, 15>(a, st);
    return launch_ladder<16, 16>(a, st);
}

}  // namespace

size_t make_labels_ws(int nq, int M, int kt)
{
    (void)kt;
    const size_t rows = (size_t)chunk_queries(nq, M) * M;
    size_t b = round_up(rows * 4, 256) * 2;                    // rows searched again
    b += round_up((size_t)nq * M * 4, 256);                    // table (when not given)
    b += round_up((size_t)nq * 4, 256);                        // flags (when not given)
    return b + 512;
}

}  // namespace ann

using namespace ann;

extern "C" size_t ann_labels_workspace_size(int32_t nq, int32_t M, int32_t kt)
{
    return make_labels_ws(nq, M, kt);
}

extern "C" ann_status ann_make_labels(const float *base, int64_t n, int32_t dim,
                                      const int32_t *graph, int32_t R, const float *queries,
                                      int32_t nq, const int32_t *truth, int32_t kt, int32_t hits,
                                      const int32_t *cand_hubs, int32_t M, const int32_t *hub_ids,
                                      const int32_t *L_ladder, int32_t n_L, int32_t *labels,
                                      int32_t *table, int32_t *flags, void *workspace,
                                      size_t ws_bytes, void *stream)
{
    ANN_REQUIRE(base && graph && workspace && L_ladder, "a required pointer is NULL");
    ANN_REQUIRE(nq == 0 || (queries && truth && cand_hubs && hub_ids && labels),
                "a required pointer is NULL");
    ANN_REQUIRE(n >= 1 && n <= 0x7FFFFFFF, "n must be in [1, 2^31)");
    ANN_SUPPORTED(dim % 4 == 0 && dim <= 1024, "dim must be a multiple of 4 and <= 1024");
    ANN_REQUIRE(R >= 1, "R must be >= 1");
    ANN_SUPPORTED(R <= 64, "R must be <= 64");
    ANN_REQUIRE(kt >= 1 && kt <= 64, "kt must be in [1, 64]");
    ANN_REQUIRE(hits >= 1 && hits <= kt, "hits must be in [1, kt]");
    ANN_REQUIRE(M >= 1, "M must be >= 1");
    ANN_REQUIRE(n_L >= 1 && n_L <= 64, "the ladder must hold 1..64 widths");
    for (int i = 0; i < n_L; ++i) {
        ANN_REQUIRE(L_ladder[i] >= kt && L_ladder[i] <= 512, "ladder widths must be in [kt, 512]");
        ANN_REQUIRE(i == 0 || L_ladder[i] > L_ladder[i - 1], "ladder must increase");
    }
    ANN_REQUIRE(aligned(base, 16) && aligned(queries, 16), "base/queries must be 16-byte aligned");
    ANN_REQUIRE(ws_bytes >= make_labels_ws(nq, M, kt), "workspace too small");
    if (nq == 0) return ANN_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Carve cv{static_cast<unsigned char *>(workspace)};
    const int cq = chunk_queries(nq, M);
    int32_t *list[2] = {cv.take<int32_t>((size_t)cq * M), cv.take<int32_t>((size_t)cq * M)};
    int32_t *tab = cv.take<int32_t>((size_t)nq * M);
    int32_t *fl = cv.take<int32_t>((size_t)nq);
    int32_t *counters = cv.take<int32_t>(64);
    if (table) tab = table;
    if (flags) fl = flags;
    hipLaunchKernelGGL(fill_value_kernel, dim3(blocks_for(nq)), dim3(256), 0, st, fl, (int64_t)nq, 0);
    ANN_LAUNCHED();
    LadderArgs a{};
    a.base = base;
    a.n = n;
    a.dim = dim;
    a.graph = graph;
    a.R = R;
    a.kt = kt;
    a.hits = hits;
    a.M = M;
    a.hub_ids = hub_ids;
    a.n_L = n_L;
    for (int i = 0; i < n_L; ++i) a.ladder[i] = (int16_t)L_ladder[i];
    const int Lmax = L_ladder[n_L - 1];
    for (int q0 = 0; q0 < nq; q0 += cq) {
        const int qn = nq - q0 < cq ? nq - q0 : cq;
        a.queries = queries + (size_t)q0 * dim;
        a.truth = truth + (size_t)q0 * kt;
        a.cand = cand_hubs + (size_t)q0 * M;
        a.rows = qn * M;
        a.table = tab + (size_t)q0 * M;
        a.flags = fl + q0;
        hipLaunchKernelGGL(fill_value_kernel, dim3(1), dim3(64), 0, st, counters, (int64_t)64, 0);
        ANN_LAUNCHED();
        // costs are distance counts, so the filter must not forget ids: 32-bit
        // ids, the rows that overflow a table searched again with a larger one
        const int tables[3] = {table_log2(Lmax, R, a.rows), LB_LOG2, LB_LOG2_MAX};
        a.list = nullptr;
        a.count = nullptr;
        for (int t = tables[0] < LB_LOG2 ? 0 : 1; t < 3; ++t) {
            a.visited_log2 = tables[t];
            beam::filter_shape(beam::kId32, tables[t], n, a.filter);
            a.wave_lds = (int)wave_lds_bytes((Lmax + 15) / 16 * 16, a.filter, false, dim);
            a.counter = reinterpret_cast<uint32_t *>(counters + t);
            a.again = t < 2 ? list[t] : nullptr;
            a.n_again = counters + 8 + t;
            ann_status s = dispatch(a, st);
            if (s != ANN_OK) return s;
            a.list = a.again;
            a.count = a.n_again;
        }
    }
    hipLaunchKernelGGL(choose_kernel, dim3(blocks_for(nq)), dim3(256), 0, st, tab, cand_hubs, nq, M,
                       labels);
    ANN_LAUNCHED();
    return ANN_OK;
}
