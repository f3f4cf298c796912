// Internal interface of the exact kNN engines (knn.hip).
#pragma once

#include "common.h"

namespace ann {

namespace knn {
struct Ent;
}

struct KnnArgs {
    const float *base;
    int64_t n;
    int dim;
    const float *queries;
    int64_t rows;
    int K;
    int exclude_self;
    const int32_t *self_col;    // column excluded for query row q (null: column q)
    const int32_t *row_list;    // query row of row g of a launch (null: row g)
    knn::Ent *buf;
    int cap;
    int32_t *out_ids;
    float *out_f;
    double *out_d;
};

// Workspace bytes for knn_run on any data, and the (smaller) bytes that a call
// is accepted with: integer data needs no more, and real-valued data then goes
// through the plain FP64 engine, or its shortlist in smaller batches of rows.
size_t knn_workspace(int64_t n, int64_t rows, int dim, int K);
size_t knn_accepts(int64_t n, int64_t rows, int dim, int K);

// Exact top-K by (squared L2, id) of `rows` query rows against `base`.
// force_engine: 0 = pick (int8 matrix cores when all values are integers in
// [0,255] and dim % 32 == 0, else the real-valued engines: the FP16 shortlist
// with FP64 distances, the plain FP64 engine for what that leaves), 1 = int8
// only, 2 = the real-valued engines only.
// With exclude_self, query row g never returns base column self_col[g]
// (column g when self_col is null).  Synchronises `st`.
ann_status knn_run(const float *base, int64_t n, int dim, const float *queries, int64_t rows,
                   int K, bool exclude_self, int32_t *out_ids, float *out_f, double *out_d,
                   void *ws, size_t ws_bytes, hipStream_t st, int force_engine,
                   const int32_t *self_col = nullptr);

// Sets *result when every value of x[0..count) is an integer in [0,255].
ann_status data_is_uint8(const float *x, int64_t count, int *flag_dev, bool *result,
                         hipStream_t st);

}  // namespace ann
