// Internal declarations of the message-passing initialiser.
#pragma once

#include <algorithm>

#include "internal.h"

namespace ffsat {

// One product on the matrix cores (k_gemm): operands, result, slices of the
// reduction and the grid (blocks of gx x gy tiles per slice).
struct GemmArgs {
    int M, N, K, lda, ldb, ldc;
    const float *A, *B, *bias;
    float *C;
    int kslice;
    size_t slice_stride;
    int vec_a, vec_b, colsum, gx, gy, blocks;
};
GemmArgs gemm_args(bool ta, bool tb, int epi, int M, int N, int K, const float *A, int lda, const float *B, int ldb,
                   float *C, int ldc, const float *bias, int splits, size_t slice_stride);
hipError_t gemm_relu(const GemmArgs &g, hipStream_t s);                              // NN, bias and ReLU
hipError_t gemm_relu2(const GemmArgs &g, const GemmArgs &g1, hipStream_t s);         // two of them
hipError_t gemm_back(const GemmArgs &weights, const GemmArgs &input, hipStream_t s); // TN with column sums, and NT
hipError_t gemm_weights2(const GemmArgs &g, const GemmArgs &g1, hipStream_t s);      // two TN with column sums
// number of reduction slices of a product for `splits` requested over K terms
int gemm_slices(int K, int splits);
// sums over slices, of all of a backward pass in one launch
struct SumJob {
    const float *part;
    size_t stride;
    int len, len_tail, S, block0;
    float *out, *tail;
};
constexpr int SUM_JOBS = 20;   // head, two input layers, two per round of up to eight
struct SumJobs {
    SumJob job[SUM_JOBS];
    int n = 0;
};
hipError_t sum_slices(SumJobs &jobs, hipStream_t s);   // and empties the list
hipError_t gather(int mode, int rows, int H, const int32_t *row_ptr, const int32_t *src_of, const int32_t *lit,
                  const float *w, const float *src, int sstride, float *dst, int dstride, const float *own, int ostride,
                  const float *y, hipStream_t s);
hipError_t relu_back(int rows, int H, float *dZ, const float *Y, const float *dx, int dxstride, hipStream_t s);
hipError_t head(int n, int H, const float *hv, const float *wo, const float *bo, float *mu, hipStream_t s);
hipError_t head_back(int n, int H, const float *mu, const float *t, const float *wo, const float *y, float *dz,
                     float *lterm, float *dZ, hipStream_t s);
constexpr int HEAD_SLICES = 128;   // part holds HEAD_SLICES * (H + 2) values
hipError_t head_sums(int n, int H, const float *dz, const float *lterm, const float *hv, float *part, float *out,
                     float *loss, SumJobs &jobs, hipStream_t s);
hipError_t adam(int64_t P, float *w, const float *g, float *m1, float *m2, float lr, float b1, float b2, float eps,
                int step, hipStream_t s);
hipError_t propose(int64_t total, int B, int nl, const float *mu, float sigma, uint64_t seed, float *x,
                   hipStream_t s);

// Incidence graph of a problem in original constraint order, on the device.
struct MpnnGraph {
    int n = 0, m = 0, nnz = 0;
    void *buf = nullptr;          // one device allocation holding every array below
    int32_t *con_ptr = nullptr;   // [m+1]
    int32_t *lit = nullptr;       // [nnz] var | negated << 31
    int32_t *var_of = nullptr;    // [nnz] variable of each slot
    float *wk = nullptr;          // [nnz] 1 / k of the slot's constraint
    float *wd = nullptr;          // [nnz] 1 / max(d, 1) of the slot's variable
    // the same in variable order (each variable's occurrences, ascending slot)
    int32_t *vptr = nullptr;      // [n+1]
    int32_t *vlit = nullptr, *vcon = nullptr;   // [nnz] literal, constraint
    float *vwk = nullptr, *vwd = nullptr;       // [nnz]
    float *fv = nullptr;          // [n][8] variable features
    float *fc = nullptr;          // [m][8] constraint features
};

}  // namespace ffsat

namespace ffsat {
hipError_t fill_f32(int64_t n, float *p, float v, hipStream_t s);
}  // namespace ffsat
