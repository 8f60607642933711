// Small calls in one launch (spd_direct.hip): both operands are read where they lie.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spd_kernels.h"

namespace spd {

struct DirectCsr { const int64_t *indptr; const int32_t *indices; const float *values; int64_t rows, nnz; };
struct DirectArgs {
    DirectCsr a, b;
    OpParams q;
    int32_t transform, norm;
    uint32_t k;                   // columns
    float *out;                   // pairwise: m x n
    int32_t knn_k;                // 0: pairwise
    int64_t *out_idx;             // k-NN: m x knn_k
    float *out_dist;
};

constexpr int kDirectRows = 4;                    // rows of A to a workgroup
constexpr int kDirectRowsB = 256;                 // rows of B that are in a workgroup together
constexpr int kDirectLanes = 4;                   // lanes to a row of B, where not one
constexpr int kDirectStagingKind = 7;             // how spd_profile_read names this kernel's staging
constexpr int64_t kDirectColumns = 2048;          // a strip of kDirectRows floats per column: 32 KB
// Rows of B: beyond, the host's look at the row pointers is most of any way's time (140,000 of 1 or 46 entries against one row: 74 us by
// lists, 167 this way).
constexpr int64_t kDirectMostRows = 1 << 15;
constexpr int64_t kDirectKnnRows = 1024;          // kDirectRows distances to a row of B: 16 KB
// The products the kernel serves (sum() = max needs the columns that B's row does not store).
SPD_HD constexpr bool direct_serves(int op) {
    return op == OP_DOT || op == OP_L1 || op == OP_CANB || op == OP_HAMM || op == OP_KL || op == OP_JS || op == OP_CNT ||
           op == OP_MINK || op == OP_MINK_ANY;
}
uint32_t direct_lds_bytes(int64_t n_cols, int64_t n, int knn_k);
hipError_t launch_direct(hipStream_t st, int op, const DirectArgs &args, int lanes);

}  // namespace spd
