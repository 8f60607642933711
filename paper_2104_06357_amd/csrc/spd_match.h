// Launch interface of the column-list kernels (spd_match*.hip).
//
// The staged scan (spd_scan_impl.h) visits every stored entry of B once per row of A and looks up
// whether the row stores the entry's column; where the rows share few columns nearly all of these
// visits meet nothing.  The column lists turn the loop round: the rows of B are cut into tiles, and
// per tile the entries are listed by column (a transpose of the tile, made on the device in each
// call).  A wavefront takes one row of A, walks the lists of that row's columns only, and adds
// product(a, b) to one sum per row of the tile, which lie in its own strip of LDS.  Work is done for
// the columns that two rows share and for nothing else.  The lists are walked in chunks of 16 entries,
// four chunks of any lists to a step.  A strip is private to its wavefront, and the sums are formed in the order of A's columns (a row of
// B appears at most once in a list, and lanes that meet in one sum are served in ascending order, which
// is that order): the results do not depend on the schedule.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spd_kernels.h"

namespace spd {

// One row of A as the kernels take them, longest first.
struct MatchRow { int64_t start; int32_t len, row; };

// Entries behind the last list, which a step may read and does not use: 15 of a chunk, and with a tile of
// 64 rows the 18 other pieces of a dense column that are summed together (half an entry a row).
constexpr int64_t kMatchSpare = 640;

// How B's rows are cut: into tiles of rows, and the columns of a tile into blocks (a power of two of them),
// each with room for its entries and for `dense_per_block` columns kept as one value per row of the tile.
struct MatchShape {
    int32_t tile_rows, n_tiles, waves;      // n_tiles 0: the product or the sizes do not fit
    int32_t block_shift, blocks, dense_per_block, dense_from;      // dense_from: entries that make a column dense
    uint32_t stage;                         // entries of a block that pass through LDS together
    int64_t ptr_stride, tile_extra;         // words of a tile's list bounds; entries beyond the tile's own
    uint32_t lds_bytes, build_lds_bytes;
    SPD_HD int64_t list_entries(int64_t nnz) const { return nnz + n_tiles * tile_extra + kMatchSpare; }
};
MatchShape match_shape(int64_t lds_budget, int op, int64_t n, int64_t n_cols, int64_t nnz);

struct MatchB {
    uint2 *list;            // {byte offset of the row's first sum in a strip, value bits}, by tile, column block and column;
                            // a dense column: tile_rows values, 0 where the row has none.  (A stored zero keeps
                            // its place in a list and points to a spare cell behind the strip's last; kMatchSpare
                            // entries at the end.)
    uint32_t *ptr;          // n_tiles * ptr_stride: where a column's list begins, from the tile's first entry on, at
                            // column + its block's number (a block has a word more for its last list's end);
                            // kMatchDense is set where the column is dense
    double *norms;          // n * 2, derived
    double *least;          // n_tiles * 2: the norms of a tile's row of the least first norm (k-NN)
    MatchShape shape;
    const uint32_t *cols;   // nullptr, or on the device how many columns there are (no more than the shape was made for)
};
constexpr uint32_t kMatchDense = 0x80000000u;

struct MatchArgs {
    const int32_t *a_indices;
    const float *a_values;
    const MatchRow *rows;
    int32_t m;
    const double *norms_a;        // m * 2, derived, by row number
    const int64_t *b_indptr;
    int64_t b_nnz;
    MatchB b;
    int64_t n;
    uint32_t k;
    int32_t transform;
    OpParams q;
    int32_t m_shared;             // the first rows, which the wavefronts of a workgroup share
    int32_t slices, groups;       // grid: groups of tiles (g, g + groups, ...) x slices of A's rows (s, s + slices, ...)
    int32_t by_xcd;               // 1: the slices of a group share an XCD
    int32_t run;                  // tiles of its group that a wavefront goes through with a row
    float *out;                   // pairwise: m x n
    int32_t knn_k;                // 0: pairwise
    KnnEntry *knn_part;           // (row * groups + group) * knn_k
    unsigned long long *knn_tau;  // per row: the tightest k-th (distance, index) key of any group
};

// Both operands over the columns that A stores (spd_match_columns.hip).
struct MatchColumns {
    uint2 *words;                 // per 32 columns: the marked ones' bits, and how many are marked before
    uint32_t *sums, *totals;      // scratch of the scans; {columns, entries of B} that stay
    uint64_t *masks;              // per 64 entries of B: which stay
    uint32_t *before;             // ... and how many stay before
    int32_t *a_indices;
    int64_t *b_indptr;
    int32_t *b_indices;
    float *b_values;
};

constexpr int64_t kMatchMostColumns = 1 << 28;    // that are renumbered (16 bytes per 64 of them)
constexpr uint32_t kBuildDense = 32;            // dense columns of a block at most
constexpr int kMatchStagingKind = 6;            // how spd_profile_read names this kernel's staging
constexpr int64_t kMatchL2Bytes = 4 << 20;      // of one XCD
// Bytes that a pair's sums take in a strip: its doubles and its count.
SPD_HD constexpr int match_doubles(int op) {
    return op == OP_DOT || op == OP_L1 || op == OP_CANB || op == OP_KL || op == OP_JS ? 1 : (op == OP_MINK || op == OP_MINK_ANY ? 2 : 0);
}
SPD_HD constexpr int match_counts(int op) { return op == OP_HAMM || op == OP_CNT || op == OP_KL || op == OP_MINK || op == OP_MINK_ANY ? 1 : 0; }
SPD_HD constexpr int match_cell_bytes(int op) { return 8 * match_doubles(op) + 4 * match_counts(op); }
SPD_HD constexpr uint32_t match_strip_bytes(int cell_bytes, int tile_rows) { return ((uint32_t)(tile_rows + 1) * (uint32_t)cell_bytes + 7u) / 8u * 8u; }
// Wavefronts of a workgroup, of which a compute unit holds one: the strips share its LDS, and where a pair's
// sums take 16 bytes or more, there are fewer and longer strips.
SPD_HD constexpr int match_waves(int cell_bytes) { return cell_bytes >= 16 ? 12 : 16; }
// Upper bound of the kernel's static __shared__ use (64 half words to a wavefront, the locks).
SPD_HD constexpr int64_t match_static_lds(int cell_bytes) { return 256 + match_waves(cell_bytes) * 128; }
// The products the column lists serve.
SPD_HD constexpr bool match_serves(int op) {
    return op == OP_DOT || op == OP_L1 || op == OP_CANB || op == OP_HAMM || op == OP_KL || op == OP_JS || op == OP_CNT ||
           op == OP_MINK || op == OP_MINK_ANY;
}

// Whether the launches for a call's lists, of which A has m rows, are below 2^32 work-items each (`renumbered`: over A's columns).
bool match_launches_fit(const MatchShape &s, int64_t m, int64_t nnz_a, bool renumbered);

hipError_t launch_match_norms(hipStream_t st, const int64_t *indptr, const float *values, int64_t n_rows, int64_t nnz,
                              int metric, int transform, int norm, float p, double k, double *norms);
// (after the norms; `b.least` nullptr: not asked for)
hipError_t launch_match_build(hipStream_t st, const int64_t *indptr, const int32_t *indices, const float *values,
                              int64_t n_rows, int64_t nnz, uint32_t k, const MatchB &b, int cell_bytes, int transform);
hipError_t launch_match_columns(hipStream_t st, const int32_t *a_indices, int64_t a_nnz, const int64_t *b_indptr, const int32_t *b_indices,
                                const float *b_values, int64_t b_rows, int64_t b_nnz, uint32_t n_cols, const MatchColumns &c);
// k-NN: the rows' bounds, and where each row's candidate lists lie.
hipError_t launch_match_knn_begin(hipStream_t st, unsigned long long *tau, int64_t *row_off, int32_t *row_lists, KnnEntry *part,
                                  int64_t m, int lists, int k);
hipError_t launch_match(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes);

}  // namespace spd
