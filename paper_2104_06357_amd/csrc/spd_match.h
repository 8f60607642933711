// Launch interface of the column-list kernels (spd_match*.hip).
//
// The staged scan (spd_scan_impl.h) visits every stored entry of B once per row of A and looks up
// whether the row stores the entry's column; where the rows share few columns nearly all of these
// visits meet nothing.  The column lists turn the loop round: the rows of B are cut into tiles, and
// per tile the entries are listed by column (a transpose of the tile, made on the device in each
// call).  A wavefront takes one row of A, walks the lists of that row's columns only, and adds
// product(a, b) to one sum per row of the tile, which lie in its own strip of LDS.  Work is done for
// the columns that two rows share and for nothing else.  The lists are walked in chunks of 16 entries,
// four chunks of any lists to a step.  A strip is private to its wavefront, but for the longest rows
// where sums are integers.  Sums in floating point are formed in the order of A's
// columns (a row of B appears at most once in a list, and lanes that meet in one sum are served in ascending order, which
// is that order), sums in fixed point come out the same in any order: the results do not depend on the schedule.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spd_kernels.h"

namespace spd {

// One row of A as the kernels take them, longest first.
struct MatchRow { int64_t start; int32_t len, row; };

// Entries behind the last list, which a step may read and does not use: 15 of a chunk, and with a tile of
// 64 rows the 18 other pieces of a dense column that are summed together (an entry a row).
constexpr int64_t kMatchSpare = 1280;

// How B's rows are cut: into tiles of rows, and the columns of a tile into blocks (a power of two of them),
// each with room for its entries; `dense_per` of 2^dense_shift columns may be kept as one value per row of the tile.
struct MatchShape {
    int32_t tile_rows, n_tiles;             // n_tiles 0: the product or the sizes do not fit
    int16_t waves, held;                    // of a workgroup of the walk; entries that a lane of the build holds
    int32_t block_shift, blocks, dense_shift, dense_per, dense_from;      // dense_from: entries that make a column dense
    uint32_t stage;                         // entries of a block that pass through LDS together
    // 1: lists of kMatchLine entries or more and dense columns begin at multiples of kMatchLine, see below.  (The walk reads it where its registers are short: from 16 bits
    // 663,000 n-grams, k-NN, take 1,828 us for 1,809.)
    int32_t aligned;
    int64_t ptr_stride, tile_extra;         // words of a tile's list bounds; entries beyond the tile's own
    uint32_t lds_bytes, build_lds_bytes;
    SPD_HD int32_t dense_before(int32_t block) const { return (int32_t)(((int64_t)block * dense_per + (1 << (dense_shift - block_shift)) - 1) >> (dense_shift - block_shift)); }
    SPD_HD int32_t dense_room() const { return tile_rows > dense_from ? tile_rows - dense_from : 0; }       // entries more than such a column has
    // The room that so many entries have in the lists: with gaps between aligned lists five sixteenths more.  (What follows one another
    // has at least its own room: the sum of two rooms is no more than the room of both.)
    SPD_HD int64_t room_of(int64_t entries) const { return aligned ? entries + (entries >> 2) + (entries >> 4) : entries; }
    SPD_HD int64_t list_entries(int64_t nnz) const { return room_of(nnz) + n_tiles * tile_extra + kMatchSpare; }
    // Of a word of the list bounds: the position, and the gap before it (entries behind the list before that are nobody's).
    SPD_HD uint32_t position_bits() const { return aligned ? 0x07FFFFFFu : 0x7FFFFFFFu; }
    SPD_HD uint32_t gap_bits() const { return aligned ? 15u : 0u; }
};
// The L1 looks a load of 64 lanes up by 16 lanes and by lines of 64 bytes: a chunk of 16 entries costs two look-ups where it begins at such a
// line (one for its values, one for its rows), and 3.4 anywhere; 64 rows of a dense column four, and eight.  (Anywhere / at lines: look-ups of 4,096 x
// 65,536 rows of 1,820, L1, 9.4e9 / 7.4e9, lines fetched from L2 4.3e9 / 3.7e9, the walk 23.4 / 21.6 ms; 1,024 x 300,000 rows of 230, cosine,
// 2.1e9 / 1.6e9 look-ups, 4.35 / 4.16 ms: its loads' addresses, five clocks and a half a load wherever they lie, take 88 % of the time.)
constexpr uint32_t kMatchLine = 16, kMatchGapShift = 27;
MatchShape match_shape(int64_t lds_budget, int op, int64_t n, int64_t n_cols, int64_t nnz);

// An entry of a list lies in two arrays, six bytes together: two loads of four and two bytes take the L1 9 clocks for 64 lanes, one
// of eight 16 (measured with everything in the L1), and a count's entries need the two bytes alone (4,096 x 500,000 sets, Jaccard,
// k-NN, 10.8 -> 8.9 ms a call).
struct MatchB {
    float *values;          // by tile, column block and column.  (A stored zero keeps its place in a list; kMatchSpare entries at the end.
                            // A dense column: tile_rows values, 0 where the row has none.)
    uint16_t *rows;         // byte offset of the row's first sum in a strip (a stored zero's: of a spare cell behind the strip's last);
                            // nothing where the column is dense
    uint32_t *ptr;          // n_tiles * ptr_stride: where a column's list begins, from the tile's first entry on, at
                            // column + its block's number (a block has a word more for its last list's end), and from bit
                            // kMatchGapShift on the gap before it where lists are aligned; kMatchDense is set where the column is dense
    double *norms;          // 2 * n, derived: the first ones, then the second ones
    double *least;          // n_tiles * 2: the norms of a tile's row of the least first norm (k-NN)
    uint8_t *ranks;         // Chebyshev: of B's entries, kRanks or more where it is not among the row's kRanks largest
    float *tops;            // ... kRanks * n: the rows' largest magnitudes, the first of all rows, the second ..., 0 where a row has no more
    MatchShape shape;
    const uint32_t *cols;   // nullptr, or on the device how many columns there are (no more than the shape was made for)
};
constexpr uint32_t kMatchDense = 0x80000000u;

struct MatchArgs {
    const int32_t *a_indices;
    const float *a_values;
    const MatchRow *rows;
    int32_t m;
    const double *norms_a;        // 2 * m, derived, likewise
    const double *norms_b;        // k-NN: those of B's that distances read first (norms_read), the first ones or the second ones
    const int16_t *scales_a;      // m: L1, the rows' exponents (match_fixed); Canberra, 1 where a row is wild
    const uint8_t *ranks_a;       // Chebyshev: of A's entries, and kRanks magnitudes of every row, one row after the other
    const float *tops_a;
    const int32_t *b_indices;     // ... and B's rows, for the pairs whose kRanks largest entries of a row were all met
    const float *b_values;
    const int64_t *b_indptr;
    int64_t b_nnz;
    MatchB b;
    int64_t n;
    uint32_t k;
    int32_t transform;
    OpParams q;
    int32_t m_shared;             // the first rows, which the wavefronts of a workgroup share
    uint32_t *next;               // per group, 0 before the launch: (tile, row)s of these rows that are taken; k-NN: behind them kMatchRowLocks locks a group
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
constexpr uint32_t kBuildDense = 64, kBuildDensePer = 32;          // dense columns of a block at most, and that have room of their own
constexpr int kBuildPerCu = 2;                  // workgroups of the build that share a compute unit's LDS
constexpr int kMatchRowLocks = 64;              // of a group, by row
constexpr int kMatchStagingKind = 6;            // how spd_profile_read names this kernel's staging
constexpr int64_t kMatchL2Bytes = 4 << 20;      // of one XCD
// Bytes that a pair's sums take in a strip: its doubles and its count.
SPD_HD constexpr int match_doubles(int op) {
    return op == OP_DOT || op == OP_L1 || op == OP_CANB || op == OP_KL || op == OP_JS ? 1 : (op == OP_MINK || op == OP_MINK_ANY ? 2 : 0);
}
SPD_HD constexpr int match_counts(int op) { return op == OP_CHEB ? 3 : op == OP_HAMM || op == OP_CNT || op == OP_KL || op == OP_MINK || op == OP_MINK_ANY ? 1 : 0; }
SPD_HD constexpr int match_cell_bytes(int op) { return 8 * match_doubles(op) + 4 * match_counts(op); }
SPD_HD constexpr uint32_t match_strip_bytes(int cell_bytes, int tile_rows) { return ((uint32_t)(tile_rows + 1) * (uint32_t)cell_bytes + 7u) / 8u * 8u; }
// Wavefronts of a workgroup, of which a compute unit holds one: the strips share its LDS, and where a pair's
// sums take 16 bytes or more, there are fewer and longer strips.
SPD_HD constexpr int match_waves(int cell_bytes) { return cell_bytes >= 16 ? 12 : 16; }
// Upper bound of the kernel's static __shared__ use (64 half words to a wavefront, the locks).
SPD_HD constexpr int64_t match_static_lds(int cell_bytes) { return 256 + match_waves(cell_bytes) * 128; }
// Sums in fixed point.  An LDS add of 64 doubles at random rows takes 25.3 clocks, of 64 integers of 64 bits 12.8 (8.1 and 6.2 without
// bank conflicts).  A term is scaled by a power of two and added to 2 in fp64, so that its last place is
// 2^-51: the words of such a sum count units of 2^-51, and adding them up as integers rounds no further.
//   L1         the scale 2^-e is the row of A's: no shared entry's min(|a|, |b|) reaches 2^(e + 1), and all of them together not 2^(e + 10).
//   Canberra   2 less the ratio, at most 2: e = 2, more for rows of A of more than 2^10 entries.
// A term has 24 bits, and a sum is exact while none reaches below a unit: L1 of rows whose entries lie within 2^28 of their largest (fp64: within
// 2^29, less the sum's growth), Canberra of rows of up to 1,023 entries (a ratio is 0 or 2^-25 at least).  Beyond that a term is
// rounded to half a unit, where a sum in fp64 is rounded with every term, to 2^-53 of what it has come to: L1 of rows whose entries lie
// 2^40 apart, 0.8 to 7e-15 of the rows' norms with fixed point and 0.2 to 2.6e-15 with fp64; Canberra of 24,000 entries
// has units of 2^-44, and a distance of such a row an ulp of 2^-38.
// Not the dot product: its terms have 48 bits, so that each is rounded, to 2^-52 of both rows' largest entries, where the norms it is
// set against are fp64 sums.  Euclidean distances of equal rows of 37 normal values came out as 3.5e-8 of the norm for
// 9e-9, rows of two values as 7e-9 for 0.
SPD_HD constexpr bool match_fixed(int op) { return op == OP_L1 || op == OP_CANB; }
// ... and the products whose sums are counts.
SPD_HD constexpr bool match_any_order(int op) { return match_fixed(op) || op == OP_HAMM || op == OP_CNT; }
// floor(log2 v), -1023 for 0, 1,024 for what is not finite.
SPD_HD int match_ilog2(double v) {
    uint64_t w;
    __builtin_memcpy(&w, &v, 8);
    return (int)((w >> 52) & 0x7ffu) - 1023;
}
// L1's exponent for a row of A from its largest entry and the sum of them.  In [-200, 200]; 0 for a row of zeros.
SPD_HD int match_scale(float largest, double sum) {
    if (!(sum > 0.0) || !(largest > 0.0f)) return 0;
    const int top = match_ilog2((double)largest), all = match_ilog2(sum);
    const int e = top > all - 9 ? top : all - 9;
    return e < -200 ? -200 : (e > 200 ? 200 : e);
}
// Canberra: whether a row of A, whose entries' magnitudes lie from `least` (but 0) to `largest`, can meet a row of finite values where |a| + |b|
// or its reciprocal is not finite in single precision, or |a - b| is not: no sum is below 2^-100 or, half an ulp of the largest number being 2^103,
// rounded to infinity else.  Such a row is walked column by column.  (Another row may meet an entry above 2^126 all the same: the reciprocal is
// 0 there and the quotient with it, as by the staged scan.)
SPD_HD bool match_wild(float least, float largest) { return !(least >= 0x1p-100f && largest < 0x1p102f); }
// Canberra's for a row of A of `len` entries: 2 len 2^(51 - e) below 2^62.
SPD_HD int match_canberra_scale(int len) { return len < (1 << 10) ? 2 : 2 + (32 - 10) - __builtin_clz((unsigned)len); }

// The products the column lists serve.
SPD_HD constexpr bool match_serves(int op) {
    return op == OP_DOT || op == OP_L1 || op == OP_CANB || op == OP_HAMM || op == OP_KL || op == OP_JS || op == OP_CNT ||
           op == OP_MINK || op == OP_MINK_ANY || op == OP_CHEB;
}
// Chebyshev: the maximum over the columns that both rows store is completed from the largest entry of either row that the other does
// not store.  The entries of a row are ranked by magnitude; a pair keeps a bit for each of the kRanks largest of either row that was
// met, so that the first one that was not is known.  Pairwise only; a (tile, row) has no distance before its bits are complete.
constexpr int kRanks = 32, kRankShift = 10, kRankedRows = 832;      // (rank and row share an entry's 16 bits; a round of finishing holds 13 x 64 rows)
SPD_HD constexpr bool match_serves_knn(int op) { return match_serves(op) && op != OP_CHEB; }

// Whether the launches for a call's lists, of which A has m rows, are below 2^32 work-items each (`renumbered`: over A's columns).
bool match_launches_fit(const MatchShape &s, int op, int64_t m, int64_t nnz_a, int64_t n, bool renumbered);

// Row pointers that the host has not seen when the kernels which go by them are launched: no row leaves the arrays, but rows may
// overlap, and all of them together be any number of times as long (0, nnz, 0, nnz, ...).  They are looked at on the device first, and these
// kernels do nothing where `*word` is `malformed` (a number that no earlier call on the word had).  word nullptr: the host has.
struct RowsVerdict { const uint32_t *word; uint32_t malformed; };
// Writes `malformed` to *word where pointers do not begin at 0, fall or do not end at nnz (`b` nullptr: of one operand alone).
hipError_t launch_match_look_at_rows(hipStream_t st, const int64_t *a, int64_t m, int64_t a_nnz, const int64_t *b, int64_t n, int64_t b_nnz,
                                     uint32_t *word, uint32_t malformed);

// (`scales` nullptr: not asked for)
hipError_t launch_match_norms(hipStream_t st, const int64_t *indptr, const float *values, int64_t n_rows, int64_t nnz,
                              int metric, int transform, int norm, float p, double k, const RowsVerdict &seen, double *norms, int16_t *scales);
// Ranks and largest magnitudes of two operands' rows (`by_row`: the magnitudes of a row one after the other, else in planes).
struct RankedRows { const int64_t *indptr; const float *values; int64_t n_rows, nnz; int by_row; uint8_t *ranks; float *tops; };
hipError_t launch_match_ranks(hipStream_t st, const RankedRows &first, const RankedRows &second, const RowsVerdict &seen);
// (after the norms; `b.least` nullptr: not asked for)
hipError_t launch_match_build(hipStream_t st, const int64_t *indptr, const int32_t *indices, const float *values,
                              int64_t n_rows, int64_t nnz, uint32_t k, const MatchB &b, int op, int transform, const RowsVerdict &seen);
hipError_t launch_match_columns(hipStream_t st, const int32_t *a_indices, int64_t a_nnz, const int64_t *b_indptr, const int32_t *b_indices,
                                const float *b_values, int64_t b_rows, int64_t b_nnz, uint32_t n_cols, const MatchColumns &c);
// k-NN: the rows' bounds, and where each row's candidate lists lie.
hipError_t launch_match_knn_begin(hipStream_t st, unsigned long long *tau, int64_t *row_off, int32_t *row_lists, KnnEntry *part,
                                  int64_t m, int lists, int k);
hipError_t launch_match(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes);

}  // namespace spd
