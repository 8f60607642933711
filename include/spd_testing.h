/*
 * Test hooks of the spd library.  They take HOST pointers and touch no GPU, so the host
 * logic (the planner, and the per-visit products and expansion functions shared with the
 * kernels) can be checked on a machine without one.  spd_pairwise / spd_knn never call
 * them and never compute on the CPU.
 */
#ifndef SPD_TESTING_H
#define SPD_TESTING_H

#include <stddef.h>
#include <stdint.h>

#include "spd.h"

#ifdef __cplusplus
extern "C" {
#endif

/* One distance from two sparse rows (host arrays, ascending columns), evaluated the way
 * the kernels do: row norms, the product g(a, b) over the stored entries of `b` with `a`
 * looked up by column (0 when absent), then the expansion function (Table 1; Section 2.2,
 * Eq. 2 in its single-sweep form).  Returns SPD_ERR_* on bad arguments. */
spd_status spd_host_pair_value(spd_metric metric, float p, int64_t n_cols, const int32_t *a_cols,
                               const float *a_vals, int64_t a_len, const int32_t *b_cols,
                               const float *b_vals, int64_t b_len, float *out);

/* Runs the planner on two row-pointer arrays (host) exactly as spd_pairwise / spd_knn
 * would (`k_neighbors` = 0 for pairwise), checks the plan's consistency, and writes a
 * JSON summary (staging kind, rows per group, workgroup size, LDS bytes, spilled rows,
 * slabs, chunks) into `json` (at most `cap` bytes, always terminated).
 * `options`: n_options pairs name/value as for spd_set_option. */
spd_status spd_host_plan_summary(const int64_t *a_indptr, int64_t a_rows, const int64_t *b_indptr,
                                 int64_t b_rows, int64_t n_cols, spd_metric metric, int k_neighbors,
                                 const char *const *option_names, const int64_t *option_values,
                                 int n_options, char *json, size_t cap);

/* Whether a call on operands of these sizes (`k_neighbors` = 0 for pairwise, `with_index` for the calls
 * on a prepared index) takes the column lists (option "match_lists"), and how it cuts them.  (Of a call that takes none: how
 * the lists over all columns would be cut.  Small calls that run in one launch: spd_host_direct_lanes.)  Besides the options,
 * "scratch": bytes that the caller lends. */
typedef struct {
    int32_t wanted;                 /* over all columns, were an index to keep them */
    int32_t tiles, tile_rows;       /* of B */
    int32_t slices, groups;         /* workgroups: slices of A's rows times groups of tiles */
    int32_t consistent;             /* what option "check_plan" finds of the cut */
    int64_t scratch_bytes;
    int64_t index_bytes;            /* what an index keeps of lists; 0: none */
    int32_t run;                    /* tiles that a wavefront goes through with a row of A */
    int32_t way;                    /* 0: the staged scan, 1: lists over all columns, 2: over the columns that A stores */
    int64_t columns;                /* that the lists are laid out for */
    int64_t block_columns;          /* of a block of the build */
    int32_t aligned, index_aligned; /* lists that begin at lines of memory: of the call's scratch, and of an index */
    int32_t staged_kind, staged_rows;   /* rows that the scan would stage together, and their kind of map */
    int64_t shared_len;             /* rows of A of more entries are shared by the wavefronts of a workgroup */
} spd_list_plan;
spd_status spd_host_list_plan(int64_t a_rows, int64_t a_nnz, int64_t b_rows, int64_t b_nnz, int64_t n_cols,
                              spd_metric metric, float p, int k_neighbors, int with_index,
                              const char *const *option_names, const int64_t *option_values, int n_options,
                              spd_list_plan *out);

/* Lanes to a row of B in the one launch that a call on operands of these sizes is by default (option "direct");
 * 0: it runs by the other ways. */
spd_status spd_host_direct_lanes(const int64_t *b_indptr, int64_t b_rows, int64_t a_rows, int64_t a_nnz, int64_t n_cols,
                                 spd_metric metric, float p, int k_neighbors, int with_index, int *lanes);

#ifdef __cplusplus
}
#endif
#endif /* SPD_TESTING_H */
