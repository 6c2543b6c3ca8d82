/*
 * libmaxk -- host-side introspection for the library's own tests.  Not part of the API: these symbols may change
 * or disappear between versions, and no caller needs them to use the path.
 */
#ifndef MAXK_TEST_HOOKS_H
#define MAXK_TEST_HOOKS_H

#include "maxk.h"

#ifdef __cplusplus
extern "C" {
#endif

/* The number of private output-row copies the forward kernel (Alg. 1's on-chip output row) keeps in LDS for
 * MaxK k: entries that share one 64-lane instruction must map to different copies.  Negative maxk_status for k < 1. */
MAXK_API int32_t maxk_fwd_private_copies(int32_t k);

/* Whether the row-by-row forward kernel works by units, not by lane groups, on `items` work items of `entries` entries (0 or 1). */
MAXK_API int32_t maxk_fwd_by_units(int32_t k, int32_t dim, int32_t value_type, int64_t items, int64_t entries);

/* Whether the pull of whole rows works by units, not by lane groups, on a graph where `beyond` of the entries have a row that is not among the most
   frequent 4 MB (0 or 1). */
MAXK_API int32_t maxk_pull_by_units(int32_t dim, int32_t k, int32_t value_type, int64_t N, int64_t nnz, double beyond);

/* Whether the expand/reduce backward kernels write and read their products past L2 at this shape (0 or 1). */
MAXK_API int32_t maxk_expand_past_l2(int64_t N, int64_t nnz, int32_t dim, int32_t k, int32_t index_bytes, int32_t dy_value_type);

/* The same for the rows that the gradient scatter writes. */
MAXK_API int32_t maxk_scatter_past_l2(int64_t N, int32_t dim);

/* How many regroupings of A^T the handle holds: slab tables (one per slab height ever needed) and visit lists of the
 * LDS-tiled backward kernel (one per destination-set size and k / 4).  They are built once and kept, so the counts
 * never go down and a repeated shape never adds one.  Either out pointer may be NULL. */
MAXK_API maxk_status maxk_graph_cached_tables(const maxk_graph* g, int32_t* n_slab_tables, int32_t* n_tiled_tables);

/* From how many entries on a visit gets a wavefront of its own (32: above 32) in a slab of `entries` whose longest has `longest`. */
MAXK_API int32_t maxk_lone_visit_line(int32_t longest, int64_t entries);

/* First entry of the batch that a kernel fetches `ahead` entries behind `base`, of a work item that ends at `end` (the last entry where
   the batch lies behind it). */
MAXK_API int64_t maxk_entry_batch(uint32_t base, uint32_t ahead, uint32_t end);

/* How many regroupings of A for the forward sweep the handle holds (kept like the tables above). */
MAXK_API int32_t maxk_graph_sweep_tables(const maxk_graph* g);

/* How many regroupings of A^T for the register-tiled backward kernel the handle holds (kept like the tables above). */
MAXK_API int32_t maxk_graph_regs_tables(const maxk_graph* g);

/* What a wavefront of that kernel copies of its list in step `step` of a tile: first record, records. */
MAXK_API maxk_status maxk_regs_step_list(uint32_t record0, uint32_t records, uint32_t step, uint32_t* first, uint32_t* copied);

/* Copies table `which` of the i-th of those regroupings to host memory (nothing where out is NULL) and returns its bytes, or a
 * negative maxk_status: 0 sizes (int64 each), 1 records, 2 headers, 3 destinations, 4 rows, 5 units, 6 parts, 7 sums, 8 splits. */
MAXK_API int64_t maxk_graph_regs_table(const maxk_graph* g, int32_t i, int32_t which, void* out, int64_t bytes);

/* From here on the handle's tables, the slice-major copy and the expand/reduce buffer are refused, as if memory had run
 * out, when they take more than `bytes` (a table: 8 an entry); negative: no limit.  Returns how many were refused so far. */
MAXK_API int64_t maxk_graph_limit_allocations(maxk_graph* g, int64_t bytes);

#ifdef __cplusplus
}
#endif
#endif /* MAXK_TEST_HOOKS_H */
