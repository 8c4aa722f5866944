// Vertices ranked by degree (rank.hip), and the exclusive scan its users share.
#pragma once

#include "common.h"

namespace sp {

// Degrees below kRankExact are ranked exactly, higher ones by their leading
// six bits, so the vertices of at least a given degree hold the first ranks
// when that degree is at most kRankExact or a power of two.
constexpr int32_t kRankExact = 256;
constexpr int32_t kRankBuckets = 1024;

// Class of a degree, 0 = heaviest: exact below 256, then 32 classes per octave.
__host__ __device__ inline int32_t rank_bucket(int32_t deg) {
    int32_t key = deg;
    if (deg >= kRankExact) {
        const int32_t e = 31 - __builtin_clz((unsigned)deg);  // 8..30
        key = kRankExact + (e - 8) * 32 + ((deg >> (e - 5)) & 31);
    }
    return kRankBuckets - 1 - key;
}

// Builds g->rank_new / g->rank_old / g->rank_first once; the caller holds g->mu.
sp_status ensure_rank_locked(sp_graph g, hipStream_t s);

// Builds g->rank_rp once, on an undirected graph; after ensure_rank_locked, the
// caller holds g->mu.
sp_status ensure_rank_rp_locked(sp_graph g, hipStream_t s);

// Vertices of degree >= deg (at most kRankExact, or a power of two); after ensure_rank_locked.
inline int32_t rank_count(sp_graph g, int32_t deg) { return g->rank_first[rank_bucket(deg) + 1]; }

// Vertices above which renumbering by rank is considered.  Weighted rows (rmat,
// edge factor 16): a query with and without 2^18 vertices 563 and 568 us, 2^19
// 736 and 746, 2^20 1,287 and 1,328, 2^21 1,634 and 1,846, 2^22 3,112 and 4,152;
// to replace the weights 97 and 71, 414 and 347, 501 and 402, 714 and 494, 1,117
// and 726.
constexpr int32_t kRenumberFrom = 1 << 20;
// PageRank (once a graph): from here on two calls of 20 iterations, and soon one,
// win back what the copy takes (rmat, edge factor 16, with and without: 410,000
// vertices first 2.4 and 2.0 ms, then 1.24 and 1.78; first, 600,000 vertices 3.0
// and 3.5, 4,000,000 12.5 and 21.1).
constexpr int32_t kPrRenumberFrom = 400000;
// Per-source passes: four sources, copy made, with and without: 600,000
// vertices 2.2 and 1.9 ms, 1,000,000 3.29 and 3.33, 2,000,000 5.4 and 6.4,
// 4,000,000 9.9 and 13.7.  The copy takes as long as four to ten of the sources
// it serves gain, so fewer than kSourceRankCount use it only where it is there
// (sp_bfs_levels, 1,000,000 vertices, first call: 2.3 and 1.1 ms).
constexpr int32_t kSourceRankFrom = 1 << 20;
constexpr int32_t kSourceRankCount = 8;

// Whether gathers concentrate enough for renumbering to pay: the eighth of the
// vertices of highest degree holds at least half of the entries (road grids
// and uniform graphs keep their numbering, which may be a local one).  After
// ensure_rank_locked.
bool rank_skewed(sp_graph g);
// Whether that can be, by the highest degree alone (flat graphs need no ranks to tell).
inline bool may_be_skewed(sp_graph g) { return 2 * ((int64_t)g->n / 8) * g->max_degree >= g->nnz; }

// Builds g->rank_ci (and g->rank_rp) once, on an undirected graph that is
// skewed; leaves it null on others and where memory is short.  The caller holds g->mu
// and has looked at the size.
sp_status ensure_rank_csr_locked(sp_graph g, hipStream_t s);

// Entries of the rows [0, rows) renumbered: row i goes to col[to[i]...], from
// the row of vertex old[order[i]] (order null: the identity).  The first
// `longer` rows take a block each, the others 16 lanes.
void launch_renumber(const int32_t *rp, const int32_t *ci, const int32_t *order, const int32_t *old,
                     const int32_t *new_id, const int32_t *to, int32_t longer, int32_t rows, int32_t *col,
                     hipStream_t s);

// Row classes by length, longest first, and a stable sort of n vertices into
// them: order[i] = the i-th vertex, first[c] = where class c starts
// (first[kRowClasses] = n).  Vertex x has the row of old[x] (x itself when old
// is null) in rp.  Class 0 holds the rows longer than `longest`.
constexpr int32_t kRowClasses = 6;
__host__ __device__ inline int32_t row_class(int32_t len, int32_t longest) {
    return len > longest ? 0 : len >= 512 ? 1 : len > 128 ? 2 : len > 32 ? 3 : len > 8 ? 4 : 5;
}
sp_status sort_rows_by_class(const int32_t *rp, const int32_t *old, int32_t n, int32_t longest, int32_t *order,
                             int32_t *first, hipStream_t s);

constexpr int32_t kScanTile = 1024;  // counts per scan tile (256 threads x 4)

// Tiles that launch_excl_scan needs for n counts.
int64_t scan_tiles(int64_t n);

// out[i] = sum of in[0..i) for i in [0, n]; out holds n + 1 values and may be
// `in` itself when that has room.  `tiles`: scan_tiles(n) values of scratch.
void launch_excl_scan(const int32_t *in, int64_t n, int32_t *out, int32_t *tiles, hipStream_t s);

// off[i] = entries of the rows before the i-th, the row of vertex old[x] for
// x = order[i] (either list null: the identity); n + 1 values.
void launch_row_offsets(const int32_t *rp, const int32_t *order, const int32_t *old, int32_t n, int32_t *off,
                        int32_t *tiles, hipStream_t s);

}  // namespace sp
