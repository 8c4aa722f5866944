// Vertices ranked by degree (rank.hip), and the exclusive scan its users share.
#pragma once

#include "common.h"

namespace sp {

// Degrees below kRankExact are ranked exactly, higher ones by their leading
// six bits; the vertices of degree >= kRankExact hold ranks [0, rank_heavy).
constexpr int32_t kRankExact = 256;

// Builds g->rank_new / g->rank_old / g->rank_heavy once; the caller holds g->mu.
sp_status ensure_rank_locked(sp_graph g, hipStream_t s);

constexpr int32_t kScanTile = 1024;  // counts per scan tile (256 threads x 4)

// Tiles that launch_excl_scan needs for n counts.
int64_t scan_tiles(int64_t n);

// out[i] = sum of in[0..i) for i in [0, n]; out holds n + 1 values and may be
// `in` itself when that has room.  `tiles`: scan_tiles(n) values of scratch.
void launch_excl_scan(const int32_t *in, int64_t n, int32_t *out, int32_t *tiles, hipStream_t s);

}  // namespace sp
