// Triangle counting (paper Appendix, Fig. "TC computation in StarPlat").
//
// The paper's node iterator counts, for every vertex v, the adjacent pairs
// (u, w) of its neighbours with u < v < w, testing adjacency by binary search
// in a sorted row; each triangle is counted once.  Its work at a vertex is
// (neighbours below) x (neighbours above): quadratic in the degree of a
// high-degree vertex.  Here each triangle is instead counted once at its
// vertex of lowest degree.  Vertices are renumbered by rank, heaviest first
// (rank.hip), and N(v) holds the neighbours of lower rank number, ascending; a
// triangle {w < u < v} is a pair (w, u) of N(v) with w in N(u).  A vertex has
// at most about sqrt(2m) heavier neighbours, so the work is bounded by
// O(m^1.5) whatever the degree mix.  The count is the same number the paper's
// loops produce.
//
// Counting goes by the middle vertex u: its N(u) is marked in a bitmap in
// LDS, and for every entry (v, u) that names it, the entries of N(v) before u
// are streamed past the bitmap, one bit test each.  rmat-22: 7.2 G tests,
// read as 16-bit ids (u < 65536: 97% of the tests), 15 GB, instead of 11.8 G
// binary searches of about ten dependent loads each.
//
// The oriented rows are built once per graph: row lengths, a scan, a
// compacting copy, each row sorted (in registers, through an LDS bitmap, or by
// a bitonic network), the entries that name each vertex, and the work units.
//
// On flat and small graphs the rows are short and that index costs more than
// it saves: they are counted by binary searches, entry by entry (tc_by_pairs).
#include <utility>

#include "blocks.h"
#include "common.h"
#include "devutil.h"
#include "levels.h"
#include "rank.h"

namespace sp {

namespace {
constexpr int32_t kTcLow = 1 << 16;    // ids below stream as 16-bit values
constexpr int32_t kTcBits = 1 << 18;   // ids below are counted with an LDS bitmap
constexpr int32_t kTcLanes = 16;       // lanes per entry
constexpr int32_t kTcUnit = 512;       // entries naming u per work unit
constexpr int32_t kTcPosCap = 4096;    // per-vertex counts of N(u) kept in LDS up to this length
constexpr int32_t kTcSortBits = 1 << 19;  // rows of lower ids are sorted through a bitmap of this size
constexpr int32_t kTcHot = 4096;      // ids whose names are counted in LDS first
constexpr int32_t kTcNamedTile = 1 << 15, kTcNamedLeast = 1 << 11;  // entries of a block's tile
constexpr int32_t kTcSortCap = 8192;   // bitonic rows (a row of a higher id holds under 4,400 entries)
constexpr int32_t kTcFlat = 48;        // see tc_by_pairs
constexpr int64_t kTcSmall = 1 << 22, kTcLight = 1 << 27;
}  // namespace

// rank(a) < rank(b): lower degree, ties broken by id.
__device__ __forceinline__ bool rank_below(int32_t da, int32_t a, int32_t db, int32_t b) {
    return da < db || (da == db && a < b);
}

// ---------------------------------------------------------------------------
// Pairs: flat and small graphs (tc_by_pairs), where an index costs more than it
// saves.  Row v keeps the neighbours above v by (degree, id), in row order, and
// every entry (v, u) searches the elements of the shorter of the two rows in
// the longer one.
// ---------------------------------------------------------------------------
// Row lengths, LPR lanes to a row.  found[0]: entries that rise by rank (as
// ensure_rank_locked orders them), found[1]: rows that are not ascending.
template <int LPR>
__global__ __launch_bounds__(256) void k_tc_pair_len(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                                     int32_t n, int32_t *odeg, unsigned long long *found) {
    __shared__ unsigned long long s_red[1];
    constexpr int kFly = LPR == 1 ? 1 : 4;  // entries of a lane in flight
    const int l = threadIdx.x % LPR;
    unsigned long long by_rank = 0;
    bool mixed = false;
    for (int64_t v = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR; v < n;
         v += (int64_t)gridDim.x * (256 / LPR)) {
        const int32_t b = rp[v], e = rp[v + 1], dv = e - b, bv = rank_bucket(dv);
        int32_t d = 0;
        for (int32_t k0 = b + l; k0 < e; k0 += kFly * LPR) {
            int32_t u[kFly], before[kFly], du[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                const int32_t k = min(k0 + q * LPR, e - 1);
                u[q] = ci[k];
                before[q] = ci[max(k - 1, b)];
            }
#pragma unroll
            for (int q = 0; q < kFly; ++q) du[q] = rp[u[q] + 1] - rp[u[q]];
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                if (k0 + q * LPR >= e) continue;
                const int32_t bu = rank_bucket(du[q]);
                d += rank_below(dv, (int32_t)v, du[q], u[q]);
                by_rank += bu < bv || (bu == bv && u[q] > v);
                mixed |= u[q] < before[q];
            }
        }
        for (int o = LPR / 2; o > 0; o >>= 1) d += __shfl_xor(d, o, kWave);
        if (l == 0) odeg[v] = d;
    }
    if (__ballot(mixed) && lane_id() == 0) atomicOr(&found[1], 1ull);
    block_add_u64<256>(by_rank, s_red, &found[0]);
}

template <int LPR>
__global__ __launch_bounds__(256) void k_tc_pair_fill(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                                      int32_t n, const int32_t *__restrict__ orp, int32_t *oci,
                                                      int32_t *osrc) {
    constexpr int kFly = LPR == 1 ? 1 : 4;
    const int l = threadIdx.x % LPR;
    for (int64_t v = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR; v < n;
         v += (int64_t)gridDim.x * (256 / LPR)) {
        const int32_t b = rp[v], e = rp[v + 1], dv = e - b;
        int32_t at = orp[v];
        for (int32_t k0 = b; k0 < e; k0 += kFly * LPR) {
            int32_t u[kFly], du[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) u[q] = ci[min(k0 + q * LPR + l, e - 1)];
#pragma unroll
            for (int q = 0; q < kFly; ++q) du[q] = rp[u[q] + 1] - rp[u[q]];
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                const bool keep = k0 + q * LPR + l < e && rank_below(dv, (int32_t)v, du[q], u[q]);
                const unsigned long long m = LPR == 1 ? (unsigned long long)keep : __ballot(keep);
                if (keep) {
                    const int32_t p = at + (LPR == 1 ? 0 : lanes_below(m));
                    oci[p] = u[q];
                    osrc[p] = (int32_t)v;
                }
                at += __popcll(m);
            }
        }
    }
}

// First position in a[lo, hi) holding a value >= x.
__device__ __forceinline__ int32_t lower_bound(const int32_t *__restrict__ a, int32_t lo, int32_t hi,
                                               int32_t x) {
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The entries of a wave, one per lane.  Where the shorter row has at most
// kTcLaneWork elements the lane walks it, the search window shrinking as the
// walk moves up; longer ones are taken by the whole wave in turn.  per: each
// triangle counts at its three vertices (those of the entry once for all of
// its triangles).
constexpr int32_t kTcLaneWork = 32;

__global__ __launch_bounds__(256) void k_tc_pairs(const int32_t *__restrict__ orp, const int32_t *__restrict__ oci,
                                                  const int32_t *__restrict__ osrc, int64_t m,
                                                  unsigned long long *total, unsigned long long *per,
                                                  unsigned long long *prof) {
    __shared__ unsigned long long s_red[1];
    const int lane = lane_id();
    unsigned long long mine = 0, probes = 0;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x - lane; e0 < m; e0 += stride) {
        const int64_t e = e0 + lane;
        int32_t v = 0, u = 0, sb = 0, se = 0, lb = 0, le = 0;
        if (e < m) {
            v = osrc[e];
            u = oci[e];
            sb = orp[v];
            se = orp[v + 1];
            lb = orp[u];
            le = orp[u + 1];
            if (se - sb > le - lb) {  // walk the shorter row
                int32_t t = sb; sb = lb; lb = t;
                t = se; se = le; le = t;
            }
        }
        const bool alone = se - sb <= kTcLaneWork;
        if (alone) {
            int32_t pos = lb;
            unsigned int hits = 0;
            for (int32_t i = sb; i < se && pos < le; ++i) {
                const int32_t w = oci[i];
                pos = lower_bound(oci, pos, le, w);
                ++probes;
                if (pos < le && oci[pos] == w) {
                    ++hits;
                    ++pos;
                    if (per) atomicAdd(&per[w], 1ull);
                }
            }
            mine += hits;
            if (per && hits) {
                atomicAdd(&per[v], (unsigned long long)hits);
                atomicAdd(&per[u], (unsigned long long)hits);
            }
        }
        unsigned long long big = __ballot(!alone);
        while (big) {
            const int src = __ffsll((long long)big) - 1;
            big &= big - 1;
            const int32_t bsb = __shfl(sb, src, kWave), bse = __shfl(se, src, kWave);
            const int32_t blb = __shfl(lb, src, kWave), ble = __shfl(le, src, kWave);
            unsigned long long hits = 0;
            for (int32_t i = bsb + lane; i < bse; i += kWave) {
                const int32_t w = oci[i];
                const int32_t pos = lower_bound(oci, blb, ble, w);
                ++probes;
                if (pos < ble && oci[pos] == w) {
                    ++hits;
                    if (per) atomicAdd(&per[w], 1ull);
                }
            }
            mine += hits;
            if (per) {
                hits = wave_sum_u64(hits);
                if (lane == src && hits) {
                    atomicAdd(&per[v], hits);
                    atomicAdd(&per[u], hits);
                }
            }
        }
    }
    block_add_u64<256>(mine, s_red, total);
    if (prof) {
        __syncthreads();
        block_add_u64<256>(probes, s_red, prof + 1);
    }
}

// Whether a vertex is counted with an LDS bitmap.  Marking and clearing one
// costs a few microseconds of a block, so it takes some entries that name u
// to pay (rmat-22: from 32 on 7.0 ms, from 16 6.5, from 8 6.2); the rest go
// entry by entry (k_tc_light), as do ids whose bitmap would not fit.
__device__ __forceinline__ bool tc_heavy(int32_t u, int32_t named) { return u < kTcBits && named >= 8; }

// The heavier neighbours of the ranked vertices [first, n): calls
// f(keep, v, w) for every entry, 16 lanes per row, or (BLOCK) a block per row.
template <bool BLOCK, class F>
__device__ __forceinline__ void tc_rows(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                        const int32_t *__restrict__ rank_new,
                                        const int32_t *__restrict__ rank_old, int32_t first, int32_t n, F f) {
    constexpr int per = BLOCK ? 256 : 16;
    const int64_t stride = BLOCK ? gridDim.x : (int64_t)gridDim.x * (256 / per);
    for (int64_t v = first + (BLOCK ? (int64_t)blockIdx.x
                                    : (int64_t)blockIdx.x * (256 / per) + threadIdx.x / per);
         v < n; v += stride) {
        const int32_t old = rank_old[v];
        const int32_t b = rp[old], e = rp[old + 1];
        f((int32_t)v, old, b, e);
    }
}

// Row lengths: odeg[v] = neighbours of v of lower rank number (and named[v]
// cleared for k_tc_named).  exact: how
// many entries rise in the (degree, id) order, which is half of them exactly
// when a graph is simple and undirected (the two orders differ only between
// vertices of degree >= kRankExact).
template <bool BLOCK>
__global__ __launch_bounds__(256) void k_tc_outdeg(const int32_t *__restrict__ rp,
                                                   const int32_t *__restrict__ ci,
                                                   const int32_t *__restrict__ rank_new,
                                                   const int32_t *__restrict__ rank_old, int32_t first,
                                                   int32_t n, int32_t heavy, int32_t *odeg, int32_t *named,
                                                   unsigned long long *exact) {
    __shared__ unsigned long long s_red[1];
    __shared__ int32_t s_sum;
    constexpr int per = BLOCK ? 256 : 16;
    const int l = threadIdx.x % per;
    unsigned long long ex = 0;
    tc_rows<BLOCK>(rp, ci, rank_new, rank_old, first, n, [&](int32_t v, int32_t old, int32_t b, int32_t e) {
        int32_t d = 0;
        for (int32_t k = b + l; k < e; k += per) {
            const int32_t w = ci[k], r = rank_new[w];
            d += r < v;
            if (v < heavy && r < heavy) ex += rank_below(e - b, old, rp[w + 1] - rp[w], w);
            else ex += r < v;
        }
        if (BLOCK) {
            if (threadIdx.x == 0) s_sum = 0;
            __syncthreads();
            if (d) atomicAdd(&s_sum, d);
            __syncthreads();
            if (threadIdx.x == 0) {
                odeg[v] = s_sum;
                named[v] = 0;
            }
            __syncthreads();
        } else {
            for (int o = 8; o > 0; o >>= 1) d += __shfl_xor(d, o, kWave);
            if (l == 0) {
                odeg[v] = d;
                named[v] = 0;
            }
        }
    });
    block_add_u64<256>(ex, s_red, exact);
}

// Rows in any order within a row (they are sorted next), each entry's row.
template <bool BLOCK>
__global__ __launch_bounds__(256) void k_tc_fill(const int32_t *__restrict__ rp,
                                                 const int32_t *__restrict__ ci,
                                                 const int32_t *__restrict__ rank_new,
                                                 const int32_t *__restrict__ rank_old, int32_t first,
                                                 int32_t n, const int32_t *__restrict__ orp, int32_t *oci,
                                                 int32_t *osrc) {
    __shared__ int32_t s_at;
    constexpr int per = BLOCK ? 256 : 16;
    const int l = threadIdx.x % per;
    const int lane = lane_id();
    tc_rows<BLOCK>(rp, ci, rank_new, rank_old, first, n, [&](int32_t v, int32_t, int32_t b, int32_t e) {
        int32_t at = orp[v];
        if (BLOCK) {
            if (threadIdx.x == 0) s_at = at;
            __syncthreads();
        }
        for (int32_t k0 = b; k0 < e; k0 += per) {
            const int32_t k = k0 + l;
            const int32_t r = k < e ? rank_new[ci[k]] : INT32_MAX;
            const bool keep = r < v;
            const unsigned long long m = __ballot(keep);
            int32_t p = 0;
            if (BLOCK) {
                if (m) {
                    const int leader = __ffsll((long long)m) - 1;
                    if (lane == leader) p = atomicAdd(&s_at, __popcll(m));
                    p = shfl_i32(p, leader) + lanes_below(m);
                }
            } else {
                const unsigned int g = (unsigned int)(m >> (lane & 48)) & 0xffffu;
                p = at + __popc(g & ((1u << l) - 1u));
                at += __popc(g);
            }
            if (keep) {
                oci[p] = r;
                osrc[p] = v;
            }
        }
        if (BLOCK) __syncthreads();
    });
}

// Rows of 2..64 entries sorted by a wave each (an entry's place is the number
// of smaller ones); longer rows listed for the block kernels.  A wave takes
// `share` rows (a power of two up to 64), one after another, the next one's
// entries loaded meanwhile: 64 of them, each waiting for its load, made a graph
// of any size wait 170 us and more (rmat-13 169 -> 15 us; rmat-22 392).
__global__ __launch_bounds__(256) void k_tc_sort_small(const int32_t *__restrict__ orp, int32_t n, int32_t share,
                                                       int32_t *oci, int32_t *big, int32_t *nbig) {
    const int lane = lane_id();
    const int64_t stride = (int64_t)gridDim.x * (256 / kWave) * share;
    for (int64_t v0 = ((int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave) * share; v0 < n; v0 += stride) {
        const int64_t v = v0 + lane;
        int32_t b = 0, len = 0;
        if (v < n && lane < share) {
            b = orp[v];
            len = orp[v + 1] - b;
        }
        const unsigned long long more = __ballot(len > kWave);
        if (more) {
            const int leader = __ffsll((long long)more) - 1;
            int32_t at = 0;
            if (lane == leader) at = atomicAdd(nbig, __popcll(more));
            at = shfl_i32(at, leader);
            if (len > kWave) big[at + lanes_below(more)] = (int32_t)v;
        }
        unsigned long long todo = __ballot(len >= 2 && len <= kWave);
        int32_t nb = 0, nl = 0, nx = 0;  // the next row and its entries
        auto take = [&]() {
            nl = 0;
            if (!todo) return;
            const int src = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            nb = __builtin_amdgcn_readlane(b, src);
            nl = __builtin_amdgcn_readlane(len, src);
            nx = lane < nl ? oci[nb + lane] : INT32_MAX;
        };
        take();
        while (nl) {
            const int32_t rb = nb, rl = nl, x = nx;
            take();
            int32_t place = 0;
            for (int32_t j = 0; j < rl; ++j) {
                const int32_t y = __builtin_amdgcn_readlane(x, j);
                place += y < x || (y == x && j < lane);
            }
            if (lane < rl) oci[rb + place] = x;
        }
    }
}

// Rows of more than 64 entries and ids in [lo, hi), hi <= 32 * WORDS: marked
// in a bitmap, read back in order.  Entries stored twice (not a simple graph)
// leave a shorter row, whose tail repeats its last entry.
template <int WORDS>
__global__ __launch_bounds__(256) void k_tc_sort_bits(const int32_t *__restrict__ orp, int32_t *oci,
                                                      const int32_t *__restrict__ big,
                                                      const int32_t *__restrict__ nbig, int32_t lo, int32_t hi) {
    __shared__ uint32_t s_bits[WORDS];
    __shared__ int32_t s_scan[256 / kWave + 1], s_last;
    const int32_t nb = *nbig;
    for (int32_t j = blockIdx.x; j < nb; j += gridDim.x) {
        const int32_t v = big[j];
        if (v < lo || v >= hi) continue;
        const int32_t b = orp[v], len = orp[v + 1] - b;
        const int32_t words = (v + 31) >> 5;  // the row's ids are below v
        for (int32_t i = threadIdx.x; i < words; i += 256) s_bits[i] = 0;
        __syncthreads();
        for (int32_t i = threadIdx.x; i < len; i += 256) {
            const int32_t w = oci[b + i];
            atomicOr(&s_bits[w >> 5], 1u << (w & 31));
        }
        __syncthreads();
        const int32_t per = (words + 255) / 256;
        const int32_t i0 = min(words, (int32_t)threadIdx.x * per), i1 = min(words, i0 + per);
        int32_t mine = 0;
        for (int32_t i = i0; i < i1; ++i) mine += __popc(s_bits[i]);
        int32_t total;
        int32_t at = b + block_excl_scan<256>(mine, s_scan, &total);
        for (int32_t i = i0; i < i1; ++i)
            for (uint32_t m = s_bits[i]; m; m &= m - 1) {
                const int32_t w = i * 32 + __ffs(m) - 1;
                oci[at++] = w;
                if (at == b + total) s_last = w;
            }
        __syncthreads();
        for (int32_t i = total + threadIdx.x; i < len; i += 256) oci[b + i] = s_last;
        __syncthreads();
    }
}

// Rows of more than 64 entries and ids from kTcSortBits up: such a vertex has
// at least kTcSortBits heavier ones, so its degree, and its row, stays under
// kTcSortCap (fewer than 2^31 entries in all).
__global__ __launch_bounds__(256) void k_tc_sort_net(const int32_t *__restrict__ orp, int32_t *oci,
                                                     const int32_t *__restrict__ big,
                                                     const int32_t *__restrict__ nbig, int32_t lo) {
    __shared__ int32_t s_x[kTcSortCap];
    const int32_t nb = *nbig;
    for (int32_t j = blockIdx.x; j < nb; j += gridDim.x) {
        const int32_t v = big[j];
        if (v < lo) continue;
        const int32_t b = orp[v], len = min(orp[v + 1] - b, kTcSortCap);
        int32_t size = 128;
        while (size < len) size <<= 1;
        for (int32_t i = threadIdx.x; i < size; i += 256) s_x[i] = i < len ? oci[b + i] : INT32_MAX;
        __syncthreads();
        for (int32_t k = 2; k <= size; k <<= 1)
            for (int32_t d = k >> 1; d > 0; d >>= 1) {
                for (int32_t i = threadIdx.x; i < size; i += 256) {
                    const int32_t p = i ^ d;
                    if (p > i) {
                        const int32_t x = s_x[i], y = s_x[p];
                        if ((x > y) == ((i & k) == 0)) {
                            s_x[i] = y;
                            s_x[p] = x;
                        }
                    }
                }
                __syncthreads();
            }
        for (int32_t i = threadIdx.x; i < len; i += 256) oci[b + i] = s_x[i];
        __syncthreads();
    }
}

// 16-bit copies of the sorted entries, and each entry's place among those
// that name the same vertex (any order: only sums are formed over them).  The
// heaviest vertices are named by most rows, so a block first counts the names
// of the ids below kTcHot in its tile in LDS and reserves each id's places
// with one atomic (rmat-22: 41% of the entries; 7.1 ms with an atomic each).
__global__ __launch_bounds__(256) void k_tc_named(const int32_t *__restrict__ oci, int64_t m, int32_t tile,
                                                  uint16_t *olo, int32_t *named, int32_t *slot) {
    __shared__ int32_t s_at[kTcHot];
    for (int64_t t0 = (int64_t)blockIdx.x * tile; t0 < m; t0 += (int64_t)gridDim.x * tile) {
        const int64_t t1 = min(m, t0 + tile);
        for (int32_t i = threadIdx.x; i < kTcHot; i += 256) s_at[i] = 0;
        __syncthreads();
        for (int64_t e = t0 + threadIdx.x; e < t1; e += 256) {
            const int32_t u = oci[e];
            olo[e] = (uint16_t)u;
            if (u < kTcHot) atomicAdd(&s_at[u], 1);
            else slot[e] = atomicAdd(&named[u], 1);
        }
        __syncthreads();
        for (int32_t i = threadIdx.x; i < kTcHot; i += 256)
            if (s_at[i]) s_at[i] = atomicAdd(&named[i], s_at[i]);
        __syncthreads();
        for (int64_t e = t0 + threadIdx.x; e < t1; e += 256) {
            const int32_t u = oci[e];
            if (u < kTcHot) slot[e] = atomicAdd(&s_at[u], 1);
        }
        __syncthreads();
    }
}

__global__ void k_tc_inlist(const int32_t *__restrict__ oci, const int32_t *__restrict__ osrc,
                            const int32_t *__restrict__ orp, const int32_t *__restrict__ iptr,
                            const int32_t *__restrict__ slot, int64_t m, int2 *inl) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride)
        inl[iptr[oci[e]] + slot[e]] = make_int2(orp[osrc[e]], (int32_t)e);
}

// Work units of the vertices counted with a bitmap: those of ids below kTcLow
// and the others, in lists of their own, by id (in the order that an atomic per
// wave gives them the count of rmat-18, edge factor 32, took 324 us, not 277).
// A block's 256 ids lie on one side of kTcLow; first its sum, then its places.
__device__ __forceinline__ int32_t tc_unit_count(const int32_t *__restrict__ iptr, int32_t u, int32_t nu) {
    if (u >= nu) return 0;
    const int32_t named = iptr[u + 1] - iptr[u];
    return tc_heavy(u, named) ? (named + kTcUnit - 1) / kTcUnit : 0;
}

__global__ __launch_bounds__(256) void k_tc_unit_sums(const int32_t *__restrict__ iptr, int32_t nu, int32_t *sums) {
    __shared__ int32_t s_scan[256 / kWave + 1];
    int32_t all;
    (void)block_excl_scan<256>(tc_unit_count(iptr, blockIdx.x * 256 + threadIdx.x, nu), s_scan, &all);
    if (threadIdx.x == 0) sums[blockIdx.x] = all;
}

__global__ __launch_bounds__(256) void k_tc_units(const int32_t *__restrict__ iptr, int32_t nu,
                                                  const int32_t *__restrict__ sums, int32_t *count, int4 *lo, int4 *hi,
                                                  int32_t lo_cap, int32_t hi_cap) {
    __shared__ int32_t s_scan[256 / kWave + 1];
    const int32_t u = blockIdx.x * 256 + threadIdx.x;
    const bool low = u < kTcLow;
    int32_t before = 0, mine = tc_unit_count(iptr, u, nu), base, all;
    for (int32_t b = (low ? 0 : kTcLow / 256) + (int32_t)threadIdx.x; b < (int32_t)blockIdx.x; b += 256)
        before += sums[b];
    (void)block_excl_scan<256>(before, s_scan, &base);
    int32_t at = base + block_excl_scan<256>(mine, s_scan, &all);
    int4 *units = low ? lo : hi;
    const int32_t cap = low ? lo_cap : hi_cap;
    if (threadIdx.x == 0 && (u + 256 >= nu || u + 256 == kTcLow)) count[low ? 0 : 1] = base + all;
    if (mine == 0) return;
    const int32_t b = iptr[u], e = iptr[u + 1];
    for (int32_t k = 0; k < mine && at + k < cap; ++k)
        units[at + k] = make_int4(u, b + k * kTcUnit, min(e, b + (k + 1) * kTcUnit), 0);
}

// Triangles by their middle vertex.  A block takes a unit {u, entries naming
// u}: N(u) goes into the bitmap, and 16 lanes per entry (v, u) stream N(v)'s
// entries before u, four per lane and load (LO: 16-bit ids, 8 bytes a lane).
// Bound by reading those entries (each row comes from L2 or the Infinity
// Cache once per heavier neighbour); eight waves per SIMD and two loads a lane
// in flight cover the latency, and 256 threads with a 8 KB bitmap leave room
// for them.  PER: per-vertex counts; hits on w are counted at w's place in
// N(u) (s_first: the row position of a bitmap word's first entry) and added
// once per unit.
template <int BITS, bool LO, bool PER>
__global__ __launch_bounds__(256) void k_tc_heavy(const int32_t *__restrict__ orp,
                                                  const int32_t *__restrict__ oci,
                                                  const uint16_t *__restrict__ olo,
                                                  const int32_t *__restrict__ osrc,
                                                  const int2 *__restrict__ inl,
                                                  const int4 *__restrict__ units, int32_t nunits,
                                                  const int32_t *__restrict__ rank_old,
                                                  unsigned long long *total, unsigned long long *per,
                                                  unsigned long long *prof) {
    constexpr int kWords = BITS / 32;
    __shared__ uint32_t s_bits[kWords];
    __shared__ uint16_t s_first[PER ? kWords : 1];
    __shared__ uint32_t s_cnt[PER ? kTcPosCap : 1];
    __shared__ int2 s_in[256];
    __shared__ unsigned long long s_red[1];
    const int l = threadIdx.x % kTcLanes, grp = threadIdx.x / kTcLanes;
    unsigned long long hits = 0, tests = 0;
    for (int32_t i = threadIdx.x; i < kWords; i += 256) s_bits[i] = 0;
    for (int32_t k = blockIdx.x; k < nunits; k += gridDim.x) {
        const int4 unit = units[k];
        const int32_t ub = orp[unit.x], un = orp[unit.x + 1] - ub;
        const bool pos = PER && un <= kTcPosCap;
        __syncthreads();  // the bitmap is clear
        for (int32_t i = threadIdx.x; i < un; i += 256) {
            const int32_t w = oci[ub + i];
            atomicOr(&s_bits[w >> 5], 1u << (w & 31));
            if (PER && pos) {
                if (i == 0 || (oci[ub + i - 1] >> 5) != (w >> 5)) s_first[w >> 5] = (uint16_t)i;
                s_cnt[i] = 0;
            }
        }
        unsigned long long unit_hits = 0;
        for (int32_t j0 = unit.y; j0 < unit.z; j0 += 256) {
            const int32_t nin = min(256, unit.z - j0);
            if ((int32_t)threadIdx.x < nin) s_in[threadIdx.x] = inl[j0 + threadIdx.x];
            __syncthreads();
            for (int32_t q = grp; q < nin; q += 256 / kTcLanes) {
                const int2 in = s_in[q];
                const int32_t b = in.x, e = in.y;  // entries [b, e) of N(v)
                uint32_t found = 0;
                // one bit of the result per entry; entries outside [b, e) masked off
                auto test4 = [&](const uint4 &x, int32_t at) {
                    const uint32_t w4[4] = {x.x, x.y, x.z, x.w};
                    uint32_t bits[4], hit = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) bits[t] = s_bits[(w4[t] >> 5) & (kWords - 1)];
#pragma unroll
                    for (int t = 0; t < 4; ++t) hit |= ((bits[t] >> (w4[t] & 31)) & 1u) << t;
                    hit &= (0xfu >> max(0, at + 4 - e)) & (0xfu << max(0, b - at));
                    found += __popc(hit);
                    if (PER) {
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            if ((hit >> t) & 1u) {
                                const uint32_t w = LO ? w4[t] & 0xffffu : w4[t];
                                const int32_t p = s_first[w >> 5] + __popc(bits[t] & ((1u << (w & 31)) - 1u));
                                if (pos && p < kTcPosCap) atomicAdd(&s_cnt[p], 1u);
                                else atomicAdd(&per[rank_old[w]], 1ull);
                            }
                    }
                };
                auto load4 = [&](int32_t at) {  // LO: odd ids keep the next one above them (masked where used)
                    if (LO) {
                        const uint2 x = *reinterpret_cast<const uint2 *>(olo + at);
                        return make_uint4(x.x, x.x >> 16, x.y, x.y >> 16);
                    }
                    return *reinterpret_cast<const uint4 *>(oci + at);
                };
                for (int32_t at = (b & ~3) + 4 * l; at < e; at += 8 * kTcLanes) {
                    const int32_t at2 = at + 4 * kTcLanes < e ? at + 4 * kTcLanes : at;
                    const uint4 x = load4(at), y = load4(at2);
                    test4(x, at);
                    if (at2 != at) test4(y, at2);
                }
                if (prof && l == 0) tests += (unsigned long long)(LO ? (e - b + 1) / 2 : e - b);  // 4-byte words
                if (PER) {
                    uint32_t f = found;
                    for (int o = kTcLanes / 2; o > 0; o >>= 1) f += __shfl_xor(f, o, kWave);
                    if (l == 0 && f) atomicAdd(&per[rank_old[osrc[e]]], (unsigned long long)f);
                }
                unit_hits += found;
            }
            __syncthreads();
        }
        hits += unit_hits;
        if (PER) {
            unit_hits = wave_sum_u64(unit_hits);
            if (lane_id() == 0 && unit_hits) atomicAdd(&per[rank_old[unit.x]], unit_hits);
        }
        for (int32_t i = threadIdx.x; i < un; i += 256) {
            const int32_t w = oci[ub + i];
            s_bits[w >> 5] = 0;
            if (PER && pos && s_cnt[i]) atomicAdd(&per[rank_old[w]], (unsigned long long)s_cnt[i]);
        }
    }
    __syncthreads();
    block_add_u64<256>(hits, s_red, total);
    if (prof) {
        __syncthreads();
        block_add_u64<256>(tests, s_red, prof + 1);
    }
}

// Triangles whose middle vertex u has no bitmap: a wave takes kTcLightIds
// consecutive vertices, and 16 lanes per entry (v, u) that names one of them
// search the elements of the shorter of N(u) and N(v)'s entries before u in
// the longer.  Few entries and short lists, so it is a matter of latency: the
// first form, an entry per lane and 64 vertices per wave, left a few waves
// with thousands of dependent searches (rmat-22: 3.0 ms).
constexpr int32_t kTcLightIds = 16;

__global__ __launch_bounds__(256) void k_tc_light(const int32_t *__restrict__ orp,
                                                  const int32_t *__restrict__ oci,
                                                  const int32_t *__restrict__ osrc,
                                                  const int32_t *__restrict__ iptr,
                                                  const int2 *__restrict__ inl, int32_t n,
                                                  const int32_t *__restrict__ rank_old,
                                                  unsigned long long *total, unsigned long long *per,
                                                  unsigned long long *prof) {
    __shared__ unsigned long long s_red[1];
    const int lane = lane_id(), l = lane & 15, grp = lane >> 4;
    unsigned long long mine = 0, tests = 0;
    constexpr int64_t per_block = kTcLightIds * (256 / kWave);
    const int64_t stride = (int64_t)gridDim.x * per_block;
    for (int64_t u0 = (int64_t)blockIdx.x * per_block + (threadIdx.x / kWave) * kTcLightIds; u0 < n; u0 += stride) {
        // lane a (< kTcLightIds) holds vertex u0 + a: its row and where its entries begin and end
        // in the wave's list
        const int64_t uu = u0 + min(lane, kTcLightIds - 1);
        int32_t named = 0, ib = 0, lb = 0, le = 0;
        if (uu < n && lane < kTcLightIds) {
            ib = iptr[uu];
            named = iptr[uu + 1] - ib;
            lb = orp[uu];
            le = orp[uu + 1];
            if (tc_heavy((int32_t)uu, named) || le == lb) named = 0;
        }
        const int32_t incl = wave_incl_scan(named);
        const int32_t all = __builtin_amdgcn_readlane(incl, kWave - 1);
        for (int32_t k0 = 0; k0 < all; k0 += 4) {
            const int32_t k = k0 + grp;
            int32_t a = 0;  // the owner: vertices whose entries all lie before k
#pragma unroll
            for (int j = 0; j < kTcLightIds - 1; ++j) a += __builtin_amdgcn_readlane(incl, j) <= k;
            const int32_t end = __shfl(incl, a, kWave), cnt = __shfl(named, a, kWave);
            const int32_t first = __shfl(ib, a, kWave);
            int32_t lo = __shfl(lb, a, kWave), hi = __shfl(le, a, kWave);
            if (k < all) {
                const int2 in = inl[first + (k - (end - cnt))];
                int32_t sb = in.x, se = in.y;
                if (se - sb > hi - lo) {  // walk the shorter list
                    int32_t t = sb; sb = lo; lo = t;
                    t = se; se = hi; hi = t;
                }
                for (int32_t i = sb + l; i < se; i += 16) {
                    const int32_t w = oci[i];
                    const int32_t at = lower_bound(oci, lo, hi, w);
                    ++tests;
                    if (at < hi && oci[at] == w) {
                        ++mine;
                        if (per) {
                            atomicAdd(&per[rank_old[osrc[in.y]]], 1ull);
                            atomicAdd(&per[rank_old[u0 + a]], 1ull);
                            atomicAdd(&per[rank_old[w]], 1ull);
                        }
                    }
                }
            }
        }
    }
    block_add_u64<256>(mine, s_red, total);
    if (prof) {
        __syncthreads();
        block_add_u64<256>(tests, s_red, prof + 1);
    }
}

__global__ void k_tc_zero(unsigned long long *p, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Which graphs are counted by pairs rather than by bitmaps: flat ones (rows of
// at most kTcFlat entries); others without an index yet, that are small (entries
// x average row at most kTcSmall; a 32nd of it where the vertices' shares are
// counted too, an atomic for every triangle) or light (entries x longest row).
// First and later counts, us, by pairs and by bitmaps, and entries x average row:
//   uniform, 2^20 vertices, 16.8 M entries, rows to 41     1426  643    2506  804
//   uniform, 2^20 vertices, 33.5 M entries, rows to 63     4742 2360    4205 1493
//   road grid, 2.25 M vertices                              205   59    1290  112
//   uniform, 8,192 vertices, 0.5 M entries, rows to 96      250  110     426  135
//   uniform, 65,536 vertices, 4.2 M entries, rows to 108    660  458     658  221
//   rmat, 65,536 vertices, 0.25 M entries                   190   84     352   98   1.0 M
//   rmat, 32,768 vertices, 0.24 M entries                   198  103     329   98   1.8 M
//   rmat, 16,384 vertices, 0.23 M entries                   213  124     334   96   3.2 M
//   rmat, 262,144 vertices, 1.0 M entries                   396  194     548  105   4.0 M
//   rmat, 8,192 vertices, 0.20 M entries                    231  142     308   98   5.1 M
//   rmat, 131,072 vertices, 1.0 M entries                   414  233     470  110   7.6 M
//   rmat, 65,536 vertices, 1.8 M entries                    715  499     494  128    51 M
// and by vertex, later counts: 8,192 vertices, 31,000 entries 113 and 123 (0.11 M),
// 2,048 vertices, 26,000 entries 183 and 136 (0.32 M).
static bool tc_by_pairs(sp_graph g, bool per) {
    if (g->tc_mixed) return false;
    if (g->max_degree <= kTcFlat || g->tc_no_index) return true;
    if (g->tc_orp) return false;
    const int64_t spread = g->nnz * g->nnz / g->n;
    return per ? spread <= kTcSmall / 32 : spread <= kTcSmall || g->nnz * g->max_degree <= kTcLight;
}

bool tc_built(sp_graph g, bool per) {
    std::lock_guard<std::mutex> lk(g->mu);
    return (tc_by_pairs(g, per) ? g->tc_pair_orp : g->tc_orp) != nullptr;
}

static sp_status refuse_csr(sp_graph g, long long kept) {
    set_error("triangle counting needs a simple undirected CSR (%lld oriented entries of %lld)", kept,
              (long long)g->nnz);
    return SP_ERR_INVALID_ARGUMENT;
}

// The oriented rows of the pair route; *mixed (rows that are not ascending)
// leaves the graph to the bitmaps, whose rows are sorted.
static sp_status ensure_pairs(sp_graph g, bool *mixed, hipStream_t s) {
    *mixed = false;
    if (g->tc_pair_orp) return SP_OK;
    const int32_t n = g->n;
    const size_t vn = (size_t)std::max(n, 1), me = (size_t)g->nnz / 2;
    const int maxb = device_cu_count() * 8;
    int32_t *orp, *oci, *osrc, *tiles;
    unsigned long long *found;
    DevBlocks keep, work;
    keep.add(&orp, vn + 1);
    keep.add(&found, 2, true);  // right behind orp: both come back in one copy
    keep.add(&oci, me + 1);
    keep.add(&osrc, me + 1);
    work.add(&tiles, (size_t)scan_tiles((int64_t)vn));
    SP_TRY(keep.alloc());
    SP_TRY(work.alloc());
    const int32_t *rp = g->row_ptr, *ci = g->col_idx;
    hipLaunchKernelGGL(k_tc_zero, dim3(1), dim3(64), 0, s, found, (int64_t)2);
    const bool wide = g->max_degree > kTcFlat;  // a wave per row, else a lane
    const dim3 grid(grid_for(n, wide ? 4 : 256, maxb));
    if (n > 0)
        hipLaunchKernelGGL(wide ? k_tc_pair_len<kWave> : k_tc_pair_len<1>, grid, dim3(256), 0, s, rp, ci, n, orp, found);
    launch_excl_scan(orp, n, orp, tiles, s);
    SP_HIP(hipGetLastError());
    char back[512];  // from orp[n], at most 256 bytes before found
    const size_t to_found = (size_t)((char *)found - (char *)(orp + n));
    SP_HIP(hipMemcpyAsync(back, orp + n, to_found + 2 * sizeof(*found), hipMemcpyDeviceToHost, s));
    SP_HIP(hipStreamSynchronize(s));
    int32_t m;
    unsigned long long got[2];
    std::memcpy(&m, back, sizeof(m));
    std::memcpy(got, back + to_found, sizeof(got));
    if ((int64_t)m * 2 != g->nnz || (int64_t)got[0] * 2 != g->nnz) return refuse_csr(g, m);
    if (got[1]) {
        *mixed = true;
        return SP_OK;
    }
    if (m > 0)
        hipLaunchKernelGGL(wide ? k_tc_pair_fill<kWave> : k_tc_pair_fill<1>, grid, dim3(256), 0, s, rp, ci, n,
                           (const int32_t *)orp, oci, osrc);
    SP_HIP(hipGetLastError());
    SP_HIP(hipStreamSynchronize(s));
    g->bytes += keep.give_to(g->tc_blocks);
    g->tc_pair_oci = oci;
    g->tc_pair_osrc = osrc;
    g->tc_m = m;
    g->tc_pair_orp = orp;
    return SP_OK;
}

// The oriented rows and the index of the bitmap route.
static sp_status ensure_index(sp_graph g, hipStream_t s) {
    if (g->tc_orp) return SP_OK;
    SP_TRY(ensure_rank_locked(g, s));
    const int32_t n = g->n, heavy = rank_count(g, kRankExact);
    const int maxb = device_cu_count() * 8;
    const size_t vn = (size_t)std::max(n, 1);
    const int32_t *rp = g->row_ptr, *ci = g->col_idx, *rn = g->rank_new, *ro = g->rank_old;
    const int32_t nu = std::min(n, kTcBits);
    int32_t *orp, *oci, *osrc, *iptr, *tiles, *big, *slot;
    uint16_t *olo;
    int2 *inl;
    int4 *units;
    unsigned long long *ctl;  // [0] entries that rise in (degree, id) order, [1] rows over 64, [2] units by list
    // Kept arrays and scratch, one block each, for half the graph's entries.
    const size_t me = (size_t)g->nnz / 2 + 1, padded = me + 8;  // 4-entry loads may run past the last row
    // units: one per kTcUnit entries, and a last one for each vertex that 8 entries or more name
    const int32_t lows = std::min(nu, kTcLow), rest = (int32_t)std::min<int64_t>(nu, (int64_t)me / 8);
    const int32_t lo_cap = (int32_t)(me / kTcUnit) + std::min(lows, rest) + 1;
    const int32_t hi_cap = nu > lows ? (int32_t)(me / kTcUnit) + std::min(nu - lows, rest) + 1 : 0;
    DevBlocks keep, work;
    keep.add(&orp, vn + 1);
    keep.add(&ctl, 3, true);  // right behind orp: both come back in one copy
    keep.add(&iptr, vn + 1);
    keep.add(&oci, padded);
    keep.add(&olo, padded);
    keep.add(&osrc, me);
    keep.add(&inl, me);
    keep.add(&units, (size_t)lo_cap + (size_t)hi_cap);
    work.add(&tiles, (size_t)scan_tiles((int64_t)vn));
    work.add(&big, vn);
    work.add(&slot, me);
    SP_TRY(keep.alloc());
    SP_TRY(work.alloc());
    hipLaunchKernelGGL(k_tc_zero, dim3(1), dim3(64), 0, s, ctl, (int64_t)3);
    const int row_grid = grid_for((int64_t)n - heavy, 16, maxb);
    if (n > 0) {
        if (heavy)
            hipLaunchKernelGGL(k_tc_outdeg<true>, dim3(std::min(heavy, maxb)), dim3(256), 0, s, rp, ci, rn, ro, 0,
                               heavy, heavy, orp, iptr, ctl);
        hipLaunchKernelGGL(k_tc_outdeg<false>, dim3(row_grid), dim3(256), 0, s, rp, ci, rn, ro, heavy, n, heavy,
                           orp, iptr, ctl);
    }
    launch_excl_scan(orp, n, orp, tiles, s);
    SP_HIP(hipGetLastError());
    char back[512];  // from orp[n], at most 256 bytes before ctl
    const size_t to_ctl = (size_t)((char *)ctl - (char *)(orp + n));
    SP_HIP(hipMemcpyAsync(back, orp + n, to_ctl + sizeof(*ctl), hipMemcpyDeviceToHost, s));
    SP_HIP(hipStreamSynchronize(s));
    int32_t m;
    unsigned long long exact;
    std::memcpy(&m, back, sizeof(m));
    std::memcpy(&exact, back + to_ctl, sizeof(exact));
    if ((int64_t)exact * 2 != g->nnz || (int64_t)m * 2 != g->nnz) {
        // a simple symmetric graph orients exactly one entry of each pair, in either order
        return refuse_csr(g, (long long)exact);
    }
    const int ent_grid = grid_for(m, 256, 2 * maxb);
    int32_t un[2] = {0, 0};
    if (n > 0) {
        if (heavy)
            hipLaunchKernelGGL(k_tc_fill<true>, dim3(std::min(heavy, maxb)), dim3(256), 0, s, rp, ci, rn, ro, 0,
                               heavy, (const int32_t *)orp, oci, osrc);
        hipLaunchKernelGGL(k_tc_fill<false>, dim3(row_grid), dim3(256), 0, s, rp, ci, rn, ro, heavy, n,
                           (const int32_t *)orp, oci, osrc);
        int32_t *nbig = (int32_t *)(ctl + 1);
        int32_t share = 4;
        while (share < kWave && (int64_t)share * (256 / kWave) * maxb < n) share *= 2;
        hipLaunchKernelGGL(k_tc_sort_small, dim3(grid_for(n, 256 / kWave * share, maxb)), dim3(256), 0, s,
                           (const int32_t *)orp, n, share, oci, big, nbig);
        hipLaunchKernelGGL(k_tc_sort_bits<kTcLow / 32>, dim3(maxb), dim3(256), 0, s, (const int32_t *)orp, oci,
                           (const int32_t *)big, (const int32_t *)nbig, 0, kTcLow);
        if (n > kTcLow)
            hipLaunchKernelGGL(k_tc_sort_bits<kTcSortBits / 32>, dim3(maxb), dim3(256), 0, s, (const int32_t *)orp,
                               oci, (const int32_t *)big, (const int32_t *)nbig, kTcLow, kTcSortBits);
        if (n > kTcSortBits)
            hipLaunchKernelGGL(k_tc_sort_net, dim3(maxb), dim3(256), 0, s, (const int32_t *)orp, oci,
                               (const int32_t *)big, (const int32_t *)nbig, kTcSortBits);
        int32_t tile = kTcNamedLeast;
        while (tile < kTcNamedTile && (int64_t)tile * device_cu_count() < m) tile *= 2;
        hipLaunchKernelGGL(k_tc_named, dim3(grid_for(m, tile, maxb)), dim3(256), 0, s, (const int32_t *)oci,
                           (int64_t)m, tile, olo, iptr, slot);
        launch_excl_scan(iptr, n, iptr, tiles, s);
        hipLaunchKernelGGL(k_tc_inlist, dim3(ent_grid), dim3(256), 0, s, (const int32_t *)oci, (const int32_t *)osrc,
                           (const int32_t *)orp, (const int32_t *)iptr, (const int32_t *)slot, (int64_t)m, inl);
        int32_t *count = (int32_t *)(ctl + 2);
        const int32_t blocks = (nu + 255) / 256;  // at most `big`'s length; the row list is done with
        hipLaunchKernelGGL(k_tc_unit_sums, dim3(blocks), dim3(256), 0, s, (const int32_t *)iptr, nu, big);
        hipLaunchKernelGGL(k_tc_units, dim3(blocks), dim3(256), 0, s, (const int32_t *)iptr, nu, (const int32_t *)big,
                           count, units, units + lo_cap, lo_cap, hi_cap);
        SP_HIP(hipGetLastError());
        SP_HIP(hipMemcpyAsync(un, count, sizeof(un), hipMemcpyDeviceToHost, s));
    }
    SP_HIP(hipStreamSynchronize(s));
    g->bytes += keep.give_to(g->tc_blocks);
    g->tc_oci = oci;
    g->tc_olo = olo;
    g->tc_osrc = osrc;
    g->tc_iptr = iptr;
    g->tc_inl = inl;
    g->tc_units = units;
    g->tc_units_hi = units + lo_cap;
    g->tc_units_n[0] = std::min(un[0], lo_cap);
    g->tc_units_n[1] = std::min(un[1], hi_cap);
    g->tc_m = m;
    g->tc_orp = orp;
    return SP_OK;
}

sp_status ensure_oriented(sp_graph g, bool per, hipStream_t s) {
    std::lock_guard<std::mutex> lk(g->mu);
    if (tc_by_pairs(g, per)) {
        SP_TRY(ensure_pairs(g, &g->tc_mixed, s));
        if (!g->tc_mixed) return SP_OK;
    }
    sp_status st = ensure_index(g, s);
    if (st == SP_ERR_OUT_OF_MEMORY && !g->tc_mixed) {  // pairs take less than half of the memory
        clear_error();
        SP_TRY(ensure_pairs(g, &g->tc_mixed, s));
        if (g->tc_mixed) return ensure_index(g, s);
        g->tc_no_index = true;
        return SP_OK;
    }
    return st;
}

template <bool PER>
static void launch_tc_count(sp_graph g, unsigned long long *d_total, unsigned long long *per, hipStream_t s) {
    const int maxb = device_cu_count() * 8;
    unsigned long long *prof = prof_counters(P_TC_COUNT);
    const int32_t lo = g->tc_units_n[0], hi = g->tc_units_n[1];
    auto heavy = [&](auto kernel, const int4 *units, int32_t count) {
        hipLaunchKernelGGL(kernel, dim3(std::min(count, maxb)), dim3(256), 0, s, (const int32_t *)g->tc_orp,
                           (const int32_t *)g->tc_oci, (const uint16_t *)g->tc_olo, (const int32_t *)g->tc_osrc,
                           (const int2 *)g->tc_inl, units, count, (const int32_t *)g->rank_old, d_total, per, prof);
    };
    if (lo > 0) heavy(k_tc_heavy<kTcLow, true, PER>, g->tc_units, lo);
    if (hi > 0) heavy(k_tc_heavy<kTcBits, false, PER>, g->tc_units_hi, hi);
    hipLaunchKernelGGL(k_tc_light, dim3(grid_for(g->n, kTcLightIds * (256 / kWave), 2 * maxb)), dim3(256), 0, s, (const int32_t *)g->tc_orp,
                       (const int32_t *)g->tc_oci, (const int32_t *)g->tc_osrc, (const int32_t *)g->tc_iptr,
                       (const int2 *)g->tc_inl, g->n, (const int32_t *)g->rank_old, d_total, per, prof);
}

sp_status tc_run(sp_graph g, unsigned long long *d_total, unsigned long long *per, hipStream_t s) {
    hipLaunchKernelGGL(k_tc_zero, dim3(1), dim3(64), 0, s, d_total, (int64_t)1);
    if (per) hipLaunchKernelGGL(k_tc_zero, dim3(grid_for(g->n, 256, 4096)), dim3(256), 0, s, per, (int64_t)g->n);
    bool pairs;
    {
        std::lock_guard<std::mutex> lk(g->mu);
        pairs = tc_by_pairs(g, per != nullptr) && g->tc_pair_orp;
    }
    if (g->tc_m > 0) {
        ProfScope ps(P_TC_COUNT, s);
        if (pairs)
            hipLaunchKernelGGL(k_tc_pairs, dim3(grid_for(g->tc_m, 256, device_cu_count() * 8)), dim3(256), 0, s,
                               (const int32_t *)g->tc_pair_orp, (const int32_t *)g->tc_pair_oci,
                               (const int32_t *)g->tc_pair_osrc, (int64_t)g->tc_m, d_total, per,
                               prof_counters(P_TC_COUNT));
        else if (per) launch_tc_count<true>(g, d_total, per, s);
        else launch_tc_count<false>(g, d_total, nullptr, s);
    }
    SP_HIP(hipGetLastError());
    return SP_OK;
}

}  // namespace sp
