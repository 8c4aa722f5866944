// Batched BC with one workgroup per source ("workgroup engine"), for graphs
// of many short levels (road-like: no vertex of degree above kExpandDeg).
//
// The arithmetic is Brandes' per source (paper Appendix, Fig. "BC computation
// in StarPlat"; DAG semantics of Section 2.3.2), as on the per-source path:
//   sigma(w) = sum over parents u (incoming row, CSR order) of sigma(u),
//   delta(v) = sum over children w (outgoing row, CSR order) of
//              (sigma(v) / sigma(w)) * (1 + delta(w))
// (rows through the CSR offsets), or, regrouped as in the bitmap engine,
//   delta(v) = sigma(v) * sum over children w of rho(w),
//   rho(w) = (1 + delta(w)) / sigma(w)
// (fixed-width rows, below).
// What differs is the schedule.  On a road-like graph a source's BFS has
// thousands of levels of a few hundred vertices each; the bitmap engine runs
// the batch's sources in lockstep, one kernel per level for the whole batch,
// and each level pays the kernel's chain of dependent memory round trips and
// its grid-wide close.  Here each source's whole pass (forward levels, then
// reverse levels) runs inside one workgroup, the level barrier is the
// workgroup barrier, and the new frontier is appended with an LDS counter:
// the batch's sources advance independently, each on its own CU.
// (One thread block per source is the coarse-grained schedule of McLaughlin
// and Bader, "Scalable and high performance betweenness centrality on the
// GPU", SC 2014.)
//
// Layout, per slot s (source-major): a 16-byte record rec[s*V + v] = {level
// (-1: unreached), value}, delta[s*V + v], the BFS-order queue
// queue[s*V + i] and the level offsets loff[s*(V+2) + l] -- 32 bytes per
// vertex and slot.  Records are filled with level -1 before each pass; every
// other field is written before it is read.  The value is sigma after the
// forward pass; the fixed-width kernel replaces it by rho once the reverse
// pass has finished the vertex, so a neighbour costs one 16-byte load (level
// and value together).  sigma itself is written out only for sp_batch_levels
// (straight into the caller's array).
// BC: for each vertex, the slots' delta in ascending slot order, skipping
// unreached vertices and the vertex's own source (level <= 0).
//
// Only the slot's own workgroup touches its arrays during the pass, so the
// claim on a level is a workgroup-scope compare-and-swap.  The CSR-offset
// kernel reads levels another wave may have claimed with workgroup-scope
// atomic loads; the fixed-width kernels read them with plain loads after the
// level barrier.  Everything else is written with plain stores by waves of
// the same workgroup and read after a barrier.
//
// Memory-level parallelism: a thread takes kEntries queue entries at once
// and walks their rows kRowStep entries at a time; for all of them the
// column ids, then the neighbours' levels, then their values (or claims) are
// each issued together, so one step of a level costs a few dependent round
// trips for kEntries x kRowStep adjacency entries.  Sums still run in CSR
// order per vertex.
//
// Fixed-width rows: on a graph whose rows hold at most 8 entries the rows
// are copied once into a fixed-width layout (W = 4 or 8 ids per vertex, -1
// padding), so a vertex's neighbours come in one load instead of an offset
// load followed by an id load.  A discovery step is then queue entry -> row
// -> claim, a path-count step queue entry -> row -> the neighbours' records,
// and a reverse step queue entry -> row (and the vertex's own record) -> the
// neighbours' records; the record of a neighbour that turns out not to be a
// parent (child) is loaded and dropped.  That is k_wg_bc_ell, for directed
// graphs and for rows that are not symmetric; symmetric rows take k_wg_bc_mesh,
// whose levels stay in LDS.
#include "common.h"
#include "devutil.h"

namespace sp {

constexpr int kRowStep = 4;   // row entries per step (road-like rows hold at most 4)
constexpr int kEntries = 4;   // queue entries a thread works on at once

// Rows of the (up to) kEntries queue entries i0, i0 + BS, ... below `end`:
// [b[u], e[u]) in the rows `rows`; returns the longest row's length.
template <int BS>
__device__ __forceinline__ int32_t rows_of_bs(const int32_t *queue, int32_t i0, int32_t end,
                                              const int32_t *__restrict__ rows, int32_t *b, int32_t *e) {
    int32_t v[kEntries];
#pragma unroll
    for (int u = 0; u < kEntries; ++u) v[u] = i0 + u * BS < end ? queue[i0 + u * BS] : -1;
    int32_t len = 0;
#pragma unroll
    for (int u = 0; u < kEntries; ++u) {
        b[u] = v[u] >= 0 ? rows[v[u]] : 0;
        e[u] = v[u] >= 0 ? rows[v[u] + 1] : 0;
        len = max(len, e[u] - b[u]);
    }
    return len;
}

__device__ __forceinline__ int32_t ld_level(const int32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// dist -1 -> lvl; returns the value found (-1 when this call claimed it).
__device__ __forceinline__ int32_t claim_level(int32_t *p, int32_t lvl) {
    int32_t expected = -1;
    __hip_atomic_compare_exchange_strong(p, &expected, lvl, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    return expected;
}

__global__ void k_wg_fill(WgRec *rec, int64_t count) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride)
        reinterpret_cast<int4 *>(rec + i)[0] = make_int4(-1, 0, 0, 0);  // level and value
}

// Fixed-width copy of the rows: ell[v * W + k] = k-th neighbour, -1 past the
// row's end (every row holds at most W entries).
template <int W>
__global__ void k_wg_ell(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, int32_t n,
                         int32_t *ell) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const int32_t b = rp[v], d = rp[v + 1] - b;
#pragma unroll
        for (int k = 0; k < W; ++k) ell[v * W + k] = k < d ? ci[b + k] : -1;
    }
}

// Whether the rows are symmetric: every u occurs in v's row as often as v in
// u's; *not_sym is set where they are not.  k_wg_bc_mesh needs it, and uploads do
// not check it.
template <int W>
__global__ void k_wg_symmetric(const int32_t *__restrict__ ell, int32_t n, int32_t *not_sym) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        int32_t x[W];
#pragma unroll
        for (int k = 0; k < W; ++k) x[k] = ell[v * W + k];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            if (x[k] < 0) continue;
            int32_t here = 0, there = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                here += x[q] == x[k];
                there += ell[(int64_t)x[k] * W + q] == (int32_t)v;
            }
            bad |= here != there;
        }
    }
    if (__ballot(bad) && lane_id() == 0) atomicOr(not_sym, 1);
}

// The loads below are issued unconditionally, from a valid address (row 0,
// vertex 0) when there is nothing to read, and their results dropped: a load
// under a branch of its own is waited for before the branch closes, which
// would turn a group of independent loads into a chain of round trips.

// queue[i] for i < end, else -1 (i < end for some lane of the call, end > 0).
__device__ __forceinline__ int32_t at_or_none(const int32_t *queue, int32_t i, int32_t end) {
    const int32_t x = queue[min(i, end - 1)];
    return i < end ? x : -1;
}

// Level barrier of the fixed-width kernels.  One workgroup's waves share their
// CU's L1, which stores and atomics keep up to date: the barrier orders all.
// (An agent-scope acquire here invalidated the L1 and the XCD's L2 at every
// level of every workgroup: a third of the whole pass.)
__device__ __forceinline__ void sync_records() {
    __syncthreads();
}

// A record in one 16-byte load (the empty asm marks the pad word used, so
// the load is not narrowed into a 4-byte and an 8-byte one: two requests).
__device__ __forceinline__ WgRec load_rec(const WgRec *p) {
    int4 x = *reinterpret_cast<const int4 *>(p);
    asm("" : "+v"(x.y));
    WgRec r;
    r.dist = x.x;
    r.pad = x.y;
    r.val = __hiloint2double(x.w, x.z);
    return r;
}

// Append x to the queue where `take` holds: one LDS add per wave reserves
// the wave's entries, lanes in lane order.
__device__ __forceinline__ void append_wave(bool take, int32_t x, int32_t *queue, int32_t *s_tail) {
    const unsigned long long bal = __ballot(take);
    if (!bal) return;
    const int first = __ffsll((long long)bal) - 1;
    int32_t at = 0;
    if (lane_id() == first) at = atomicAdd(s_tail, __popcll(bal));  // LDS
    at = __shfl(at, first, kWave);
    const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    if (take) queue[at + r] = x;
}

// Row of v in the fixed-width layout (v < 0: an empty row).
template <int W>
__device__ __forceinline__ void ell_row(const int32_t *__restrict__ ell, int32_t v, int32_t (&nb)[W]) {
    const int4 *r = reinterpret_cast<const int4 *>(ell + (int64_t)max(v, 0) * W);
#pragma unroll
    for (int q = 0; q < W / 4; ++q) {
        const int4 x = r[q];
        nb[4 * q + 0] = v >= 0 ? x.x : -1;
        nb[4 * q + 1] = v >= 0 ? x.y : -1;
        nb[4 * q + 2] = v >= 0 ? x.z : -1;
        nb[4 * q + 3] = v >= 0 ? x.w : -1;
    }
}

// k_wg_bc over fixed-width rows (see the latency note above): the same sums
// in the same order.
template <int BS, int W>
__global__ __launch_bounds__(BS) void k_wg_bc_ell(const int32_t *__restrict__ ell,
                                                  const int32_t *__restrict__ ell_in,
                                                  const int32_t *__restrict__ slot_src, int32_t n,
                                                  WgRec *rec_all, double *delta_all, double *sigma_out,
                                                  int32_t *queue_all, int32_t *loff_all, WgSlotResult *res,
                                                  unsigned long long *prof) {
    constexpr int E = W == 8 ? 2 : kEntries;  // entries in flight per thread (registers)
    const int32_t slot = blockIdx.x;
    const int64_t base = (int64_t)slot * n;
    WgRec *rec = rec_all + base;
    double *delta = delta_all + base;
    double *sig_out = sigma_out ? sigma_out + base : nullptr;  // sp_batch_levels' sigma
    int32_t *queue = queue_all + base;
    int32_t *loff = loff_all + (int64_t)slot * ((int64_t)n + 2);
    const int32_t src = slot_src[slot];
    __shared__ int32_t s_tail, s_flag;
    __shared__ double s_max[BS / kWave];
    __shared__ unsigned long long s_red[1];
    if (threadIdx.x == 0) {
        rec[src].dist = 0;
        rec[src].val = 1.0;
        if (sig_out) sig_out[src] = 1.0;
        queue[0] = src;
        loff[0] = 0;
        loff[1] = 1;
        s_tail = 1;
        s_flag = 0;
    }
    sync_records();
    int32_t lo = 0, hi = 1, level = 0;
    double my_max = 1.0;
    unsigned long long my_edges = 0, my_pairs = 0;
    for (;;) {
        // Discovery of level + 1 from the frontier [lo, hi): the claim
        // (dist -1 -> level + 1) decides who appends the vertex; a wave
        // reserves its appends with one LDS add.
        for (int32_t i0 = lo + (int32_t)threadIdx.x; i0 < hi; i0 += BS * E) {
            int32_t v[E], nb[E][W], old[E][W];
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = at_or_none(queue, i0 + u * BS, hi);
#pragma unroll
            for (int u = 0; u < E; ++u) ell_row<W>(ell, v[u], nb[u]);
#pragma unroll
            for (int u = 0; u < E; ++u)
#pragma unroll
                for (int k = 0; k < W; ++k) old[u][k] = nb[u][k] >= 0 ? claim_level(&rec[nb[u][k]].dist, level + 1) : 0;
#pragma unroll
            for (int u = 0; u < E; ++u)
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    if (nb[u][k] >= 0) ++my_edges;
                    append_wave(nb[u][k] >= 0 && old[u][k] == -1, nb[u][k], queue, &s_tail);
                }
        }
        sync_records();
        const int32_t tail = s_tail;
        if (tail == hi) break;  // block-uniform: every thread read the same tail
        // Path counts of the new vertices [hi, tail): parents over incoming
        // rows, added in row order; one record load per neighbour.
        for (int32_t j0 = hi + (int32_t)threadIdx.x; j0 < tail; j0 += BS * E) {
            int32_t w[E], p[E][W];
            WgRec r[E][W];
#pragma unroll
            for (int u = 0; u < E; ++u) w[u] = at_or_none(queue, j0 + u * BS, tail);
#pragma unroll
            for (int u = 0; u < E; ++u) ell_row<W>(ell_in, w[u], p[u]);
#pragma unroll
            for (int u = 0; u < E; ++u)
#pragma unroll
                for (int k = 0; k < W; ++k) r[u][k] = load_rec(&rec[max(p[u][k], 0)]);
#pragma unroll
            for (int u = 0; u < E; ++u) {
                double acc = 0.0;
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (p[u][k] >= 0 && r[u][k].dist == level) {
                        acc += r[u][k].val;
                        ++my_pairs;
                    }
                if (w[u] >= 0) {
                    rec[w[u]].val = acc;
                    if (sig_out) sig_out[w[u]] = acc;
                    my_max = fmax(my_max, acc);
                    if (sigma_is_large(acc)) s_flag = 1;
                }
            }
        }
        if (threadIdx.x == 0) loff[level + 2] = tail;
        sync_records();
        lo = hi;
        hi = tail;
        ++level;
    }
    // Reverse sweep from the deepest level up to level 1 (the deepest has no
    // children: its delta is 0); children over outgoing rows, in row order.
    // A finished vertex's record holds rho = (1 + delta) / sigma, so a parent
    // reads one record per neighbour: delta(v) = sigma(v) * sum of its
    // children's rho (the regrouping of the bitmap engine).
    for (int32_t l = level; l >= 1; --l) {
        const int32_t a = loff[l], z = loff[l + 1];
        for (int32_t j0 = a + (int32_t)threadIdx.x; j0 < z; j0 += BS * E) {
            int32_t v[E], nb[E][W];
            double sv[E];
            WgRec r[E][W];
#pragma unroll
            for (int u = 0; u < E; ++u) v[u] = at_or_none(queue, j0 + u * BS, z);
#pragma unroll
            for (int u = 0; u < E; ++u) {
                ell_row<W>(ell, v[u], nb[u]);
                sv[u] = rec[max(v[u], 0)].val;  // sigma(v)
            }
#pragma unroll
            for (int u = 0; u < E; ++u)
#pragma unroll
                for (int k = 0; k < W; ++k) r[u][k] = load_rec(&rec[max(nb[u][k], 0)]);
#pragma unroll
            for (int u = 0; u < E; ++u) {
                double acc = 0.0;
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (nb[u][k] >= 0 && r[u][k].dist == l + 1) {
                        acc += r[u][k].val;
                        ++my_pairs;
                    }
                if (v[u] >= 0) {
                    const double dv = sv[u] * acc;
                    delta[v[u]] = dv;
                    rec[v[u]].val = (1.0 + dv) / sv[u];
                }
            }
        }
        sync_records();
    }
    my_max = wave_max_f64(my_max);
    if (lane_id() == 0) s_max[threadIdx.x / kWave] = my_max;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int w = 0; w < BS / kWave; ++w) m = fmax(m, s_max[w]);
        res[slot] = WgSlotResult{level + 1, hi, m, s_flag};
    }
    if (prof) {
        __syncthreads();
        block_add_u64<BS>(threadIdx.x == 0 ? (unsigned long long)hi : 0ull, s_red, prof + 0);
        __syncthreads();
        block_add_u64<BS>(my_edges, s_red, prof + 1);
        __syncthreads();
        block_add_u64<BS>(my_pairs, s_red, prof + 2);
    }
}

// The pass over symmetric fixed-width rows (k_wg_symmetric).  Everything a level
// needs of the one before stays in LDS: a frontier entry holds its vertex, its
// path count and its row, with the parent that claimed it marked there; a
// finished entry of the reverse sweep its rho, by position in the level.  In
// memory there are, per vertex, its position in BFS order (pos; -1 unreached)
// and, per position, the vertex (queue), the path count (sig) and a link to the
// children.
//
// Forward, a level is one round trip: the rows of an entry's neighbours but the
// parent and, in the same breath, the positions of those that may be reached
// already.  A neighbour of a vertex lies at most a level away (the rows being
// symmetric: a vertex claimed again would run the positions past n), so these are the
// ones whose hash is in the filter of this level or the one before (s_seen), one
// in ten on a road grid.  An unreached one is claimed in an LDS hash table (by
// compare-and-swap on pos, to -2, if its place there is crowded or the level is
// past kMeshCap): an atomic on memory is performed behind the L2, and at four a vertex they alone moved
// 70 GB of the pass.  A claimed vertex takes the claimer's path count.  A child
// that another entry claimed too is marked by its hash (s_shared), and adds its
// parents' counts up in row order when its own turn comes, its row's positions
// having been loaded with its neighbours' rows; a mark met by chance only adds
// up a single parent.
//
// The children a vertex claimed have consecutive positions, in row order: link
// holds the first (relative to its level), a bit per claimed neighbour, and
// whether others claimed some.  The reverse sweep therefore reads queue, sig and
// link in order, three levels ahead of use; the vertices with shared children
// (8 in a hundred) have their rows, then their row's positions, loaded in the
// two levels between.
//
// Sums run in row order on every path, whoever claimed a vertex: the same bits.
// Entries of a level past kMeshCap live in memory only.
//
// What bounds it: on the largest grids the one CU a source has -- per level of
// 1,400 entries some 5,000 lines in and out of its L1 -- and on small ones the
// instructions of one wave's turn (2 us a level forward, 1.4 in reverse).
// Spanning tree and 2% more of a grid, blocks of 1,024, 64 sources (300 x 300:
// 16), whole call:
//   grid                                           300    512   1000   2048
//   a record per vertex, claimed by atomics, an
//   invalidation after each level                                   168 ms
//   levels in LDS, positions                                           125
//   without the invalidation                                            95
//   atomics on the neighbours in question only     3.7    7.7   19.5    61
//   claims in LDS                                  3.8    7.7   17.9    54
//   shared children in their own turn, the reverse
//   sweep's loads three levels ahead               3.4    6.6   15.9  53.5
//   the filter                                     3.6    6.9   15.6  51.3
// (a table of each level's positions in LDS in place of pos, forward: 5.0, 9.5,
// 21.3 and 73.7 ms -- more instructions than the round trip it saves; two
// entries in flight per thread: 3.7, 7.1, 16.9 and 56.7.)
constexpr int kMeshTable = 4096;   // entries of the claims' hash table
constexpr int kMeshProbes = 64;    // a key lies this close behind its hash, or not in the table
constexpr int kMeshSeen = 32768;   // bits of a level's filter
constexpr int kMeshOffsets = 4096;  // level offsets held in LDS by the reverse sweep
constexpr uint32_t kLinkSlow = 1u << 24;
template <int W>
constexpr int kMeshCap = W == 4 ? 2048 : 1024;  // entries of a level held in LDS

// Workgroup barrier that orders LDS only: stores to memory stay in flight.
__device__ __forceinline__ void sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint32_t mesh_hash(int32_t v) { return (uint32_t)v * 0x9E3779B1u >> 16; }

template <int BS, int W>
__global__ __launch_bounds__(BS) void k_wg_bc_mesh(const int32_t *__restrict__ ell,
                                                   const int32_t *__restrict__ slot_src, int32_t n,
                                                   int32_t *pos_all, uint32_t *link_all, double *sig_all,
                                                   double *delta_all, double *sigma_out, int32_t *queue_all,
                                                   int32_t *loff_all, WgSlotResult *res,
                                                   unsigned long long *prof) {
    constexpr int kCap = kMeshCap<W>;
    struct Row {
        int32_t x[W];
    };
    __shared__ __attribute__((aligned(16))) int32_t s_key[kMeshTable];  // claimed for the next level; -1 empty
    __shared__ uint32_t s_seen[3][kMeshSeen / 32];  // hashes of a level's vertices
    __shared__ uint32_t s_shared[2][kMeshTable / 32];  // hashes of a level's vertices with several parents
    __shared__ __attribute__((aligned(16))) Row s_row[2][kCap];  // the parent that claimed the entry: -2 - parent
    __shared__ int32_t s_v[2][kCap];
    __shared__ double s_val[3][kCap];  // sigma forward, rho in reverse
    __shared__ int32_t s_tail, s_flag;
    __shared__ double s_max[BS / kWave];
    __shared__ unsigned long long s_red[1];
    const int32_t slot = blockIdx.x, tid = threadIdx.x;
    const int64_t base = (int64_t)slot * n;
    int32_t *pos = pos_all + base;
    uint32_t *link = link_all + base;
    double *sig = sig_all + base;
    double *delta = delta_all + base;
    double *sig_out = sigma_out ? sigma_out + base : nullptr;  // sp_batch_levels' sigma
    int32_t *queue = queue_all + base;
    int32_t *loff = loff_all + (int64_t)slot * ((int64_t)n + 2);
    const int32_t src = slot_src[slot];
    const int lane = lane_id(), wave0 = tid - lane;

    auto row_of = [&](int32_t v) {
        Row r;
        const int4 *p = reinterpret_cast<const int4 *>(ell + (int64_t)v * W);
#pragma unroll
        for (int q = 0; q < W / 4; ++q) {
            const int4 y = p[q];
            r.x[4 * q] = y.x, r.x[4 * q + 1] = y.y, r.x[4 * q + 2] = y.z, r.x[4 * q + 3] = y.w;
        }
        return r;
    };
    for (int32_t i = 4 * tid; i < kMeshTable; i += 4 * BS)
        *reinterpret_cast<int4 *>(&s_key[i]) = make_int4(-1, -1, -1, -1);
    for (int32_t i = tid; i < kMeshTable / 32; i += BS) s_shared[0][i] = s_shared[1][i] = 0;
    for (int32_t i = tid; i < kMeshSeen / 32; i += BS) s_seen[0][i] = s_seen[1][i] = s_seen[2][i] = 0;
    __syncthreads();
    if (tid == 0) {
        const uint32_t h = mesh_hash(src) & (kMeshSeen - 1);
        s_seen[0][h >> 5] = 1u << (h & 31);
        pos[src] = 0;
        loff[0] = 0;
        loff[1] = 1;
        s_v[0][0] = src;
        s_val[0][0] = 1.0;
        s_row[0][0] = row_of(src);
        s_tail = 1;
        s_flag = 0;
    }
    __syncthreads();

    // Forward.
    struct Entry {
        int32_t v;
        double sv;
        Row row, at;         // neighbours and their positions
        Row next[W == 4 ? W : 1];  // the neighbours' rows
        bool shared;         // several parents
    };
    int32_t plo = 0, lo = 0, hi = 1, level = 0, t = 0, mask = 63;  // t: level % 3
    double my_max = 1.0;
    unsigned long long my_edges = 0, my_pairs = 0;
    auto fetch = [&](Entry &e, int32_t k) {  // entry k of the level
        if (lo + k >= hi) return;
        const int tp = t == 0 ? 2 : t - 1;
        if (k < kCap) {
            e.v = s_v[level & 1][k];
            e.sv = s_val[t][k];
            e.row = s_row[level & 1][k];
        } else {
            e.v = queue[lo + k];
            e.sv = sig[lo + k];
            e.row = row_of(e.v);
        }
        const uint32_t h = mesh_hash(e.v) & (kMeshTable - 1);
        e.shared = (s_shared[level & 1][h >> 5] >> (h & 31)) & 1u;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            int32_t u = e.row.x[q];
            e.at.x[q] = -2;
            my_edges += u != -1;
            if (u < -1 && e.shared) u = -2 - u;
            if (u >= 0) {
                const uint32_t g = mesh_hash(u) & (kMeshSeen - 1);
                if (((s_seen[tp][g >> 5] | s_seen[t][g >> 5]) >> (g & 31)) & 1u) e.at.x[q] = pos[u];
                else e.at.x[q] = -1;
                if (W == 4) e.next[q % (W == 4 ? W : 1)] = row_of(u);
            }
        }
    };
    Entry e;
    fetch(e, tid);
    for (;;) {
        const int tp = t == 0 ? 2 : t - 1, tn = t == 2 ? 0 : t + 1, nx = (level + 1) & 1;
        const int probes = hi - lo <= kCap ? kMeshProbes : 0;
        auto process = [&](Entry &x, int32_t k) {
            const int32_t i = lo + k;
            const bool has = i < hi;
            uint32_t claimed = 0, shared = 0;
            if (has) {
                if (x.shared) {
                    double acc = 0.0;
#pragma unroll
                    for (int q = 0; q < W; ++q) {
                        const int32_t p = x.at.x[q];
                        if (p >= plo && p < lo) acc += p - plo < kCap ? s_val[tp][p - plo] : sig[p];
                    }
                    x.sv = acc;
                    if (k < kCap) s_val[t][k] = acc;
                    my_max = fmax(my_max, acc);
                    if (sigma_is_large(acc)) s_flag = 1;
                }
                queue[i] = x.v;
                sig[i] = x.sv;
                if (sig_out) sig_out[x.v] = x.sv;
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const int32_t u = x.row.x[q];
                    int32_t found = x.at.x[q];
                    if (found == -1) {
                        uint32_t h = mesh_hash(u);
                        for (int step = 0;; ++step, ++h) {
                            if (step == probes) {  // no room
                                found = claim_level(&pos[u], -2);
                                break;
                            }
                            found = atomicCAS(&s_key[h & mask], -1, u);  // LDS
                            if (found == -1) break;
                            if (found == u) {
                                found = hi;
                                break;
                            }
                        }
                    }
                    claimed |= (uint32_t)(found == -1) << q;
                    shared |= (uint32_t)(u >= 0 && (found == -2 || found >= hi)) << q;
                }
            }
            int32_t cnt = __popc(claimed);
            const int32_t incl = wave_incl_scan(cnt);
            const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
            int32_t at = 0;
            if (lane == 0 && total) at = atomicAdd(&s_tail, total);  // LDS
            at = __builtin_amdgcn_readfirstlane(at) + incl - cnt;
            if (at + cnt > n) {  // no position is given out past the arrays (symmetric rows never ask for one)
                while (cnt && at + cnt > n) claimed &= ~(0x80000000u >> __clz((int)claimed)), --cnt;
            }
            if (has) {
                const int32_t first = at - hi;
                link[i] = cnt && first > 0xffff ? kLinkSlow
                                                : (uint32_t)(cnt ? first : 0) | claimed << 16 | (shared ? kLinkSlow : 0u);
                my_pairs += cnt + __popc(shared);
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const int32_t u = x.row.x[q];
                    if ((claimed >> q) & 1u) {
                        pos[u] = at;
                        const uint32_t g = mesh_hash(u) & (kMeshSeen - 1);
                        atomicOr(&s_seen[tn][g >> 5], 1u << (g & 31));  // LDS
                        const int32_t j = at - hi;
                        if (j < kCap) {
                            Row r = W == 4 ? x.next[q % (W == 4 ? W : 1)] : row_of(u);
#pragma unroll
                            for (int w = 0; w < W; ++w) r.x[w] = r.x[w] == x.v ? -2 - x.v : r.x[w];
                            s_v[nx][j] = u;
                            s_val[tn][j] = x.sv;
                            s_row[nx][j] = r;
                        } else {
                            queue[at] = u;
                            sig[at] = x.sv;
                        }
                        ++at;
                    }
                    if ((shared >> q) & 1u) {
                        const uint32_t h = mesh_hash(u) & (kMeshTable - 1);
                        atomicOr(&s_shared[nx][h >> 5], 1u << (h & 31));  // LDS
                    }
                }
            }
        };
        for (int32_t b = wave0; b < hi - lo; b += BS) {
            if (b != wave0) fetch(e, b + lane);
            process(e, b + lane);
        }
        __syncthreads();
        const int32_t tail = min(s_tail, n);
        if (tid == 0) loff[level + 2] = tail;
        if (tail == hi) break;
        plo = lo;
        lo = hi;
        hi = tail;
        ++level;
        t = tn;
        fetch(e, tid);
        for (int32_t i = 4 * tid; i <= mask; i += 4 * BS)
            *reinterpret_cast<int4 *>(&s_key[i]) = make_int4(-1, -1, -1, -1);
        for (int32_t i = tid; i < kMeshTable / 32; i += BS) s_shared[(level + 1) & 1][i] = 0;
        for (int32_t i = tid; i < kMeshSeen / 32; i += BS) s_seen[tp][i] = 0;
        mask = 63;
        while (mask < (hi - lo) * 8 && mask < kMeshTable - 1) mask = 2 * mask + 1;
        sync_lds();
    }

    // Reverse, from the deepest level up to level 1.  A level's entries go
    // through three stages of loads, a level apart, before their turn: the
    // entry itself, the row and the row's positions (of those with shared
    // children).
    struct Stage {
        int32_t v;
        uint32_t lk;
        double sv;
        Row row;
    };
    int32_t *s_off = s_key, off0 = max(0, level + 3 - kMeshOffsets);
    __syncthreads();
    for (int32_t i = tid; i < kMeshOffsets; i += BS) s_off[i] = loff[min(off0 + i, level + 2)];
    __syncthreads();
    auto off = [&](int32_t l) { return s_off[l - off0]; };
    auto stage1 = [&](Stage &x, int32_t l) {
        if (l < 1) return;
        const int32_t i = min(off(l) + tid, off(l + 1) - 1);
        x.v = queue[i];
        x.lk = link[i];
        x.sv = sig[i];
    };
    auto stage2 = [&](Stage &x, int32_t l) {
        if (l >= 1 && (x.lk & kLinkSlow)) x.row = row_of(x.v);
    };
    auto stage3 = [&](Stage &x, int32_t l) {
        if (l >= 1 && (x.lk & kLinkSlow)) {
#pragma unroll
            for (int q = 0; q < W; ++q)
                if (x.row.x[q] >= 0) x.row.x[q] = pos[x.row.x[q]];
        }
    };
    auto finish = [&](const Stage &x, int32_t i, int32_t l) {
        const int32_t a = off(l), z = off(l + 1), z2 = off(l + 2);
        auto rho = [&](int32_t k) { return k < kCap ? s_val[(l + 1) & 1][k] : sig[z + k]; };
        double acc = 0.0;
        if (x.lk & kLinkSlow) {
#pragma unroll
            for (int q = 0; q < W; ++q)
                if (x.row.x[q] >= z && x.row.x[q] < z2) {
                    acc += rho(x.row.x[q] - z);
                    ++my_pairs;
                }
        } else {
            const int32_t first = (int32_t)(x.lk & 0xffffu), c = __popc((x.lk >> 16) & 0xffu);
            for (int32_t q = 0; q < c; ++q) acc += rho(first + q);
            my_pairs += c;
        }
        const double dv = x.sv * acc;
        delta[x.v] = dv;
        const double r = (1.0 + dv) / x.sv;
        if (i - a < kCap) s_val[l & 1][i - a] = r;
        else sig[i] = r;
    };
    Stage st[4];
    stage1(st[0], level);
    stage1(st[1], level - 1);
    stage1(st[2], level - 2);
    stage2(st[0], level);
    stage2(st[1], level - 1);
    stage3(st[0], level);
    for (int32_t l = level; l >= 1;) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (l < 1) break;
            if (l - 3 < off0 && off0 > 0) {
                __syncthreads();
                off0 = max(0, l + 3 - kMeshOffsets);
                for (int32_t i = tid; i < kMeshOffsets; i += BS) s_off[i] = loff[min(off0 + i, level + 2)];
                __syncthreads();
            }
            stage3(st[(u + 1) & 3], l - 1);
            stage2(st[(u + 2) & 3], l - 2);
            stage1(st[(u + 3) & 3], l - 3);
            const int32_t a = off(l), z = off(l + 1);
            if (a + tid < z) finish(st[u], a + tid, l);
            for (int32_t i = a + tid + BS; i < z; i += BS) {
                Stage x{queue[i], link[i], sig[i], {}};
                stage2(x, l);
                stage3(x, l);
                finish(x, i, l);
            }
            if (z - a > kCap) __syncthreads();
            else sync_lds();
            --l;
        }
    }
    my_max = wave_max_f64(my_max);
    if (lane == 0) s_max[tid / kWave] = my_max;
    __syncthreads();
    if (tid == 0) {
        double m = 0.0;
        for (int w = 0; w < BS / kWave; ++w) m = fmax(m, s_max[w]);
        res[slot] = WgSlotResult{level + 1, hi, m, s_flag};
    }
    if (prof) {
        __syncthreads();
        block_add_u64<BS>(tid == 0 ? (unsigned long long)hi : 0ull, s_red, prof + 0);
        __syncthreads();
        block_add_u64<BS>(my_edges, s_red, prof + 1);
        __syncthreads();
        block_add_u64<BS>(my_pairs, s_red, prof + 2);
    }
}

// Positions -1 (unreached).
__global__ void k_wg_fill_pos(int2 *pos, int64_t pairs) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < pairs; i += stride)
        pos[i] = make_int2(-1, -1);
}

// k_wg_extract by position: the level of position p is the last whose offset
// is at most p.
__global__ void k_wg_extract_mesh(int32_t n, int32_t nslots, const int32_t *__restrict__ pos,
                                  const int32_t *__restrict__ loff, const WgSlotResult *__restrict__ res,
                                  const double *__restrict__ delta, int32_t *out_dist, double *out_sigma,
                                  double *out_delta) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (int64_t)n * nslots; i += stride) {
        const int32_t s = (int32_t)(i / n), p = pos[i];
        int32_t d = -1;
        if (p >= 0) {
            const int32_t *off = loff + (int64_t)s * ((int64_t)n + 2);
            int32_t lo = 0, hi = res[s].levels - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (off[mid] <= p) lo = mid; else hi = mid - 1;
            }
            d = lo;
        }
        if (out_dist) out_dist[i] = d;
        if (out_sigma && d < 0) out_sigma[i] = 0.0;  // reached: written by the pass
        if (out_delta) out_delta[i] = d > 0 ? delta[i] : 0.0;
    }
}

// One source per workgroup: blockIdx.x = slot.
template <int BS>
__global__ __launch_bounds__(BS) void k_wg_bc(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                              const int32_t *__restrict__ rpi,
                                              const int32_t *__restrict__ cii,
                                              const int32_t *__restrict__ slot_src, int32_t n,
                                              WgRec *rec_all, double *delta_all, double *sigma_out,
                                              int32_t *queue_all, int32_t *loff_all, WgSlotResult *res,
                                              unsigned long long *prof) {
    const int32_t slot = blockIdx.x;
    const int64_t base = (int64_t)slot * n;
    WgRec *rec = rec_all + base;
    double *delta = delta_all + base;
    double *sig_out = sigma_out ? sigma_out + base : nullptr;  // sp_batch_levels' sigma
    int32_t *queue = queue_all + base;
    int32_t *loff = loff_all + (int64_t)slot * ((int64_t)n + 2);
    const int32_t src = slot_src[slot];
    __shared__ int32_t s_tail, s_flag;
    __shared__ double s_max[BS / kWave];
    __shared__ unsigned long long s_red[1];
    if (threadIdx.x == 0) {
        rec[src].dist = 0;
        rec[src].val = 1.0;
        if (sig_out) sig_out[src] = 1.0;
        queue[0] = src;
        loff[0] = 0;
        loff[1] = 1;
        s_tail = 1;
        s_flag = 0;
    }
    __syncthreads();
    int32_t lo = 0, hi = 1, level = 0;
    double my_max = 1.0;
    unsigned long long my_edges = 0, my_pairs = 0;
    for (;;) {
        // Discovery of level + 1 from the frontier [lo, hi), outgoing rows;
        // the claim (dist -1 -> level + 1) decides who appends the vertex.
        for (int32_t i0 = lo + (int32_t)threadIdx.x; i0 < hi; i0 += BS * kEntries) {
            int32_t b[kEntries], e[kEntries];
            int32_t len = rows_of_bs<BS>(queue, i0, hi, rp, b, e);
            for (int32_t k0 = 0; k0 < len; k0 += kRowStep) {
                int32_t w[kEntries][kRowStep], d[kEntries][kRowStep], old[kEntries][kRowStep];
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) w[u][t] = b[u] + k0 + t < e[u] ? ci[b[u] + k0 + t] : -1;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) d[u][t] = w[u][t] >= 0 ? ld_level(&rec[w[u][t]].dist) : 0;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t)
                        old[u][t] = d[u][t] < 0 ? claim_level(&rec[w[u][t]].dist, level + 1) : 0;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t)
                        if (d[u][t] < 0 && old[u][t] == -1) queue[atomicAdd(&s_tail, 1)] = w[u][t];  // LDS
            }
#pragma unroll
            for (int u = 0; u < kEntries; ++u) my_edges += (unsigned long long)(e[u] - b[u]);
        }
        __syncthreads();
        const int32_t tail = s_tail;
        if (tail == hi) break;  // block-uniform: every thread read the same tail
        // Path counts of the new vertices [hi, tail): parents over incoming
        // rows, added in row order.
        for (int32_t j0 = hi + (int32_t)threadIdx.x; j0 < tail; j0 += BS * kEntries) {
            int32_t b[kEntries], e[kEntries];
            const int32_t len = rows_of_bs<BS>(queue, j0, tail, rpi, b, e);
            double acc[kEntries] = {};
            for (int32_t k0 = 0; k0 < len; k0 += kRowStep) {
                int32_t p[kEntries][kRowStep];
                bool par[kEntries][kRowStep];
                double x[kEntries][kRowStep];
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) p[u][t] = b[u] + k0 + t < e[u] ? cii[b[u] + k0 + t] : -1;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) par[u][t] = p[u][t] >= 0 && ld_level(&rec[p[u][t]].dist) == level;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) x[u][t] = par[u][t] ? rec[p[u][t]].val : 0.0;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t)
                        if (par[u][t]) {
                            acc[u] += x[u][t];
                            ++my_pairs;
                        }
            }
#pragma unroll
            for (int u = 0; u < kEntries; ++u) {
                const int32_t j = j0 + u * BS;
                if (j < tail) {
                    rec[queue[j]].val = acc[u];
                    if (sig_out) sig_out[queue[j]] = acc[u];
                    my_max = fmax(my_max, acc[u]);
                    if (sigma_is_large(acc[u])) s_flag = 1;
                }
            }
        }
        if (threadIdx.x == 0) loff[level + 2] = tail;
        __syncthreads();
        lo = hi;
        hi = tail;
        ++level;
    }
    // `level` is the deepest level; reverse sweep from it up to level 1
    // (the deepest has no children: its delta is 0).  Children over outgoing
    // rows, added in row order.
    for (int32_t l = level; l >= 1; --l) {
        const int32_t a = loff[l], z = loff[l + 1];
        for (int32_t j0 = a + (int32_t)threadIdx.x; j0 < z; j0 += BS * kEntries) {
            int32_t b[kEntries], e[kEntries], v[kEntries];
            double sv[kEntries], acc[kEntries] = {};
#pragma unroll
            for (int u = 0; u < kEntries; ++u) v[u] = j0 + u * BS < z ? queue[j0 + u * BS] : -1;
            int32_t len = 0;
#pragma unroll
            for (int u = 0; u < kEntries; ++u) {
                b[u] = v[u] >= 0 ? rp[v[u]] : 0;
                e[u] = v[u] >= 0 ? rp[v[u] + 1] : 0;
                sv[u] = v[u] >= 0 ? rec[v[u]].val : 0.0;
                len = max(len, e[u] - b[u]);
            }
            for (int32_t k0 = 0; k0 < len; k0 += kRowStep) {
                int32_t w[kEntries][kRowStep];
                bool ch[kEntries][kRowStep];
                double sw[kEntries][kRowStep], dw[kEntries][kRowStep];
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) w[u][t] = b[u] + k0 + t < e[u] ? ci[b[u] + k0 + t] : -1;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) ch[u][t] = w[u][t] >= 0 && ld_level(&rec[w[u][t]].dist) == l + 1;
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t) {
                        sw[u][t] = ch[u][t] ? rec[w[u][t]].val : 1.0;
                        dw[u][t] = ch[u][t] ? delta[w[u][t]] : 0.0;
                    }
#pragma unroll
                for (int u = 0; u < kEntries; ++u)
#pragma unroll
                    for (int t = 0; t < kRowStep; ++t)
                        if (ch[u][t]) {
                            acc[u] += (sv[u] / sw[u][t]) * (1.0 + dw[u][t]);
                            ++my_pairs;
                        }
            }
#pragma unroll
            for (int u = 0; u < kEntries; ++u)
                if (v[u] >= 0) delta[v[u]] = acc[u];
        }
        __syncthreads();
    }
    my_max = wave_max_f64(my_max);
    if (lane_id() == 0) s_max[threadIdx.x / kWave] = my_max;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        for (int w = 0; w < BS / kWave; ++w) m = fmax(m, s_max[w]);
        res[slot] = WgSlotResult{level + 1, hi, m, s_flag};
    }
    if (prof) {
        __syncthreads();
        block_add_u64<BS>(threadIdx.x == 0 ? (unsigned long long)hi : 0ull, s_red, prof + 0);
        __syncthreads();
        block_add_u64<BS>(my_edges, s_red, prof + 1);
        __syncthreads();
        block_add_u64<BS>(my_pairs, s_red, prof + 2);
    }
}

// BC[v] += delta of v for every slot that reached v from another vertex, in
// ascending slot order; consecutive slots with the same output array are
// summed in a register.
// MESH: whether a slot reached v comes from v's position (the source's is 0),
// else from its record's level.
template <int BS, bool MESH>
__global__ __launch_bounds__(BS) void k_wg_bc_sum(int32_t n, int32_t nslots, const WgRec *__restrict__ rec,
                                                  const int32_t *__restrict__ pos,
                                                  const double *__restrict__ delta, SlotTable tbl,
                                                  unsigned long long *prof) {
    __shared__ unsigned long long s_red[1];
    unsigned long long my_items = 0;
    for (int32_t v = blockIdx.x * BS + threadIdx.x; v < n; v += gridDim.x * BS) {
        double *cur = nullptr;
        double acc = 0.0;
        for (int32_t s = 0; s < nslots; ++s) {
            double *out = tbl.out[s];
            if (!out) continue;
            if (out != cur) {
                if (cur) cur[v] = acc;
                cur = out;
                acc = out[v];
            }
            const int64_t o = (int64_t)s * n + v;
            if ((MESH ? pos[o] : rec[o].dist) > 0) {
                acc += delta[o];
                ++my_items;
            }
        }
        if (cur) cur[v] = acc;
    }
    if (prof) block_add_u64<BS>(my_items, s_red, prof + 3);
}

// Per-slot results into the caller's source-major arrays (sp_batch_levels):
// dist as is, sigma of reached vertices, delta of vertices below the source.
__global__ void k_wg_extract(int64_t count, const WgRec *__restrict__ rec, const double *__restrict__ delta,
                             int32_t *out_dist, double *out_sigma,
                             double *out_delta) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const int32_t d = rec[i].dist;
        if (out_dist) out_dist[i] = d;
        if (out_sigma && d < 0) out_sigma[i] = 0.0;  // reached: written by the pass
        if (out_delta) out_delta[i] = d > 0 ? delta[i] : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Width of the fixed-width rows for g: 4 or 8 when every row fits, else 0.
static int32_t ell_width(sp_graph g) {
    return g->max_degree <= 4 ? 4 : g->max_degree <= 8 ? 8 : 0;
}

size_t wg_ws_bytes(sp_graph g, int32_t width) {
    const size_t V = (size_t)std::max(g->n, 1);
    const size_t ell = V * (size_t)ell_width(g) * 4 * (g->directed ? 2 : 1);
    return (size_t)width * (V * (sizeof(WgRec) + 8 + 4) + (V + 2) * 4) + (size_t)width * sizeof(WgSlotResult) + ell;
}

sp_status wg_ws_alloc(sp_graph g, int32_t width, BatchWorkspace &ws) {
    const size_t V = (size_t)std::max(g->n, 1), W = (size_t)width;
    SP_TRY(dev_alloc((void **)&ws.wg_rec, W * V * sizeof(WgRec)));
    SP_TRY(dev_alloc((void **)&ws.wg_delta, W * V * 8));
    SP_TRY(dev_alloc((void **)&ws.wg_queue, W * V * 4));
    SP_TRY(dev_alloc((void **)&ws.wg_loff, W * (V + 2) * 4));
    SP_TRY(dev_alloc((void **)&ws.wg_res, W * sizeof(WgSlotResult)));
    SP_HIP(hipHostMalloc((void **)&ws.wg_res_host, W * sizeof(WgSlotResult), hipHostMallocDefault));
    ws.wg_ell_w = ell_width(g);
    ws.wg_ell_built = false;
    if (ws.wg_ell_w) {
        const size_t cells = V * (size_t)ws.wg_ell_w;
        SP_TRY(dev_alloc((void **)&ws.wg_ell, cells * 4));
        if (g->directed) SP_TRY(dev_alloc((void **)&ws.wg_ell_in, cells * 4));
    }
    return SP_OK;
}

void wg_ws_free(BatchWorkspace &ws) {
    dev_free(ws.wg_rec);
    dev_free(ws.wg_delta);
    dev_free(ws.wg_queue);
    dev_free(ws.wg_loff);
    dev_free(ws.wg_res);
    dev_free(ws.wg_ell);
    dev_free(ws.wg_ell_in);
    ws.wg_ell = ws.wg_ell_in = nullptr;
    ws.wg_ell_w = 0;
    ws.wg_ell_built = false;
    if (ws.wg_res_host) (void)hipHostFree(ws.wg_res_host);
    ws.wg_rec = nullptr;
    ws.wg_delta = nullptr;
    ws.wg_queue = ws.wg_loff = nullptr;
    ws.wg_res = ws.wg_res_host = nullptr;
}

// Whether g's rows are symmetric, looked at on the graph's first pass (one
// kernel over ws.wg_ell and a wait: 64 bytes read per entry at most).
static sp_status rows_symmetric(sp_graph g, BatchWorkspace &ws, hipStream_t s, bool *out) {
    int32_t known = g->wg_symmetric.load();
    if (known < 0) {
        int32_t *not_sym = ws.wg_loff;  // free until the pass
        SP_TRY(launch_fill_i32(not_sym, 1, 0, s));
        auto look = ws.wg_ell_w == 4 ? k_wg_symmetric<4> : k_wg_symmetric<8>;
        hipLaunchKernelGGL(look, dim3(grid_for(g->n, 256, 4096)), dim3(256), 0, s, (const int32_t *)ws.wg_ell, g->n,
                           not_sym);
        SP_HIP(hipGetLastError());
        int32_t bad = 0;
        SP_HIP(hipMemcpyAsync(&bad, not_sym, sizeof(bad), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        known = bad == 0;
        g->wg_symmetric.store(known);
    }
    *out = known == 1;
    return SP_OK;
}

template <int BS>
static sp_status wg_run_bs(sp_graph g, BatchWorkspace &ws, const int32_t *srcs, int32_t nslots,
                           double *const *bc_of_slot, hipStream_t s, BatchResult *res,
                           const BatchExtract *ex) {
    const int32_t n = g->n;
    const int64_t count = (int64_t)nslots * n;
    int32_t *h_src = (int32_t *)ws.staging;
    for (int32_t i = 0; i < kSlots; ++i) h_src[i] = i < nslots ? srcs[i] : -1;
    SP_HIP(hipMemcpyAsync(ws.slot_src, h_src, kSlots * 4, hipMemcpyHostToDevice, s));
    const int ew = ws.wg_ell_w;
    if (ew && !ws.wg_ell_built) {
        auto build = ew == 4 ? k_wg_ell<4> : k_wg_ell<8>;
        hipLaunchKernelGGL(build, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, (const int32_t *)g->row_ptr,
                           (const int32_t *)g->col_idx, n, ws.wg_ell);
        if (g->directed)
            hipLaunchKernelGGL(build, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, (const int32_t *)g->rp_in,
                               (const int32_t *)g->ci_in, n, ws.wg_ell_in);
        SP_HIP(hipGetLastError());
        ws.wg_ell_built = true;
    }
    // symmetric fixed-width rows: k_wg_bc_mesh, whose positions, links and values share the records' memory
    bool mesh = ew != 0 && !g->directed;
    if (mesh) SP_TRY(rows_symmetric(g, ws, s, &mesh));
    const int64_t cells = (int64_t)ws.width * n;
    double *sig = (double *)ws.wg_rec;
    int32_t *pos = (int32_t *)(sig + cells);
    uint32_t *link = (uint32_t *)(pos + cells);
    if (mesh)  // (in pairs: of an odd count the entry behind, a link or an unused position, is cleared too)
        hipLaunchKernelGGL(k_wg_fill_pos, dim3(grid_for((count + 1) / 2, 256, 4096)), dim3(256), 0, s, (int2 *)pos,
                           (count + 1) / 2);
    else
        hipLaunchKernelGGL(k_wg_fill, dim3(grid_for(count, 256, 4096)), dim3(256), 0, s, ws.wg_rec, count);
    {
        ProfScope ps(P_WG_BC, s);
        if (mesh) {
            auto pass = ew == 4 ? k_wg_bc_mesh<BS, 4> : k_wg_bc_mesh<BS, 8>;
            hipLaunchKernelGGL(pass, dim3(nslots), dim3(BS), 0, s, (const int32_t *)ws.wg_ell,
                               (const int32_t *)ws.slot_src, n, pos, link, sig, ws.wg_delta, ex ? ex->sigma : nullptr,
                               ws.wg_queue, ws.wg_loff, ws.wg_res, prof_counters(P_WG_BC));
        } else if (ew) {
            auto pass = ew == 4 ? k_wg_bc_ell<BS, 4> : k_wg_bc_ell<BS, 8>;
            const int32_t *ell_in = g->directed ? ws.wg_ell_in : ws.wg_ell;
            hipLaunchKernelGGL(pass, dim3(nslots), dim3(BS), 0, s, (const int32_t *)ws.wg_ell, ell_in,
                               (const int32_t *)ws.slot_src, n, ws.wg_rec, ws.wg_delta,
                               ex ? ex->sigma : nullptr, ws.wg_queue, ws.wg_loff, ws.wg_res, prof_counters(P_WG_BC));
        } else
            hipLaunchKernelGGL(k_wg_bc<BS>, dim3(nslots), dim3(BS), 0, s, (const int32_t *)g->row_ptr,
                               (const int32_t *)g->col_idx, (const int32_t *)g->rp_in, (const int32_t *)g->ci_in,
                               (const int32_t *)ws.slot_src, n, ws.wg_rec, ws.wg_delta, ex ? ex->sigma : nullptr,
                               ws.wg_queue, ws.wg_loff, ws.wg_res, prof_counters(P_WG_BC));
    }
    SP_HIP(hipGetLastError());
    if (ex && mesh)
        hipLaunchKernelGGL(k_wg_extract_mesh, dim3(grid_for(count, 256, 4096)), dim3(256), 0, s, n, nslots,
                           (const int32_t *)pos, (const int32_t *)ws.wg_loff, (const WgSlotResult *)ws.wg_res,
                           (const double *)ws.wg_delta, ex->dist, ex->sigma, ex->delta);
    else if (ex)
        hipLaunchKernelGGL(k_wg_extract, dim3(grid_for(count, 256, 4096)), dim3(256), 0, s, count,
                           (const WgRec *)ws.wg_rec, (const double *)ws.wg_delta, ex->dist, ex->sigma,
                           ex->delta);
    SlotTable tbl{};
    bool any_out = false;
    for (int32_t i = 0; i < kSlots; ++i) {
        tbl.out[i] = (bc_of_slot && i < nslots) ? bc_of_slot[i] : nullptr;
        any_out |= tbl.out[i] != nullptr;
    }
    if (any_out) {
        ProfScope ps(P_MS_BC, s);
        auto sum = mesh ? k_wg_bc_sum<BS, true> : k_wg_bc_sum<BS, false>;
        hipLaunchKernelGGL(sum, dim3(grid_for(n, BS, device_cu_count() * 8)), dim3(BS), 0, s, n, nslots,
                           (const WgRec *)ws.wg_rec, (const int32_t *)pos, (const double *)ws.wg_delta, tbl,
                           prof_counters(P_MS_BC));
    }
    SP_HIP(hipGetLastError());
    SP_HIP(hipMemcpyAsync(ws.wg_res_host, ws.wg_res, (size_t)nslots * sizeof(WgSlotResult),
                          hipMemcpyDeviceToHost, s));
    SP_HIP(hipStreamSynchronize(s));
    if (res) {
        *res = BatchResult{};
        for (int32_t i = 0; i < nslots; ++i) {
            const WgSlotResult &r = ws.wg_res_host[i];
            res->levels = std::max(res->levels, r.levels);
            res->reached += r.reached;
            res->entries += r.reached;
            res->sigma_max = std::max(res->sigma_max, r.sigma_max);
            if (r.flagged) {
                res->flagged++;
                res->flagged_mask |= 1ull << i;
            }
            res->td += r.levels - 1;  // every level expanded top-down
        }
    }
    return SP_OK;
}

sp_status wg_run(sp_graph g, BatchWorkspace &ws, const int32_t *srcs, int32_t nslots,
                 double *const *bc_of_slot, const BatchRunOpts &o, hipStream_t s, BatchResult *res,
                 const BatchExtract *ex) {
    switch (o.block) {
        case 128: return wg_run_bs<128>(g, ws, srcs, nslots, bc_of_slot, s, res, ex);
        case 256: return wg_run_bs<256>(g, ws, srcs, nslots, bc_of_slot, s, res, ex);
        case 512: return wg_run_bs<512>(g, ws, srcs, nslots, bc_of_slot, s, res, ex);
        default: return wg_run_bs<1024>(g, ws, srcs, nslots, bc_of_slot, s, res, ex);
    }
}

}  // namespace sp
