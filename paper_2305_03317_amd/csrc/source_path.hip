// Per-source Brandes pass on the GPU: one source at a time.
//
// Forward (paper Section 2.3.2 "iterateInBFS", Appendix Fig. "BC computation
// in StarPlat"): levels are expanded one after another.  A level is
//   discover: the next frontier F_{l+1} = unreached vertices adjacent to F_l,
//             either top-down (scan the adjacency of F_l, claim with a CAS on
//             dist) or bottom-up (every unreached vertex scans its own
//             adjacency and stops once it finds a neighbour in F_l);
//   sigma:    every w in F_{l+1} sums sigma over its DAG parents (neighbours
//             at level l) -- a pull, so no floating-point atomics; its last
//             block moves the frontier window and picks the direction of the
//             next level from the frontier's and the unreached vertices'
//             adjacency sizes;
//   hubs:     path counts of the new level's hubs (see kHubDeg), chunk by
//             chunk, beside the next level's discovery; the last chunk of a
//             hub to arrive adds them up.
// The queue holds the vertices in level order; level_off[l] is where level l
// starts, so the reverse pass replays the levels without a second BFS.
//
// Reverse ("iterateInReverse"): for l = L-1 down to 1 each v in F_l sums
// (sigma[v] / sigma[w]) * (1 + delta[w]) over its DAG children w (level l+1)
// and adds delta[v] to BC[v]; the source (level 0) is skipped.  One launch per
// level, the hubs' chunks beside the other rows.  A row is summed by 1, 4 or 16
// lanes, a chunk by 64, in an order its length fixes (row_sum), so every
// vertex's value is independent of where it sits in the queue.
//
// sigma and delta of a vertex sit side by side, so that a child's two values
// come in one line.  On large skewed graphs (ensure_rank_csr_locked) the pass
// runs on rows numbered by degree rank: most of what a level reads then stays in
// L2.  The rows keep their entries' order, so the results are the same bits.
//
// Level loops run on the device: the host enqueues a chunk of levels, whose
// kernels return at once after the control block says `done`, and reads the
// control block back once per chunk.
#include "common.h"
#include "devutil.h"
#include "levels.h"
#include "rank.h"

namespace sp {

// ---------------------------------------------------------------------------
// Fills
// ---------------------------------------------------------------------------
__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_fill_f64(double *p, int64_t n, double v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

sp_status launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return SP_OK;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

sp_status launch_fill_f64(double *p, int64_t n, double v, hipStream_t s) {
    if (n <= 0) return SP_OK;
    hipLaunchKernelGGL(k_fill_f64, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, p, n, v);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------
// Rows, lists and arrays of a pass, as every kernel sees them.
struct SrcView {
    const int32_t *rp, *ci;        // outgoing rows (discovery, reverse pass)
    const int32_t *rpi, *cii;      // incoming rows (bottom-up, path counts)
    int32_t *dist;
    double2 *sd;                   // {sigma, delta}
    int32_t *queue, *level_off;
    HubEntry *hub_list;            // `entry` counts the chunks that have arrived
    HubEntry *in_hub_list;         // directed graphs only: a level's long incoming rows
    int32_t *hub_off, *hub_end;    // per level: first hub, end of its chunk ids over all levels
    int32_t *owner;                // hub of each chunk id over all levels; null: searched for
    double *partial;
    long long hub_cap, in_hub_cap, owner_cap;
};

// First chunk id, over all levels, of level l.
__device__ __forceinline__ int32_t chunk_start(const SrcView &p, int32_t l) { return l > 0 ? p.hub_end[l - 1] : 0; }

// The hub of a level's chunk k: through the owner map, else a search over the
// level's hubs.
__device__ __forceinline__ int32_t hub_of(const SrcView &p, int32_t start, int32_t lo, int32_t hi, int32_t k) {
    if (p.owner) return p.owner[start + k];
    return hub_find(p.hub_list, lo, hi, k);
}

__global__ void k_src_init(LevelCtl *c, SrcView p, int32_t src, const int32_t *__restrict__ new_id, int32_t n,
                           long long nnz, double alpha, double beta) {
    if (new_id) src = new_id[src];
    const int32_t deg = p.rp[src + 1] - p.rp[src];
    const bool hub = deg > kHubDeg;
    const int32_t nch = hub ? split_hub_nchunks(deg) : 0;
    if (p.owner)
        for (int32_t q = threadIdx.x; q < nch && q < p.owner_cap; q += blockDim.x) p.owner[q] = 0;
    if (threadIdx.x != 0) return;
    c->level = 0;
    c->lo = 0;
    c->hi = 1;
    c->tail_.v = 1;
    c->done = 0;
    c->mode = MODE_TOPDOWN;
    c->overflow_.v = 0;
    c->blocks_done_.v = 0;
    c->front_deg = (unsigned long long)deg;
    c->next_deg_.v = 0;
    c->unset_deg = (unsigned long long)(nnz - deg);
    c->reached_pairs = 1;
    c->sigma_max_bits_.v = (unsigned long long)__double_as_longlong(1.0);
    c->flagged_slots_.v = 0;
    c->settled_deg_.v = 0;
    c->alpha = alpha;
    c->beta = beta;
    c->n_vertices = n;
    c->topdown_levels = 0;
    c->bottomup_levels = 0;
    if (hub) p.hub_list[0] = HubEntry{src, 0, 0, nch};
    c->hub_pack_.v = 0;
    c->in_hub_n = 0;
    c->in_hub_nchunks = 0;
    c->in_hub_pack_.v = 0;
    c->hub_lo = 0;
    c->hub_hi = hub ? 1 : 0;
    c->hub_nchunks = nch;
    c->hub_next = c->hub_hi;
    c->chunk_next = nch;
    p.hub_off[0] = 0;
    p.hub_off[1] = c->hub_hi;
    p.hub_end[0] = nch;
    c->seg_off[0] = 0;
    c->seg_off[1] = 1;
    c->seg_chunks[0] = nch;
    p.dist[src] = 0;
    p.sd[src].x = 1.0;
    p.queue[0] = src;
    p.level_off[0] = 0;
    p.level_off[1] = 1;
}

// ---------------------------------------------------------------------------
// Row sums.  A term of row v: for a neighbour u at level `lvl`, sigma[u]
// (forward) or (sigma[v] / sigma[u]) * (1 + delta[u]) (reverse).
// ---------------------------------------------------------------------------
template <bool REV>
struct RowTerms {
    const int32_t *ci, *dist;
    const double2 *sd;
    int32_t lvl;
};

// Sum over the entries [beg, beg + len) by LPR lanes, all of which receive it:
// lane l adds entries l, l + LPR, ... four at a time, in pairs, then a fixed tree
// (one after another: mean error against 80-bit sums on a road grid 2.72e-17 of a
// dependency, so 2.68e-17).  The four are in flight together, ids, then levels,
// then values: a lane past the row's end reads the last entry again, and a
// neighbour at another level sends its value's read to the row's own vertex (one
// line, in L1), so no load sits under a condition; both are dropped (+0.0 leaves
// a sum that is never negative unchanged).  own: the row's vertex; sv: its sigma
// (reverse).
template <int LPR, bool REV>
__device__ __forceinline__ double row_sum(const RowTerms<REV> &t, int32_t beg, int32_t len, int32_t l, int32_t own,
                                          double sv, unsigned long long &pairs) {
    constexpr int kFly = 4;
    double s = 0.0;
    for (int32_t k = l; __ballot(k < len); k += kFly * LPR) {
        if (k < len) {
            int32_t u[kFly];
            bool hit[kFly];
            double2 x[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) u[q] = t.ci[beg + min(k + q * LPR, len - 1)];
#pragma unroll
            for (int q = 0; q < kFly; ++q) hit[q] = t.dist[u[q]] == t.lvl && k + q * LPR < len;
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                const double2 *at = t.sd + (hit[q] ? u[q] : own);
                if (REV) x[q] = *at;
                else x[q].x = at->x;
            }
            double term[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                term[q] = REV ? (sv / x[q].x) * (1.0 + x[q].y) : x[q].x;
                if (!hit[q]) term[q] = 0.0;
                pairs += hit[q];
            }
            s += (term[0] + term[1]) + (term[2] + term[3]);
        }
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    return s;
}

// Rows of at least `least` and at most `most` entries, LPR lanes each: the
// lanes that hold one are listed, and the wave takes 64 / LPR of them at a
// time.  Their sums go to sum[lane that holds the row].
template <int LPR, bool REV>
__device__ __forceinline__ void rows_by(const RowTerms<REV> &t, int32_t least, int32_t most, int32_t beg,
                                        int32_t deg, int32_t own, double sv, int32_t *list, double *sum,
                                        unsigned long long &pairs) {
    const unsigned long long m = __ballot(deg >= least && deg <= most);
    if (!m) return;
    const int lane = lane_id(), n = __popcll(m);
    if (deg >= least && deg <= most) list[lanes_below(m)] = lane;
    __builtin_amdgcn_wave_barrier();
    for (int i0 = 0; i0 < n; i0 += kWave / LPR) {
        const int i = i0 + lane / LPR;
        const int src = i < n ? list[i] : lane;
        const int32_t rb = __shfl(beg, src, kWave), rl = __shfl(deg, src, kWave), ro = __shfl(own, src, kWave);
        const double rs = REV ? __shfl(sv, src, kWave) : 0.0;
        const double x = row_sum<LPR, REV>(t, rb, i < n ? rl : 0, lane % LPR, ro, rs, pairs);
        if (i < n && lane % LPR == 0) sum[src] = x;
    }
    __builtin_amdgcn_wave_barrier();
}

// The sum of each lane's row (deg 0: none; at most kHubDeg).  list, sum: 64
// values of LDS for the wave.
template <bool REV>
__device__ __forceinline__ double rows_sum(const RowTerms<REV> &t, int32_t beg, int32_t deg, int32_t own, double sv,
                                           int32_t *list, double *sum, unsigned long long &pairs) {
    double s = 0.0;
    if (__ballot(deg > 0 && deg <= 8))
        s = row_sum<1, REV>(t, beg, deg <= 8 ? deg : 0, 0, own, sv, pairs);
    rows_by<4, REV>(t, 9, 32, beg, deg, own, sv, list, sum, pairs);
    rows_by<16, REV>(t, 33, kHubDeg, beg, deg, own, sv, list, sum, pairs);
    return deg > 8 ? sum[lane_id()] : s;
}

// One chunk of a hub, by a wave: its sum is kept, and the hub's last chunk to
// arrive adds them all in a fixed order.  True, with the hub's sum, on every
// lane of that wave.  The sums pass through memory that every XCD sees (agent
// scope), and a chunk is counted once its sum is there.
template <bool REV>
__device__ __forceinline__ bool hub_piece(const RowTerms<REV> &t, const int32_t *__restrict__ rp, HubEntry *slot,
                                          const HubEntry &h, int32_t k, double sv, double *partial, double *total,
                                          unsigned long long &edges, unsigned long long &pairs) {
    int32_t beg, end;
    if (!hub_chunk_range(h, k, rp, beg, end)) return false;
    const int lane = lane_id();
    edges += lane == 0 ? (unsigned long long)(end - beg) : 0ull;
    const double x = row_sum<kWave, REV>(t, beg, end - beg, lane, h.v, sv, pairs);
    int32_t before = 0;
    if (lane == 0) {
        __hip_atomic_store(&partial[k], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_s_waitcnt(0);
        before = atomicAdd(&slot->entry, 1);
    }
    if (__builtin_amdgcn_readfirstlane(before) != h.nchunks - 1) return false;
    double s = 0.0;
    for (int32_t q = lane; q < h.nchunks; q += kWave) s += ld_agent(&partial[h.chunk_base + q]);
    *total = wave_sum_f64(s);
    if (lane == 0) slot->entry = 0;  // for the reverse pass
    return true;
}

// Fewer rows per wave where a level would leave waves without any.
template <int BS>
__device__ __forceinline__ int32_t rows_per_wave(int64_t cnt) {
    const int64_t waves = (int64_t)min((int)gridDim.x, 1024) * (BS / kWave);
    int32_t e = 4;
    while (e < kWave && waves * e < cnt) e <<= 1;
    return e;
}

// Top-down discovery.  blockIdx.y == 0: the block takes BS frontier vertices
// (hubs excluded), scans their degrees, and walks the concatenated adjacency BS
// entries at a time, one entry per lane.  blockIdx.y == 1: blocks walk the
// chunks of the frontier's hubs.
template <int BS>
__device__ __forceinline__ void src_topdown(LevelCtl *c, const SrcView &p, unsigned long long *prof) {
    const int32_t *__restrict__ rp = p.rp, *__restrict__ ci = p.ci;
    int32_t *dist = p.dist, *queue = p.queue;
    __shared__ int32_t s_beg[BS], s_off[BS], s_scan[BS / kWave + 1];
    __shared__ int32_t s_qbuf[4 * BS], s_meta[2];
    __shared__ unsigned long long s_red[1];
    StagedQueue<BS, 4 * BS> q;
    q.init(s_qbuf, s_meta);
    const int32_t lo = c->lo, hi = c->hi, nl = c->level + 1, n = c->n_vertices;
    unsigned long long my_items = 0, my_edges = 0;
    if (blockIdx.y == 0) {
        for (int32_t b = lo + blockIdx.x * BS; b < hi; b += gridDim.x * BS) {
            const int32_t i = b + threadIdx.x;
            int32_t beg = 0, deg = 0;
            if (i < hi) {
                const int32_t v = queue[i];
                beg = rp[v];
                deg = rp[v + 1] - beg;
                if (deg > kHubDeg) deg = 0;  // chunks handled by blockIdx.y == 1
                ++my_items;
                my_edges += deg;
            }
            int32_t total;
            const int32_t off = block_excl_scan<BS>(deg, s_scan, &total);
            s_beg[threadIdx.x] = beg;
            s_off[threadIdx.x] = off;
            __syncthreads();
            for (int32_t k0 = 0; k0 < total; k0 += BS) {
                const int32_t k = k0 + threadIdx.x;
                bool claim = false;
                int32_t w = 0;
                if (k < total) {
                    int32_t a = 0, z = BS - 1;  // last j with s_off[j] <= k
                    while (a < z) {
                        const int32_t mid = (a + z + 1) >> 1;
                        if (s_off[mid] <= k) a = mid; else z = mid - 1;
                    }
                    w = ci[s_beg[a] + (k - s_off[a])];
                    if (dist[w] < 0) claim = atomicCAS(&dist[w], -1, nl) == -1;
                }
                q.stage(claim, w, &c->tail_.v, queue, n, &c->overflow_.v);
            }
            __syncthreads();
        }
    } else {
        const int32_t hlo = c->hub_lo, hhi = c->hub_hi, nch = c->hub_nchunks, start = chunk_start(p, c->level);
        for (int32_t k = blockIdx.x; k < nch; k += gridDim.x) {
            const HubEntry h = p.hub_list[hub_of(p, start, hlo, hhi, k)];
            int32_t beg, end;
            if (!hub_chunk_range(h, k, rp, beg, end)) continue;
            my_edges += (threadIdx.x == 0) ? (unsigned long long)(end - beg) : 0ull;
            for (int32_t e0 = beg; e0 < end; e0 += BS) {
                const int32_t e = e0 + threadIdx.x;
                bool claim = false;
                int32_t w = 0;
                if (e < end) {
                    w = ci[e];
                    if (dist[w] < 0) claim = atomicCAS(&dist[w], -1, nl) == -1;
                }
                q.stage(claim, w, &c->tail_.v, queue, n, &c->overflow_.v);
            }
        }
    }
    q.finish(&c->tail_.v, queue, n, &c->overflow_.v);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
}

// Bottom-up discovery: every unreached vertex looks for a neighbour on the
// current level, 8 entries per lane group, and stops once it finds one.
template <int BS>
__device__ __forceinline__ void src_bottomup(LevelCtl *c, const SrcView &p, unsigned long long *prof) {
    const int32_t *__restrict__ rp = p.rpi, *__restrict__ ci = p.cii;
    int32_t *dist = p.dist, *queue = p.queue;
    __shared__ int32_t s_qbuf[4 * BS], s_meta[2];
    __shared__ int32_t s_coff[BS], s_beg[BS], s_deg[BS];
    __shared__ double s_acc[BS];
    __shared__ unsigned long long s_red[1];
    StagedQueue<BS, 4 * BS> q;
    q.init(s_qbuf, s_meta);
    const int wbase = threadIdx.x & ~(kWave - 1);
    const WaveScratch ws{s_coff + wbase, s_beg + wbase, s_deg + wbase, s_acc + wbase};
    const int32_t lvl = c->level, n = c->n_vertices;
    unsigned long long my_items = 0, my_edges = 0;
    for (int32_t b = blockIdx.x * BS; b < n; b += gridDim.x * BS) {
        const int32_t v = b + threadIdx.x;
        int32_t beg = 0, deg = 0;
        if (v < n && dist[v] < 0) {
            beg = rp[v];
            deg = rp[v + 1] - beg;
            ++my_items;
        }
        const bool found = wave_chunk_any(beg, deg, ws, [&](int32_t e, int32_t) {
            ++my_edges;
            return dist[ci[e]] == lvl;
        });
        if (found) dist[v] = lvl + 1;
        q.stage(found, v, &c->tail_.v, queue, n, &c->overflow_.v);
    }
    q.finish(&c->tail_.v, queue, n, &c->overflow_.v);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
}

// Path counts of the current level's hubs (parents one level up).
// Undirected: the level's hub segment; directed: the incoming-row list.
template <int BS>
__device__ __forceinline__ void src_sigma_hub(LevelCtl *c, const SrcView &p, unsigned long long *prof) {
    const bool in = p.in_hub_list != nullptr;
    const int32_t hlo = c->hub_lo, hhi = c->hub_hi, start = in ? 0 : chunk_start(p, c->level);
    const int32_t nch = in ? c->in_hub_nchunks : c->hub_nchunks;
    HubEntry *hubs = in ? p.in_hub_list : p.hub_list;
    const RowTerms<false> terms{p.cii, p.dist, p.sd, c->level - 1};
    __shared__ unsigned long long s_red[1];
    unsigned long long my_edges = 0, my_pairs = 0;
    for_xcd_chunks<BS>(nch, [&](int64_t k) {
        const int32_t j = in ? hub_find(hubs, 0, c->in_hub_n, (int32_t)k) : hub_of(p, start, hlo, hhi, (int32_t)k);
        const HubEntry h = hubs[j];
        double s;
        if (hub_piece<false>(terms, p.rpi, hubs + j, h, (int32_t)k, 0.0, p.partial, &s, my_edges, my_pairs) &&
            lane_id() == 0) {
            p.sd[h.v].x = s;
            atomic_max_nonneg_f64(&c->sigma_max_bits_.v, s);
            if (sigma_is_large(s)) atomicOr(&c->flagged_slots_.v, 1ull);
        }
    });
    flush_counters<BS>(prof, 0, my_edges, my_pairs, s_red);
}

// The first kernel of a level: what discovers the next one, in the direction
// chosen, and beside it the path counts of this level's hubs, which nothing
// reads before the next level's k_src_sigma (three launches cost 4.5 us each
// where they had nothing to do).  blockIdx.y == 0: top-down without the hubs,
// or bottom-up; 1: the frontier's hub chunks, top-down; 2: hub path counts.
// WHICH takes them apart for timing (1: top-down, 2: bottom-up, 4: hubs, 7: all).
template <int BS, int WHICH>
__global__ __launch_bounds__(BS) void k_src_discover(LevelCtl *c, SrcView p, unsigned long long *prof_td,
                                                     unsigned long long *prof_bu, unsigned long long *prof_hub) {
    if (c->done) return;
    if (blockIdx.y == 2) {
        if ((WHICH & 4) && c->level >= 1) src_sigma_hub<BS>(c, p, prof_hub);  // level 0 was given its count
    } else if (c->mode == MODE_TOPDOWN) {
        if (WHICH & 1) src_topdown<BS>(c, p, prof_td);
    } else if (blockIdx.y == 0) {
        if (WHICH & 2) src_bottomup<BS>(c, p, prof_bu);
    }
}

// End of a forward level (one thread of k_src_sigma's last block).
__device__ void src_advance(LevelCtl *c, const SrcView &p) {
    if (c->mode == MODE_TOPDOWN) c->topdown_levels++; else c->bottomup_levels++;
    const int32_t tail = ld_agent(&c->tail_.v);
    const int32_t nf = tail - c->hi;
    if (nf <= 0) {
        c->done = 1;
        return;
    }
    const int32_t nl = c->level + 1;
    p.level_off[nl + 1] = tail;
    const unsigned long long hp = ld_agent(&c->hub_pack_.v);
    c->hub_lo = c->hub_next;
    c->hub_hi = c->hub_next + (int32_t)(hp >> 40);
    c->hub_nchunks = (int32_t)(hp & ((1ull << 40) - 1));
    c->hub_next = c->hub_hi;
    c->hub_pack_.v = 0;
    c->chunk_next += c->hub_nchunks;
    p.hub_off[nl + 1] = c->hub_hi;
    p.hub_end[nl] = c->chunk_next;
    if (nl < kSegLevels) {
        c->seg_off[nl + 1] = tail;
        c->seg_chunks[nl] = c->hub_nchunks;
    }
    const unsigned long long ip = ld_agent(&c->in_hub_pack_.v);
    c->in_hub_n = (int32_t)(ip >> 40);
    c->in_hub_nchunks = (int32_t)(ip & ((1ull << 40) - 1));
    c->in_hub_pack_.v = 0;
    const unsigned long long deg = ld_agent(&c->next_deg_.v);
    c->front_deg = deg;
    c->unset_deg -= deg;
    c->next_deg_.v = 0;
    c->reached_pairs += (unsigned long long)nf;
    c->lo = c->hi;
    c->hi = tail;
    c->level = nl;
    if (c->mode == MODE_TOPDOWN) {
        if ((double)c->front_deg * c->alpha > (double)c->unset_deg) c->mode = MODE_BOTTOMUP;
    } else {
        if ((double)nf * c->beta < (double)c->n_vertices) c->mode = MODE_TOPDOWN;
    }
}

// Path counts of the new frontier: sigma[w] = sum of sigma[u] over neighbours
// u on the current level.  Hubs are registered for k_src_discover: by
// outgoing length (discovery, reverse pass) and, on a directed graph, by
// incoming length in a list of this level's own.  The last block closes the level.
template <int BS>
__global__ __launch_bounds__(BS, 8) void k_src_sigma(LevelCtl *c, SrcView p, unsigned long long *prof) {
    if (c->done) return;
    __shared__ int32_t s_list[BS];
    __shared__ double s_sum[BS];
    __shared__ unsigned long long s_red[1];
    const int lane = lane_id();
    int32_t *list = s_list + (threadIdx.x - lane);
    double *sum = s_sum + (threadIdx.x - lane);
    const int32_t lvl = c->level, hi = c->hi, tail = min(c->tail_.v, c->n_vertices);
    const RowTerms<false> terms{p.cii, p.dist, p.sd, lvl};
    unsigned long long my_deg = 0, my_items = 0, my_pairs = 0, my_scan = 0;
    double my_max = 0.0;
    bool large = false;
    const int32_t share = rows_per_wave<BS>((int64_t)tail - hi), per = BS / kWave * share;
    for (int64_t b = hi + (int64_t)blockIdx.x * per + threadIdx.x / kWave * share; b < tail;
         b += (int64_t)gridDim.x * per) {
        const int64_t i = b + lane;
        int32_t w = -1, beg = 0, deg = 0;
        if (i < tail && lane < share) {
            w = p.queue[i];
            beg = p.rpi[w];
            deg = p.rpi[w + 1] - beg;
        }
        const bool hub = deg > kHubDeg;
        const double s = rows_sum<false>(terms, beg, hub ? 0 : deg, max(w, 0), 0.0, list, sum, my_pairs);
        if (w >= 0) {
            my_deg += (unsigned long long)deg;
            ++my_items;
            const int32_t dout = p.in_hub_list ? p.rp[w + 1] - p.rp[w] : deg;
            if (dout > kHubDeg)
                hub_register(&c->hub_pack_.v, p.hub_list, p.hub_cap, c->hub_next, w, 0, dout, p.owner, c->chunk_next,
                             p.owner_cap);
            if (p.in_hub_list && hub) hub_register(&c->in_hub_pack_.v, p.in_hub_list, p.in_hub_cap, 0, w, 0, deg);
            if (!hub) {
                my_scan += (unsigned long long)deg;
                p.sd[w].x = s;
                my_max = fmax(my_max, s);
                large |= sigma_is_large(s);
            }
        }
    }
    my_max = wave_max_f64(my_max);
    if (lane == 0) atomic_max_nonneg_f64(&c->sigma_max_bits_.v, my_max);
    if (__ballot(large) && lane == 0) atomicOr(&c->flagged_slots_.v, 1ull);
    block_add_u64<BS>(my_deg, s_red, &c->next_deg_.v);
    flush_counters<BS>(prof, my_items, my_scan, my_pairs, s_red);
    if (last_block(c, working_blocks((int64_t)tail - hi, per)) && threadIdx.x == 0) src_advance(c, p);
}

// Reverse sweep over one level.  blockIdx.y == 0: its rows without the hubs;
// blockIdx.y == 1: the chunks of its hubs.  WHICH takes them apart for timing
// (1: rows, 2: hubs, 3: both).
template <int BS, int WHICH>
__global__ __launch_bounds__(BS, 8) void k_src_delta(SrcView p, int32_t lvl, double *bc, unsigned long long *prof,
                                                     unsigned long long *prof_hub) {
    __shared__ int32_t s_list[BS];
    __shared__ double s_sum[BS];
    __shared__ unsigned long long s_red[1];
    const int lane = lane_id();
    const RowTerms<true> terms{p.ci, p.dist, p.sd, lvl + 1};
    unsigned long long my_items = 0, my_edges = 0, my_pairs = 0;
    const bool rows = WHICH == 1 || (WHICH == 3 && blockIdx.y == 0);
    if (rows) {
        int32_t *list = s_list + (threadIdx.x - lane);
        double *sum = s_sum + (threadIdx.x - lane);
        const int32_t lo = p.level_off[lvl], hi = p.level_off[lvl + 1];
        const int32_t share = rows_per_wave<BS>((int64_t)hi - lo), per = BS / kWave * share;
        for (int64_t b = lo + (int64_t)blockIdx.x * per + threadIdx.x / kWave * share; b < hi;
             b += (int64_t)gridDim.x * per) {
            const int64_t i = b + lane;
            int32_t v = -1, beg = 0, deg = 0;
            double sv = 0.0;
            if (i < hi && lane < share) {
                v = p.queue[i];
                beg = p.rp[v];
                deg = p.rp[v + 1] - beg;
                sv = p.sd[v].x;
            }
            const bool hub = deg > kHubDeg;
            const double acc = rows_sum<true>(terms, beg, hub ? 0 : deg, max(v, 0), sv, list, sum, my_pairs);
            if (v >= 0 && !hub) {
                p.sd[v].y = acc;
                if (bc) bc[v] += acc;
                ++my_items;
                my_edges += (unsigned long long)deg;
            }
        }
    } else {
        const int32_t hlo = p.hub_off[lvl], hhi = p.hub_off[lvl + 1], start = chunk_start(p, lvl);
        for_xcd_chunks<BS>(p.hub_end[lvl] - start, [&](int64_t k) {
            const int32_t j = hub_of(p, start, hlo, hhi, (int32_t)k);
            const HubEntry h = p.hub_list[j];
            const double sv = p.sd[h.v].x;
            double s;
            if (hub_piece<true>(terms, p.rp, p.hub_list + j, h, (int32_t)k, sv, p.partial, &s, my_edges, my_pairs) &&
                lane == 0) {
                p.sd[h.v].y = s;
                if (bc) bc[h.v] += s;
            }
        });
    }
    flush_counters<BS>(rows ? prof : prof_hub, my_items, my_edges, my_pairs, s_red);
}

// BC of the ranks to the caller's vertices.
__global__ void k_src_unrank(const double *__restrict__ bc, const int32_t *__restrict__ new_id, int32_t n,
                             double *out) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) out[v] = bc[new_id[v]];
}

sp_status launch_unrank(sp_graph g, const double *bc, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_src_unrank, dim3(grid_for(g->n, 256, 4096)), dim3(256), 0, s, bc,
                       (const int32_t *)g->rank_new, g->n, out);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
sp_status source_ws_create(sp_graph g, SourceWorkspace &ws) {
    ws.device = g->device;
    ws.n = g->n;
    const size_t n = (size_t)std::max(g->n, 1);
    SP_TRY(dev_alloc((void **)&ws.dist, n * sizeof(int32_t)));
    SP_TRY(dev_alloc((void **)&ws.sd, n * sizeof(double2)));
    SP_TRY(dev_alloc((void **)&ws.queue, n * sizeof(int32_t)));
    ws.level_cap = (int32_t)n + 2;
    SP_TRY(dev_alloc((void **)&ws.level_off, (size_t)ws.level_cap * sizeof(int32_t)));
    SP_TRY(dev_alloc((void **)&ws.hub_off, (size_t)ws.level_cap * sizeof(int32_t)));
    SP_TRY(dev_alloc((void **)&ws.hub_end, (size_t)ws.level_cap * sizeof(int32_t)));
    SP_TRY(dev_alloc((void **)&ws.hub_list, ((size_t)g->n_hubs + 1) * sizeof(HubEntry)));
    if (g->directed) SP_TRY(dev_alloc((void **)&ws.in_hub_list, ((size_t)g->n_hubs_in + 1) * sizeof(HubEntry)));
    ws.owner_cap = g->split_hub_chunks + 1;
    SP_TRY(dev_alloc((void **)&ws.owner, (size_t)ws.owner_cap * sizeof(int32_t)));
    SP_TRY(dev_alloc((void **)&ws.partial,
                     ((size_t)std::max(g->split_hub_chunks, g->split_hub_chunks_in) + 1) * sizeof(double)));
    SP_TRY(dev_alloc((void **)&ws.ctl, sizeof(LevelCtl)));
    SP_HIP(hipHostMalloc((void **)&ws.ctl_host, sizeof(LevelCtl), hipHostMallocDefault));
    SP_HIP(hipEventCreate(&ws.ev0));
    SP_HIP(hipEventCreate(&ws.ev1));
    return SP_OK;
}

void source_ws_destroy(SourceWorkspace &ws) {
    dev_free(ws.dist);
    dev_free(ws.sd);
    dev_free(ws.queue);
    dev_free(ws.level_off);
    dev_free(ws.hub_off);
    dev_free(ws.hub_end);
    dev_free(ws.hub_list);
    dev_free(ws.in_hub_list);
    dev_free(ws.owner);
    dev_free(ws.partial);
    dev_free(ws.bc);
    dev_free(ws.ctl);
    if (ws.ctl_host) (void)hipHostFree(ws.ctl_host);
    if (ws.ev0) (void)hipEventDestroy(ws.ev0);
    if (ws.ev1) (void)hipEventDestroy(ws.ev1);
    ws = SourceWorkspace{};
}

bool source_ranked(sp_graph g, int32_t n_sources, hipStream_t s) {
    if (g->n < kSourceRankFrom) return false;
    std::lock_guard<std::mutex> lk(g->mu);
    if (!g->rank_ci && n_sources < kSourceRankCount) return false;
    return ensure_rank_csr_locked(g, s) == SP_OK && g->rank_ci != nullptr;
}

template <int BS>
static sp_status source_run_bs(sp_graph g, SourceWorkspace &ws, int32_t src, double *bc,
                               bool with_backward, const SourceRunOpts &o, hipStream_t s,
                               SourceResult *res) {
    const int32_t n = g->n;
    const int maxb = device_cu_count() * 8;
    // a block per BS vertices, or what a small level spreads over (rows_per_wave)
    auto level_grid = [&](int64_t cnt) {
        return std::max(grid_for(cnt, BS, maxb), grid_for(cnt, BS / kWave * 4, std::min(maxb, 1024)));
    };
    const int grid = grid_for((int64_t)n, BS, maxb);
    // Hub rows: discovery and the reverse pass walk outgoing rows, the path
    // counts incoming ones.  On an undirected graph they are the same rows and
    // one hub list serves all passes; a directed graph keeps a second list of
    // the level's long incoming rows for the path counts.
    const bool hubs = g->n_hubs > 0;
    const bool hubs_in = g->n_hubs_in > 0;
    const bool may_pull = o.alpha > 0 && g->max_degree > 8;  // sparse meshes never pull
    SrcView p{};
    p.rp = o.ranked ? g->rank_rp : g->row_ptr;
    p.ci = o.ranked ? g->rank_ci : g->col_idx;
    p.rpi = o.ranked ? g->rank_rp : g->rp_in;  // (only undirected graphs are ranked)
    p.cii = o.ranked ? g->rank_ci : g->ci_in;
    p.dist = ws.dist;
    p.sd = ws.sd;
    p.queue = ws.queue;
    p.level_off = ws.level_off;
    p.hub_list = ws.hub_list;
    p.in_hub_list = g->directed ? ws.in_hub_list : nullptr;
    p.hub_off = ws.hub_off;
    p.hub_end = ws.hub_end;
    p.owner = ws.owner;
    p.partial = ws.partial;
    p.hub_cap = (long long)g->n_hubs + 1;
    p.in_hub_cap = (long long)g->n_hubs_in + 1;
    p.owner_cap = ws.owner_cap;
    SP_TRY(launch_fill_i32(ws.dist, n, -1, s));
    hipLaunchKernelGGL(k_src_init, dim3(1), dim3(256), 0, s, ws.ctl, p, src,
                       o.ranked ? (const int32_t *)g->rank_new : nullptr, n, (long long)g->nnz,
                       may_pull ? o.alpha : 0.0, o.beta);  // alpha 0: never switch to bottom-up
    SP_HIP(hipGetLastError());
    const int hub_grid = hubs_in ? grid_for(g->split_hub_chunks_in * kWave, BS, maxb) : 1;
    const dim3 discover_grid(hubs || hubs_in ? xcd_grid(std::max(grid, hub_grid), maxb) : grid,
                             hubs_in ? 3 : hubs ? 2 : 1);
    auto discover = [&](int kind, auto kernel) {
        ProfScope ps(kind, s);
        hipLaunchKernelGGL(kernel, discover_grid, dim3(BS), 0, s, ws.ctl, p,
                           prof_counters(P_SRC_TOPDOWN), prof_counters(P_SRC_BOTTOMUP),
                           prof_counters(P_SRC_SIGMA_HUB));
    };
    int32_t enqueued = 0;
    for (;;) {
        const int chunk = std::max(1, std::abs(o.chunk_levels));
        for (int k = 0; k < chunk; ++k) {
            if (prof_enabled()) {
                discover(P_SRC_TOPDOWN, k_src_discover<BS, 1>);
                if (may_pull) discover(P_SRC_BOTTOMUP, k_src_discover<BS, 2>);
                if (hubs_in) discover(P_SRC_SIGMA_HUB, k_src_discover<BS, 4>);
            } else {
                discover(P_SRC_TOPDOWN, k_src_discover<BS, 7>);
            }
            {
                ProfScope ps(P_SRC_SIGMA, s);
                hipLaunchKernelGGL(k_src_sigma<BS>, dim3(level_grid(n)), dim3(BS), 0, s, ws.ctl, p,
                                   prof_counters(P_SRC_SIGMA));
            }
        }
        SP_HIP(hipGetLastError());
        enqueued += chunk;
        SP_HIP(hipMemcpyAsync(ws.ctl_host, ws.ctl, sizeof(LevelCtl), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        if (ws.ctl_host->done) break;
        if (enqueued > n + 2) {
            set_error("BFS did not terminate after %d levels", enqueued);
            return SP_ERR_DEVICE;
        }
    }
    const LevelCtl &c = *ws.ctl_host;
    const int32_t levels = c.level + 1;
    // Reverse pass, deepest level first.  The level offsets and hub chunk
    // counts that size its launches come with the control block where the
    // levels are few, else a window of kRevWindow levels at a time, into fixed
    // buffers (no host allocation per call; one synchronisation per window).
    constexpr int32_t kRevWindow = 1024;
    int32_t off_w[kRevWindow + 1], end_w[kRevWindow + 1];
    for (int32_t top = with_backward ? levels - 1 : 0; top >= 1; top -= kRevWindow) {
        const int32_t lo = std::max(1, top - kRevWindow + 1);  // window: levels lo..top
        const bool at_hand = levels <= kSegLevels;
        if (!at_hand) {
            SP_HIP(hipMemcpyAsync(off_w, ws.level_off + lo, sizeof(int32_t) * (top - lo + 2),
                                  hipMemcpyDeviceToHost, s));
            SP_HIP(hipMemcpyAsync(end_w, ws.hub_end + lo - 1, sizeof(int32_t) * (top - lo + 2),
                                  hipMemcpyDeviceToHost, s));
            SP_HIP(hipStreamSynchronize(s));
        }
        for (int32_t l = top; l >= lo; --l) {
            const int32_t cnt = at_hand ? c.seg_off[l + 1] - c.seg_off[l] : off_w[l + 1 - lo] - off_w[l - lo];
            const int32_t chunks = at_hand ? c.seg_chunks[l] : end_w[l + 1 - lo] - end_w[l - lo];
            const bool both = hubs && chunks > 0;
            int gx = level_grid((int64_t)cnt);
            if (both) gx = xcd_grid(std::max(gx, grid_for((int64_t)chunks * kWave, BS, maxb)), maxb);
            auto delta = [&](int kind, int gy, auto kernel) {
                ProfScope ps(kind, s);
                hipLaunchKernelGGL(kernel, dim3(gx, gy), dim3(BS), 0, s, p, l, bc, prof_counters(P_SRC_DELTA),
                                   prof_counters(P_SRC_DELTA_HUB));
            };
            if (!both || prof_enabled()) delta(P_SRC_DELTA, 1, k_src_delta<BS, 1>);
            if (both && prof_enabled()) delta(P_SRC_DELTA_HUB, 1, k_src_delta<BS, 2>);
            if (both && !prof_enabled()) delta(P_SRC_DELTA, 2, k_src_delta<BS, 3>);
        }
        SP_HIP(hipGetLastError());
    }
    if (res) {
        res->levels = levels;
        res->reached = c.hi;
        std::memcpy(&res->sigma_max, &c.sigma_max_bits_.v, sizeof(double));
        res->flagged = c.flagged_slots_.v != 0;
        res->td = c.topdown_levels;
        res->bu = c.bottomup_levels;
    }
    return SP_OK;
}

sp_status source_run(sp_graph g, SourceWorkspace &ws, int32_t src, double *bc, bool with_backward,
                     const SourceRunOpts &o, hipStream_t s, SourceResult *res) {
    switch (o.block) {
        case 128: return source_run_bs<128>(g, ws, src, bc, with_backward, o, s, res);
        case 512: return source_run_bs<512>(g, ws, src, bc, with_backward, o, s, res);
        default: return source_run_bs<256>(g, ws, src, bc, with_backward, o, s, res);
    }
}

}  // namespace sp
