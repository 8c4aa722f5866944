// Single-source shortest paths on a weighted graph (paper Section 2.2, Fig.
// "SSSP computation in StarPlat"; the pull form in the Appendix).
//
// The paper's method is a Bellman-Ford variant driven by a `modified` flag:
// in each round every vertex modified in the previous round relaxes its edges
// with an atomic Min (push), or every vertex takes the Min over its modified
// neighbours (pull), until a round modifies nothing.  Here:
//
//   * the `modified` set of a round is a frontier queue, which push rounds
//     read; a stamp per vertex, the last round whose frontier holds it, keeps
//     it free of repeats.  Distances and stamps are arrays of their own, since
//     relaxations read distances only;
//   * a push relaxation lowers dist[u] with atomicMin; the first thread in a
//     round whose atomicMin lowered it raises u's stamp to the next round with
//     atomicMax and appends u to the next frontier, so a vertex joins a
//     frontier at most once per round;
//   * a pull round walks every vertex's row, takes the least candidate over
//     the neighbours that have a distance (more than the modified ones: what
//     the others offer was taken before and lowers nothing), and stores it
//     when lower;
//   * rows longer than kHubDeg entries ("hubs") are cut into chunks of
//     kHubChunk entries that blocks take one at a time: in push rounds the
//     frontier's hubs (registered when they join it), in pull rounds every
//     hub of the graph (a fixed list built with the weights);
//   * adjacency entries are packed {neighbour, weight}; one load per entry;
//   * each round is one kernel per direction.  The direction is chosen on the
//     device: a round pulls when its frontier's adjacency entries times alpha
//     exceed the graph's; the other direction's kernel returns at once.  The
//     last working block of a round's kernel closes the round, so chunks of
//     rounds are captured once as HIP graphs and replayed until a round
//     lowers nothing.
//
// Every round only lowers distances toward the same least fixed point, so
// the result does not depend on scheduling: it is the shortest-path distance
// (INT32_MAX where unreached), bit for bit.
#include <type_traits>

#include "capture.h"
#include "common.h"
#include "devutil.h"
#include "levels.h"
#include "rank.h"

namespace sp {

namespace {
constexpr int32_t kInf = INT32_MAX;
}

// d + w, or kInf with `ovf` set when the sum reaches INT32_MAX.  d and w lie
// in [0, INT32_MAX), so the unsigned sum cannot wrap.  A saturated candidate
// lowers nothing (kInf is the unreached mark).  It only matters if it is the
// sole way to reach a vertex, which the check after the last round decides
// (k_sssp_unfit), so `ovf` merely asks for that check.
__device__ __forceinline__ int32_t candidate(int32_t d, int32_t w, bool &ovf) {
    const uint32_t s = (uint32_t)d + (uint32_t)w;
    if (s >= (uint32_t)kInf) {
        ovf = true;
        return kInf;
    }
    return (int32_t)s;
}

// Push relaxation of u to nd in round r.  True for exactly one caller per
// vertex and round: the first whose atomicMin lowered u's distance in this
// round; it puts u into the next frontier.  A stale plain read can only be
// too large, so skipping on it is safe.
__device__ __forceinline__ bool relax_push(int32_t *dist, int32_t *stamp, int32_t u, int32_t nd, int32_t r, bool &lowered) {
    lowered = false;
    if (nd >= dist[u]) return false;
    const int32_t old = atomicMin(&dist[u], nd);
    if (nd >= old) return false;
    lowered = true;
    return atomicMax(&stamp[u], r + 1) < r + 1;
}

// Entries of a block's local frontier (see k_sssp_push_hops).
constexpr int kLocalCap = 512;

// Fewest frontier vertices a wave of k_sssp_mesh starts with.
constexpr int kMeshLeast = 8;

// Entries a wave of k_sssp_push takes at least of a frontier's rows, on average
// (1, 64, 128, 256: 262,144 vertices of three entries 635, 569, 568, 593 us;
// uniform, 65,536 vertices, 498, 501, 503, 518).
constexpr int kPushStep = 128;

// The round state word (SsspCtl::state).
struct RoundState {
    int32_t cnt;      // frontier size
    int32_t chunks;   // chunks of the frontier's hubs
    int32_t parity;   // round & 1
    bool pull, done;
    int32_t share;    // fewest frontier vertices a wave of k_sssp_push takes
};

// deg: the frontier's entries.
__device__ __forceinline__ unsigned long long pack_state(int32_t cnt, int32_t chunks, int32_t round,
                                                         int32_t mode, bool done, unsigned long long deg) {
    const float rows = (float)kPushStep * (float)cnt / (float)max(deg, 1ull);  // of a step, on average
    const int32_t lg = rows >= 64.0f ? 6 : max(1, 31 - __clz((int)rows | 1));
    return (unsigned long long)(uint32_t)cnt | ((unsigned long long)(uint32_t)chunks << 31) |
           ((unsigned long long)(round & 1) << 55) | ((unsigned long long)(mode == SSSP_PULL) << 56) |
           ((unsigned long long)done << 57) | ((unsigned long long)lg << 58);
}

__device__ __forceinline__ RoundState unpack_state(unsigned long long w) {
    return RoundState{(int32_t)(w & 0x7fffffffull), (int32_t)((w >> 31) & 0xffffffull),
                      (int32_t)((w >> 55) & 1ull), ((w >> 56) & 1ull) != 0, ((w >> 57) & 1ull) != 0,
                      1 << (int32_t)((w >> 58) & 7ull)};
}

// Largest frontier hub chunk count the state word holds (24 bits).
constexpr int64_t kMaxStateChunks = (1 << 24) - 1;

// Block-uniform snapshot of the round state: one load by thread 0, shared
// through LDS.  A block of round r's kernel that starts after the round was
// closed sees round r + 1, whose parity differs from the kernel's: it returns.
__device__ __forceinline__ RoundState read_state(SsspCtl *c) {
    __shared__ unsigned long long s_state;
    if (threadIdx.x == 0) s_state = ld_agent(&c->state);
    __syncthreads();
    return unpack_state(s_state);
}

// Bookkeeping of a vertex that joined the next frontier: its adjacency
// entries count toward the next round's direction choice, and a hub is
// registered for the next round's chunk blocks (list entry plus the owner of
// each of its chunks).
__device__ __forceinline__ void joined(SsspCtl *c, int32_t deg, HubEntry *hn,
                                       int32_t *on, int32_t hub_cap, int32_t chunk_cap, int32_t u,
                                       unsigned long long &my_deg) {
    my_deg += (unsigned long long)deg;
    if (deg > kHubDeg) {
        const int32_t nch = (deg + kHubChunk - 1) / kHubChunk;
        const unsigned long long old =
            atomicAdd(&c->hub_pack_.v, (1ull << 40) | (unsigned long long)nch);
        const int64_t idx = (int64_t)(old >> 40);
        const int64_t base = (int64_t)(old & ((1ull << 40) - 1));
        if (idx >= hub_cap || base + nch > chunk_cap) {
            atomicOr(&c->capacity_.v, 1);
            return;
        }
        hn[idx] = HubEntry{u, 0, (int32_t)base, nch};
        for (int32_t q = 0; q < nch; ++q) on[base + q] = (int32_t)idx;
    }
}

// Last j with off[j] <= k (off ascending, off[0] = 0).
template <int BS>
__device__ __forceinline__ int32_t owner_of(const int32_t *off, int32_t k) {
    int32_t a = 0, z = BS - 1;
    while (a < z) {
        const int32_t mid = (a + z + 1) >> 1;
        if (off[mid] <= k) a = mid; else z = mid - 1;
    }
    return a;
}

template <int BS>
__device__ __forceinline__ int32_t block_min_i32(int32_t x, int32_t *lds) {
    for (int o = 32; o > 0; o >>= 1) x = min(x, __shfl_xor(x, o, kWave));
    if (lane_id() == 0) lds[threadIdx.x / kWave] = x;
    __syncthreads();
    int32_t m = lds[0];
    for (int w = 1; w < BS / kWave; ++w) m = min(m, lds[w]);
    __syncthreads();
    return m;
}

// End of a round (one thread of the last working block): the next frontier
// becomes current, its hubs' chunks become the chunk work, the direction of
// the next round is chosen, or the run ends.  The state word is stored last.
__device__ void close_round(SsspCtl *c, int32_t mode, int32_t n, int32_t hub_cap, int32_t chunk_cap) {
    if (mode == SSSP_PUSH) c->push_rounds++; else c->pull_rounds++;
    const int32_t tail = ld_agent(&c->tail_.v);
    const unsigned long long hp = ld_agent(&c->hub_pack_.v);
    const int64_t nh = (int64_t)(hp >> 40), nch = (int64_t)(hp & ((1ull << 40) - 1));
    const unsigned long long deg = ld_agent(&c->next_deg_.v);
    const int32_t r = c->round + 1;
    c->round = r;
    c->tail_.v = 0;
    c->next_deg_.v = 0;
    c->hub_pack_.v = 0;
    if (tail > n || nh > hub_cap || nch > chunk_cap || nch > kMaxStateChunks) c->capacity_.v = 1;
    const bool done = tail <= 0 || c->capacity_.v;
    int32_t next = SSSP_PUSH;
    if (c->forced >= 0) next = c->forced;
    else if ((double)deg * c->alpha > (double)c->nnz) next = SSSP_PULL;
    c->done = done;
    __hip_atomic_store(&c->state, pack_state(done ? 0 : tail, done ? 0 : (int32_t)nch, r, next, done, deg),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void k_sssp_fill(int32_t *dist, int32_t *stamp, int32_t n) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        dist[v] = kInf;
        stamp[v] = -1;
    }
}

__global__ void k_sssp_init(SsspCtl *c, const int32_t *__restrict__ rp, int32_t *dist, int32_t *stamp, int32_t *q0,
                            HubEntry *h0, int32_t *o0, int32_t src, const int32_t *__restrict__ new_id, int32_t n, long long nnz,
                            int32_t forced, double alpha, int32_t static_chunks) {
    if (new_id) src = new_id[src];
    const int32_t deg = rp[src + 1] - rp[src];
    dist[src] = 0;
    stamp[src] = 0;
    q0[0] = src;
    c->round = 0;
    c->done = 0;
    c->n_vertices = n;
    c->forced = forced;
    c->push_rounds = 0;
    c->pull_rounds = 0;
    c->static_chunks = static_chunks;
    c->nnz = nnz;
    c->alpha = alpha;
    const int32_t nch = deg > kHubDeg ? (deg + kHubChunk - 1) / kHubChunk : 0;
    if (nch) h0[0] = HubEntry{src, 0, 0, nch};
    for (int32_t q = 0; q < nch; ++q) o0[q] = 0;
    c->tail_.v = 0;
    c->overflow_.v = 0;
    c->capacity_.v = 0;
    c->next_deg_.v = 0;
    c->hub_pack_.v = 0;
    c->blocks_done_.v = 0;
    c->reached_.v = 0;
    int32_t mode = SSSP_PUSH;
    if (forced >= 0) mode = forced;
    else if ((double)deg * alpha > (double)nnz) mode = SSSP_PULL;
    c->state = pack_state(1, nch, 0, mode, false, (unsigned long long)deg);
}

// Push round.  Waves work by themselves, without barriers but the last.
// blockIdx.y == 0: a wave takes frontier vertices (hubs excluded; up to 64, fewer
// where that leaves waves idle, but of about kPushStep entries together), lays
// their rows end to end, and walks them 256 entries per step: a lane takes four
// consecutive entries, whose rows one search and a short walk find, so four
// packed entries and then four distances are in flight.  blockIdx.y == 1: a wave
// per chunk of the frontier's hubs.  Entries that may lower their vertex are
// gathered in LDS and settled up to 256 together, the vertices that join the next
// frontier written out in batches, the last one of all the block's waves with
// one atomic: one on the shared tail takes 5 ns of every wave's time (an atomic
// per wave, 262,144 vertices of three entries: 0.93 ms, so 0.53; uniform, 2^20
// vertices, 2.73 and 2.19; rmat-20 1.54 and 1.29).  Against blocks of 256 that
// took an entry per thread between barriers: rmat-22, rows not numbered by rank,
// 4.9 -> 4.15 ms per source, rmat with 8,192 vertices 0.69 -> 0.31.
template <int BS>
__global__ __launch_bounds__(BS) void k_sssp_push(SsspCtl *c, const int32_t *__restrict__ rp,
                                                  const int2 *__restrict__ adj, int32_t *dist,
                                                  int32_t *stamp, int32_t *q0, int32_t *q1, HubEntry *h0,
                                                  HubEntry *h1, int32_t *o0, int32_t *o1,
                                                  int32_t hub_cap, int32_t chunk_cap, int32_t n,
                                                  int32_t parity, unsigned long long *prof) {
    const RoundState st = read_state(c);
    if (st.done || st.pull || st.parity != parity) return;
    constexpr int kWaves = BS / kWave, kFly = 4, kStep = kFly * kWave;
    constexpr int kCand = kStep + kWave, kOut = kStep + kWave;
    __shared__ int32_t s_off[kWaves][kWave + 1], s_beg[kWaves][kWave], s_d[kWaves][kWave];
    __shared__ int2 s_cand[kWaves][kCand];
    __shared__ int32_t s_out[kWaves][kOut], s_left[kWaves], s_base;
    __shared__ unsigned long long s_red[1], s_deg[kWaves];
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int32_t cnt = st.cnt, nch = st.chunks;
    int32_t share = st.share;
    while (share < kWave && (int64_t)gridDim.x * kWaves * share < cnt) share <<= 1;
    const int32_t per = kWaves * share;
    const int nb0 = working_blocks(cnt, per), nb1 = working_blocks(nch, kWaves);
    if ((int)blockIdx.x >= (blockIdx.y == 0 ? nb0 : nb1)) return;
    const int32_t r = c->round;
    const int32_t *qc = parity ? q1 : q0;
    int32_t *qn = parity ? q0 : q1;
    const HubEntry *hc = parity ? h1 : h0;
    HubEntry *hn = parity ? h0 : h1;
    const int32_t *oc = parity ? o1 : o0;
    int32_t *on = parity ? o0 : o1;
    unsigned long long my_deg = 0, my_items = 0, my_edges = 0;
    bool ovf = false;
    int32_t ncand = 0, nout = 0;  // the same in every lane
    auto write_out = [&](int32_t base) {
        for (int32_t i = lane; i < nout; i += kWave) {
            if (base + i < n) qn[base + i] = s_out[wv][i];
            else atomicOr(&c->capacity_.v, 1);
        }
        nout = 0;
    };
    auto flush = [&]() {
        if (nout == 0) return;
        int32_t base = 0;
        if (lane == 0) base = atomicAdd(&c->tail_.v, nout);
        write_out(__builtin_amdgcn_readfirstlane(base));
        __builtin_amdgcn_wave_barrier();
    };
    // settles the last `groups` x 64 candidates together (of the last group, what is there)
    auto settle = [&](auto groups) {
        constexpr int G = decltype(groups)::value;
        const int32_t take_n = min(ncand, (int32_t)(G * kWave));
        ncand -= take_n;
        int2 x[G];
        int32_t deg[G], old[G];
        bool take[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            x[g] = s_cand[wv][ncand + min(g * kWave + lane, take_n - 1)];
            if (G == 1 && lane >= take_n) x[g].y = kInf;  // lowers nothing
        }
#pragma unroll
        for (int g = 0; g < G; ++g) deg[g] = rp[x[g].x + 1] - rp[x[g].x];
#pragma unroll
        for (int g = 0; g < G; ++g) old[g] = dist[x[g].x];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (x[g].y < old[g]) old[g] = atomicMin(&dist[x[g].x], x[g].y);
#pragma unroll
        for (int g = 0; g < G; ++g) take[g] = x[g].y < old[g] && atomicMax(&stamp[x[g].x], r + 1) < r + 1;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (take[g]) joined(c, deg[g], hn, on, hub_cap, chunk_cap, x[g].x, my_deg);
            const unsigned long long m = __ballot(take[g]);
            if (take[g]) s_out[wv][nout + lanes_below(m)] = x[g].x;
            nout += __popcll(m);
            __builtin_amdgcn_wave_barrier();
            if (nout > kOut - kWave) flush();
        }
    };
    auto offer = [&](bool may, int32_t u, int32_t nd) {
        const unsigned long long m = __ballot(may);
        if (may) s_cand[wv][ncand + lanes_below(m)] = make_int2(u, nd);
        ncand += __popcll(m);
    };
    // four entries per lane, loaded together; an entry that is none reads `adj[some]`
    auto relax4 = [&](const int32_t (&e)[kFly], const int32_t (&d)[kFly], int32_t some) {
        int2 x[kFly];
        int32_t old[kFly];
#pragma unroll
        for (int q = 0; q < kFly; ++q) x[q] = adj[e[q] >= 0 ? e[q] : some];
#pragma unroll
        for (int q = 0; q < kFly; ++q) old[q] = dist[x[q].x];
#pragma unroll
        for (int q = 0; q < kFly; ++q) {
            const int32_t nd = e[q] >= 0 ? candidate(d[q], x[q].y, ovf) : kInf;
            offer(nd < old[q], x[q].x, nd);
        }
        __builtin_amdgcn_wave_barrier();
        if (ncand >= 4 * kWave) settle(std::integral_constant<int, 4>{});
        if (ncand >= 2 * kWave) settle(std::integral_constant<int, 2>{});
        while (ncand >= kWave) settle(std::integral_constant<int, 1>{});
    };
    if (blockIdx.y == 0) {
        for (int64_t b = (int64_t)blockIdx.x * per + wv * share; b < cnt; b += (int64_t)gridDim.x * per) {
            const int64_t i = b + lane;
            int32_t beg = 0, deg = 0, d = 0;
            if (i < cnt && lane < share) {
                const int32_t v = qc[i];
                beg = rp[v];
                deg = rp[v + 1] - beg;
                if (deg > kHubDeg) deg = 0;  // its chunks are taken by blockIdx.y == 1
                d = dist[v];
                ++my_items;
                my_edges += (unsigned long long)deg;
            }
            const int32_t incl = wave_incl_scan(deg);
            const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
            s_off[wv][lane] = incl - deg;
            if (lane == 0) s_off[wv][kWave] = total;
            s_beg[wv][lane] = beg;
            s_d[wv][lane] = d;
            __builtin_amdgcn_wave_barrier();
            const int32_t some = __builtin_amdgcn_readlane(beg, __ffsll((long long)(__ballot(deg > 0) | 1ull << 63)) - 1);
            for (int32_t k0 = 0; k0 < total; k0 += kStep) {
                const int32_t k = k0 + lane * kFly;
                int32_t e[kFly], dk[kFly];
                int32_t a = 0, z = kWave - 1;
                while (a < z) {
                    const int32_t mid = (a + z + 1) >> 1;
                    if (s_off[wv][mid] <= k) a = mid; else z = mid - 1;
                }
#pragma unroll
                for (int q = 0; q < kFly; ++q) {
                    e[q] = -1;
                    dk[q] = 0;
                    if (k + q < total) {
                        while (s_off[wv][a + 1] <= k + q) ++a;
                        e[q] = s_beg[wv][a] + (k + q - s_off[wv][a]);
                        dk[q] = s_d[wv][a];
                    }
                }
                relax4(e, dk, some);
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        for (int32_t k = blockIdx.x * kWaves + wv; k < nch; k += gridDim.x * kWaves) {
            const HubEntry h = hc[oc[k]];
            const int32_t beg = rp[h.v] + (k - h.chunk_base) * kHubChunk;
            const int32_t end = min(rp[h.v + 1], beg + kHubChunk);
            const int32_t d = dist[h.v];
            my_edges += lane == 0 ? (unsigned long long)(end - beg) : 0ull;
            for (int32_t e0 = beg; e0 < end; e0 += kStep) {
                int32_t e[kFly], dk[kFly];
#pragma unroll
                for (int q = 0; q < kFly; ++q) {
                    const int32_t at = e0 + q * kWave + lane;
                    e[q] = at < end ? at : -1;
                    dk[q] = d;
                }
                relax4(e, dk, beg);
            }
        }
    }
    while (ncand > 0) settle(std::integral_constant<int, 1>{});
    // what the block's waves have left goes out with one atomic
    const unsigned long long deg = wave_sum_u64(my_deg);
    if (lane == 0) {
        s_left[wv] = nout;
        s_deg[wv] = deg;
    }
    __syncthreads();
    int32_t before = 0;
    for (int w = 0; w < wv; ++w) before += s_left[w];
    if (threadIdx.x == 0) {
        int32_t all = 0;
        unsigned long long all_deg = 0;
        for (int w = 0; w < kWaves; ++w) {
            all += s_left[w];
            all_deg += s_deg[w];
        }
        if (all_deg) atomicAdd(&c->next_deg_.v, all_deg);
        if (all) s_base = atomicAdd(&c->tail_.v, all);
    }
    __syncthreads();
    write_out(s_base + before);
    if (__ballot(ovf) && lane == 0) atomicOr(&c->overflow_.v, 1);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
    if (last_working_block(&c->blocks_done_.v, true, nb0 + nb1) && threadIdx.x == 0)
        close_round(c, SSSP_PUSH, n, hub_cap, chunk_cap);
}

// Push round whose blocks also follow their own lowerings (long rows and an
// explicit local_hops).  blockIdx.y == 0: a block takes BS frontier vertices
// (hubs excluded), scans their row lengths and walks the concatenated rows BS
// entries at a time, one entry per lane.  blockIdx.y == 1: blocks take the
// chunks of the frontier's hubs.
//
// A block follows its own lowerings for up to HOPS more hops inside the
// round: every vertex it lowered goes, with the distance it wrote, into an
// LDS list, and the list is expanded the same way.  Every lowering still
// puts its vertex into the next frontier (first lowering in the round) or
// finds it there already, so the next round expands it with its current
// distance whatever happened locally; the local hops only add relaxations
// from valid path lengths, and the improvements travel up to HOPS + 1 edges
// per round instead of one.
template <int BS, int HOPS>
__global__ __launch_bounds__(BS) void k_sssp_push_hops(SsspCtl *c, const int32_t *__restrict__ rp,
                                                  const int2 *__restrict__ adj, int32_t *dist,
                                                  int32_t *stamp,
                                                  int32_t *q0, int32_t *q1, HubEntry *h0,
                                                  HubEntry *h1, int32_t *o0, int32_t *o1,
                                                  int32_t hub_cap, int32_t chunk_cap, int32_t n,
                                                  int32_t parity, unsigned long long *prof) {
    const RoundState st = read_state(c);
    if (st.done || st.pull || st.parity != parity) return;
    static_assert(HOPS > 0, "k_sssp_push runs rounds without local hops");
    constexpr int kLists = 2, kCap = kLocalCap;
    __shared__ int32_t s_beg[BS], s_off[BS], s_d[BS], s_scan[BS / kWave + 1];
    __shared__ int32_t s_qbuf[4 * BS], s_meta[2];
    __shared__ int32_t s_lv[kLists][kCap], s_ld[kLists][kCap], s_ln[2];
    __shared__ unsigned long long s_red[1];
    const int32_t r = c->round, cnt = st.cnt, nch = st.chunks;
    const int32_t *qc = parity ? q1 : q0;
    int32_t *qn = parity ? q0 : q1;
    const HubEntry *hc = parity ? h1 : h0;
    HubEntry *hn = parity ? h0 : h1;
    const int32_t *oc = parity ? o1 : o0;
    int32_t *on = parity ? o0 : o1;
    StagedQueue<BS, 4 * BS> q;
    q.init(s_qbuf, s_meta);
    unsigned long long my_deg = 0, my_items = 0, my_edges = 0;
    bool ovf = false;
    const int nb0 = working_blocks(cnt, BS);
    const int nb1 = (int)min((int64_t)gridDim.x, (int64_t)nch);
    // Expands the rows held by the block's threads (row start, length, the
    // distance to extend): scan, walk one entry per lane, relax; lowered
    // vertices go to local list `dst` when dst >= 0.  All threads call it.
    auto walk = [&](int32_t beg, int32_t deg, int32_t d, int dst) {
        int32_t total;
        const int32_t off = block_excl_scan<BS>(deg, s_scan, &total);
        s_beg[threadIdx.x] = beg;
        s_off[threadIdx.x] = off;
        s_d[threadIdx.x] = d;
        __syncthreads();
        for (int32_t k0 = 0; k0 < total; k0 += BS) {
            const int32_t k = k0 + threadIdx.x;
            bool take = false;
            int32_t u = 0;
            if (k < total) {
                const int32_t a = owner_of<BS>(s_off, k);
                const int2 e = adj[s_beg[a] + (k - s_off[a])];
                u = e.x;
                const int32_t nd = candidate(s_d[a], e.y, ovf);
                bool lowered;
                take = relax_push(dist, stamp, u, nd, r, lowered);
                if (take) joined(c, rp[u + 1] - rp[u], hn, on, hub_cap, chunk_cap, u, my_deg);
                if (dst >= 0 && lowered) {
                    const int32_t at = atomicAdd(&s_ln[dst], 1);
                    if (at < kCap) {
                        s_lv[dst][at] = u;
                        s_ld[dst][at] = nd;
                    }
                }
            }
            q.stage(take, u, &c->tail_.v, qn, n, &c->capacity_.v);
        }
        __syncthreads();
    };
    bool working;
    if (blockIdx.y == 0) {
        working = (int)blockIdx.x < nb0;
        for (int32_t b = blockIdx.x * BS; b < cnt; b += gridDim.x * BS) {
            const int32_t i = b + threadIdx.x;
            int32_t beg = 0, deg = 0, d = 0;
            if (i < cnt) {
                const int32_t v = qc[i];
                beg = rp[v];
                deg = rp[v + 1] - beg;
                if (deg > kHubDeg) deg = 0;  // its chunks are taken by blockIdx.y == 1
                d = dist[v];
                ++my_items;
                my_edges += (unsigned long long)deg;
            }
            if (threadIdx.x == 0) s_ln[0] = 0;  // seen after the scan's barrier
            walk(beg, deg, d, 0);
            int cur = 0;
            for (int hop = 0; hop < HOPS; ++hop) {
                const int32_t ln = min(s_ln[cur], kCap);
                if (ln == 0) break;
                const int nxt = cur ^ 1;
                if (threadIdx.x == 0) s_ln[nxt] = 0;
                for (int32_t lb = 0; lb < ln; lb += BS) {
                    const int32_t j = lb + threadIdx.x;
                    int32_t lbeg = 0, ldeg = 0, ld = 0;
                    if (j < ln) {
                        const int32_t v = s_lv[cur][j];
                        ld = s_ld[cur][j];
                        lbeg = rp[v];
                        ldeg = rp[v + 1] - lbeg;
                        if (ldeg > kHubDeg) ldeg = 0;  // already in the next frontier
                        ++my_items;
                        my_edges += (unsigned long long)ldeg;
                    }
                    walk(lbeg, ldeg, ld, hop + 1 < HOPS ? nxt : -1);
                }
                cur = nxt;
            }
        }
    } else {
        working = (int)blockIdx.x < nb1;
        for (int32_t k = blockIdx.x; k < nch; k += gridDim.x) {
            const HubEntry h = hc[oc[k]];
            const int32_t beg = rp[h.v] + (k - h.chunk_base) * kHubChunk;
            const int32_t end = min(rp[h.v + 1], beg + kHubChunk);
            const int32_t d = dist[h.v];
            my_edges += threadIdx.x == 0 ? (unsigned long long)(end - beg) : 0ull;
            for (int32_t e0 = beg; e0 < end; e0 += BS) {
                const int32_t e = e0 + threadIdx.x;
                bool take = false;
                int32_t u = 0;
                if (e < end) {
                    const int2 x = adj[e];
                    u = x.x;
                    bool lowered;
                    take = relax_push(dist, stamp, u, candidate(d, x.y, ovf), r, lowered);
                    if (take) joined(c, rp[u + 1] - rp[u], hn, on, hub_cap, chunk_cap, u, my_deg);
                }
                q.stage(take, u, &c->tail_.v, qn, n, &c->capacity_.v);
            }
        }
    }
    q.finish(&c->tail_.v, qn, n, &c->capacity_.v);
    if (__ballot(ovf) && lane_id() == 0) atomicOr(&c->overflow_.v, 1);
    block_add_u64<BS>(my_deg, s_red, &c->next_deg_.v);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
    if (last_working_block(&c->blocks_done_.v, working, nb0 + nb1) && threadIdx.x == 0)
        close_round(c, SSSP_PUSH, n, hub_cap, chunk_cap);
}

// Push round on graphs whose rows all hold at most 8 entries (sssp_mesh_rows),
// where rounds are many and small, and what a round costs is the length of
// its chain of dependent memory operations.  Each wave works by itself, without
// barriers: it takes up to 64 frontier vertices, then follows its own lowerings
// for `hops` more steps through a ring in LDS.  A step is one memory round
// trip: a lane holds {vertex, distance, row}, lowers its neighbours with
// atomicMin, and loads the neighbours' rows in the same breath, so that a
// lowered neighbour enters the ring with its row (W = 4; rows of 8 are loaded
// on the next step).  The fixed-width rows spare the offsets, the value that
// atomicMin returns the read before it, and only what the ring cannot hold or
// the last step lowered is put into the next frontier: every lowering is
// expanded at its distance by the wave that made it or, from the frontier, at
// the distance then current, so the rounds end at the same least fixed point.
// road-1501: a hop took 4 us in the general kernel's chain of six operations
// and two barriers, 13.7 ms in all; here a
// step takes 1.6 us, 4.8 ms in all (starting waves on 32, 16, 8, 4 vertices: 5.4, 5.0, 4.8, 4.8 ms).
constexpr int kMeshRing = 128;  // entries per wave
template <int BS, int W>
__global__ __launch_bounds__(BS) void k_sssp_mesh(SsspCtl *c, const int2 *__restrict__ ell, int32_t *dist,
                                                  int32_t *stamp,
                                                  int32_t *q0, int32_t *q1, int32_t n, int32_t hops,
                                                  int32_t parity, unsigned long long *prof) {
    const RoundState st = read_state(c);
    if (st.done || st.pull || st.parity != parity) return;
    constexpr int kWaves = BS / kWave;
    constexpr bool kCarry = W <= 4;  // rows travel with the ring's entries
    struct Row {
        int4 part[W / 2];  // {id, weight, id, weight}; id -1 past the row's end
    };
    __shared__ int2 s_vd[kWaves][kMeshRing];
    __shared__ Row s_row[kCarry ? kWaves : 1][kCarry ? kMeshRing : 1];
    __shared__ unsigned long long s_red[1];
    const int lane = lane_id(), wv = threadIdx.x / kWave;
    const int32_t r = c->round, cnt = st.cnt;
    const int32_t *qc = parity ? q1 : q0;
    int32_t *qn = parity ? q0 : q1;
    unsigned long long my_items = 0, my_edges = 0;
    bool ovf = false;
    // frontier vertices per wave: few enough to use every wave, from kMeshLeast up
    int32_t share = kMeshLeast;
    while (share < kWave && (int64_t)gridDim.x * kWaves * share < cnt) share <<= 1;
    const int32_t per = kWaves * share;
    auto row_of = [&](int32_t v) {
        Row x;
        const int4 *p = reinterpret_cast<const int4 *>(ell + (int64_t)v * W);
#pragma unroll
        for (int k = 0; k < W / 2; ++k) x.part[k] = p[k];
        return x;
    };
    // the lanes' vertices join the next frontier, each once per round
    auto leave = [&](bool take, int32_t u) {
        if (take) take = atomicMax(&stamp[u], r + 1) < r + 1;
        const unsigned long long m = __ballot(take);
        if (!m) return;
        const int leader = __ffsll((long long)m) - 1;
        int32_t at = 0;
        if (lane == leader) at = atomicAdd(&c->tail_.v, __popcll(m));
        at = shfl_i32(at, leader) + lanes_below(m);
        if (take) {
            if (at < n) qn[at] = u;
            else atomicOr(&c->capacity_.v, 1);
        }
    };
    for (int64_t b = (int64_t)blockIdx.x * per; b < cnt; b += (int64_t)gridDim.x * per) {
        const int64_t i = b + wv * share + lane;
        bool has = i < cnt && lane < share;
        int32_t v = 0, d = 0;
        Row row;
        if (has) {
            v = qc[i];
            d = dist[v];
            row = row_of(v);
        }
        uint32_t head = 0, tail = 0;  // ring positions, the same in every lane
        for (int32_t step = 0; __ballot(has); ++step) {
            int32_t to[W], nd[W], old[W];
            Row nrow[kCarry ? W : 1];
            if (has) {
                ++my_items;
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    const int4 q = row.part[k / 2];
                    const int32_t id = k & 1 ? q.z : q.x, w = k & 1 ? q.w : q.y;
                    my_edges += id >= 0;
                    // past the row's end: the vertex itself, which INT32_MAX does not lower
                    to[k] = id >= 0 ? id : v;
                    nd[k] = id >= 0 ? candidate(d, w, ovf) : kInf;
                }
#pragma unroll
                for (int k = 0; k < W; ++k) old[k] = atomicMin(&dist[to[k]], nd[k]);
                if (kCarry) {
#pragma unroll
                    for (int k = 0; k < W; ++k) nrow[k] = row_of(to[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const bool low = has && nd[k] < old[k];
                const unsigned long long m = __ballot(low);
                if (!m) continue;
                const uint32_t at = tail + (uint32_t)lanes_below(m);
                const bool fits = at - head < (uint32_t)kMeshRing;
                if (low && fits) {
                    s_vd[wv][at % kMeshRing] = make_int2(to[k], nd[k]);
                    if (kCarry) s_row[wv][at % kMeshRing] = nrow[k];
                }
                tail = min(tail + (uint32_t)__popcll(m), head + (uint32_t)kMeshRing);
                if (__ballot(low && !fits)) leave(low && !fits, to[k]);
            }
            __builtin_amdgcn_wave_barrier();
            if (step >= hops) break;
            const uint32_t left = min(tail - head, (uint32_t)kWave);
            has = (uint32_t)lane < left;
            if (has) {
                const int2 x = s_vd[wv][(head + lane) % kMeshRing];
                v = x.x;
                d = x.y;
                row = kCarry ? s_row[wv][(head + lane) % kMeshRing] : row_of(v);
            }
            head += left;
            __builtin_amdgcn_wave_barrier();
        }
        while (head != tail) {
            const uint32_t left = min(tail - head, (uint32_t)kWave);
            const bool mine = (uint32_t)lane < left;
            leave(mine, mine ? s_vd[wv][(head + lane) % kMeshRing].x : 0);
            head += left;
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (__ballot(ovf) && lane == 0) atomicOr(&c->overflow_.v, 1);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
    const int nb = working_blocks(cnt, per);
    if (last_working_block(&c->blocks_done_.v, (int)blockIdx.x < nb, nb) && threadIdx.x == 0)
        close_round(c, SSSP_PUSH, n, 1, 1);
}

// Rows of at most W entries at a fixed width: {neighbour, weight}, {-1, 0} past the end.
template <int W>
__global__ void k_sssp_mesh_rows(const int32_t *__restrict__ rp, const int2 *__restrict__ adj, int32_t n,
                                 int2 *ell) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (int64_t)n * W; i += stride) {
        const int32_t v = (int32_t)(i / W), k = (int32_t)(i % W);
        const int32_t b = rp[v];
        ell[i] = k < rp[v + 1] - b ? adj[b + k] : make_int2(-1, 0);
    }
}

// Pull round.  blockIdx.y == 0: a block takes BS consecutive vertices (hubs
// excluded), walks their concatenated rows one entry per lane, and folds each
// entry's candidate into its vertex's LDS minimum; each vertex then stores
// the minimum when it is lower (only its own thread writes it).
// blockIdx.y == 1: blocks take the chunks of every hub of the graph, reduce a
// chunk to its minimum and lower the hub with atomicMin.
//
// An entry takes one gather, the neighbour's distance.  Passing over neighbours
// that were not lowered takes their stamps too, two gathers for most entries of
// the rounds that are worth a pull, and a compare with the vertex's minimum drops
// their offers as well.  All rounds pulled, and alpha 50, us: rmat-20 3,053 and
// 2,217, so 2,772 and 1,786; rmat, 10^6 vertices, 2,471 and 2,084, so 2,179 and
// 1,657; 750,000 vertices, 1,833 and 1,241, so 1,671 and 1,091.
template <int BS>
__global__ __launch_bounds__(BS) void k_sssp_pull(SsspCtl *c, const int32_t *__restrict__ rp,
                                                  const int2 *__restrict__ adj, int32_t *dist,
                                                  int32_t *stamp,
                                                  int32_t *q0, int32_t *q1, HubEntry *h0,
                                                  HubEntry *h1, int32_t *o0, int32_t *o1,
                                                  int32_t hub_cap, int32_t chunk_cap, int32_t n,
                                                  const HubEntry *__restrict__ hs,
                                                  const int32_t *__restrict__ os, int32_t heavy, int32_t parity,
                                                  unsigned long long *prof) {
    const RoundState st = read_state(c);
    if (st.done || !st.pull || st.parity != parity) return;
    __shared__ int32_t s_beg[BS], s_off[BS], s_best[BS], s_scan[BS / kWave + 1];
    __shared__ int32_t s_qbuf[4 * BS], s_meta[2], s_min[BS / kWave];
    __shared__ unsigned long long s_red[1];
    const int32_t r = c->round, nch = c->static_chunks;
    int32_t *qn = parity ? q0 : q1;
    HubEntry *hn = parity ? h0 : h1;
    int32_t *on = parity ? o0 : o1;
    StagedQueue<BS, 4 * BS> q;
    q.init(s_qbuf, s_meta);
    unsigned long long my_deg = 0, my_items = 0, my_edges = 0;
    bool ovf = false;
    // rows numbered by rank: few of the `heavy` first ones a tile, which hold the long ones side by side
    // (from 16 entries on; all pulled, like the others and so: rmat-21 5.3 and 4.6 ms, rmat-22 11.5 and 11.1,
    // 2^21 vertices and edge factor 4 3.8 and 1.9)
    constexpr int kFew = BS / 8;
    const int32_t heavy_tiles = (heavy + kFew - 1) / kFew;
    const int32_t tiles = heavy_tiles + (n - heavy + BS - 1) / BS;
    const int nb0 = working_blocks(tiles, 1);
    const int nb1 = (int)min((int64_t)gridDim.x, (int64_t)nch);
    bool working;
    if (blockIdx.y == 0) {
        working = (int)blockIdx.x < nb0;
        for (int32_t b = blockIdx.x; b < tiles; b += gridDim.x) {
            const bool few = b < heavy_tiles;
            const int32_t v = few ? b * kFew + (int32_t)threadIdx.x : heavy + (b - heavy_tiles) * BS + (int32_t)threadIdx.x;
            int32_t beg = 0, deg = 0;
            if (few ? (int)threadIdx.x < kFew && v < heavy : v < n) {
                beg = rp[v];
                deg = rp[v + 1] - beg;
                if (deg > kHubDeg) deg = 0;  // its chunks are taken by blockIdx.y == 1
                ++my_items;
                my_edges += (unsigned long long)deg;
            }
            int32_t total;
            const int32_t off = block_excl_scan<BS>(deg, s_scan, &total);
            const int32_t own = deg > 0 ? dist[v] : kInf;
            s_beg[threadIdx.x] = beg;
            s_off[threadIdx.x] = off;
            s_best[threadIdx.x] = own;
            __syncthreads();
            for (int32_t k0 = 0; k0 < total; k0 += BS) {
                const int32_t k = k0 + threadIdx.x;
                if (k < total) {
                    const int32_t a = owner_of<BS>(s_off, k);
                    const int2 e = adj[s_beg[a] + (k - s_off[a])];
                    const int32_t d = dist[e.x];
                    const int32_t nd = d != kInf ? candidate(d, e.y, ovf) : kInf;
                    if (nd < s_best[a]) atomicMin(&s_best[a], nd);
                }
            }
            __syncthreads();
            bool take = false;
            if (deg > 0) {
                const int32_t best = s_best[threadIdx.x];
                if (best < own) {
                    dist[v] = best;
                    stamp[v] = r + 1;
                    take = true;
                    joined(c, deg, hn, on, hub_cap, chunk_cap, v, my_deg);
                }
            }
            q.stage(take, v, &c->tail_.v, qn, n, &c->capacity_.v);
        }
    } else {
        working = (int)blockIdx.x < nb1;
        for (int32_t k = blockIdx.x; k < nch; k += gridDim.x) {
            const HubEntry h = hs[os[k]];
            const int32_t beg = rp[h.v] + (k - h.chunk_base) * kHubChunk;
            const int32_t end = min(rp[h.v + 1], beg + kHubChunk);
            my_edges += threadIdx.x == 0 ? (unsigned long long)(end - beg) : 0ull;
            int32_t m = kInf;
            for (int32_t e = beg + threadIdx.x; e < end; e += BS) {
                const int2 x = adj[e];
                const int32_t du = dist[x.x];
                if (du != kInf) m = min(m, candidate(du, x.y, ovf));
            }
            m = block_min_i32<BS>(m, s_min);
            bool take = false;
            if (threadIdx.x == 0 && m < dist[h.v]) {
                const int32_t old = atomicMin(&dist[h.v], m);
                take = m < old && atomicMax(&stamp[h.v], r + 1) < r + 1;
                if (take) joined(c, rp[h.v + 1] - rp[h.v], hn, on, hub_cap, chunk_cap, h.v, my_deg);
            }
            q.stage(take, h.v, &c->tail_.v, qn, n, &c->capacity_.v);
        }
    }
    q.finish(&c->tail_.v, qn, n, &c->capacity_.v);
    if (__ballot(ovf) && lane_id() == 0) atomicOr(&c->overflow_.v, 1);
    block_add_u64<BS>(my_deg, s_red, &c->next_deg_.v);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
    if (last_working_block(&c->blocks_done_.v, working, nb0 + nb1) && threadIdx.x == 0)
        close_round(c, SSSP_PULL, n, hub_cap, chunk_cap);
}

// After the rounds, when some candidate saturated: a reached vertex with an
// unreached neighbour means that neighbour's distance is INT32_MAX or more
// (every relaxation into it saturated), which int32 cannot hold.
__global__ void k_sssp_unfit(SsspCtl *c, const int32_t *__restrict__ rp,
                             const int2 *__restrict__ adj, const int32_t *__restrict__ dist, int32_t n) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t u = blockIdx.x * blockDim.x + threadIdx.x; u < n; u += stride) {
        if (dist[u] == kInf) continue;
        for (int32_t e = rp[u]; e < rp[u + 1]; ++e)
            if (dist[adj[e].x] == kInf) {
                atomicOr(&c->capacity_.v, 2);
                return;
            }
    }
}

// Distances to the caller's buffer, and the count of reached vertices.
__global__ void k_sssp_export(SsspCtl *c, const int32_t *__restrict__ dist,
                              const int32_t *__restrict__ new_id, int32_t *out, int32_t n) {
    __shared__ unsigned long long s_red[1];
    unsigned long long reached = 0;
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const int32_t d = dist[new_id ? new_id[v] : v];
        out[v] = d;
        reached += d != kInf;
    }
    block_add_u64<256>(reached, s_red, &c->reached_.v);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Rows [first, last) of the rank numbering, PER lanes each: {rank of the
// neighbour, weight}; counts weights outside [0, INT32_MAX - 1].  The ranks are
// those of the earlier weights' rows, where there are some (`before`).
template <int BS, int PER>
__global__ __launch_bounds__(BS) void k_sssp_pack_ranked(const int32_t *__restrict__ rp,
                                                          const int32_t *__restrict__ ci,
                                                          const int32_t *__restrict__ w,
                                                          const int32_t *__restrict__ rank_new,
                                                          const int32_t *__restrict__ rank_old,
                                                          const int32_t *__restrict__ wrp,
                                                          const int2 *__restrict__ before, int32_t first,
                                                          int32_t last, int2 *adjw, unsigned int *bad) {
    unsigned int b = 0;
    const int64_t stride = (int64_t)gridDim.x * (BS / PER);
    for (int64_t r = first + (int64_t)blockIdx.x * (BS / PER) + threadIdx.x / PER; r < last; r += stride) {
        const int32_t at = rp[rank_old[r]], to = wrp[r], len = wrp[r + 1] - to;
        constexpr int kFly = 4;  // a long row is one block's: with a load at a time rmat-20 took 330 us for them, not 190
        for (int32_t k = threadIdx.x % PER; k < len; k += kFly * PER) {
            int32_t x[kFly], u[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) {
                const int32_t j = min(k + q * PER, len - 1);
                x[q] = w[at + j];
                u[q] = before ? before[to + j].x : ci[at + j];
            }
            if (!before) {
#pragma unroll
                for (int q = 0; q < kFly; ++q) u[q] = rank_new[u[q]];
            }
#pragma unroll
            for (int q = 0; q < kFly; ++q)
                if (k + q * PER < len) {
                    if (x[q] < 0 || x[q] == kInf) ++b;
                    adjw[to + k + q * PER] = make_int2(u[q], x[q]);
                }
        }
    }
    if (b) atomicAdd(bad, b);
}

// Pushes on a large skewed graph are bound by their reads of the neighbours'
// distances, mostly those of the heaviest vertices: numbered by rank these
// fill consecutive lines, and the distances of the first million ranks (98% of
// the entries on rmat-22) fit an XCD's 4 MB L2.  rmat-22: 4.15 -> 3.11 ms per
// source (kRenumberFrom).
sp_status sssp_pack_ranked(sp_graph g, const int32_t *weights, int2 *adjw, unsigned int *bad, bool *ranked,
                           hipStream_t s) {
    const int32_t n = g->n;
    if (n <= kRenumberFrom || g->max_degree <= 8 || !may_be_skewed(g)) return SP_OK;
    {
        std::lock_guard<std::mutex> lk(g->mu);
        sp_status st = ensure_rank_locked(g, s);
        if (st == SP_OK && !rank_skewed(g)) return SP_OK;
        if (st == SP_OK) st = ensure_rank_rp_locked(g, s);
        if (st == SP_ERR_OUT_OF_MEMORY) {
            clear_error();
            return SP_OK;
        }
        if (st != SP_OK) return st;
    }
    const int2 *before = g->sssp_ranked ? g->adjw : nullptr;
    const int maxb = device_cu_count() * 8;
    auto pack = [&](auto kernel, int block, int rows_per_block, int32_t first, int32_t last) {
        if (last > first)
            hipLaunchKernelGGL(kernel, dim3(grid_for((int64_t)last - first, rows_per_block, maxb)), dim3(block), 0, s,
                               (const int32_t *)g->row_ptr, (const int32_t *)g->col_idx, weights,
                               (const int32_t *)g->rank_new, (const int32_t *)g->rank_old,
                               (const int32_t *)g->rank_rp, before, first, last, adjw, bad);
    };
    const int32_t longest = rank_count(g, 8192), longer = rank_count(g, kRankExact);
    pack(k_sssp_pack_ranked<1024, 1024>, 1024, 1, 0, longest);
    pack(k_sssp_pack_ranked<256, 256>, 256, 1, longest, longer);
    pack(k_sssp_pack_ranked<256, 16>, 256, 16, longer, n);
    SP_HIP(hipGetLastError());
    *ranked = true;
    return SP_OK;
}

// Offsets of the rows of g->adjw.
static const int32_t *weighted_rows(sp_graph g) { return g->sssp_ranked ? g->rank_rp : g->row_ptr; }

int32_t sssp_mesh_width(sp_graph g) { return g->max_degree > 8 || g->n == 0 ? 0 : g->max_degree <= 4 ? 4 : 8; }

void launch_mesh_rows(sp_graph g, const int2 *adjw, int32_t width, int2 *ell, hipStream_t s) {
    auto fill = width == 4 ? k_sssp_mesh_rows<4> : k_sssp_mesh_rows<8>;
    hipLaunchKernelGGL(fill, dim3(grid_for((int64_t)g->n * width, 256, 8192)), dim3(256), 0, s,
                       (const int32_t *)g->row_ptr, adjw, g->n, ell);
}

sp_status sssp_ws_create(sp_graph g, SsspWorkspace &ws) {
    const int32_t n = std::max(g->n, 1);
    const size_t hubs = (size_t)g->n_hubs + 1, chunks = (size_t)g->hub_chunks + 1;
    ws.n = g->n;
    SP_HIP(hipGetDevice(&ws.device));
    auto fail = [&](sp_status st) {
        sssp_ws_destroy(ws);
        return st;
    };
    sp_status st = dev_alloc((void **)&ws.dist, sizeof(int32_t) * (size_t)n);
    if (st == SP_OK) st = dev_alloc((void **)&ws.stamp, sizeof(int32_t) * (size_t)n);
    if (st == SP_OK) st = dev_alloc((void **)&ws.queue[0], sizeof(int32_t) * (size_t)n);
    if (st == SP_OK) st = dev_alloc((void **)&ws.queue[1], sizeof(int32_t) * (size_t)n);
    if (st == SP_OK) st = dev_alloc((void **)&ws.hubs[0], sizeof(HubEntry) * hubs);
    if (st == SP_OK) st = dev_alloc((void **)&ws.hubs[1], sizeof(HubEntry) * hubs);
    if (st == SP_OK) st = dev_alloc((void **)&ws.owner[0], sizeof(int32_t) * chunks);
    if (st == SP_OK) st = dev_alloc((void **)&ws.owner[1], sizeof(int32_t) * chunks);
    if (st == SP_OK) st = dev_alloc((void **)&ws.ctl, sizeof(SsspCtl));
    if (st != SP_OK) return fail(st);
    if (hipHostMalloc((void **)&ws.ctl_host, sizeof(SsspCtl), hipHostMallocDefault) != hipSuccess) {
        ws.ctl_host = nullptr;
        set_error("pinned host allocation failed");
        return fail(SP_ERR_OUT_OF_MEMORY);
    }
    if (hipEventCreate(&ws.ev0) != hipSuccess || hipEventCreate(&ws.ev1) != hipSuccess) {
        set_error("hipEventCreate failed");
        return fail(SP_ERR_DEVICE);
    }
    return SP_OK;
}

void sssp_ws_destroy(SsspWorkspace &ws) {
    if (ws.rounds_short.exec) (void)hipGraphExecDestroy(ws.rounds_short.exec);
    if (ws.rounds_long.exec) (void)hipGraphExecDestroy(ws.rounds_long.exec);
    if (ws.cap_stream) (void)hipStreamDestroy(ws.cap_stream);
    dev_free(ws.dist);
    dev_free(ws.stamp);
    dev_free(ws.queue[0]);
    dev_free(ws.queue[1]);
    dev_free(ws.hubs[0]);
    dev_free(ws.hubs[1]);
    dev_free(ws.owner[0]);
    dev_free(ws.owner[1]);
    dev_free(ws.ctl);
    if (ws.ctl_host) (void)hipHostFree(ws.ctl_host);
    if (ws.ev0) (void)hipEventDestroy(ws.ev0);
    if (ws.ev1) (void)hipEventDestroy(ws.ev1);
    ws = SsspWorkspace{};
}

// `rounds` rounds starting at an even round: each round launches its push
// and/or pull kernel with the round's parity, and a kernel runs only while the
// control block is at a round of that parity.  A block of round r's kernel
// that starts after the round was closed therefore sees round r + 1 and
// returns, instead of taking part in a round that is not its own.
template <int BS, int HOPS>
static void enqueue_rounds(sp_graph g, SsspWorkspace &ws, int rounds, int grid, bool hubs,
                           bool may_pull, bool may_push, hipStream_t s) {
    const int32_t hub_cap = g->n_hubs + 1, chunk_cap = (int32_t)g->hub_chunks + 1, n = g->n;
    const int32_t *rp = weighted_rows(g);
    for (int k = 0; k < rounds; ++k) {
        const int32_t parity = k & 1;
        if (HOPS > 0 && g->sssp_ell && may_push) {  // rows of at most 8 entries, local hops
            ProfScope ps(P_SSSP_PUSH, s);
            auto mesh = g->sssp_ell_w == 4 ? k_sssp_mesh<BS, 4> : k_sssp_mesh<BS, 8>;
            hipLaunchKernelGGL(mesh, dim3(grid), dim3(BS), 0, s, ws.ctl, (const int2 *)g->sssp_ell, ws.dist, ws.stamp, ws.queue[0],
                               ws.queue[1], n, (int32_t)HOPS, parity, prof_counters(P_SSSP_PUSH));
        } else if (may_push) {
            ProfScope ps(P_SSSP_PUSH, s);
            auto push = k_sssp_push<BS>;
            if constexpr (HOPS > 0) push = k_sssp_push_hops<BS, HOPS>;
            hipLaunchKernelGGL(push, dim3(grid, hubs ? 2 : 1), dim3(BS), 0, s, ws.ctl,
                               (const int32_t *)rp, (const int2 *)g->adjw, ws.dist, ws.stamp, ws.queue[0],
                               ws.queue[1], ws.hubs[0], ws.hubs[1], ws.owner[0], ws.owner[1],
                               hub_cap, chunk_cap, n, parity, prof_counters(P_SSSP_PUSH));
        }
        if (may_pull) {
            ProfScope ps(P_SSSP_PULL, s);
            hipLaunchKernelGGL(k_sssp_pull<BS>, dim3(grid, hubs ? 2 : 1), dim3(BS), 0, s, ws.ctl,
                               (const int32_t *)rp, (const int2 *)g->adjw, ws.dist, ws.stamp, ws.queue[0],
                               ws.queue[1], ws.hubs[0], ws.hubs[1], ws.owner[0], ws.owner[1],
                               hub_cap, chunk_cap, n, (const HubEntry *)g->hub_static,
                               (const int32_t *)g->owner_static, g->sssp_ranked ? rank_count(g, 16) : 0, parity,
                               prof_counters(P_SSSP_PULL));
        }
    }
}

template <int BS, int HOPS>
static sp_status sssp_run_bs(sp_graph g, SsspWorkspace &ws, int32_t src, int32_t *out_dist,
                             const SsspOpts &o, hipStream_t s, SsspResult *res) {
    const int32_t n = g->n;
    const int maxb = o.max_blocks > 0 ? o.max_blocks : device_cu_count() * 8;
    const int grid = grid_for((int64_t)n, BS, maxb);
    const bool hubs = g->n_hubs > 0;
    // Automatic choice never pulls on sparse meshes (every row at most 8 long),
    // nor when alpha <= 1 (a frontier's entries never exceed the graph's).
    const bool may_pull = o.forced == SSSP_PULL || (o.forced < 0 && o.alpha > 1.0 && g->max_degree > 8);
    const bool may_push = o.forced != SSSP_PULL;
    const int forced = may_pull ? o.forced : SSSP_PUSH;
    hipLaunchKernelGGL(k_sssp_fill, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, ws.dist, ws.stamp, n);
    const int32_t *rp = weighted_rows(g), *new_id = g->sssp_ranked ? (const int32_t *)g->rank_new : nullptr;
    hipLaunchKernelGGL(k_sssp_init, dim3(1), dim3(1), 0, s, ws.ctl, rp, ws.dist, ws.stamp, ws.queue[0], ws.hubs[0],
                       ws.owner[0], src, new_id, n, (long long)g->nnz,
                       forced, o.alpha, (int32_t)g->hub_chunks);
    SP_HIP(hipGetLastError());
    const bool capture = o.chunk_rounds > 0 && !prof_enabled();
    int32_t enqueued = 0, chunks = 0, graph_launches = 0;
    for (;;) {
        const bool deep = chunks >= 4;
        const int base = std::max(1, std::abs(o.chunk_rounds));
        const int chunk = (base + (base & 1)) * (deep ? 4 : 1);  // even: parity holds
        if (capture) {
            const std::array<long long, 12> key = {
                BS * 16 + HOPS, grid, hubs, may_pull, may_push, chunk, (long long)(intptr_t)ws.dist,
                (long long)(intptr_t)ws.ctl, g->weight_gen, 0, 0, 0};
            SP_TRY(replay_captured(&ws.cap_stream, deep ? ws.rounds_long : ws.rounds_short, key,
                                   [&](hipStream_t cs) {
                                       enqueue_rounds<BS, HOPS>(g, ws, chunk, grid, hubs, may_pull, may_push, cs);
                                   },
                                   s));
            ++graph_launches;
        } else {
            enqueue_rounds<BS, HOPS>(g, ws, chunk, grid, hubs, may_pull, may_push, s);
            SP_HIP(hipGetLastError());
        }
        enqueued += chunk;
        ++chunks;
        SP_HIP(hipMemcpyAsync(ws.ctl_host, ws.ctl, sizeof(SsspCtl), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        if (ws.ctl_host->done) break;
        // Round k leaves every distance of a shortest path of at most k + 1
        // edges final, so n + 1 rounds always suffice.
        if (enqueued > n + 2 + chunk) {
            set_error("SSSP did not converge after %d rounds", enqueued);
            return SP_ERR_DEVICE;
        }
    }
    const SsspCtl &c = *ws.ctl_host;
    if (res) {
        res->rounds = c.push_rounds + c.pull_rounds;
        res->push_rounds = c.push_rounds;
        res->pull_rounds = c.pull_rounds;
        res->graph_launches = graph_launches;
    }
    if (c.capacity_.v) {
        set_error("SSSP frontier capacity exceeded (internal error)");
        return SP_ERR_DEVICE;
    }
    if (c.overflow_.v) {
        hipLaunchKernelGGL(k_sssp_unfit, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, ws.ctl,
                           rp, (const int2 *)g->adjw, (const int32_t *)ws.dist, n);
        SP_HIP(hipGetLastError());
        int32_t unfit = 0;
        SP_HIP(hipMemcpyAsync(&unfit, &ws.ctl->capacity_.v, sizeof(unfit), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        if (unfit) {
            if (res) res->overflow = true;
            set_error("a shortest-path length reaches INT32_MAX; distances do not fit in int32");
            return SP_ERR_NOT_SUPPORTED;
        }
    }
    // (512 blocks: each ends in an atomic on one counter, 4,096 of them took 55 us)
    hipLaunchKernelGGL(k_sssp_export, dim3(grid_for(n, 256, 512)), dim3(256), 0, s, ws.ctl,
                       (const int32_t *)ws.dist, new_id, out_dist, n);
    SP_HIP(hipGetLastError());
    if (res) {
        unsigned long long reached = 0;
        SP_HIP(hipMemcpyAsync(&reached, &ws.ctl->reached_.v, sizeof(reached), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        res->reached = (int32_t)reached;
    }
    return SP_OK;
}

template <int HOPS>
static sp_status sssp_run_hops(sp_graph g, SsspWorkspace &ws, int32_t src, int32_t *out_dist,
                               const SsspOpts &o, hipStream_t s, SsspResult *res) {
    switch (o.block) {
        case 128: return sssp_run_bs<128, HOPS>(g, ws, src, out_dist, o, s, res);
        case 512: return sssp_run_bs<512, HOPS>(g, ws, src, out_dist, o, s, res);
        default: return sssp_run_bs<256, HOPS>(g, ws, src, out_dist, o, s, res);
    }
}

int sssp_local_hops(sp_graph g, int requested) {
    if (requested < 0) return 0;
    if (requested > 0) return requested;
    // automatic: graphs of short rows only (many small rounds); hub rows
    // never go through the local lists
    // (measured on road-4096: 4 hops 98 ms per source, 8: 73, 16: 51, 32: 43,
    // 64: 44, 128: 52; on rmat-22 any local hops cost time)
    return (g->max_degree <= 8 && g->n_hubs == 0) ? 32 : 0;
}

sp_status sssp_run(sp_graph g, SsspWorkspace &ws, int32_t src, int32_t *out_dist, const SsspOpts &o,
                   hipStream_t s, SsspResult *res) {
    switch (sssp_local_hops(g, o.local_hops)) {
        case 0: return sssp_run_hops<0>(g, ws, src, out_dist, o, s, res);
        case 1: return sssp_run_hops<1>(g, ws, src, out_dist, o, s, res);
        case 2: return sssp_run_hops<2>(g, ws, src, out_dist, o, s, res);
        case 4: return sssp_run_hops<4>(g, ws, src, out_dist, o, s, res);
        case 8: return sssp_run_hops<8>(g, ws, src, out_dist, o, s, res);
        case 16: return sssp_run_hops<16>(g, ws, src, out_dist, o, s, res);
        case 32: return sssp_run_hops<32>(g, ws, src, out_dist, o, s, res);
        case 64: return sssp_run_hops<64>(g, ws, src, out_dist, o, s, res);
        default: return sssp_run_hops<128>(g, ws, src, out_dist, o, s, res);
    }
}

}  // namespace sp
