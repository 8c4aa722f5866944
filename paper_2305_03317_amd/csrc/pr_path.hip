// PageRank, pull form, double buffered (paper Appendix, Fig. "PR computation
// in StarPlat").  Every vertex starts at 1/N; an iteration computes
//     val[v] = (1 - delta) / N + delta * sum over in-neighbours u of pr[u] / outdeg(u)
// from the previous iteration's values, and the run stops once the sum over
// vertices of |val - pr| is at most beta or max_iter iterations have run
// (the absolute difference is this library's reading of the paper's `diff`).
// A vertex's in-neighbours are its row on an undirected graph and its row of
// the reversed graph on a directed one; outdeg is always the outgoing row's
// length, and a vertex without outgoing arcs passes nothing on.
//
// Design: each iteration is one pass over the entries and one launch.  The
// producer of a value also stores share = val / outdeg, so the gather reads one
// double per entry.  A plan made once per graph (ensure_pr_plan) lists the rows by
// length class, and each class gives a row the lanes its length fills: 1 for up to
// 8 entries (summed in row order), 4 up to 32, 16 up to 128, 64 below 512, a
// block from there on; rows of 8,192 entries and more are cut into pieces of that
// many, and the last piece of a row to arrive adds their sums.  Flat graphs (no
// row over 64 entries) are not listed: 4 lanes a row, 1 where no row holds more
// than 8.  A lane adds entries j, j + lanes, ... in order, four loads in flight,
// and a fixed tree adds the lanes, so a vertex's sum depends only on its row.
//
// On large skewed graphs the plan renumbers the vertices by degree rank: the
// shares that most entries gather then fill consecutive lines that stay in
// each XCD's 4 MB L2 (rmat-22: the first eighth of the ranks holds 92% of the
// entries), where random numbers spread them over 33 MB.  What is left then is L2
// bandwidth: 93 M requests of a 128-byte line per iteration, 17 TB/s; blocks
// therefore keep the shares of the first 9,216 ranks (a third of the gathers)
// in LDS.  rmat-22: 1.09 -> 0.68 ms per iteration; rmat-15, where latency and
// the number of launches count: 43 -> 13 us.
//
// The stopping test sums |val - pr| per block in a fixed order (the rows cut into
// pieces each by themselves) and adds these sums as fixed-point integers, so the
// total and the decision do not depend on scheduling.  The last working block
// closes the iteration;
// chunks of iterations are captured as HIP graphs and replayed until the
// device reports done.
#include <type_traits>

#include "blocks.h"
#include "capture.h"
#include "common.h"
#include "devutil.h"
#include "levels.h"
#include "rank.h"

namespace sp {

static_assert(kPrRowClasses == kRowClasses, "one tile range per row class");

__device__ __forceinline__ unsigned long long diff_fixed(double x) { return __double2ull_rn(x * kPrDiffUnit); }

// Block-uniform read of the iteration state (iteration * 2 + done).
__device__ __forceinline__ int32_t read_pr_state(PrCtl *c) {
    __shared__ int32_t s_state;
    if (threadIdx.x == 0) s_state = ld_agent(&c->state);
    __syncthreads();
    return s_state;
}

// Sum of the block's per-thread |change| in a fixed order, added to the
// iteration's total as a fixed-point integer.
template <int BS>
__device__ __forceinline__ void add_block_diff(PrCtl *c, double x, double *lds) {
    x = wave_sum_f64(x);
    if (lane_id() == 0) lds[threadIdx.x / kWave] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < BS / kWave; ++w) s += lds[w];
        if (s > 0.0) atomicAdd(&c->diff_.v, diff_fixed(s));
    }
}

// End of an iteration (one thread of the last working block).
__device__ void close_iteration(PrCtl *c) {
    const int32_t it = (c->state >> 1) + 1;
    const double diff = (double)ld_agent(&c->diff_.v) * (1.0 / kPrDiffUnit);
    c->diff_.v = 0;
    c->last_diff = diff;
    const bool done = !(diff > c->beta && it < c->max_iter);
    __hip_atomic_store(&c->state, it * 2 + (done ? 1 : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// rp: outgoing row offsets; old: vertex of an id (null: the id).
__global__ void k_pr_init(PrCtl *c, const int32_t *__restrict__ rp, const int32_t *__restrict__ old,
                          double *pr, double *share, int32_t n, double beta, int32_t max_iter,
                          int32_t *arrived, int32_t n_split) {
    const double x = 1.0 / (double)n;
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t v = old ? old[i] : i;
        const int32_t deg = rp[v + 1] - rp[v];
        pr[i] = x;
        share[i] = deg > 0 ? x / (double)deg : 0.0;
        if (i < n_split) arrived[i] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        c->state = 0;
        c->max_iter = max_iter;
        c->beta = beta;
        c->last_diff = 0.0;
        c->diff_.v = 0;
        c->blocks_done_.v = 0;
    }
}

// Shares by id: the first HOT of them from LDS.  Both sides are read without
// a branch: ids in LDS send their memory read to one common line.
template <int HOT>
struct Shares {
    const double *sh, *hot;
    __device__ __forceinline__ double get(int32_t u) const {
        if (HOT == 0) return sh[u];
        const double far = sh[max(u, HOT)], near = hot[min(u, HOT - 1)];
        return u < HOT ? near : far;
    }
};

// Sum of sh over the entries col[beg + lane], col[beg + lane + LPR], ... by LPR
// lanes, all of which receive it.  Four entries per lane are in flight: a lane
// past the row's end reads the last entry again and drops it, so that the
// loads are issued together (under a condition each would be waited for).
template <int LPR, int FLY, class S>
__device__ __forceinline__ double lanes_sum(const int32_t *__restrict__ col, const S &sh,
                                            int32_t beg, int32_t len, int32_t l) {
    double s = 0.0;
    for (int32_t t = l; __ballot(t < len); t += FLY * LPR) {
        if (t < len) {
            int32_t u[FLY];
            double x[FLY];
#pragma unroll
            for (int q = 0; q < FLY; ++q) u[q] = __builtin_nontemporal_load(&col[beg + min(t + q * LPR, len - 1)]);
#pragma unroll
            for (int q = 0; q < FLY; ++q) x[q] = sh.get(u[q]);
#pragma unroll
            for (int q = 0; q < FLY; ++q)
                if (t + q * LPR < len) s += x[q];
        }
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kWave);
    return s;
}

// The same by 512 lanes whatever the block size (each thread of a smaller
// block stands for 512 / BS of them, a block of 1024 sums two rows), their
// waves added in order; the sum arrives on the first of the row's threads.
template <int BS, int FLY, class S>
__device__ __forceinline__ double block_row_sum(const int32_t *__restrict__ col, const S &sh,
                                                int32_t beg, int32_t len, double *lds) {
    constexpr int kLanes = 512, T = BS < kLanes ? BS : kLanes, V = kLanes / T;
    constexpr int U = V >= FLY ? 1 : FLY / V;  // steps in flight
    const int32_t tid = threadIdx.x % T;
    double *mine = lds + threadIdx.x / T * (kLanes / kWave);
    double acc[V];
#pragma unroll
    for (int a = 0; a < V; ++a) acc[a] = 0.0;
    for (int32_t t = tid; t < len; t += kLanes * U) {
        int32_t u[U * V];
        double x[U * V];
#pragma unroll
        for (int q = 0; q < U * V; ++q) u[q] = __builtin_nontemporal_load(&col[beg + min(t + q * T, len - 1)]);
#pragma unroll
        for (int q = 0; q < U * V; ++q) x[q] = sh.get(u[q]);
#pragma unroll
        for (int q = 0; q < U * V; ++q)
            if (t + q * T < len) acc[q % V] += x[q];
    }
#pragma unroll
    for (int a = 0; a < V; ++a) {
        const double s = wave_sum_f64(acc[a]);
        if (lane_id() == 0) mine[a * (T / kWave) + tid / kWave] = s;
    }
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
        for (int k = 0; k < kLanes / kWave; ++k) s += mine[k];
    __syncthreads();
    return s;
}

// One iteration's gather: blocks walk the tiles of the row classes, heaviest
// first (a tile: one piece or row of the block classes, BS / lanes rows of the
// others), and the last block closes the iteration.
template <int BS, int HOT>
__global__ __launch_bounds__(BS, 8) void k_pr_pull(PrCtl *c, PrView p, double *pr0, double *pr1, double *sh0,
                                                   double *sh1, double *partial, int32_t *arrived, double teleport,
                                                   double delta, int32_t parity, unsigned long long *prof) {
    const int32_t st = read_pr_state(c);
    if ((st & 1) || ((st >> 1) & 1) != parity) return;
    __shared__ double s_w[BS > 512 ? BS / kWave : 8];  // (of 512 lanes, of the block's waves at the end)
    constexpr int kTeam = BS > 512 ? 512 : BS;  // threads per row of the block classes
    __shared__ unsigned long long s_red[1];
    const double *pr = parity ? pr1 : pr0;
    constexpr int FLY = 4;  // entries in flight per lane (8: rmat-22 13.7 -> 14.7 ms, road-2500 1.8 -> 2.2)
    __shared__ double s_hot[HOT ? HOT : 1];
    const Shares<HOT> sh{parity ? sh1 : sh0, s_hot};
    double *pr_n = parity ? pr0 : pr1;
    double *sh_n = parity ? sh0 : sh1;
    if (HOT) {
        for (int32_t k = threadIdx.x; k < HOT; k += BS) s_hot[k] = sh.sh[k];
        __syncthreads();
    }
    unsigned long long my_items = 0, my_edges = 0;
    double my_diff = 0.0;  // over the block's tiles, which are the same in every run
    auto row_at = [&](int32_t i) { return p.rows ? p.rows[i] : make_int2(p.rp[i], p.rp[i + 1] - p.rp[i]); };
    auto settle = [&](int32_t i, int32_t len, double sum) {
        const int32_t x = p.order ? p.order[i] : i;
        const int32_t dout = p.out_deg ? p.out_deg[x] : len;
        const double val = teleport + delta * sum;
        const double change = fabs(val - pr[x]);
        pr_n[x] = val;
        sh_n[x] = dout > 0 ? val / (double)dout : 0.0;
        ++my_items;
        my_edges += (unsigned long long)len;
        return change;
    };
    auto rows_of = [&](auto lanes, int cls, int32_t tile) {
        constexpr int LPR = decltype(lanes)::value;
        const int32_t i = p.row0[cls] + (tile - p.tile0[cls]) * (BS / LPR) + (int32_t)threadIdx.x / LPR;
        const int32_t l = threadIdx.x % LPR;
        const bool mine = i < p.row0[cls + 1];
        const int2 row = mine ? row_at(i) : make_int2(0, 0);
        const double sum = lanes_sum<LPR, FLY>(p.col, sh, row.x, row.y, l);
        if (mine && l == 0) my_diff += settle(i, row.y, sum);
    };
    const int32_t ntiles = p.tile0[kPrRowClasses];
    for (int32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (tile >= p.tile0[5]) rows_of(std::integral_constant<int, 1>{}, 5, tile);
        else if (tile >= p.tile0[4]) rows_of(std::integral_constant<int, 4>{}, 4, tile);
        else if (tile >= p.tile0[3]) rows_of(std::integral_constant<int, 16>{}, 3, tile);
        else if (tile >= p.tile0[2]) rows_of(std::integral_constant<int, 64>{}, 2, tile);
        else {
            const bool whole = tile >= p.tile0[1];  // a row, or a piece of one
            const int32_t k = (tile - (whole ? p.tile0[1] : 0)) * (BS / kTeam) + (int32_t)threadIdx.x / kTeam;
            const int32_t i = whole ? p.row0[1] + k : k;
            const bool mine = whole ? i < p.row0[2] : i < p.n_pieces;
            int2 row = make_int2(0, 0);
            if (mine) row = whole ? row_at(i) : p.pieces[i];
            const double sum = block_row_sum<BS, FLY>(p.col, sh, row.x, row.y, s_w);
            if (whole && mine && threadIdx.x % kTeam == 0) my_diff += settle(i, row.y, sum);
            if (!whole) {  // the last piece of a row to arrive settles it, on its team's first wave
                int32_t r = -1;
                if (mine && threadIdx.x % kTeam == 0) {
                    const int32_t owner = p.piece_row[i];
                    __hip_atomic_store(&partial[i], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __builtin_amdgcn_s_waitcnt(0);  // the sum is where every block reads it before it is counted
                    if (atomicAdd(&arrived[owner], 1) == p.split[owner].y - 1) {
                        arrived[owner] = 0;
                        r = owner;
                    }
                }
                r = __shfl(r, 0, kWave);
                if (r >= 0 && threadIdx.x % kTeam < kWave) {
                    const int2 h = p.split[r];
                    double s = 0.0;
                    for (int32_t k2 = lane_id(); k2 < h.y; k2 += kWave) s += ld_agent(&partial[h.x + k2]);
                    s = wave_sum_f64(s);
                    // whichever block that is: its |change| is rounded by itself
                    if (lane_id() == 0) {
                        const unsigned long long d = diff_fixed(settle(r, row_at(r).y, s));
                        if (d) atomicAdd(&c->diff_.v, d);
                    }
                }
            }
        }
    }
    add_block_diff<BS>(c, my_diff, s_w);
    flush_counters<BS>(prof, my_items, my_edges, 0, s_red);
    if (last_block(c, working_blocks((int64_t)ntiles, 1)) && threadIdx.x == 0) close_iteration(c);
}

// Values of the ids to the caller's vertices.
__global__ void k_pr_export(const double *__restrict__ pr, const int32_t *__restrict__ new_id, int32_t n,
                            double *out) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) out[v] = pr[new_id[v]];
}

// ---------------------------------------------------------------------------
// The plan
// ---------------------------------------------------------------------------
__global__ void k_pr_out_deg(const int32_t *__restrict__ rp, const int32_t *__restrict__ old, int32_t n,
                             int32_t *out_deg) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
        const int32_t v = old ? old[x] : x;
        out_deg[x] = rp[v + 1] - rp[v];
    }
}

// {first entry, entries} of the i-th row: at off[i] in a renumbered copy, else
// where the graph has it.
__global__ void k_pr_rows(const int32_t *__restrict__ rp, const int32_t *__restrict__ order,
                          const int32_t *__restrict__ old, const int32_t *__restrict__ off, int32_t n,
                          int2 *rows) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t x = order ? order[i] : i, v = old ? old[x] : x;
        const int32_t b = rp[v];
        rows[i] = make_int2(off ? off[i] : b, rp[v + 1] - b);
    }
}

namespace {
constexpr int kPrHotPerThread = 9;  // shares in LDS per thread of a renumbered run: 144 KB of a CU's 160 at 32 waves
constexpr int32_t kPrFlat = 64;     // rows of at most this many entries are not told apart
constexpr int32_t kPrPiece = 8192;  // rows from here on are split into pieces (a power of two: whole rank classes)
}  // namespace

void pr_plan_free(PrPlan *p) {
    if (!p) return;
    for (void *b : p->blocks) dev_free(b);
    delete p;
}

sp_status ensure_pr_plan(sp_graph g, hipStream_t s) {
    std::lock_guard<std::mutex> lk(g->mu);
    if (g->pr_plan) return SP_OK;
    const int32_t n = g->n;
    const int32_t *rp = g->rp_in, *ci = g->ci_in;
    struct Guard {
        PrPlan *p = new PrPlan;
        ~Guard() { pr_plan_free(p); }
    } gd;
    PrPlan &pl = *gd.p;
    constexpr int32_t longest = kPrPiece - 1;
    const size_t vn = (size_t)n;
    // renumbered when it pays and its copy fits; the graph's own rows do otherwise
    bool renum = false;
    const bool large = n > kPrRenumberFrom && g->max_degree > 8 && may_be_skewed(g);
    if (large && !g->directed) {  // the copy that the per-source path runs on too
        SP_TRY(ensure_rank_csr_locked(g, s));
        renum = g->rank_ci != nullptr;
        if (renum) {
            rp = g->rank_rp;
            ci = g->rank_ci;
        }
    } else if (large) {
        const sp_status st = ensure_rank_locked(g, s);
        if (st != SP_OK && st != SP_ERR_OUT_OF_MEMORY) return st;
        if (st != SP_OK) clear_error();
        renum = st == SP_OK && rank_skewed(g);
    }
    // undirected ranks list the rows by length already, and rows of one class need no list: rows of up to 8
    // entries, and those of flat graphs, four lanes each (a list costs their first call 0.3 ms and more)
    int2 *rows = nullptr;  // null: the rows' own offsets serve
    int32_t *order = nullptr, *out_deg = nullptr, *col = nullptr;
    bool listed;
    for (;; renum = false) {
        listed = renum ? g->directed : g->max_degree > kPrFlat;
        DevBlocks keep;
        if (listed) {
            keep.add(&rows, vn);
            keep.add(&order, vn);
        }
        if (g->directed) keep.add(&out_deg, vn + 1 + (size_t)scan_tiles(n));  // the copied rows' offsets first
        if (g->directed && renum) keep.add(&col, (size_t)std::max<int64_t>(g->nnz, 1));
        const sp_status st = keep.alloc();
        if (st == SP_ERR_OUT_OF_MEMORY && g->directed && renum) {
            clear_error();
            continue;
        }
        if (st != SP_OK) return st;
        pl.bytes = keep.give_to(pl.blocks);
        break;
    }
    if (renum) {
        pl.old_id = g->rank_old;
        pl.new_id = g->rank_new;
    }
    int32_t *row0 = pl.view.row0;
    if (listed) {
        SP_TRY(sort_rows_by_class(rp, pl.old_id, n, longest, order, row0, s));
    } else if (renum) {
        const int32_t at_least[kRowClasses - 1] = {kPrPiece, 512, 129, 33, 9};
        row0[0] = 0;
        for (int c = 1; c < kRowClasses; ++c) row0[c] = rank_count(g, at_least[c - 1]);
        row0[kRowClasses] = n;
    } else {
        row0[kRowClasses] = n;  // every row in the last class, or in the one before
        if (g->max_degree > 8) row0[kRowClasses - 1] = n;
    }
    const int maxb = device_cu_count() * 8;
    const int vgrid = grid_for(n, 256, maxb);
    int32_t *off = nullptr;
    if (col) {
        off = out_deg;
        launch_row_offsets(rp, order, pl.old_id, n, off, off + n + 1, s);
        launch_renumber(rp, ci, order, pl.old_id, pl.new_id, off, row0[2], n, col, s);
    }
    if (rows)
        hipLaunchKernelGGL(k_pr_rows, dim3(vgrid), dim3(256), 0, s, rp, (const int32_t *)order, pl.old_id,
                           (const int32_t *)off, n, rows);
    if (out_deg)
        hipLaunchKernelGGL(k_pr_out_deg, dim3(vgrid), dim3(256), 0, s, (const int32_t *)g->row_ptr, pl.old_id, n,
                           out_deg);
    SP_HIP(hipGetLastError());
    const int32_t ns = row0[1];  // a row per kPrPiece entries at most
    if (ns > 0) {
        std::vector<int2> srow((size_t)ns), split((size_t)ns), pieces;
        std::vector<int32_t> owner;
        if (rows) {
            SP_HIP(hipMemcpyAsync(srow.data(), rows, sizeof(int2) * (size_t)ns, hipMemcpyDeviceToHost, s));
            SP_HIP(hipStreamSynchronize(s));
        } else {
            std::vector<int32_t> first((size_t)ns + 1);
            SP_HIP(hipMemcpyAsync(first.data(), rp, sizeof(int32_t) * first.size(), hipMemcpyDeviceToHost, s));
            SP_HIP(hipStreamSynchronize(s));
            for (int32_t j = 0; j < ns; ++j) srow[j] = make_int2(first[j], first[j + 1] - first[j]);
        }
        for (int32_t j = 0; j < ns; ++j) {
            split[j].x = (int32_t)pieces.size();
            for (int64_t k = 0; k < srow[j].y; k += kPrPiece) {
                pieces.push_back(make_int2(srow[j].x + (int32_t)k, (int32_t)std::min<int64_t>(kPrPiece, srow[j].y - k)));
                owner.push_back(j);
            }
            split[j].y = (int32_t)pieces.size() - split[j].x;
        }
        int2 *d_split, *d_pieces;
        int32_t *d_owner;
        DevBlocks keep;
        keep.add(&d_split, split.size());
        keep.add(&d_pieces, pieces.size());
        keep.add(&d_owner, owner.size());
        SP_TRY(keep.alloc());
        SP_HIP(hipMemcpyAsync(d_split, split.data(), sizeof(int2) * split.size(), hipMemcpyHostToDevice, s));
        SP_HIP(hipMemcpyAsync(d_pieces, pieces.data(), sizeof(int2) * pieces.size(), hipMemcpyHostToDevice, s));
        SP_HIP(hipMemcpyAsync(d_owner, owner.data(), sizeof(int32_t) * owner.size(), hipMemcpyHostToDevice, s));
        SP_HIP(hipStreamSynchronize(s));
        pl.view.split = d_split;
        pl.view.pieces = d_pieces;
        pl.view.piece_row = d_owner;
        pl.bytes += keep.give_to(pl.blocks);
        pl.view.n_pieces = (int32_t)pieces.size();
        pl.n_split = ns;
    }
    SP_HIP(hipStreamSynchronize(s));
    pl.view.col = col ? col : ci;
    pl.view.rows = rows;
    pl.view.rp = rp;
    pl.view.order = order;
    pl.view.out_deg = out_deg;
    g->bytes += pl.bytes;
    g->pr_plan = gd.p;
    gd.p = nullptr;
    return SP_OK;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
sp_status pr_ws_create(sp_graph g, PrWorkspace &ws) {
    const size_t n = (size_t)std::max(g->n, 1);
    SP_HIP(hipGetDevice(&ws.device));
    DevBlocks keep;
    for (int p = 0; p < 2; ++p) {
        keep.add(&ws.pr[p], n);
        keep.add(&ws.share[p], n);
    }
    keep.add(&ws.partial, (size_t)g->pr_plan->view.n_pieces + 1);
    keep.add(&ws.arrived, (size_t)g->pr_plan->n_split + 1);
    keep.add(&ws.ctl, 1);
    SP_TRY(keep.alloc());
    keep.give_to(ws.blocks);
    if (hipHostMalloc((void **)&ws.ctl_host, sizeof(PrCtl), hipHostMallocDefault) != hipSuccess) {
        ws.ctl_host = nullptr;
        pr_ws_destroy(ws);
        set_error("pinned host allocation failed");
        return SP_ERR_OUT_OF_MEMORY;
    }
    if (hipEventCreate(&ws.ev0) != hipSuccess || hipEventCreate(&ws.ev1) != hipSuccess) {
        pr_ws_destroy(ws);
        set_error("hipEventCreate failed");
        return SP_ERR_DEVICE;
    }
    return SP_OK;
}

void pr_ws_destroy(PrWorkspace &ws) {
    if (ws.iters.exec) (void)hipGraphExecDestroy(ws.iters.exec);
    if (ws.cap_stream) (void)hipStreamDestroy(ws.cap_stream);
    for (void *b : ws.blocks) dev_free(b);
    if (ws.ctl_host) (void)hipHostFree(ws.ctl_host);
    if (ws.ev0) (void)hipEventDestroy(ws.ev0);
    if (ws.ev1) (void)hipEventDestroy(ws.ev1);
    ws = PrWorkspace{};
}

// `count` iterations starting at an even iteration (parity = k & 1).
template <int BS>
static void enqueue_iterations(const PrPlan &pl, const PrView &view, PrWorkspace &ws, int count, int grid,
                               double teleport, double delta, hipStream_t s) {
    auto pull = pl.new_id ? k_pr_pull<BS, kPrHotPerThread * BS> : k_pr_pull<BS, 0>;
    for (int k = 0; k < count; ++k) {
        ProfScope ps(P_PR_PULL, s);
        hipLaunchKernelGGL(pull, dim3(grid), dim3(BS), 0, s, ws.ctl, view, ws.pr[0], ws.pr[1], ws.share[0],
                           ws.share[1], ws.partial, ws.arrived, teleport, delta, (int32_t)(k & 1),
                           prof_counters(P_PR_PULL));
    }
}

static long long bits_of(double x) {
    long long b;
    std::memcpy(&b, &x, sizeof(b));
    return b;
}

template <int BS>
static sp_status pr_run_bs(sp_graph g, PrWorkspace &ws, double beta, double delta, int32_t max_iter,
                           double *out_pr, const PrOpts &o, hipStream_t s, PrResult *res) {
    const int32_t n = g->n;
    const PrPlan &pl = *g->pr_plan;
    PrView view = pl.view;
    constexpr int team = BS > 512 ? 512 : BS, team_rows = BS / team;
    constexpr int lanes[kPrRowClasses] = {team, team, 64, 16, 4, 1};
    view.tile0[0] = 0;
    view.tile0[1] = (view.n_pieces + team_rows - 1) / team_rows;
    for (int k = 1; k < kPrRowClasses; ++k) {
        const int32_t rows = view.row0[k + 1] - view.row0[k], per = BS / lanes[k];
        view.tile0[k + 1] = view.tile0[k] + (int32_t)(((int64_t)rows + per - 1) / per);
    }
    // Renumbered: twice the blocks that fit at once, which evens out their rows (small blocks up to 2 M vertices: as
    // many as fit).  Else as many as fit, and half of that up to 2 M vertices: every block ends in two atomics to one
    // line each, which take 5 ns a block (road-1000, 20 iterations: 587 -> 488 us; directed rmat-20, blocks of 256:
    // 2.52 -> 2.28 ms).
    const int threads_per_cu = pl.new_id ? (BS >= 512 || n > (1 << 21) ? 4096 : 2048) : n > (1 << 21) ? 2048 : 1024;
    const int grid = grid_for(view.tile0[kPrRowClasses], 1, device_cu_count() * threads_per_cu / BS);
    const double teleport = (1.0 - delta) / (double)n;
    hipLaunchKernelGGL(k_pr_init, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s, ws.ctl,
                       (const int32_t *)g->row_ptr, pl.old_id, ws.pr[0], ws.share[0], n, beta, max_iter, ws.arrived,
                       pl.n_split);
    SP_HIP(hipGetLastError());
    const bool capture = o.chunk_iters > 0 && !prof_enabled();
    const int base = std::max(1, std::abs(o.chunk_iters));
    const int chunk = base + (base & 1);  // even: every chunk starts at an even iteration
    int32_t enqueued = 0, graph_launches = 0;
    for (;;) {
        if (capture) {
            const std::array<long long, 12> key = {
                BS, grid, chunk, (long long)(intptr_t)ws.pr[0], (long long)(intptr_t)ws.ctl,
                (long long)(intptr_t)g->pr_plan, bits_of(teleport), bits_of(delta), pl.n_split, 0, 0, 0};
            SP_TRY(replay_captured(&ws.cap_stream, ws.iters, key,
                                   [&](hipStream_t cs) {
                                       enqueue_iterations<BS>(pl, view, ws, chunk, grid, teleport, delta, cs);
                                   },
                                   s));
            ++graph_launches;
        } else {
            enqueue_iterations<BS>(pl, view, ws, chunk, grid, teleport, delta, s);
            SP_HIP(hipGetLastError());
        }
        enqueued += chunk;
        SP_HIP(hipMemcpyAsync(ws.ctl_host, ws.ctl, sizeof(PrCtl), hipMemcpyDeviceToHost, s));
        SP_HIP(hipStreamSynchronize(s));
        if (ws.ctl_host->state & 1) break;
        if (enqueued >= max_iter + chunk) {
            set_error("PageRank did not stop after %d iterations", enqueued);
            return SP_ERR_DEVICE;
        }
    }
    const int32_t iters = ws.ctl_host->state >> 1;
    if (pl.new_id) {
        hipLaunchKernelGGL(k_pr_export, dim3(grid_for(n, 256, 4096)), dim3(256), 0, s,
                           (const double *)ws.pr[iters & 1], pl.new_id, n, out_pr);
        SP_HIP(hipGetLastError());
    } else {
        SP_HIP(hipMemcpyAsync(out_pr, ws.pr[iters & 1], sizeof(double) * (size_t)n, hipMemcpyDeviceToDevice, s));
    }
    if (res) {
        res->iterations = iters;
        res->diff = ws.ctl_host->last_diff;
        res->graph_launches = graph_launches;
    }
    return SP_OK;
}

sp_status pr_run(sp_graph g, PrWorkspace &ws, double beta, double delta, int32_t max_iter,
                 double *out_pr, const PrOpts &o, hipStream_t s, PrResult *res) {
    // blocks of 1024 hold the most shares per copy: rmat-22, 20 iterations: 15.2, 14.9 and 13.7 ms with 256,
    // 512 and 1024 threads; the others measured best with 512 (rmat-15 337, 267, 254 us, uniform with 8 M edges
    // 2.42, 2.47, 2.63 ms)
    switch (o.block ? o.block : g->pr_plan->new_id ? 1024 : 512) {
        case 128: return pr_run_bs<128>(g, ws, beta, delta, max_iter, out_pr, o, s, res);
        case 1024: return pr_run_bs<1024>(g, ws, beta, delta, max_iter, out_pr, o, s, res);
        case 512: return pr_run_bs<512>(g, ws, beta, delta, max_iter, out_pr, o, s, res);
        default: return pr_run_bs<256>(g, ws, beta, delta, max_iter, out_pr, o, s, res);
    }
}

}  // namespace sp
