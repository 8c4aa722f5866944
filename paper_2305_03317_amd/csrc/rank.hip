// Vertices ranked by degree, highest first: rank_new[v] is v's rank, rank_old
// its inverse.  Ties of equal degree go to the higher id first.  Degrees of
// 256 and more are ranked by their leading six bits (the order only has to
// put heavy vertices first; any fixed total order orients a graph).  The same
// sort lists rows by length class (sort_rows_by_class).
//
// A stable counting sort: a wave per tile of items counts its buckets in LDS,
// the counts are scanned bucket by bucket, and the same walk hands out the
// places.  About 0.2 ms for the degrees of 4.2 M vertices, once per graph.
#include "common.h"
#include "devutil.h"
#include "rank.h"

namespace sp {

namespace {
constexpr int32_t kRankTile = 256;  // items per wave; longer where that would be over 2048 tiles

// What is sorted: item i's bucket, and what to do with its place.
struct ByDegree {  // item i is vertex n - 1 - i (ties rank the higher id first)
    static constexpr int32_t kBuckets = kRankBuckets;
    const int32_t *rp;
    int32_t n;
    int32_t *rank_new, *rank_old;
    int32_t skip;  // buckets of higher degrees than any
    __device__ int32_t bucket(int64_t i) const {
        const int32_t v = (int32_t)(n - 1 - i);
        return rank_bucket(rp[v + 1] - rp[v]) - skip;
    }
    __device__ void place(int64_t i, int32_t r) const {
        const int32_t v = (int32_t)(n - 1 - i);
        rank_new[v] = r;
        rank_old[r] = v;
    }
};
struct ByRowClass {
    static constexpr int32_t kBuckets = kRowClasses;
    const int32_t *rp, *old;
    int32_t n, longest;
    int32_t *order;
    int32_t skip = 0;
    __device__ int32_t bucket(int64_t i) const {
        const int32_t v = old ? old[i] : (int32_t)i;
        return row_class(rp[v + 1] - rp[v], longest);
    }
    __device__ void place(int64_t i, int32_t r) const { order[r] = (int32_t)i; }
};
}  // namespace

template <class Item>
__global__ __launch_bounds__(kWave) void k_sort_count(Item it, int32_t tile, int32_t ntiles, int32_t *hist) {
    __shared__ int32_t s_cnt[Item::kBuckets];
    const int32_t nb = Item::kBuckets - it.skip;
    for (int32_t b = threadIdx.x; b < nb; b += kWave) s_cnt[b] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * tile, i1 = min((int64_t)it.n, i0 + tile);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kWave) atomicAdd(&s_cnt[it.bucket(i)], 1);
    __syncthreads();
    for (int32_t b = threadIdx.x; b < nb; b += kWave) hist[(int64_t)b * ntiles + blockIdx.x] = s_cnt[b];
}

template <class Item>
__global__ __launch_bounds__(kWave) void k_sort_place(Item it, int32_t tile, int32_t ntiles,
                                                      const int32_t *__restrict__ first) {
    __shared__ int32_t s_at[Item::kBuckets];
    for (int32_t b = threadIdx.x; b < Item::kBuckets - it.skip; b += kWave)
        s_at[b] = first[(int64_t)b * ntiles + blockIdx.x];
    __syncthreads();
    const int lane = lane_id();
    const int64_t i0 = (int64_t)blockIdx.x * tile, i1 = min((int64_t)it.n, i0 + tile);
    for (int64_t b = i0; b < i1; b += kWave) {
        const int64_t i = b + lane;
        const int32_t mine = i < i1 ? it.bucket(i) : -1;
        unsigned long long todo = __ballot(i < i1);
        int32_t r = 0;
        while (todo) {  // one bucket of this step at a time, its lanes in order
            const int leader = __ffsll((long long)todo) - 1;
            const int32_t bk = __builtin_amdgcn_readlane(mine, leader);
            const unsigned long long same = __ballot(mine == bk);
            const int32_t at = s_at[bk];
            if (mine == bk) r = at + lanes_below(same);
            __builtin_amdgcn_wave_barrier();
            if (lane == leader) s_at[bk] = at + __popcll(same);
            __builtin_amdgcn_wave_barrier();
            todo &= ~same;
        }
        if (i < i1) it.place(i, r);
    }
}

// ---------------------------------------------------------------------------
// Exclusive scan of int32 counts (sums below 2^31): tiles of kScanTile, the
// tile totals by one block, then the tile offsets added.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_scan_tiles(const int32_t *__restrict__ in, int64_t n,
                                                    int32_t *out, int32_t *tile_sum) {
    __shared__ int32_t s_scan[256 / kWave + 1];
    const int64_t i0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
    int32_t d[4];
    int32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        d[q] = i0 + q < n ? in[i0 + q] : 0;
        mine += d[q];
    }
    int32_t total;
    int32_t off = block_excl_scan<256>(mine, s_scan, &total);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (i0 + q < n) out[i0 + q] = off;
        off += d[q];
    }
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_totals(int32_t *tile_sum, int32_t ntiles, int32_t *total_out) {
    __shared__ int32_t s_scan[256 / kWave + 1];
    int32_t carry = 0;
    for (int32_t b = 0; b < ntiles; b += 256) {
        const int32_t i = b + threadIdx.x;
        const int32_t x = i < ntiles ? tile_sum[i] : 0;
        int32_t total;
        const int32_t off = block_excl_scan<256>(x, s_scan, &total);
        if (i < ntiles) tile_sum[i] = carry + off;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total_out = carry;
}

__global__ __launch_bounds__(256) void k_scan_add(int32_t *out, int64_t n,
                                                  const int32_t *__restrict__ tile_base) {
    const int64_t i0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
    const int32_t t = tile_base[blockIdx.x];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (i0 + q < n) out[i0 + q] += t;
}

int64_t scan_tiles(int64_t n) { return std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile); }

void launch_excl_scan(const int32_t *in, int64_t n, int32_t *out, int32_t *tiles, hipStream_t s) {
    const int32_t nt = (int32_t)scan_tiles(n);
    hipLaunchKernelGGL(k_scan_tiles, dim3(nt), dim3(256), 0, s, in, n, out, tiles);
    hipLaunchKernelGGL(k_scan_totals, dim3(1), dim3(256), 0, s, tiles, nt, out + n);
    hipLaunchKernelGGL(k_scan_add, dim3(nt), dim3(256), 0, s, out, n, (const int32_t *)tiles);
}

// start[b] = first[b * stride] for b in [0, count).
__global__ void k_sort_starts(const int32_t *__restrict__ first, int32_t stride, int32_t count, int32_t *start) {
    for (int32_t b = threadIdx.x; b < count; b += blockDim.x) start[b] = first[(int64_t)b * stride];
}

// Stable counting sort of `it`; start[b] receives where bucket b begins
// (start[kBuckets] = n).  Synchronises the stream.
template <class Item>
static sp_status counting_sort(const Item &it, int32_t *start, hipStream_t s) {
    const int32_t nb = Item::kBuckets - it.skip;
    const int32_t n = it.n;
    const int32_t tile = std::max(kRankTile, (n / 2048 / kWave + 1) * kWave);
    const int32_t ntiles = (int32_t)std::max<int64_t>(1, ((int64_t)n + tile - 1) / tile);
    const int64_t cells = (int64_t)nb * ntiles;
    int32_t *hist = nullptr;  // counts, scanned in place (one more for the total); the scan's tiles; the starts
    SP_TRY(dev_alloc((void **)&hist, sizeof(int32_t) * (size_t)(cells + 1 + scan_tiles(cells) + nb + 1)));
    int32_t *tiles = hist + cells + 1, *starts = tiles + scan_tiles(cells);
    for (int32_t b = 0; b <= Item::kBuckets; ++b) start[b] = 0;
    hipError_t e = hipSuccess;
    if (n > 0) {
        hipLaunchKernelGGL((k_sort_count<Item>), dim3(ntiles), dim3(kWave), 0, s, it, tile, ntiles, hist);
        launch_excl_scan(hist, cells, hist, tiles, s);
        hipLaunchKernelGGL((k_sort_place<Item>), dim3(ntiles), dim3(kWave), 0, s, it, tile, ntiles,
                           (const int32_t *)hist);
        hipLaunchKernelGGL(k_sort_starts, dim3(1), dim3(256), 0, s, (const int32_t *)hist, ntiles, nb + 1, starts);
        e = hipGetLastError();
        if (e == hipSuccess)
            e = hipMemcpyAsync(start + it.skip, starts, sizeof(int32_t) * (size_t)(nb + 1), hipMemcpyDeviceToHost, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    dev_free(hist);
    if (e != hipSuccess) {
        set_error("sorting the vertices failed: %s", hipGetErrorString(e));
        return SP_ERR_DEVICE;
    }
    return SP_OK;
}

sp_status ensure_rank_locked(sp_graph g, hipStream_t s) {
    if (g->rank_new) return SP_OK;
    const size_t vn = (size_t)std::max(g->n, 1);
    const size_t bytes = sizeof(int32_t) * (g->directed ? 2 * vn : 3 * vn + 1);  // undirected: room for rank_rp
    int32_t *rn = nullptr;
    SP_TRY(dev_alloc((void **)&rn, bytes));
    std::vector<int32_t> start(kRankBuckets + 1);
    const sp_status st = counting_sort(ByDegree{g->row_ptr, g->n, rn, rn + vn, rank_bucket(g->max_degree)}, start.data(), s);
    if (st < 0) {
        dev_free(rn);
        return st;
    }
    g->rank_first = std::move(start);
    g->rank_new = rn;
    g->rank_old = rn + vn;
    g->bytes += bytes;
    return SP_OK;
}

sp_status ensure_rank_rp_locked(sp_graph g, hipStream_t s) {
    if (g->rank_rp) return SP_OK;
    int32_t *rp = g->rank_old + std::max(g->n, 1), *tiles = nullptr;
    SP_TRY(dev_alloc((void **)&tiles, sizeof(int32_t) * (size_t)scan_tiles(g->n)));
    launch_row_offsets(g->row_ptr, nullptr, g->rank_old, g->n, rp, tiles, s);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    dev_free(tiles);
    if (e != hipSuccess) {
        set_error("numbering the rows by rank failed: %s", hipGetErrorString(e));
        return SP_ERR_DEVICE;
    }
    g->rank_rp = rp;
    return SP_OK;
}

bool rank_skewed(sp_graph g) {
    int64_t seen = 0, entries = 0;
    for (int32_t b = 0; b < kRankBuckets && seen < g->n / 8; ++b) {
        const int32_t key = kRankBuckets - 1 - b, k = key - kRankExact;
        const int64_t deg = k < 0 ? key : (int64_t)(32 + k % 32) << (k / 32 + 3);  // the class's least
        const int64_t count = std::min<int64_t>(g->rank_first[b + 1] - g->rank_first[b], g->n / 8 - seen);
        seen += count;
        entries += count * deg;
    }
    return 2 * entries >= g->nnz;
}

__global__ void k_row_len(const int32_t *__restrict__ rp, const int32_t *__restrict__ order,
                          const int32_t *__restrict__ old, int32_t n, int32_t *len) {
    const int32_t stride = gridDim.x * blockDim.x;
    for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t x = order ? order[i] : i, v = old ? old[x] : x;
        len[i] = rp[v + 1] - rp[v];
    }
}

void launch_row_offsets(const int32_t *rp, const int32_t *order, const int32_t *old, int32_t n, int32_t *off,
                        int32_t *tiles, hipStream_t s) {
    hipLaunchKernelGGL(k_row_len, dim3(grid_for(n, 256, device_cu_count() * 8)), dim3(256), 0, s, rp, order, old, n,
                       off);
    launch_excl_scan(off, n, off, tiles, s);
}

template <int PER>
__global__ __launch_bounds__(256) void k_renumber(const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                                                  const int32_t *__restrict__ order,
                                                  const int32_t *__restrict__ old,
                                                  const int32_t *__restrict__ new_id,
                                                  const int32_t *__restrict__ to, int32_t first, int32_t last,
                                                  int32_t *col) {
    const int64_t stride = (int64_t)gridDim.x * (256 / PER);
    for (int64_t i = first + (int64_t)blockIdx.x * (256 / PER) + threadIdx.x / PER; i < last; i += stride) {
        const int32_t v = old[order ? order[i] : i];
        const int32_t b = rp[v], len = rp[v + 1] - b, at = to[i];
        for (int32_t k = threadIdx.x % PER; k < len; k += PER) col[at + k] = new_id[ci[b + k]];
    }
}

void launch_renumber(const int32_t *rp, const int32_t *ci, const int32_t *order, const int32_t *old,
                     const int32_t *new_id, const int32_t *to, int32_t longer, int32_t rows, int32_t *col,
                     hipStream_t s) {
    const int maxb = device_cu_count() * 8;
    if (longer > 0)
        hipLaunchKernelGGL(k_renumber<256>, dim3(std::min(longer, maxb)), dim3(256), 0, s, rp, ci, order, old, new_id,
                           to, 0, longer, col);
    if (rows > longer)
        hipLaunchKernelGGL(k_renumber<16>, dim3(grid_for((int64_t)rows - longer, 16, maxb)), dim3(256), 0, s, rp, ci,
                           order, old, new_id, to, longer, rows, col);
}

sp_status ensure_rank_csr_locked(sp_graph g, hipStream_t s) {
    if (g->rank_ci || g->directed || g->max_degree <= 8 || !may_be_skewed(g)) return SP_OK;
    int32_t *ci = nullptr;
    sp_status st = ensure_rank_locked(g, s);
    if (st == SP_OK && !rank_skewed(g)) return SP_OK;
    const size_t eb = sizeof(int32_t) * (size_t)std::max<int64_t>(g->nnz, 1);
    if (st == SP_OK) st = ensure_rank_rp_locked(g, s);
    if (st == SP_OK) st = dev_alloc((void **)&ci, eb);
    if (st == SP_OK) {
        launch_renumber(g->row_ptr, g->col_idx, nullptr, g->rank_old, g->rank_new, g->rank_rp,
                        rank_count(g, kRankExact), g->n, ci, s);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            dev_free(ci);
            set_error("numbering the rows by rank failed: %s", hipGetErrorString(e));
            return SP_ERR_DEVICE;
        }
        g->rank_ci = ci;
        g->bytes += eb;
    }
    if (st == SP_ERR_OUT_OF_MEMORY) {
        clear_error();
        return SP_OK;
    }
    return st;
}

sp_status sort_rows_by_class(const int32_t *rp, const int32_t *old, int32_t n, int32_t longest, int32_t *order,
                             int32_t *first, hipStream_t s) {
    return counting_sort(ByRowClass{rp, old, n, longest, order}, first, s);
}

}  // namespace sp
