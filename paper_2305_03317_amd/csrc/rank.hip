// Vertices ranked by degree, highest first: rank_new[v] is v's rank, rank_old
// its inverse.  Ties of equal degree go to the higher id first.  Degrees of
// 256 and more are ranked by their leading six bits (the order only has to
// put heavy vertices first; any fixed total order orients a graph).
//
// A stable counting sort over kRankBuckets degree classes: a wave per tile of
// kRankTile ids counts its classes in LDS, the counts are scanned class by
// class, and the same walk hands out the ranks.  About 0.2 ms for 4.2 M
// vertices, once per graph.
#include "common.h"
#include "devutil.h"
#include "rank.h"

namespace sp {

namespace {
constexpr int32_t kRankBuckets = 1024;
constexpr int32_t kRankTile = 256;  // ids per wave; longer where that would be over 2048 tiles
}  // namespace

// Class of a degree, 0 = heaviest: exact below 256, then 32 classes per octave.
__device__ __forceinline__ int32_t rank_bucket(int32_t deg) {
    int32_t key = deg;
    if (deg >= kRankExact) {
        const int32_t e = 31 - __clz(deg);  // 8..30
        key = kRankExact + (e - 8) * 32 + ((deg >> (e - 5)) & 31);
    }
    return kRankBuckets - 1 - key;
}

// Tile t covers the ids n-1-i for i in [t, t+1) * tile (descending, so
// that ties rank the higher id first).
__global__ __launch_bounds__(kWave) void k_rank_count(const int32_t *__restrict__ rp, int32_t n,
                                                      int32_t tile, int32_t ntiles, int32_t *hist) {
    __shared__ int32_t s_cnt[kRankBuckets];
    for (int32_t b = threadIdx.x; b < kRankBuckets; b += kWave) s_cnt[b] = 0;
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * tile, i1 = min((int64_t)n, i0 + tile);
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kWave) {
        const int32_t v = (int32_t)(n - 1 - i);
        atomicAdd(&s_cnt[rank_bucket(rp[v + 1] - rp[v])], 1);
    }
    __syncthreads();
    for (int32_t b = threadIdx.x; b < kRankBuckets; b += kWave)
        hist[(int64_t)b * ntiles + blockIdx.x] = s_cnt[b];
}

__global__ __launch_bounds__(kWave) void k_rank_place(const int32_t *__restrict__ rp, int32_t n,
                                                      int32_t tile, int32_t ntiles,
                                                      const int32_t *__restrict__ first,
                                                      int32_t *rank_new, int32_t *rank_old) {
    __shared__ int32_t s_at[kRankBuckets];
    for (int32_t b = threadIdx.x; b < kRankBuckets; b += kWave)
        s_at[b] = first[(int64_t)b * ntiles + blockIdx.x];
    __syncthreads();
    const int lane = lane_id();
    const int64_t i0 = (int64_t)blockIdx.x * tile, i1 = min((int64_t)n, i0 + tile);
    for (int64_t b = i0; b < i1; b += kWave) {
        const int64_t i = b + lane;
        const int32_t v = (int32_t)(n - 1 - i);
        const int32_t mine = i < i1 ? rank_bucket(rp[v + 1] - rp[v]) : -1;
        unsigned long long todo = __ballot(i < i1);
        int32_t r = 0;
        while (todo) {  // one class of this step at a time, its lanes in order
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
        if (i < i1) {
            rank_new[v] = r;
            rank_old[r] = v;
        }
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

sp_status ensure_rank_locked(sp_graph g, hipStream_t s) {
    if (g->rank_new) return SP_OK;
    const int32_t n = g->n;
    const int32_t tile = std::max(kRankTile, (n / 2048 / kWave + 1) * kWave);
    const int32_t ntiles = (int32_t)std::max<int64_t>(1, ((int64_t)n + tile - 1) / tile);
    const int64_t cells = (int64_t)kRankBuckets * ntiles;
    const size_t vn = (size_t)std::max(n, 1);
    int32_t *rn = nullptr, *tmp = nullptr;
    auto fail = [&](sp_status st) {
        dev_free(rn);
        dev_free(tmp);
        return st;
    };
    sp_status st = dev_alloc((void **)&rn, 2 * sizeof(int32_t) * vn);
    int32_t *ro = rn ? rn + vn : nullptr;
    // counts, their scan (one more for the total), the scan's tiles
    if (st == SP_OK) st = dev_alloc((void **)&tmp, sizeof(int32_t) * (size_t)(2 * cells + 1 + scan_tiles(cells)));
    if (st != SP_OK) return fail(st);
    int32_t *hist = tmp, *first = tmp + cells, *tiles = first + cells + 1;
    if (n > 0) {
        hipLaunchKernelGGL(k_rank_count, dim3(ntiles), dim3(kWave), 0, s, (const int32_t *)g->row_ptr, n, tile,
                           ntiles, hist);
        launch_excl_scan(hist, cells, first, tiles, s);
        hipLaunchKernelGGL(k_rank_place, dim3(ntiles), dim3(kWave), 0, s, (const int32_t *)g->row_ptr, n, tile,
                           ntiles, (const int32_t *)first, rn, ro);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        set_error("ranking the vertices failed: %s", hipGetErrorString(e));
        return fail(SP_ERR_DEVICE);
    }
    dev_free(tmp);
    g->rank_new = rn;
    g->rank_old = ro;
    g->bytes += 2 * sizeof(int32_t) * vn;
    int32_t heavy = 0;
    for (int32_t v = 0; v < n; ++v) heavy += g->host_deg[v] >= kRankExact;
    g->rank_heavy = heavy;
    return SP_OK;
}

}  // namespace sp
