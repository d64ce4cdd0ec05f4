// Ragged batches: chains of different lengths in one call (the networks of Section 5 range from
// n = 15 to n = 1001 layers).  Chain c occupies elements offsets[c] .. offsets[c+1]-1 of one flat
// array.  The host counts the chains of every length (launch planning, no arithmetic of the
// method) and decides where each length's group is staged; a kernel hands every chain a place in
// its group; a tiled transposition through LDS brings all groups into position-major staging at
// once; eval_peak, eval_timeline and solve_linear then take every group in one launch (a wave looks
// up the group its chains belong to), the cubic solver group by group; a second
// transposition puts the results where the flat layout wants them.  Everything is enqueued on
// the caller's stream.
#include <vector>

#include "linear_wave.h"
#include "ragged_plan.h"

namespace ckpt {
namespace {

constexpr int kTile = 64;         // chains and positions per transposition tile
constexpr int kTileThreads = 256; // four waves

// ---- the plan made on the device ------------------------------------------------------------
// When the caller has the offsets in device memory, the lengths are counted here instead of on the
// host: ragged_count_kernel checks every offset and counts the chains of every length (hist[n]),
// ragged_layout_kernel turns the counts into the table of groups, exactly as the host would
// (ragged_next_group), and the host reads back the totals only: how many waves, tiles and bytes of
// staging the launches that follow need.
constexpr int kCountThreads = 1024;
constexpr int kCountLds = 4096;  // lengths below this are first added up per workgroup in LDS

__global__ __launch_bounds__(kCountThreads) void ragged_count_kernel(const int64_t *__restrict__ off, int64_t batch,
                                                                     int max_layers, uint32_t *__restrict__ hist,
                                                                     RaggedTotals *__restrict__ totals)
{
    __shared__ uint32_t near_count[kCountLds];
    __shared__ int longest;
    for (int b = threadIdx.x; b < kCountLds; b += kCountThreads) near_count[b] = 0;
    if (threadIdx.x == 0) longest = 0;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * kCountThreads + threadIdx.x;
    const int lane = threadIdx.x % kWave;
    constexpr uint64_t kMaxOffset = (uint64_t)(INT64_MAX / 64);
    bool ok = false;
    uint32_t n = 0;
    if (c < batch) {
        // every offset in 0 .. INT64_MAX / 64 (a negative one reads as huge), so the difference is
        // exact, and a decreasing pair wraps to a huge length
        const uint64_t lo = (uint64_t)off[c], hi = (uint64_t)off[c + 1];
        const uint64_t below = hi - lo - 2;  // n - 1
        ok = below <= (uint64_t)(max_layers - 1) && hi <= kMaxOffset && lo <= kMaxOffset;
        n = (uint32_t)below + 1u;
        if (!ok) totals->bad = 1;  // (every writer writes the same value)
    }
    // the lanes of a wave that hold the same length count together
    uint64_t todo = __builtin_amdgcn_ballot_w64(ok);
    while (todo) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const uint32_t nl = (uint32_t)__builtin_amdgcn_readlane((int)n, leader);
        const uint64_t same = __builtin_amdgcn_ballot_w64(ok && n == nl);
        if (lane == leader) {
            const uint32_t many = (uint32_t)__popcll((unsigned long long)same);
            if (nl < (uint32_t)kCountLds) atomicAdd(near_count + nl, many); else atomicAdd(hist + nl, many);
            atomicMax(&longest, (int)nl);
        }
        todo &= ~same;
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kCountLds && b <= longest; b += kCountThreads) {
        const uint32_t many = near_count[b];
        if (many) atomicAdd(hist + b, many);
    }
    if (threadIdx.x == 0 && longest > 0) atomicMax(&totals->max_layers, longest);
}

// Exclusive prefix sums of N values per thread over the workgroup (kCountThreads threads), and their totals.
constexpr int kSums = 7;
__device__ inline void block_exclusive_sums(int64_t (&v)[kSums], int64_t (&total)[kSums],
                                            int64_t (&wave_sum)[kCountThreads / kWave][kSums])
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    int64_t incl[kSums];
#pragma unroll
    for (int q = 0; q < kSums; ++q) incl[q] = v[q];
#pragma unroll 1
    for (int s = 1; s < kWave; s <<= 1) {
#pragma unroll
        for (int q = 0; q < kSums; ++q) {
            const int64_t up = __shfl_up(incl[q], s, kWave);
            if (lane >= s) incl[q] += up;
        }
    }
    __syncthreads();  // (the previous call's readers are done with wave_sum)
    if (lane == kWave - 1) {
#pragma unroll
        for (int q = 0; q < kSums; ++q) wave_sum[wave][q] = incl[q];
    }
    __syncthreads();
    int64_t before[kSums] = {};
#pragma unroll
    for (int q = 0; q < kSums; ++q) total[q] = 0;
#pragma unroll 1
    for (int k = 0; k < kCountThreads / kWave; ++k) {
#pragma unroll
        for (int q = 0; q < kSums; ++q) {
            const int64_t x = wave_sum[k][q];
            before[q] += k < wave ? x : 0;
            total[q] += x;
        }
    }
#pragma unroll
    for (int q = 0; q < kSums; ++q) v[q] = before[q] + incl[q] - v[q];
}

// One workgroup: the lengths in tiles of kCountThreads, a length per thread.  Most of the 65,535 possible lengths do
// not occur, so the tiles that hold none are found first (every thread reads its length of every tile up to the longest
// that was counted, the loads in flight together) and passed over; in a tile that holds some, every thread adds up what its
// group contributes to the totals and, knowing the totals before it, writes the group's descriptor.  13 us with 1,001
// layers at most; 18 where all 64 tiles are looked at, 65 with a thread per stretch of 64 lengths, each walked twice.
__global__ __launch_bounds__(kCountThreads) void ragged_layout_kernel(const uint32_t *__restrict__ hist,
                                                                      int64_t batch, RaggedGroupDev *__restrict__ groups,
                                                                      int64_t *__restrict__ tile_first2,
                                                                      RaggedTotals *__restrict__ totals)
{
    __shared__ int64_t wave_sum[kCountThreads / kWave][kSums];
    __shared__ unsigned long long used;  // bit k: some length of tile k occurs
    __shared__ unsigned long long wave_layers, lane_waves, layers, deep_layers;
    __shared__ int wave_longest, lane_longest, deep_chains;
    const int max_layers = totals->max_layers;
    constexpr int kTiles = (CKPT_MAX_LAYERS + kCountThreads - 1) / kCountThreads;
    static_assert(kTiles <= 64, "one bit per tile");
    if (threadIdx.x == 0) {
        wave_longest = lane_longest = deep_chains = 0;
        used = wave_layers = lane_waves = layers = deep_layers = 0;
    }
    __syncthreads();
    unsigned long long mine = 0;
#pragma unroll 16
    for (int k = 0; k < (max_layers + kCountThreads - 1) / kCountThreads; ++k) {  // (a load behind a branch would wait for the one before it)
        const int n = 1 + k * kCountThreads + (int)threadIdx.x;
        const bool some = hist[n <= max_layers ? n : max_layers] != 0 && n <= max_layers;
        mine |= some ? 1ull << k : 0;
    }
    if (mine) atomicOr(&used, mine);
    __syncthreads();
    RaggedTotals at = {};  // the totals before the tile
    RaggedTotals own = {};  // of the thread's groups: only their sums are wanted
    for (unsigned long long todo = used; todo != 0; todo &= todo - 1) {
        const int n = 1 + (__ffsll(todo) - 1) * kCountThreads + (int)threadIdx.x;
        const int64_t many = n <= max_layers ? hist[n] : 0;
        RaggedTotals one = {};
        int64_t first2;
        if (many) (void)ragged_next_group(one, n, many, &first2);
        int64_t v[kSums] = {one.n_groups, one.chains, one.waves, one.linear_waves, one.tiles, one.tiles2, one.staged};
        int64_t all[kSums];
        block_exclusive_sums(v, all, wave_sum);
        if (many) {
            RaggedTotals t = {};
            t.n_groups = at.n_groups + (int32_t)v[0];
            t.chains = at.chains + v[1];
            t.waves = at.waves + v[2];
            t.linear_waves = at.linear_waves + v[3];
            t.tiles = at.tiles + v[4];
            t.tiles2 = at.tiles2 + v[5];
            t.staged = at.staged + v[6];
            const int slot = t.n_groups;
            const RaggedGroupDev g = ragged_next_group(t, n, many, &first2);
            groups[slot] = g;
            tile_first2[slot] = first2;
            if (g.first < batch - kLongest && batch - kLongest <= t.chains) totals->rows_longest = n;
        }
        at.n_groups += (int32_t)all[0];
        at.chains += all[1];
        at.waves += all[2];
        at.linear_waves += all[3];
        at.tiles += all[4];
        at.tiles2 += all[5];
        at.staged += all[6];
        own.wave_longest = one.wave_longest ? one.wave_longest : own.wave_longest;  // (ascending)
        own.lane_longest = one.lane_longest ? one.lane_longest : own.lane_longest;
        own.wave_layers += one.wave_layers;
        own.lane_waves += one.lane_waves;
        own.deep_chains += one.deep_chains;
        own.deep_layers += one.deep_layers;
        own.layers += one.layers;
    }
    // (what no thread of a wave has is passed over; with shuffles of all of it the launch took 3 us longer)
    const bool last = threadIdx.x % kWave == kWave - 1;
    if (__any(own.layers != 0)) {
        const int64_t all = sum_up_to(own.layers);
        const int deepest = max_up_to(own.lane_longest);
        if (last) {
            atomicAdd(&layers, (unsigned long long)all);
            atomicMax(&lane_longest, deepest);
        }
    }
    if (__any(own.wave_layers != 0)) {
        const int64_t all = sum_up_to(own.wave_layers), waves = sum_up_to(own.lane_waves);
        const int deepest = max_up_to(own.wave_longest);
        if (last) {
            atomicAdd(&wave_layers, (unsigned long long)all);
            atomicAdd(&lane_waves, (unsigned long long)waves);
            atomicMax(&wave_longest, deepest);
        }
    }
    if (__any(own.deep_layers != 0)) {
        const int64_t all = sum_up_to(own.deep_layers);
        const int chains = sum_up_to(own.deep_chains);
        if (last) {
            atomicAdd(&deep_layers, (unsigned long long)all);
            atomicAdd(&deep_chains, chains);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        totals->n_groups = at.n_groups;
        totals->chains = at.chains;
        totals->waves = at.waves;
        totals->linear_waves = at.linear_waves;
        totals->tiles = at.tiles;
        totals->tiles2 = at.tiles2;
        totals->staged = at.staged;
        totals->wave_longest = wave_longest;
        totals->lane_longest = lane_longest;
        totals->wave_layers = (int64_t)wave_layers;
        totals->lane_waves = (int64_t)lane_waves;
        totals->deep_chains = deep_chains;
        totals->deep_layers = (int64_t)deep_layers;
        totals->layers = (int64_t)layers;
    }
}

// Hands every chain a place among the chains of its length: perm[first(group) + k] = chain, k
// taken from a counter per group.  The lanes of a wave that belong to one group take their
// places together; with few groups (at most kPermLdsGroups) the waves of a workgroup first add
// up in LDS, so that a group's counter in memory is touched once per workgroup (a few lengths
// shared by a million chains would otherwise queue up on a handful of addresses).  The order
// inside a group is whatever the waves make it; everything downstream goes through perm, so the
// results do not depend on it.
constexpr int kPermThreads = 1024;
constexpr int kPermLdsGroups = 64;

__global__ __launch_bounds__(kPermThreads) void ragged_perm_kernel(const int64_t *__restrict__ off, int64_t batch,
                                                                   const RaggedGroupDev *__restrict__ groups,
                                                                   int n_groups, int32_t *__restrict__ cursor,
                                                                   int32_t *__restrict__ perm)
{
    __shared__ int32_t block_count[kPermLdsGroups];  // chains of the workgroup per group, then its base
    const bool in_lds = n_groups <= kPermLdsGroups;
    const int64_t c = (int64_t)blockIdx.x * kPermThreads + threadIdx.x;
    const int lane = threadIdx.x % kWave;
    const bool valid = c < batch;
    if (threadIdx.x < kPermLdsGroups) block_count[threadIdx.x] = 0;
    __syncthreads();
    int g = -1;
    if (valid) {
        const int32_t n = (int32_t)(off[c + 1] - off[c] - 1);
        int lo = 0, hi = n_groups - 1;  // the group of length n: it exists, the host counted this chain
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (groups[mid].n < n) lo = mid + 1; else hi = mid;
        }
        g = lo;
    }
    // a place inside the wave's share of its group, and the share's start (in the workgroup's
    // share if in_lds, else in the group)
    int32_t place = 0;
    uint64_t todo = __builtin_amdgcn_ballot_w64(valid);
    while (todo) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const int gl = __builtin_amdgcn_readlane(g, leader);
        const uint64_t same = __builtin_amdgcn_ballot_w64(valid && g == gl);
        const int32_t many = (int32_t)__popcll((unsigned long long)same);
        int32_t base = 0;
        if (lane == leader) base = in_lds ? atomicAdd(block_count + gl, many) : atomicAdd(cursor + gl, many);
        base = __builtin_amdgcn_readlane(base, leader);
        if (valid && g == gl) place = base + (int32_t)__popcll((unsigned long long)(same & ((1ull << lane) - 1ull)));
        todo &= ~same;
    }
    if (in_lds) {
        __syncthreads();
        if ((int)threadIdx.x < n_groups) {
            const int32_t many = block_count[threadIdx.x];
            block_count[threadIdx.x] = many > 0 ? atomicAdd(cursor + threadIdx.x, many) : 0;
        }
        __syncthreads();
        if (valid) place += block_count[g];
    }
    if (valid) perm[groups[g].first + place] = (int32_t)c;
}

// (counts: three more words, or null)
__global__ void ragged_clear_kernel(int32_t *cursor, int n_groups, int32_t *counts)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < n_groups) cursor[g] = 0;
    if (counts && g < 3) counts[g] = 0;
}

// Flat -> position-major, every group in one launch.  A workgroup takes one tile of 64 chains x 64
// rows of one group (found from the tile's number).  Element k of chain c is src[mult*off[c] + k],
// k < rows = mult * (n + 1); it goes to stage[mult*stage_off + k*pitch + j], j the chain's place
// in its group.  Reads run along a chain (several short chains to a wave), writes along the
// chains: both are contiguous per wave.
struct TileAt {
    RaggedGroupDev g;
    int64_t j0;  // first chain of the tile within the group
    int k0;      // first row
    int rows;
};

__device__ inline TileAt tile_at(const RaggedGroupDev *groups, const int64_t *tile_first2, int n_groups, int mult)
{
    TileAt t;
    int gi;
    int64_t local;
    if (mult == 1) {
        gi = ragged_group_of_tile(groups, n_groups, blockIdx.x);
        local = (int64_t)blockIdx.x - groups[gi].tile_first;
    } else {  // the tiles of the arrays with 2n+2 rows per chain are numbered on their own
        int lo = 0, hi = n_groups - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tile_first2[mid] <= (int64_t)blockIdx.x) lo = mid; else hi = mid - 1;
        }
        gi = lo;
        local = (int64_t)blockIdx.x - tile_first2[gi];
    }
    t.g = groups[gi];
    t.rows = mult * (t.g.n + 1);
    t.j0 = (local % t.g.tiles_x) * kTile;
    t.k0 = (int)(local / t.g.tiles_x) * kTile;
    return t;
}

// Where the tile's part of each of its 64 chains starts in the flat array (element index), looked
// up once per tile; the caller synchronises before use.
__device__ inline void tile_chains(const TileAt &t, const int64_t *__restrict__ off, const int32_t *__restrict__ perm,
                                   int mult, int64_t *chain_at)
{
    if (threadIdx.x < kTile) {
        const int64_t j = t.j0 + threadIdx.x;
        chain_at[threadIdx.x] = j < t.g.count ? (int64_t)mult * off[perm[t.g.first + j]] + t.k0 : 0;
    }
}

// The workgroup's threads laid along the chains of a tile `width` rows wide (1..64): a thread keeps
// one row k of the tile and walks the chains; width is rounded up to a power of two so that a
// thread's chain and row are a shift and a mask away.
struct AlongChain {
    int shift, width;
    __device__ explicit AlongChain(int w) : shift(w > 1 ? 32 - __builtin_clz((unsigned)w - 1u) : 0), width(w) {}
    __device__ int k() const { return (int)threadIdx.x & ((1 << shift) - 1); }
    __device__ bool active() const { return k() < width; }
    __device__ int first_chain() const { return (int)threadIdx.x >> shift; }
    __device__ int chains_per_pass() const { return kTileThreads >> shift; }
};

template <typename T>
__global__ __launch_bounds__(kTileThreads) void ragged_gather_kernel(const T *__restrict__ src,
                                                                     const int64_t *__restrict__ off,
                                                                     const int32_t *__restrict__ perm,
                                                                     const RaggedGroupDev *__restrict__ groups,
                                                                     const int64_t *__restrict__ tile_first2,
                                                                     int n_groups, int mult, T *__restrict__ stage)
{
    __shared__ T tile[kTile][kTile + 1];
    __shared__ int64_t chain_at[kTile];
    const TileAt t = tile_at(groups, tile_first2, n_groups, mult);
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int64_t count = t.g.count;
    tile_chains(t, off, perm, mult, chain_at);
    __syncthreads();
    const AlongChain a(min(kTile, t.rows - t.k0));
    for (int r = a.first_chain(); r < kTile; r += a.chains_per_pass())
        if (a.active() && t.j0 + r < count) tile[r][a.k()] = src[chain_at[r] + a.k()];
    __syncthreads();
    T *out = stage + (int64_t)mult * t.g.stage_off;
    for (int r = wave; r < kTile; r += kTileThreads / kWave) {
        const int k = t.k0 + r;
        const int64_t j = t.j0 + lane;
        if (k < t.rows && j < count) out[(int64_t)k * t.g.pitch + j] = tile[lane][r];
    }
}

// Position-major -> flat: the inverse.
template <typename T>
__global__ __launch_bounds__(kTileThreads) void ragged_scatter_kernel(const T *__restrict__ stage,
                                                                      const int64_t *__restrict__ off,
                                                                      const int32_t *__restrict__ perm,
                                                                      const RaggedGroupDev *__restrict__ groups,
                                                                      const int64_t *__restrict__ tile_first2,
                                                                      int n_groups, int mult, T *__restrict__ dst)
{
    __shared__ T tile[kTile][kTile + 1];
    __shared__ int64_t chain_at[kTile];
    const TileAt t = tile_at(groups, tile_first2, n_groups, mult);
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    const int64_t count = t.g.count;
    tile_chains(t, off, perm, mult, chain_at);
    const T *in = stage + (int64_t)mult * t.g.stage_off;
    for (int r = wave; r < kTile; r += kTileThreads / kWave) {
        const int k = t.k0 + r;
        const int64_t j = t.j0 + lane;
        if (k < t.rows && j < count) tile[lane][r] = in[(int64_t)k * t.g.pitch + j];
    }
    __syncthreads();
    const AlongChain a(min(kTile, t.rows - t.k0));
    for (int r = a.first_chain(); r < kTile; r += a.chains_per_pass())
        if (a.active() && t.j0 + r < count) dst[chain_at[r] + a.k()] = tile[r][a.k()];
}

// One value per chain from its place back to the chain's own index, all groups at once.
template <typename T>
__global__ __launch_bounds__(kTileThreads) void ragged_scatter_value_kernel(const T *__restrict__ stage,
                                                                            const int32_t *__restrict__ perm,
                                                                            int64_t batch, T *__restrict__ dst)
{
    const int64_t p = (int64_t)blockIdx.x * kTileThreads + threadIdx.x;
    if (p < batch) dst[perm[p]] = stage[p];
}

template <typename T>
void scatter_value(const T *stage, const int32_t *perm, int64_t batch, T *dst, hipStream_t s)
{
    if (!dst) return;
    hipLaunchKernelGGL(ragged_scatter_value_kernel<T>, dim3((unsigned)((batch + kTileThreads - 1) / kTileThreads)),
                       dim3(kTileThreads), 0, s, stage, perm, batch, dst);
}

}  // namespace

int ragged_plan_on_device(const int64_t *offsets_dev, int64_t batch, int max_layers, const RaggedWorkspace &w,
                          void *ws, hipStream_t stream, RaggedPlan &p)
{
    char *base = (char *)ws;
    RaggedTotals *totals = (RaggedTotals *)(base + w.totals);
    uint32_t *hist = (uint32_t *)(base + w.hist);
    static_assert(sizeof(RaggedTotals) % 4 == 0, "cleared as 32-bit words");
    // the totals and the counts lie behind each other: one fill clears both
    const int64_t words = (int64_t)((w.hist - w.totals) / 4) + max_layers + 1;
    hipLaunchKernelGGL(ragged_clear_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream,
                       (int32_t *)totals, (int)words, (int32_t *)nullptr);
    hipLaunchKernelGGL(ragged_count_kernel, dim3((unsigned)((batch + kCountThreads - 1) / kCountThreads)),
                       dim3(kCountThreads), 0, stream, offsets_dev, batch, max_layers, hist, totals);
    hipLaunchKernelGGL(ragged_layout_kernel, dim3(1), dim3(kCountThreads), 0, stream, hist, batch,
                       (RaggedGroupDev *)(base + w.groups), (int64_t *)(base + w.tiles2), totals);
    if (hipGetLastError() != hipSuccess) return CKPT_ERR_DEVICE;
    // the call's one wait: the launches that follow are sized by the totals
    if (hipMemcpyAsync(&p.t, totals, sizeof(RaggedTotals), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return CKPT_ERR_DEVICE;
    if (p.t.bad) return CKPT_ERR_SHAPE;
    return ragged_check_totals(p.t, batch);
}

int ragged_run(int which, const int64_t *d, const uint8_t *mask_in, const int64_t *offsets_host,
               const int64_t *offsets_dev, int64_t batch, int objective, uint8_t *mask_out, int64_t *peak_out,
               int64_t *budget_out, int64_t *timeline_out, int32_t *status_out, const RaggedPlan &p,
               const RaggedWorkspace &w, void *ws, hipStream_t stream)
{
    const bool eval = which == CKPT_CALL_EVAL_PEAK || which == CKPT_CALL_EVAL_TIMELINE;
    char *base = (char *)ws;
    const int64_t *off = offsets_dev ? offsets_dev : (const int64_t *)(base + w.off);
    int32_t *perm = (int32_t *)(base + w.perm);
    const RaggedGroupDev *groups = (const RaggedGroupDev *)(base + w.groups);
    const int64_t *tile_first2 = (const int64_t *)(base + w.tiles2);
    int32_t *cursor = (int32_t *)(base + w.cursor);
    int64_t *sd = (int64_t *)(base + w.d), *swide = (int64_t *)(base + w.wide);
    int64_t *speak = (int64_t *)(base + w.peak), *sbudget = (int64_t *)(base + w.budget);
    uint8_t *smask = (uint8_t *)(base + w.mask);
    int32_t *sstatus = (int32_t *)(base + w.status);
    const int n_groups = p.t.n_groups;
    if (which == CKPT_CALL_SOLVE_CUBIC && p.t.max_layers <= kSearchMaxLayers) {
        // Short chains are solved one by one where they lie: nothing is grouped, staged or put back (1,000
        // chains of 2 to 152 layers: 0.11 ms; group after group, 136 of them, it took 6.7 ms).
        if (!offsets_dev) {
            if (hipMemcpyAsync(base + w.off, offsets_host, (size_t)(batch + 1) * 8, hipMemcpyHostToDevice, stream) !=
                    hipSuccess ||
                hipStreamSynchronize(stream) != hipSuccess)  // the caller's offsets may end with the call
                return CKPT_ERR_DEVICE;
        }
        SearchClass classes[kSearchClasses];
        for (const RaggedGroupDev &g : p.groups) {
            int k = 0;
            while (g.n > search_class_limit(k)) ++k;
            classes[k].longest = g.n;  // (the groups ascend in n)
            classes[k].us += (float)g.count * search_us(g.n);
        }
        const hipError_t e = launch_cubic_search_ragged(d, off, batch, classes, mask_out, peak_out, budget_out,
                                                        status_out, (int32_t *)(base + w.totals), perm, stream);
        return e == hipSuccess ? CKPT_OK : CKPT_ERR_DEVICE;
    }
    if (!p.groups.empty()) {
        // The host made the plan.  The group table lives in host memory that ends with this call (and
        // the caller's offsets may end with it too): wait until the copies have read them.
        if (hipMemcpyAsync(base + w.groups, p.groups.data(), p.groups.size() * sizeof(RaggedGroupDev),
                           hipMemcpyHostToDevice, stream) != hipSuccess ||
            hipMemcpyAsync(base + w.tiles2, p.tile_first2.data(), p.tile_first2.size() * 8, hipMemcpyHostToDevice,
                           stream) != hipSuccess)
            return CKPT_ERR_DEVICE;
        if (!offsets_dev && hipMemcpyAsync(base + w.off, offsets_host, (size_t)(batch + 1) * 8,
                                           hipMemcpyHostToDevice, stream) != hipSuccess)
            return CKPT_ERR_DEVICE;
        if (hipStreamSynchronize(stream) != hipSuccess) return CKPT_ERR_DEVICE;
    }
    const bool flat = which == CKPT_CALL_SOLVE_LINEAR && linear_takes_flat(batch, p.t.max_layers);
    hipLaunchKernelGGL(ragged_clear_kernel, dim3((unsigned)((n_groups + 255) / 256)), dim3(256), 0, stream, cursor,
                       n_groups, flat ? (int32_t *)(base + w.inner) : nullptr);
    hipLaunchKernelGGL(ragged_perm_kernel, dim3((unsigned)((batch + kPermThreads - 1) / kPermThreads)),
                       dim3(kPermThreads), 0, stream, off, batch, groups, n_groups, cursor, perm);
    if (flat) {
        // few chains: a row of lanes or a wave reads a chain where it lies, nothing is staged or put back
        const hipError_t e = launch_solve_linear_flat(d, off, perm, batch, p.t, mask_out, peak_out, status_out,
                                                      base + w.inner, stream);
        return e == hipSuccess ? CKPT_OK : CKPT_ERR_DEVICE;
    }
    // every group's chains into the position-major staging
    hipLaunchKernelGGL(ragged_gather_kernel<int64_t>, dim3((unsigned)p.t.tiles), dim3(kTileThreads), 0, stream, d, off, perm,
                       groups, tile_first2, n_groups, 1, sd);
    if (eval)
        hipLaunchKernelGGL(ragged_gather_kernel<uint8_t>, dim3((unsigned)p.t.tiles), dim3(kTileThreads), 0, stream, mask_in,
                           off, perm, groups, tile_first2, n_groups, 1, smask);
    hipError_t e = hipSuccess;
    if (which == CKPT_CALL_EVAL_PEAK) {
        e = launch_eval_peak_ragged(sd, smask, groups, p.t, batch, objective, speak, sstatus, stream);
    } else if (which == CKPT_CALL_SOLVE_LINEAR) {
        e = launch_solve_linear_ragged(sd, groups, p.t, batch, smask, speak, sstatus, base + w.inner, stream);
    } else if (which == CKPT_CALL_EVAL_TIMELINE) {
        e = launch_eval_timeline_ragged(sd, smask, groups, n_groups, p.t.waves, objective, swide, sstatus, stream);
    } else {
        // the cubic solver takes the groups one after the other, each where it is staged (its tables
        // and launches are sized by the group's length)
        for (const RaggedGroupDev &g : p.groups) {
            e = launch_solve_cubic(sd + g.stage_off, g.count, g.n, Strides{1, g.pitch}, smask + g.stage_off,
                                   speak + g.first, sbudget + g.first, sstatus + g.first, false, nullptr, nullptr,
                                   nullptr, base + w.inner, stream);
            if (e != hipSuccess) return CKPT_ERR_DEVICE;
        }
    }
    if (e != hipSuccess) return CKPT_ERR_DEVICE;
    if (which == CKPT_CALL_EVAL_TIMELINE) {
        hipLaunchKernelGGL(ragged_scatter_kernel<int64_t>, dim3((unsigned)p.t.tiles2), dim3(kTileThreads), 0, stream, swide,
                           off, perm, groups, tile_first2, n_groups, 2, timeline_out);
    } else {
        if (!eval)
            hipLaunchKernelGGL(ragged_scatter_kernel<uint8_t>, dim3((unsigned)p.t.tiles), dim3(kTileThreads), 0, stream,
                               smask, off, perm, groups, tile_first2, n_groups, 1, mask_out);
        scatter_value(speak, perm, batch, peak_out, stream);
        if (which == CKPT_CALL_EVAL_PEAK && objective == CKPT_OBJ_BOTH)  // the dynamic peaks behind the static ones
            scatter_value(speak + batch, perm, batch, peak_out + batch, stream);
        if (which == CKPT_CALL_SOLVE_CUBIC) scatter_value(sbudget, perm, batch, budget_out, stream);
    }
    scatter_value(sstatus, perm, batch, status_out, stream);
    return hipGetLastError() == hipSuccess ? CKPT_OK : CKPT_ERR_DEVICE;
}

}  // namespace ckpt
