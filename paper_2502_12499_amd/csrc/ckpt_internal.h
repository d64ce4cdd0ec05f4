// Internal launch interface between the C-ABI entry points (ckpt_api.hip) and
// the kernel translation units.  Host code only validates and launches; every
// step of the path runs in the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <initializer_list>

#include "../../include/ckpt.h"

namespace ckpt {

constexpr int kWave = 64;

// Chain c, position k of an array laid out by a ckpt_layout.
struct Strides {
    int64_t chain;
    int64_t pos;
};

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Dynamic LDS beyond 64 KB has to be allowed per kernel and device.  The limit is state that all host threads share, so
// it is raised once, to the most that any call of the kernels asks for, and not to what the present call does.
// `raised`: a flag per device, of the calling file.
constexpr int kMaxDevices = 64;
constexpr size_t kDefaultLdsLimit = 65536;
inline hipError_t raise_lds_limit(std::atomic<bool> (&raised)[kMaxDevices], std::initializer_list<const void *> kernels,
                                  size_t most)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (raised[dev].load(std::memory_order_acquire)) return hipSuccess;
    for (const void *f : kernels) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) return e;
    }
    raised[dev].store(true, std::memory_order_release);
    return hipSuccess;
}

// Whether sum(d) + max(d) is beyond INT64_MAX, for kernels that add the sizes of a chain up in no particular order.
// `sum` is their sum modulo 2^64, `high` that of their upper halves: from 2^31 on the sum is at least 2^63, and below
// that it is less than 2^63 + 2^48, so it has not wrapped.  (The sum and the largest size together may wrap: one
// size near INT64_MAX beside small ones.)
__host__ __device__ inline bool chain_overflows(uint64_t sum, uint64_t high, uint64_t largest)
{
    return high >= (1ull << 31) || sum > (uint64_t)INT64_MAX || largest > (uint64_t)INT64_MAX - sum;
}

// Workgroups are handed to the eight XCDs of the chip in turn, and each XCD has its own L2.  A
// one-wave workgroup of a lane-per-chain kernel touches 64 bytes of a mask row, half a 128-byte
// line; its neighbour, which holds the other half, would run on the next XCD and fetch the line
// again.  This maps the workgroup index so that, within every 16 consecutive workgroups, the two
// that one XCD receives take neighbouring groups of chains.  A bijection on [0, grid).
__device__ inline unsigned xcd_paired_block(unsigned b, unsigned grid)
{
    constexpr unsigned kXcds = 8;
    if (b >= grid / (2 * kXcds) * (2 * kXcds)) return b;  // the ragged end keeps its order
    return (b / (2 * kXcds)) * (2 * kXcds) + (b % kXcds) * 2 + (b / kXcds) % 2;
}

// Workgroups go to the eight XCDs in turn, and each XCD has its own L2; a wave of one chain (four)
// reads 8 (32) of the 128 bytes of a line of a position-major batch.  Within every 512 workgroups the 64 that one XCD
// receives take neighbouring ones.  A bijection on [0, grid).
__device__ inline unsigned xcd_blocked(unsigned b, unsigned grid)
{
    if (b >= grid / 512 * 512) return b;
    return b / 512 * 512 + (b % 8) * 64 + (b / 8) % 64;
}

// ---- wave reductions on the data-parallel-primitive path (no LDS traffic) --------------------------

constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr4 = 0x114, kDppRowShr8 = 0x118;
constexpr int kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;

// One step of a wave reduction: every lane whose DPP source exists (and whose
// row is in ROW_MASK) joins its value with the source's; the others keep theirs.
template <int CTRL, int ROW_MASK>
__device__ inline uint64_t dpp_min_step_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    const uint32_t olo = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, CTRL, ROW_MASK, 0xf, false);
    const uint32_t ohi = (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, CTRL, ROW_MASK, 0xf, false);
    const uint64_t o = ((uint64_t)ohi << 32) | olo;
    return o < v ? o : v;
}

// Minimum over the wave, returned to every lane.  Shifts by 1, 2, 4, 8 inside
// each row of 16 lanes leave the row's minimum in its last lane; lane 15 is
// then broadcast into row 1 and lane 47 into row 3, lane 31 into rows 2 and 3,
// and lane 63 holds the minimum of all 64.
__device__ inline uint64_t wave_min_u64(uint64_t v)
{
    v = dpp_min_step_u64<kDppRowShr1, 0xf>(v);
    v = dpp_min_step_u64<kDppRowShr2, 0xf>(v);
    v = dpp_min_step_u64<kDppRowShr4, 0xf>(v);
    v = dpp_min_step_u64<kDppRowShr8, 0xf>(v);
    v = dpp_min_step_u64<kDppRowBcast15, 0xa>(v);
    v = dpp_min_step_u64<kDppRowBcast31, 0xc>(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// (one instruction a step: a lane without a source keeps its value; the value a DPP source reads must be two wait
// states old)
__device__ inline uint32_t wave_min_u32(uint32_t v)
{
    asm("s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 0"
        : "+v"(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Lexicographic minimum of (a, b) over the wave; every lane gets the result.  Both values are
// non-negative wherever this is used (costs, budgets, indices, kInf), so they order as unsigned:
// the smallest a, then the smallest b among the lanes that hold it.
__device__ inline void wave_min_pair(int64_t &a, int64_t &b)
{
    const uint64_t am = wave_min_u64((uint64_t)a);
    const uint64_t bm = wave_min_u64((uint64_t)a == am ? (uint64_t)b : ~0ull);
    a = (int64_t)am;
    b = (int64_t)bm;
}

// ---- a first bound for the cubic search ------------------------------------------------------------
//
// For a segment length, a checkpoint wherever the interior prefix sums pass a multiple of it: what lies between two of
// them adds up to the length at most, so checkpoints + length bounds the optimum from above.  In floats, on prefix
// sums of the INTERIOR sizes: the size in front is subtracted as an integer first (in a float it would swallow interior
// sizes 2^24 times smaller), and no sum that is rounded exceeds `all`, the sum of the interior sizes.
__host__ __device__ inline float bound_prefix(uint64_t prefix, uint64_t first) { return (float)(prefix - first); }
// What layer i adds to the checkpoints: before, at: bound_prefix at i - 1 and i; inv: 1 / length.
__host__ __device__ inline float bound_layer(float before, float at, float inv)
{
    return floorf(before * inv) != floorf(at * inv) ? at - before : 0.0f;
}
// The cost from the sum of those over the n - 1 interior layers, without the sizes at the ends.  A difference of two
// rounded prefix sums is off by up to 2^-24 of `all` for each, on either side of a checkpoint, and the 1/512 covers the
// roundings of their sum, of the length and of its reciprocal.
__host__ __device__ inline float bound_cost(float kept, float length, uint64_t all, int n)
{
    return (kept + length) * (1.0f + 1.0f / 512.0f) + (float)all * (float)n * 0x1p-22f;
}

// ---- eval_peak ---------------------------------------------------------------
hipError_t launch_eval_peak(const int64_t *d, const uint8_t *mask, int64_t batch, int n, Strides st,
                            int objective, int64_t *peak_out, int32_t *status_out, hipStream_t stream);

// ---- eval_timeline, select_baseline ------------------------------------------
hipError_t launch_eval_timeline(const int64_t *d, const uint8_t *mask, int64_t batch, int n, Strides st,
                                int objective, int64_t *out, Strides out_st, int32_t *status_out,
                                hipStream_t stream);
hipError_t launch_select_baseline(int64_t batch, int n, Strides st, int kind, uint8_t *mask_out,
                                  hipStream_t stream);

// ---- solve_linear ------------------------------------------------------------
size_t linear_workspace_bytes(int64_t batch, int n);
hipError_t launch_solve_linear(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                               int64_t *peak_out, int32_t *status_out, void *ws, hipStream_t stream);
// the same launches with the lists in an array of the library's own (batch and n within the
// CKPT_NOALLOC_* limits, checked by the caller); no allocation, no other library call
hipError_t launch_solve_linear_noalloc(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                                       int64_t *peak_out, int32_t *status_out, hipStream_t stream);

// ---- solve_quadratic ---------------------------------------------------------
hipError_t launch_solve_quadratic(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                                  int64_t *peak_out, int64_t *value_out, int32_t *status_out,
                                  hipStream_t stream);

// ---- solve_cubic -------------------------------------------------------------
size_t cubic_workspace_bytes(int64_t batch, int n);
// pruned: budgets that a sample of the budgets shows cannot be optimal are skipped (same results);
// evaluated_out (may be null) receives the number of budgets whose recurrence was run, per chain
// trace_s, trace_cost (may be null): per budget lane, the budget and its cost s + c_s in bytes
hipError_t launch_solve_cubic(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                              int64_t *peak_out, int64_t *budget_out, int32_t *status_out, bool pruned,
                              int64_t *evaluated_out, int64_t *trace_s, int64_t *trace_cost, void *ws,
                              hipStream_t stream);
// the unpruned call without the costs, for chains of up to kSearchMaxLayers layers; ws: 256 + 4 * batch bytes
constexpr int kSearchMaxLayers = 256;
hipError_t launch_cubic_search(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                               int64_t *peak_out, int64_t *budget_out, int32_t *status_out, void *ws,
                               hipStream_t stream);
// ... and for longer ones; ws: cubic_search_long_bytes() bytes
size_t cubic_search_long_bytes(int64_t batch, int n);
hipError_t launch_cubic_search_long(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                                    int64_t *peak_out, int64_t *budget_out, int32_t *status_out, void *ws,
                                    hipStream_t stream);
// The same for a ragged batch whose chains all have up to kSearchMaxLayers layers, on the flat arrays
// themselves, in one launch with the LDS of the longest chain or in one per class of lengths.  count: one value,
// list: `batch` values of scratch.
constexpr int kSearchClasses = 4;
__host__ __device__ inline int search_class_limit(int k) { return 32 << k; }
static_assert((32 << (kSearchClasses - 1)) == kSearchMaxLayers, "the last class ends where the search does");
// About what a chain of n layers takes a wave, us (aligned ones; 24 layers 13, 64 32, 152 102, 256 234).
inline float search_us(int n) { return 6.0f + 0.25f * (float)n + 0.0025f * (float)n * (float)n; }
struct SearchClass {
    int longest = 0;      // 0: no chain
    float us = 0.0f;      // search_us of all its chains
};
hipError_t launch_cubic_search_ragged(const int64_t *d, const int64_t *offsets_dev, int64_t batch,
                                      const SearchClass (&classes)[kSearchClasses], uint8_t *mask_out, int64_t *peak_out,
                                      int64_t *budget_out, int32_t *status_out, int32_t *count, int32_t *list, hipStream_t stream);
// entries per chain of the two trace arrays: one per lane of the chain's waves of 64 budgets
int64_t cubic_trace_len(int n);

// ---- ragged batches ----------------------------------------------------------
// What the kernels are told about the chains of one length (a "group") when all groups of a call
// are staged side by side and taken by one launch.  Groups ascend in n; their chains have the
// places first .. first + count - 1, their waves of 64 chains the numbers wave_first .., their
// transposition tiles the numbers tile_first ..; the group's staging (position-major, `pitch`
// elements from one position to the next) starts stage_off elements into the staging arrays.
struct RaggedGroupDev {
    int32_t n;
    int32_t count;
    int32_t first;
    int32_t wave_first;
    int64_t tile_first;
    int64_t stage_off;
    int64_t pitch;
    int32_t tiles_x;  // tiles across the chains: ceil(count / 64)
    int32_t linear_first;  // the linear solver's first wave of the group, where it gives some chains a wave each
};

// The sums over the groups laid out so far (all of them at the end); `bad` is set by the device's
// count of the lengths when an offset is out of range.
struct RaggedTotals {
    int32_t n_groups, bad, max_layers;
    int32_t wave_longest;  // of the groups that ragged_wave_per_chain takes: the longest chains' length ...
    int32_t deep_chains;   // those of more than kDeepLayers layers
    int32_t rows_longest;  // the longest chain but for the kLongest longest
    int32_t lane_longest;  // ... and of the groups that ragged_wave_per_chain does not take
    int64_t chains, waves, linear_waves, tiles, tiles2, staged;
    int64_t wave_layers;   // ... the layers of all their chains ...
    int64_t lane_waves;    // ... and the waves that they take with a lane per chain
    int64_t layers, deep_layers;  // of all chains, of the deep ones
};

// A row of lanes' chain has its steps in the wave's LDS, and up to kDeepLayers layers that leaves a SIMD four waves.
// Longer chains among many get a wave each, as the kLongest longest always do.
constexpr int kDeepLayers = 1023, kLongest = 64;
// They are few enough for that: a wave takes 40 to 110 ps a layer of the whole chip, rows 9 to 15, and 18 to 26 where
// their LDS leaves a SIMD one wave.
inline bool deep_ones_alone(const RaggedTotals &t) { return 8 * t.deep_layers <= t.layers; }

// Groups of a large ragged batch (linear_takes_flat takes the others) whose chains the linear solver gives a wave each
// instead of a lane each, if all such groups together are small enough (ragged_waves_pay): few chains (they would fill a
// handful of waves) and long ones (whose lane-per-chain form takes 660 ns a position, a wave per chain 40).
__host__ __device__ inline bool ragged_wave_per_chain(int n, int64_t count)
{
    return n > 256 && n <= 4095 && count <= 1024;
}
__host__ __device__ inline int64_t ragged_linear_waves(int n, int64_t count)
{
    return ragged_wave_per_chain(n, count) ? count : (count + 63) / 64;
}

// With a wave per chain these groups take 40 ps a layer once they fill the chip (110 in 64 bits); with a lane per chain
// 660 ns a layer of the longest, and in proportion more from about five waves to four SIMDs on (unrounded ones, whose
// 64 bits are taken by rows, 100 ps a layer).  A line at 16,384 chains instead: 66,000 chains of up to 1,001 layers
// 883 -> 708 us, unrounded ones 675 -> 1,029, and of up to 600 layers 131,072 unrounded ones 828 -> 1,249.
inline bool ragged_waves_pay(const RaggedTotals &t)
{
    constexpr int64_t kChains = 6144, kLaneWaves = 1280;
    return t.wave_layers <= kChains * t.wave_longest * std::max(t.lane_waves, kLaneWaves) / kLaneWaves;
}

// Elements from one position to the next in a group's staging: rows start on 256 bytes for groups
// of 32 chains or more, on 64 bytes for smaller ones (a lone long chain is not blown up 32 times).
__host__ __device__ inline int64_t ragged_pitch(int64_t count)
{
    return count >= 32 ? (count + 31) / 32 * 32 : (count + 7) / 8 * 8;
}

// The descriptor of the group of `many` chains of n layers that follows the groups summed up in
// t, which it then joins; *tile_first2 receives the number of its first tile among those of the
// arrays with 2n+2 rows per chain.  The host's plan and the device's are both built with this.
__host__ __device__ inline RaggedGroupDev ragged_next_group(RaggedTotals &t, int n, int64_t many, int64_t *tile_first2)
{
    RaggedGroupDev g;
    g.n = n;
    g.count = (int32_t)many;
    g.first = (int32_t)t.chains;
    g.wave_first = (int32_t)t.waves;
    g.tile_first = t.tiles;
    g.stage_off = t.staged;
    g.pitch = ragged_pitch(many);
    g.tiles_x = (int32_t)((many + 63) / 64);
    g.linear_first = (int32_t)t.linear_waves;
    *tile_first2 = t.tiles2;
    t.n_groups += 1;
    t.max_layers = n;
    t.chains += many;
    t.waves += (many + 63) / 64;
    t.linear_waves += ragged_linear_waves(n, many);
    t.layers += n * many;
    if (n > kDeepLayers) {
        t.deep_chains += (int32_t)many;
        t.deep_layers += n * many;
    }
    if (ragged_wave_per_chain(n, many)) {
        t.wave_longest = n;
        t.wave_layers += n * many;
        t.lane_waves += (many + 63) / 64;
    } else {
        t.lane_longest = n;
    }
    t.tiles += (int64_t)g.tiles_x * ((n + 1 + 63) / 64);
    t.tiles2 += (int64_t)g.tiles_x * ((2 * n + 2 + 63) / 64);
    t.staged += ((int64_t)(n + 1) * g.pitch + 31) / 32 * 32;  // the next group starts on 256 bytes
    return g;
}

// The group that holds wave `wave`, place `place` or tile `tile` (each exists).
__device__ inline int ragged_group_of_wave(const RaggedGroupDev *g, int n_groups, int64_t wave)
{
    int lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)g[mid].wave_first <= wave) lo = mid; else hi = mid - 1;
    }
    return lo;
}
__device__ inline int ragged_group_of_linear_wave(const RaggedGroupDev *g, int n_groups, int64_t wave)
{
    int lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)g[mid].linear_first <= wave) lo = mid; else hi = mid - 1;
    }
    return lo;
}
__device__ inline int ragged_group_of_place(const RaggedGroupDev *g, int n_groups, int64_t place)
{
    int lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)g[mid].first <= place) lo = mid; else hi = mid - 1;
    }
    return lo;
}
__device__ inline int ragged_group_of_tile(const RaggedGroupDev *g, int n_groups, int64_t tile)
{
    int lo = 0, hi = n_groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (g[mid].tile_first <= tile) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// All groups of a ragged call in one launch each (the staging arrays hold every group).
// batch: chains in all groups (with CKPT_OBJ_BOTH peak_stage holds 2 * batch values)
hipError_t launch_eval_peak_ragged(const int64_t *d_stage, const uint8_t *mask_stage, const RaggedGroupDev *groups,
                                   const RaggedTotals &t, int64_t batch, int objective, int64_t *peak_stage,
                                   int32_t *status_stage, hipStream_t stream);
hipError_t launch_eval_timeline_ragged(const int64_t *d_stage, const uint8_t *mask_stage,
                                       const RaggedGroupDev *groups, int n_groups, int64_t waves, int objective,
                                       int64_t *wide_stage, int32_t *status_stage, hipStream_t stream);
// batch: chains in all groups.  ws as for launch_solve_linear(batch, t.max_layers).
hipError_t launch_solve_linear_ragged(const int64_t *d_stage, const RaggedGroupDev *groups, const RaggedTotals &t,
                                      int64_t batch, uint8_t *mask_stage, int64_t *peak_stage, int32_t *status_stage,
                                      void *ws, hipStream_t stream);
// The same for few enough chains, where they lie in the flat arrays; perm: the chains in order of their lengths;
// ws as above, its first three 32-bit words 0.
bool linear_takes_flat(int64_t batch, int n);
hipError_t launch_solve_linear_flat(const int64_t *d, const int64_t *off, const int32_t *perm, int64_t batch,
                                    const RaggedTotals &t, uint8_t *mask_out, int64_t *peak_out, int32_t *status_out, void *ws,
                                    hipStream_t stream);

// which: a ckpt_call; offsets_host: batch + 1 element offsets in host memory
size_t ragged_workspace_bytes(int which, const int64_t *offsets_host, int64_t batch);
// Returns a ckpt_status.  Copies the group table (and the offsets, if offsets_dev is null) to the
// workspace and waits for the copies; everything else is enqueued on the stream.
int launch_ragged(int which, const int64_t *d, const uint8_t *mask_in, const int64_t *offsets_host,
                  const int64_t *offsets_dev, int64_t batch,
                  int objective, uint8_t *mask_out, int64_t *peak_out, int64_t *budget_out, int64_t *timeline_out,
                  int32_t *status_out, void *ws, size_t ws_bytes, hipStream_t stream);

}  // namespace ckpt
