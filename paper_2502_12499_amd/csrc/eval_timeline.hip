// Memory per training phase index for a given checkpoint set (Section 5.1,
// "training phase index": 0 before training, 1..n the forward stage of layer
// i, n+1..2n the backward stages of layers n..1, 2n+1 after training), under
// the memory behaviour of Algorithm 2 (static objective) or Algorithm 3
// (dynamic objective), one lane per chain.
//
// A stage's value is the live memory after the stage's allocations and before
// the release at its end:
//   forward stage i     sum_{c in C, c <= i-1} d_c + d_i + [i-1 not in C] d_{i-1}
//   backward stage of layer i, with h the last checkpoint below i and nx the
//   first checkpoint at or above i:
//     Algorithm 3       sum_{c in C, c <= h} d_c + sum_{k=h+1}^{i} d_k + max_{h<=k<nx} d_k
//                       (Equation (memory) for i = nx, Equation (iprime) otherwise)
//     Algorithm 2       sum_{c in C} d_c + sum_{h<k<nx} d_k
//   index 0 and 2n+1    d_0
// so the largest backward stage is the peak that ckpt_eval_peak returns.
//
// A backward stage needs something from each side of position i: the part of
// its segment below i (running sums from the pass itself) and the part above,
// max or sum of d_i..d_{nx-1}; Algorithm 2's stages also contain the sum of ALL
// checkpoints.  Chains of up to kTwiceMaxLayers layers are divided among the
// waves of a workgroup, which hold their rows in registers: see
// eval_timeline_parts_kernel.  Both objectives then read 9(n+1) bytes and write
// 16(n+1) per chain (beyond kOnceMaxLayers layers the chain is read twice),
// which is what the stages themselves have to move.
// Longer chains, the groups of a ragged call, and under Algorithm 3 large
// batches of more than kOnceMaxLayers layers take the walk (timeline_walk), a
// lane per chain: it walks the chain once, upwards, in
// chunks of kChunk rows held in registers, with the next chunk already loaded
// and the one after it in flight.  For a chunk it first finds what lies above
// the chunk's last row (it scans the next chunk's registers up to the first
// checkpoint; while some lane of the wave has found none, the wave goes on
// with the rows in flight and then with eight further rows at a time),
// then sweeps the chunk downwards in registers to get the part above every
// row, then upwards to write both stages of every row.  For Algorithm 2 it
// passes over the chain once more beforehand, to add up the checkpoints.
#include "ckpt_internal.h"

namespace ckpt {
namespace {

constexpr int kBlock = 64;
constexpr int kChunk = 8;
// The parts of a chain.  32 rows are 112 registers a lane, so that four waves fit a SIMD: with 64 (two waves) and 16
// (seven) 1,048,576 chains of 256 layers take as long within 5 %, 997 chains of 300 layers 23 us instead of 18.
constexpr int kPartRows = 32, kPartWaves = 16;
constexpr int kOnceMaxLayers = kPartRows * kPartWaves, kTwiceMaxLayers = 2 * kOnceMaxLayers;
// Under Algorithm 3 the walk reads a chain once: beyond kOnceMaxLayers layers it is the faster one when its waves fill
// the chip (1,001 layers: 50,000 chains 551 us against 456 of the parts, 200,000 chains 1.08 ms against 1.52).
constexpr int64_t kTwiceMaxBatch = 49152;
extern __shared__ __align__(16) uint64_t timeline_parts[];

// The walk up the chain that writes both stages of every row.
template <int OBJ>
__device__ __forceinline__ void timeline_walk(const int64_t *__restrict__ dp, const uint8_t *__restrict__ mp,
                                              const int64_t pstride, const int n, const bool bad_mask,
                                              const uint64_t ckpt_all, int64_t *__restrict__ op, const int64_t opstride,
                                              int32_t *__restrict__ status_out, const int64_t c)
{
    auto ld = [&](int r) -> int64_t { return dp[(int64_t)r * pstride]; };
    auto lm = [&](int r) -> uint8_t { return mp[(int64_t)r * pstride]; };
    const int64_t x0 = dp[0];
    const int64_t last = 2 * (int64_t)n + 1;
    // the part of a segment above a row: its largest size (Algorithm 3) or its sum (Algorithm 2).
    // Sums are unsigned so that an invalid chain cannot trip signed overflow.
    auto join = [](uint64_t acc, int64_t x) -> uint64_t {
        return OBJ == CKPT_OBJ_STATIC ? acc + (uint64_t)x : ((uint64_t)x > acc ? (uint64_t)x : acc);
    };

    // rows beyond n re-read row n and are not used
    // the masks of a chunk that has arrived are kept as one bit per row
    int64_t cur_d[kChunk], nxt_d[kChunk];
    uint32_t cur_m = 0, nxt_m = 0;
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
        const int a = min(1 + u, n), b = min(1 + kChunk + u, n);
        cur_d[u] = ld(a); cur_m |= (uint32_t)(lm(a) != 0) << u;
        nxt_d[u] = ld(b); nxt_m |= (uint32_t)(lm(b) != 0) << u;
    }

    bool bad_size = x0 <= 0, ovf = false;
    uint64_t total = (uint64_t)x0;
    int64_t dmax = x0;

    op[0] = x0;
    uint64_t below = (uint64_t)x0;  // checkpoints up to the last one below the row
    uint64_t seg = 0;               // non-checkpoints since then
    int64_t segmax = x0;            // largest size from that checkpoint up to the row before
    int64_t prev = 0;               // the row before, if it is no checkpoint, else 0

    for (int k0 = 1; k0 <= n; k0 += kChunk) {
        int64_t far_d[kChunk];
        uint8_t far_m[kChunk];
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const int a = min(k0 + 2 * kChunk + u, n);
            far_d[u] = ld(a); far_m[u] = lm(a);
        }

        // what lies above the chunk's last row: d from the next chunk's first row up to (not
        // including) the first checkpoint.  Most lanes find it among the next chunk's rows; as
        // long as some lane of the wave has not, the whole wave looks at eight more rows: first
        // the ones already requested for the chunk after next, then further ones, eight loads
        // at a time (one memory latency per round instead of one per row).
        uint64_t acc = 0;
        bool found = false;
        auto bits = [](const uint8_t(&mm)[kChunk]) -> uint32_t {
            uint32_t b = 0;
#pragma unroll
            for (int u = 0; u < kChunk; ++u) b |= (uint32_t)(mm[u] != 0) << u;
            return b;
        };
        auto scan = [&](const int64_t(&dd)[kChunk], const uint32_t mm, const int first_row) {
#pragma unroll
            for (int u = 0; u < kChunk; ++u) {
                const bool ck = (mm >> u) & 1u;
                const bool open = !found && (first_row + u) <= n;
                found |= (first_row + u) > n || ck;
                if (open && !ck) acc = join(acc, dd[u]);
            }
        };
        scan(nxt_d, nxt_m, k0 + kChunk);
        if (__builtin_amdgcn_ballot_w64(!found) != 0) {
            scan(far_d, bits(far_m), k0 + 2 * kChunk);
            for (int kb = k0 + 3 * kChunk; __builtin_amdgcn_ballot_w64(!found) != 0; kb += kChunk) {
                int64_t more_d[kChunk];
                uint8_t more_m[kChunk];
#pragma unroll
                for (int u = 0; u < kChunk; ++u) {
                    const int a = min(kb + u, n);
                    more_d[u] = ld(a); more_m[u] = lm(a);
                }
                scan(more_d, bits(more_m), kb);
            }
        }

        // downwards: the part above each row of the chunk (the row itself included)
        uint64_t above[kChunk];
#pragma unroll
        for (int u = kChunk - 1; u >= 0; --u) {
            if (k0 + u <= n) acc = ((cur_m >> u) & 1u) ? 0 : join(acc, cur_d[u]);
            above[u] = acc;
        }

        // upwards: both stages of each row
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const int i = k0 + u;
            if (i > n) break;
            const int64_t x = cur_d[u];
            bad_size |= x <= 0;
            total += (uint64_t)x;
            ovf |= total > (uint64_t)INT64_MAX;
            dmax = x > dmax ? x : dmax;
            __builtin_nontemporal_store((int64_t)(below + (uint64_t)x + (uint64_t)prev), op + (int64_t)i * opstride);
            uint64_t b;
            if (OBJ == CKPT_OBJ_STATIC)
                b = ckpt_all + seg + above[u];
            else
                b = below + seg + (uint64_t)x + ((uint64_t)segmax > above[u] ? (uint64_t)segmax : above[u]);
            __builtin_nontemporal_store((int64_t)b, op + (last - i) * opstride);
            if ((cur_m >> u) & 1u) {
                below += (uint64_t)x;
                seg = 0;
                segmax = x;
                prev = 0;
            } else {
                seg += (uint64_t)x;
                segmax = x > segmax ? x : segmax;
                prev = x;
            }
        }
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            cur_d[u] = nxt_d[u];
            nxt_d[u] = far_d[u];
        }
        cur_m = nxt_m;
        nxt_m = bits(far_m);
    }
    op[last * opstride] = x0;
    ovf |= (total + (uint64_t)dmax) > (uint64_t)INT64_MAX;

    int32_t status = CKPT_OK;
    if (bad_size) status = CKPT_ERR_SIZE;
    else if (ovf) status = CKPT_ERR_OVERFLOW;
    else if (bad_mask) status = CKPT_ERR_MASK;
    if (status_out) status_out[c] = status;
    if (status != CKPT_OK)
        for (int64_t t = 0; t <= last; ++t) op[t * opstride] = -1;
}

// The timeline of chain c of a batch laid out by the strides (the lanes of a wave call it together).
template <int OBJ>
__device__ __forceinline__ void eval_timeline_chain(const int64_t *__restrict__ d, const uint8_t *__restrict__ mask,
                                                    int64_t batch, int n, int64_t cstride, int64_t pstride,
                                                    int64_t *__restrict__ out, int64_t ocstride, int64_t opstride,
                                                    int32_t *__restrict__ status_out, const int64_t c)
{
    if (c >= batch) return;
    const int64_t *dp = d + c * cstride;
    const uint8_t *mp = mask + c * cstride;

    uint64_t ckpt_all = 0;  // sum of all checkpoints (Algorithm 2 only)
    if (OBJ == CKPT_OBJ_STATIC) {
        // both loads of a row are issued whatever the mask says, so that sixteen rows are in flight
#pragma unroll 16
        for (int k = 0; k <= n; ++k) {
            const uint8_t on = mp[(int64_t)k * pstride];
            const int64_t x = dp[(int64_t)k * pstride];
            ckpt_all += on ? (uint64_t)x : 0;
        }
    }
    const bool bad_mask = mp[0] == 0 || mp[(int64_t)n * pstride] == 0;
    timeline_walk<OBJ>(dp, mp, pstride, n, bad_mask, ckpt_all, out + c * ocstride, opstride, status_out, c);
}

template <int OBJ>
__global__ __launch_bounds__(kBlock) void eval_timeline_kernel(const int64_t *__restrict__ d,
                                                               const uint8_t *__restrict__ mask, int64_t batch,
                                                               int n, int64_t cstride, int64_t pstride,
                                                               int64_t *__restrict__ out, int64_t ocstride,
                                                               int64_t opstride, int32_t *__restrict__ status_out)
{
    const int64_t c = (int64_t)xcd_paired_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    eval_timeline_chain<OBJ>(d, mask, batch, n, cstride, pstride, out, ocstride, opstride, status_out, c);
}

// The rows of 64 chains are divided into parts among the waves of a workgroup.  A wave holds its part in registers, all
// loads in flight at once, and sums it up; the parts' summaries meet in LDS; then each wave writes the stages of its own
// rows: what a row needs from outside its part is a few values per chain.  Up to kOnceMaxLayers layers a wave has one
// part and reads it once (TWICE = false); beyond, each has two, read again to write their stages.
// Bound by memory: 1,048,576 chains of 256 layers move 6.75 GB in 1.38 to 1.41 ms, 4.8 to 4.9 TB/s, what a large copy
// reaches (Algorithm 2 by the walk, which reads every chain twice: 1.97 ms).  With few chains, by one memory latency a
// pass: 997 chains of 300 layers 18 us (116), one of 152 layers 17 (35), 997 of 1,001 layers 72 (371).
// (Loads that bypass the caches: 2 % faster at that size, up to 40 % slower where the sizes fit the memory-side cache.)
struct Part {
    int64_t x[kPartRows];
    uint8_t on[kPartRows];
    int first, rows;
    __device__ __forceinline__ Part(int q, int per, int n) : first(1 + q * per), rows(min(per, n - q * per)) {}
};
struct Stages {
    int64_t *op;
    int64_t opstride, last;
    uint64_t ckpt_all;
};

template <int OBJ>
__device__ __forceinline__ uint64_t timeline_join(uint64_t acc, uint64_t v)
{
    return OBJ == CKPT_OBJ_STATIC ? acc + v : (v > acc ? v : acc);
}

// Eight rows at a time; rows past the part's end re-read its last one.
__device__ __forceinline__ void part_load(Part &p, const int64_t *__restrict__ dp, const uint8_t *__restrict__ mp,
                                          const int64_t pstride)
{
#pragma unroll
    for (int b = 0; b < kPartRows; b += 8) {
        if (b >= p.rows) break;
#pragma unroll
        for (int u = b; u < b + 8; ++u) {
            const int64_t r = p.first + (u < p.rows ? u : p.rows - 1);
            p.on[u] = mp[r * pstride];
            p.x[u] = dp[r * pstride];
        }
    }
}

// The mask of a part, a bit a row.
__device__ __forceinline__ uint32_t part_bits(const Part &p)
{
    uint32_t on = 0;
#pragma unroll
    for (int b = 0; b < kPartRows; b += 8) {
        if (b >= p.rows) break;
#pragma unroll
        for (int u = b; u < b + 8; ++u) on |= (uint32_t)(p.on[u] != 0) << u;
    }
    return on;
}

// Both stages of a part's rows.  below, seg, segmax, prev: of the rows before it; acc: what lies above it.
template <int OBJ>
__device__ __forceinline__ void part_write(const Part &p, const uint32_t on, const Stages &o, uint64_t below, uint64_t seg,
                                           int64_t segmax, int64_t prev, uint64_t acc)
{
    // what lies above the last row of each eight
    uint64_t above8[kPartRows / 8];
#pragma unroll
    for (int b = kPartRows - 8; b >= 0; b -= 8) {
        above8[b / 8] = acc;
        if (b >= p.rows || b == 0) continue;
#pragma unroll
        for (int u = b + 7; u >= b; --u)
            if (u < p.rows) acc = ((on >> u) & 1u) ? 0 : timeline_join<OBJ>(acc, (uint64_t)p.x[u]);
    }
#pragma unroll
    for (int b = 0; b < kPartRows; b += 8) {
        if (b >= p.rows) break;
        uint64_t above[8];
        acc = above8[b / 8];
#pragma unroll
        for (int u = b + 7; u >= b; --u) {
            if (u < p.rows) acc = ((on >> u) & 1u) ? 0 : timeline_join<OBJ>(acc, (uint64_t)p.x[u]);
            above[u - b] = acc;
        }
#pragma unroll
        for (int u = b; u < b + 8; ++u) {
            if (u >= p.rows) break;
            const int64_t i = p.first + u, x = p.x[u];
            __builtin_nontemporal_store((int64_t)(below + (uint64_t)x + (uint64_t)prev), o.op + i * o.opstride);
            uint64_t back;
            if (OBJ == CKPT_OBJ_STATIC)
                back = o.ckpt_all + seg + above[u - b];
            else
                back = below + seg + (uint64_t)x + ((uint64_t)segmax > above[u - b] ? (uint64_t)segmax : above[u - b]);
            __builtin_nontemporal_store((int64_t)back, o.op + (o.last - i) * o.opstride);
            const bool ck = (on >> u) & 1u;
            below += ck ? (uint64_t)x : 0;
            seg = ck ? 0 : seg + (uint64_t)x;
            if (OBJ != CKPT_OBJ_STATIC) segmax = ck || x > segmax ? x : segmax;
            prev = ck ? 0 : x;
        }
    }
}

enum { kCkpt, kTail, kTailMax, kHead, kTotal, kLargest, kPrev, kPartWords };  // a part's summary in LDS, [word][part][lane]
enum : uint32_t { kHas = 1, kBadSize = 2, kOverflow = 4, kBadMask = 8 };      // and its flags behind them, [part][lane]
size_t parts_lds_bytes(int parts) { return (size_t)parts * kBlock * (kPartWords * 8 + 4); }

template <int OBJ, bool TWICE>
__global__ __launch_bounds__(kBlock *kPartWaves) void eval_timeline_parts_kernel(
    const int64_t *__restrict__ d, const uint8_t *__restrict__ mask, int64_t batch, int n, int parts, int64_t cstride,
    int64_t pstride, int64_t *__restrict__ out, int64_t ocstride, int64_t opstride, int32_t *__restrict__ status_out)
{
    const int lane = threadIdx.x % kBlock, waves = blockDim.x / kBlock;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock);
    const int64_t chain = (int64_t)xcd_paired_block(blockIdx.x, gridDim.x) * kBlock + lane;
    const int64_t c = chain < batch ? chain : batch - 1;  // (lanes past the batch repeat the last chain, writing nothing)
    const int64_t *dp = d + c * cstride;
    const uint8_t *mp = mask + c * cstride;
    const int per = (n + parts - 1) / parts;  // rows 1 + q * per .. of part q
    uint32_t *const flags = (uint32_t *)(timeline_parts + (size_t)kPartWords * parts * kBlock);
    auto word = [&](int field, int q) -> uint64_t & { return timeline_parts[(field * parts + q) * kBlock + lane]; };

    const int64_t x0 = dp[0];
    auto sum_up = [&](const Part &p, const uint32_t on, const int q) {
        uint64_t ckpt = 0, tail = 0, head = 0, total = 0;
        int64_t tail_max = 0, largest = 0, prev = 0;
        uint32_t f = 0;
#pragma unroll
        for (int b = 0; b < kPartRows; b += 8) {
            if (b >= p.rows) break;
#pragma unroll
            for (int u = b; u < b + 8; ++u) {
                if (u >= p.rows) break;
                const int64_t x = p.x[u];
                const bool ck = (on >> u) & 1u;
                f |= x <= 0 ? kBadSize : 0;
                total += (uint64_t)x;
                f |= total > (uint64_t)INT64_MAX ? kOverflow : 0;
                largest = x > largest ? x : largest;
                f |= ck ? kHas : 0;
                head = (f & kHas) ? head : timeline_join<OBJ>(head, (uint64_t)x);
                ckpt += ck ? (uint64_t)x : 0;
                tail = ck ? 0 : tail + (uint64_t)x;
                if (OBJ != CKPT_OBJ_STATIC) tail_max = ck || x > tail_max ? x : tail_max;
                prev = ck ? 0 : x;
            }
        }
        if (q == 0) f |= (x0 <= 0 ? kBadSize : 0) | (mp[0] == 0 ? kBadMask : 0);
        if (q == parts - 1) f |= (on >> (p.rows - 1)) & 1u ? 0 : kBadMask;
        word(kCkpt, q) = ckpt;
        word(kTail, q) = tail;
        if (OBJ != CKPT_OBJ_STATIC) word(kTailMax, q) = (uint64_t)tail_max;
        word(kHead, q) = head;
        word(kTotal, q) = total;
        word(kLargest, q) = (uint64_t)largest;
        word(kPrev, q) = (uint64_t)prev;
        flags[q * kBlock + lane] = f;
    };
    int64_t *op = out + c * ocstride;
    Stages o{op, opstride, 2 * (int64_t)n + 1, 0};
    auto write = [&](const Part &p, const uint32_t on, const int mine) {
        uint64_t below = (uint64_t)x0, seg = 0, acc = 0, total = (uint64_t)x0;
        int64_t segmax = x0, prev = 0, largest = x0;
        uint32_t seen = 0;
        bool open = true;
        o.ckpt_all = (uint64_t)x0;
        for (int q = 0; q < parts; ++q) {
            const uint32_t f = flags[q * kBlock + lane];
            const uint64_t ck = word(kCkpt, q);
            o.ckpt_all += ck;
            if (q < mine) {
                below += ck;
                seg = (f & kHas) ? word(kTail, q) : seg + word(kTail, q);
                if (OBJ != CKPT_OBJ_STATIC) {
                    const int64_t m = (int64_t)word(kTailMax, q);
                    segmax = (f & kHas) || m > segmax ? m : segmax;
                }
                if (q == mine - 1) prev = (int64_t)word(kPrev, q);
            } else if (q > mine) {
                if (open) acc = timeline_join<OBJ>(acc, word(kHead, q));
                open = open && !(f & kHas);
            }
            // (the sum of the parts so far and a part are at most INT64_MAX each, or the flag is up)
            total += word(kTotal, q);
            seen |= f | (total > (uint64_t)INT64_MAX ? kOverflow : 0);
            const int64_t m = (int64_t)word(kLargest, q);
            largest = m > largest ? m : largest;
        }
        if (total + (uint64_t)largest > (uint64_t)INT64_MAX) seen |= kOverflow;
        const int32_t status = (seen & kBadSize)    ? CKPT_ERR_SIZE
                               : (seen & kOverflow) ? CKPT_ERR_OVERFLOW
                               : (seen & kBadMask)  ? CKPT_ERR_MASK
                                                    : CKPT_OK;
        if (chain >= batch) return;
        if (mine == 0) {
            op[0] = status == CKPT_OK ? x0 : -1;
            op[o.last * opstride] = status == CKPT_OK ? x0 : -1;
            if (status_out) status_out[c] = status;
        }
        if (status == CKPT_OK) {
            part_write<OBJ>(p, on, o, below, seg, segmax, prev, acc);
        } else {
            for (int64_t i = p.first; i < p.first + p.rows; ++i) {
                op[i * opstride] = -1;
                op[(o.last - i) * opstride] = -1;
            }
        }
    };

    if constexpr (TWICE) {
#pragma unroll 1
        for (int q = wave; q < parts; q += waves) {
            Part p(q, per, n);
            part_load(p, dp, mp, pstride);
            sum_up(p, part_bits(p), q);
        }
        __syncthreads();
#pragma unroll 1
        for (int q = wave; q < parts; q += waves) {
            Part p(q, per, n);
            part_load(p, dp, mp, pstride);
            write(p, part_bits(p), q);
        }
    } else {
        Part p(wave, per, n);
        part_load(p, dp, mp, pstride);
        const uint32_t on = part_bits(p);
        sum_up(p, on, wave);
        __syncthreads();
        write(p, on, wave);
    }
}

// Every group of a ragged call in one launch: a wave looks up the group its 64 chains belong to and
// writes their timelines (2n+2 rows, position-major) where the group's share of the wide staging
// lies, which is twice as far in as in the staging of the sizes.
template <int OBJ>
__global__ __launch_bounds__(kBlock) void eval_timeline_ragged_kernel(const int64_t *__restrict__ d_stage,
                                                                      const uint8_t *__restrict__ mask_stage,
                                                                      const RaggedGroupDev *__restrict__ groups,
                                                                      int n_groups, int64_t *__restrict__ wide_stage,
                                                                      int32_t *__restrict__ status_stage)
{
    const RaggedGroupDev g = groups[ragged_group_of_wave(groups, n_groups, blockIdx.x)];
    const int64_t c = ((int64_t)blockIdx.x - g.wave_first) * kBlock + threadIdx.x;
    eval_timeline_chain<OBJ>(d_stage + g.stage_off, mask_stage + g.stage_off, g.count, g.n, 1, g.pitch,
                                    wide_stage + 2 * g.stage_off, 1, g.pitch, status_stage + g.first, c);
}

// Checkpoint sets that do not depend on the sizes: the two ends only, every
// position, or segments of ceil(sqrt(n)) layers (the sqrt(n) rule of Section
// 2.1 as Section 5 applies it: n = 24 gives {5,10,15,20,24}).  The byte of a
// position is the same for every chain, so with chains next to each other in
// memory (chain stride 1) a lane writes the bytes of PACK chains as one word.
template <int PACK>
__global__ __launch_bounds__(kBlock) void select_baseline_kernel(int64_t batch, int n, int64_t cstride,
                                                                 int64_t pstride, int kind, int seg_len,
                                                                 uint8_t *__restrict__ mask_out)
{
    const int64_t c = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * PACK;
    if (c >= batch) return;
    uint8_t *mp = mask_out + c * cstride;
    int next_multiple = 0;
    for (int k = 0; k <= n; ++k) {
        bool on = k == 0 || k == n || kind == CKPT_SELECT_ALL;
        if (k == next_multiple) {
            on |= kind == CKPT_SELECT_SQRT;
            next_multiple += seg_len;
        }
        if (PACK == 8)
            __builtin_nontemporal_store(on ? 0x0101010101010101ull : 0ull, (uint64_t *)(mp + (int64_t)k * pstride));
        else
            mp[(int64_t)k * pstride] = on ? 1 : 0;
    }
}

std::atomic<bool> parts_lds_raised[kMaxDevices];

}  // namespace

hipError_t launch_eval_timeline(const int64_t *d, const uint8_t *mask, int64_t batch, int n, Strides st,
                                int objective, int64_t *out, Strides out_st, int32_t *status_out,
                                hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    const unsigned grid = (unsigned)((batch + kBlock - 1) / kBlock);
    if (n <= kOnceMaxLayers || (n <= kTwiceMaxLayers && (objective == CKPT_OBJ_STATIC || batch <= kTwiceMaxBatch))) {
        const int parts = (n + kPartRows - 1) / kPartRows, waves = parts < kPartWaves ? parts : kPartWaves;
        const size_t lds = parts_lds_bytes(parts);
        auto go = [&](auto kernel) -> hipError_t {
            if (lds > kDefaultLdsLimit) {  // (two parts to a wave)
                const hipError_t e = raise_lds_limit(parts_lds_raised,
                                                     {(const void *)eval_timeline_parts_kernel<CKPT_OBJ_STATIC, true>,
                                                      (const void *)eval_timeline_parts_kernel<CKPT_OBJ_DYNAMIC, true>},
                                                     parts_lds_bytes(kTwiceMaxLayers / kPartRows));
                if (e != hipSuccess) return e;
            }
            hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * kBlock), lds, stream, d, mask, batch, n, parts, st.chain,
                               st.pos, out, out_st.chain, out_st.pos, status_out);
            return hipGetLastError();
        };
        if (objective == CKPT_OBJ_STATIC)
            return parts <= kPartWaves ? go(eval_timeline_parts_kernel<CKPT_OBJ_STATIC, false>)
                                       : go(eval_timeline_parts_kernel<CKPT_OBJ_STATIC, true>);
        return parts <= kPartWaves ? go(eval_timeline_parts_kernel<CKPT_OBJ_DYNAMIC, false>)
                                   : go(eval_timeline_parts_kernel<CKPT_OBJ_DYNAMIC, true>);
    }
    if (objective == CKPT_OBJ_STATIC)
        hipLaunchKernelGGL(eval_timeline_kernel<CKPT_OBJ_STATIC>, dim3(grid), dim3(kBlock), 0, stream, d, mask,
                           batch, n, st.chain, st.pos, out, out_st.chain, out_st.pos, status_out);
    else
        hipLaunchKernelGGL(eval_timeline_kernel<CKPT_OBJ_DYNAMIC>, dim3(grid), dim3(kBlock), 0, stream, d, mask,
                           batch, n, st.chain, st.pos, out, out_st.chain, out_st.pos, status_out);
    return hipGetLastError();
}

hipError_t launch_eval_timeline_ragged(const int64_t *d_stage, const uint8_t *mask_stage,
                                       const RaggedGroupDev *groups, int n_groups, int64_t waves, int objective,
                                       int64_t *wide_stage, int32_t *status_stage, hipStream_t stream)
{
    if (waves == 0) return hipSuccess;
    static_assert(kBlock == kWave, "a workgroup is one of the groups' waves");
    if (objective == CKPT_OBJ_STATIC)
        hipLaunchKernelGGL(eval_timeline_ragged_kernel<CKPT_OBJ_STATIC>, dim3((unsigned)waves), dim3(kBlock), 0, stream,
                           d_stage, mask_stage, groups, n_groups, wide_stage, status_stage);
    else
        hipLaunchKernelGGL(eval_timeline_ragged_kernel<CKPT_OBJ_DYNAMIC>, dim3((unsigned)waves), dim3(kBlock), 0, stream,
                           d_stage, mask_stage, groups, n_groups, wide_stage, status_stage);
    return hipGetLastError();
}

hipError_t launch_select_baseline(int64_t batch, int n, Strides st, int kind, uint8_t *mask_out,
                                  hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    int seg_len = 1;  // ceil(sqrt(n))
    while ((int64_t)seg_len * seg_len < n) ++seg_len;
    // eight chains per lane when every row of eight bytes is contiguous and 8-byte aligned
    const bool packed = st.chain == 1 && batch % 8 == 0 && st.pos % 8 == 0 && ((uintptr_t)mask_out & 7u) == 0;
    if (packed) {
        const unsigned grid = (unsigned)((batch / 8 + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(select_baseline_kernel<8>, dim3(grid), dim3(kBlock), 0, stream, batch, n, st.chain, st.pos,
                           kind, seg_len, mask_out);
    } else {
        const unsigned grid = (unsigned)((batch + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(select_baseline_kernel<1>, dim3(grid), dim3(kBlock), 0, stream, batch, n, st.chain, st.pos,
                           kind, seg_len, mask_out);
    }
    return hipGetLastError();
}

}  // namespace ckpt
