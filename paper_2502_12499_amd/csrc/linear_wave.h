// The dynamic recurrence of one chain by one wave (solve_linear.hip: the wave kernel and ragged calls).
//
// Positions are taken in blocks, lane l = position hi - l.  Within a block the recurrence is a triangular system:
//   B(i) = min over j > i of max(M(j), U(i,j)),  M(j) = d_j + B(j),
// and U(i,j) = T(i) - T(j) + max(d_i..d_{j-1}) needs the sizes only.  So the block's U(i,j) are laid out first, a
// register per position j (the range maxima are a running maximum while j moves up through the block), then the
// positions are settled from the highest j down: M(j) is read from its lane, and all lanes take it in with a maximum and a
// minimum.  Four dependent instructions a position; the settled lanes need no mask, for M(j) > B(i) whenever j < i:
// the best way from j either stops at i, or passes over it by a step k1 -> k2, which from i costs no more.
// What lies beyond the block is the queue of Algorithm 6, an entry per lane: positions j with M(j) strictly decreasing
// and U(i,j) increasing in j.  Each lane takes its minimum over the entries before its block is settled; the entries
// after the first with U(lowest position,j) >= M(j) are dead for good (Lemma 4), and a block's own entries are those
// whose M is below that of all smaller positions of the block.
//
// What bounds it is instructions: a wave issues one every five cycles, and other waves on its SIMD take turns with it.
// 32 bits, cycles of a block of 64 positions (1,001 aligned sizes): sizes and their prefixes 310, the queue 790, the table
// 1,600, the positions one after the other 2,240, the new queue 960; 95 a position.  (2,460 for the table while each
// lane's value was read just before its use, 1,000 for the queue an entry at a time.)
#pragma once
#include "ckpt_internal.h"

#include <limits>

// v_writelane_b32 (the compiler has an intrinsic for it, but no builtin)
extern "C" __device__ int ckpt_write_lane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace ckpt {
namespace {

__device__ inline int32_t lane_value(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ inline int64_t lane_value(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ inline int32_t with_lane(int32_t v, int32_t x, int lane) { return ckpt_write_lane(x, lane, v); }
__device__ inline int64_t with_lane(int64_t v, int64_t x, int lane)
{
    const uint32_t lo = (uint32_t)ckpt_write_lane((int)(uint32_t)(uint64_t)x, lane, (int)(uint32_t)(uint64_t)v);
    const uint32_t hi = (uint32_t)ckpt_write_lane((int)((uint64_t)x >> 32), lane, (int)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <int CTRL, int ROWS>
__device__ inline int32_t dpp_value(int32_t old, int32_t v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ inline int64_t dpp_value(int64_t old, int64_t v)
{
    const uint32_t lo = (uint32_t)dpp_value<CTRL, ROWS>((int32_t)(uint32_t)(uint64_t)old, (int32_t)(uint32_t)(uint64_t)v);
    const uint32_t hi = (uint32_t)dpp_value<CTRL, ROWS>((int32_t)((uint64_t)old >> 32), (int32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ inline uint64_t lane_value(uint64_t v, int lane) { return (uint64_t)lane_value((int64_t)v, lane); }
__device__ inline uint64_t with_lane(uint64_t v, uint64_t x, int lane) { return (uint64_t)with_lane((int64_t)v, (int64_t)x, lane); }
template <int CTRL, int ROWS>
__device__ inline uint64_t dpp_value(uint64_t old, uint64_t v)
{
    return (uint64_t)dpp_value<CTRL, ROWS>((int64_t)old, (int64_t)v);
}

__device__ inline double lane_value(double v, int lane)
{
    return __builtin_bit_cast(double, lane_value(__builtin_bit_cast(int64_t, v), lane));
}
__device__ inline double with_lane(double v, double x, int lane)
{
    return __builtin_bit_cast(double, with_lane(__builtin_bit_cast(int64_t, v), __builtin_bit_cast(int64_t, x), lane));
}
template <int CTRL, int ROWS>
__device__ inline double dpp_value(double old, double v)
{
    return __builtin_bit_cast(double, dpp_value<CTRL, ROWS>(__builtin_bit_cast(int64_t, old), __builtin_bit_cast(int64_t, v)));
}

template <class S> __device__ inline S larger(S a, S b) { return a > b ? a : b; }
template <class S> __device__ inline S smaller(S a, S b) { return a < b ? a : b; }
// (one instruction; the compiler quiets NaNs first, or compares and selects.  The results are not DPP operands: the
// compiler does not count the wait states those need after an assembly statement.)
template <class S> __device__ inline S top_of(S a, S b) { return a > b ? a : b; }
template <class S> __device__ inline S least_of(S a, S b) { return a < b ? a : b; }
__device__ inline double top_of(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double least_of(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}


// Sums and maxima over the lanes up to this one.  (A lane without a source gets the operation's neutral value, which lets
// the compiler make one instruction of a step.)
template <class S>
__device__ inline S sum_up_to(S v)
{
    v += dpp_value<kDppRowShr1, 0xf>((S)0, v);
    v += dpp_value<kDppRowShr2, 0xf>((S)0, v);
    v += dpp_value<kDppRowShr4, 0xf>((S)0, v);
    v += dpp_value<kDppRowShr8, 0xf>((S)0, v);
    v += dpp_value<kDppRowBcast15, 0xa>((S)0, v);
    v += dpp_value<kDppRowBcast31, 0xc>((S)0, v);
    return v;
}
template <class S>
__device__ inline S max_up_to(S v)
{
    constexpr S kNone = std::numeric_limits<S>::lowest();
    v = larger(v, dpp_value<kDppRowShr1, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShr2, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShr4, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShr8, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowBcast15, 0xa>(kNone, v));
    v = larger(v, dpp_value<kDppRowBcast31, 0xc>(kNone, v));
    return v;
}
// Bits that some lane up to this one has set.
__device__ inline int64_t bits_up_to(int64_t v)
{
    v |= dpp_value<kDppRowShr1, 0xf>((int64_t)0, v);
    v |= dpp_value<kDppRowShr2, 0xf>((int64_t)0, v);
    v |= dpp_value<kDppRowShr4, 0xf>((int64_t)0, v);
    v |= dpp_value<kDppRowShr8, 0xf>((int64_t)0, v);
    v |= dpp_value<kDppRowBcast15, 0xa>((int64_t)0, v);
    v |= dpp_value<kDppRowBcast31, 0xc>((int64_t)0, v);
    return v;
}

constexpr int kDppRowShl1 = 0x101, kDppRowShl2 = 0x102, kDppRowShl4 = 0x104, kDppRowShl8 = 0x108;
// The maximum over the lanes above this one, `none` (the least there is) for the last.
template <class S>
__device__ inline S max_above(S v, const S none)
{
    constexpr S kNone = std::numeric_limits<S>::lowest();
    const int row = threadIdx.x % kWave / 16;
    v = larger(v, dpp_value<kDppRowShl1, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShl2, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShl4, 0xf>(kNone, v));
    v = larger(v, dpp_value<kDppRowShl8, 0xf>(kNone, v));
    const S r3 = lane_value(v, 48), r2 = larger(r3, lane_value(v, 32)), r1 = larger(r2, lane_value(v, 16));
    const S over = row == 0 ? r1 : row == 1 ? r2 : row == 2 ? r3 : none;
    return larger(over, dpp_value<kDppRowShl1, 0xf>(kNone, v));
}

// Positions of a block: a register (pair) of the table for each.
template <class S> constexpr int kBlockOf = sizeof(S) == 4 ? 64 : 32;
// Values the recurrence may reach: (sum(d) + max(d)) >> shift stays below.
template <class S> constexpr S kBeyond = (S)1 << 30;
template <> constexpr double kBeyond<double> = (double)((int64_t)1 << 52);  // (integers, exact to 2^53)
template <> constexpr uint64_t kBeyond<uint64_t> = (uint64_t)1 << 63;       // (twice as much fits: every checked chain)

// Turns the order around: the smallest of values is what the largest of these is turned back.
template <class S> __device__ inline S turned(S v) { return -v; }
__device__ inline uint64_t turned(uint64_t v) { return ~v; }

constexpr int kQueueBytes = 2048;
// Bytes of LDS: the queue while it is put together, the steps of a chain.
__host__ __device__ inline size_t wave_lds_bytes(int n) { return kQueueBytes + ((size_t)n + 1) * 2; }

// Sizes come from `load` (scaled, kBeyond bounds their sum and largest); the chosen step of every position goes to nxt.
// Returns false if more than 64 entries are live at the end of a block.
template <typename S, class Load>
__device__ __forceinline__ bool wave_steps(const Load load, const int n, unsigned char *lds, uint16_t *nxt, S &result)
{
    constexpr int kBlock = kBlockOf<S>, kGroup = 8, kEntries = 4;
    constexpr S kTop = kBeyond<S>;
    struct alignas(16) Entry { S M, minus_T, G, j; };
    static_assert(sizeof(Entry) * kWave <= kQueueBytes, "the queue's place in LDS");
    Entry *const queue = (Entry *)lds;
    const int lane = threadIdx.x % kWave;

    // the queue: lane p its entry p from the head, M(j), -T(j), G = the largest size from the block's end (hi + 1) to j - 1;
    // the lanes beyond the entries an M that is no minimum
    S qM = load(n), q_minus_T = 0, qG = 0;
    int qJ = n;
    int entries = 1;
    S base = lane_value(qM, 0);  // T(hi)
    qM = lane == 0 ? qM : kTop;
    S rows = load(n - 1 - lane);
    for (int hi = n - 1;; hi -= kBlock) {
        const int many = hi + 1 < kBlock ? hi + 1 : kBlock;
        const S d = lane < many ? rows : 0;
        rows = load(hi - kBlock - lane);  // (positions below 0 repeat position 0 and are not used)
        const S sums = sum_up_to(d), front = max_up_to(d);
        const S T = base + sums - d, minus_T = -T;

        // Beyond the block, until no lane has U(i,j) below what it has found: from there on U(i,j) only grows.
        S B = kTop - 1;
        int back = 0;  // hi - j of the choice
        for (int p0 = 0; p0 < entries; p0 += kEntries) {
            S M[kEntries], G[kEntries], minus[kEntries];
            int j[kEntries];
#pragma unroll
            for (int p = 0; p < kEntries; ++p) {
                M[p] = lane_value(qM, p0 + p);
                G[p] = lane_value(qG, p0 + p);
                minus[p] = lane_value(q_minus_T, p0 + p);
                j[p] = __builtin_amdgcn_readlane(qJ, p0 + p);
            }
            __builtin_amdgcn_sched_barrier(0);
            S u;
#pragma unroll
            for (int p = 0; p < kEntries; ++p) {
                u = top_of(front, G[p]) + T + minus[p];
                const S v = top_of(u, M[p]);
                back = v < B ? hi - j[p] : back;  // ties go to the lower index
                B = least_of(v, B);
            }
            if (__builtin_amdgcn_ballot_w64(u < B) == 0) break;
        }

        // U(i,j) of the block: lanes l > m hold T(i) - T(j) + max(d_i..d_{j-1}) for the position j of lane m; the others hold
        // what is not used.
        S table[kBlock];
        S R = 0;
#pragma unroll
        for (int g = kBlock / kGroup - 1; g >= 0; --g) {
            if (g * kGroup < many) {
                S minus[kGroup], dm[kGroup];
#pragma unroll
                for (int k = 0; k < kGroup; ++k) {
                    minus[k] = lane_value(minus_T, g * kGroup + k);
                    dm[k] = lane_value(d, g * kGroup + k);
                }
                __builtin_amdgcn_sched_barrier(0);  // (a lane's value can be used two instructions later)
#pragma unroll
                for (int k = kGroup - 1; k >= 0; --k) {
                    table[g * kGroup + k] = R + T + minus[k];
                    R = with_lane(top_of(R, dm[k]), dm[k], g * kGroup + k);
                }
            }
        }

        // The block, from its highest position down.  (Lanes without a position: sizes that no lane takes as M.)
        const S weight = lane < many ? d : kTop;
#pragma unroll
        for (int g = 0; g < kBlock / kGroup; ++g) {
            if (g * kGroup < many) {
#pragma unroll
                for (int m = g * kGroup; m < g * kGroup + kGroup; ++m) {
                    const S v = top_of(table[m], lane_value((S)(B + weight), m));
                    back = v <= B ? m : back;
                    B = least_of(v, B);
                }
            }
        }
        const S M = B + weight;
        if (lane < many) nxt[hi - lane] = (uint16_t)(hi - back);
        if (many == hi + 1) {
            result = lane_value(M, hi);
            return true;
        }

        // The queue seen from the next block: this block's entries, then those of the old ones whose M is smaller.
        const S below = max_above(d, (S)0);                             // max(d_lowest..d_{j-1})
        const S next = turned(max_above(turned(lane < kBlock ? M : kTop), turned(kTop)));  // the smallest M of the positions below
        const S Tlow = lane_value(T, kBlock - 1);
        uint64_t fresh = __builtin_amdgcn_ballot_w64(lane < kBlock && M < next);
        const uint64_t fresh_sat = __builtin_amdgcn_ballot_w64(below + (Tlow - T) >= M) & fresh;
        const S least = lane_value(smaller(M, next), 0);
        qG = larger(qG, lane_value(front, kBlock - 1));
        uint64_t old = __builtin_amdgcn_ballot_w64(lane < entries && qM < least);
        const int dropped = entries - (int)__popcll((unsigned long long)old);
        const uint64_t old_sat = __builtin_amdgcn_ballot_w64(qG + Tlow + q_minus_T >= qM) & old;
        if (fresh_sat) {  // (the queue goes through the block from its last lane)
            fresh &= ~0ull << (63 - __clzll((unsigned long long)fresh_sat));
            old = 0;
        } else if (old_sat) {
            old &= old_sat ^ (old_sat - 1);
        }
        const int ahead = (int)__popcll((unsigned long long)fresh);
        entries = ahead + (int)__popcll((unsigned long long)old);
        if (entries > kWave) return false;
        if ((fresh >> lane) & 1) {
            const int at = ahead - 1 - (int)__popcll((unsigned long long)(fresh & ((1ull << lane) - 1)));
            queue[at] = Entry{M, minus_T, below, (S)(hi - lane)};
        }
        if ((old >> lane) & 1) queue[ahead + lane - dropped] = Entry{qM, q_minus_T, qG, (S)qJ};
        __syncthreads();
        const Entry e = queue[lane];
        __syncthreads();
        qM = lane < entries ? e.M : kTop;
        q_minus_T = e.minus_T;
        qG = e.G;
        qJ = (int)e.j;
        base += lane_value(sums, kBlock - 1);
    }
}

}  // namespace
}  // namespace ckpt
