// The dynamic recurrence of four chains by one wave, a row of 16 lanes each (solve_linear.hip).
//
// The blocks of linear_wave.h with 16 positions to a block: the same table of U(i,j), the same order, the same queue, at
// most 16 entries of it live when a block ends.  What a lane has to tell its chain goes through the row broadcast of
// a DPP operand (row_newbcast), so a position costs nine instructions for four chains at once, no scalar register is
// passed, and nothing diverges; the work around a block (about 150 instructions) falls on 16 positions instead of 64.
// Values are unsigned 32-bit integers, or doubles as exact 53-bit integers (one instruction for a sum, a maximum or a
// comparison; a 64-bit maximum is three), or unsigned 64-bit integers where the sizes, divided by their common power of
// two, need them.  Where a queue outgrows its row, or a size is not positive, the chain is left to the form of a wave per chain.
//
// What bounds it is issue again, and alone on a SIMD the wait states around DPP operands: 72 ns a position (32 bits;
// 105 in doubles) with one wave there, 150 with four.  65,536 chains of 64 unrounded layers 45 us (62 in
// doubles, 66 with a move for each half of one), where a lane per chain took 137 (a try in 32 bits, then 64-bit integers
// with a queue in LDS, 1.8 us a position).
#pragma once
#include <type_traits>
#include <utility>

#include "ckpt_internal.h"
#include "linear_wave.h"

// v_mov_b64_dpp (the builtin takes a double, but not where its control depends on a template's argument)
extern "C" __device__ double ckpt_update_dpp(double old, double value, int control, int rows, int banks, bool bound)
    __asm("llvm.amdgcn.update.dpp.f64");

namespace ckpt {
namespace {

constexpr int kRow = 16;             // lanes of a chain, positions of a block
constexpr int kRowsOfWave = kWave / kRow;

// The value of lane LANE of the row, in all its lanes (8 bytes: one instruction too, as a double).
template <int LANE, class S>
__device__ inline S row_value(S v)
{
    constexpr int kRowNewBcast = 0x150;
    if constexpr (sizeof(S) == 4) {
        return __builtin_bit_cast(S, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), kRowNewBcast + LANE, 0xf, 0xf, true));
    } else {
        const double x = __builtin_bit_cast(double, v);
        return __builtin_bit_cast(S, ckpt_update_dpp(x, x, kRowNewBcast + LANE, 0xf, 0xf, true));
    }
}
// The value of the lane CTRL names, `none` in lanes without one.
template <int CTRL, class S>
__device__ inline S row_or(S none, S v)
{
    if constexpr (sizeof(S) == 4) {
        return __builtin_bit_cast(S, dpp_value<CTRL, 0xf>(__builtin_bit_cast(int32_t, none), __builtin_bit_cast(int32_t, v)));
    } else {
        return __builtin_bit_cast(S, dpp_value<CTRL, 0xf>(__builtin_bit_cast(int64_t, none), __builtin_bit_cast(int64_t, v)));
    }
}

// op over the lanes of the row up to this one, or from this one on
template <class S, class Op>
__device__ inline S row_up_to(S v, const S none, const Op op)
{
    v = op(v, row_or<kDppRowShr1>(none, v));
    v = op(v, row_or<kDppRowShr2>(none, v));
    v = op(v, row_or<kDppRowShr4>(none, v));
    return op(v, row_or<kDppRowShr8>(none, v));
}
template <class S, class Op>
__device__ inline S row_from(S v, const S none, const Op op)
{
    v = op(v, row_or<kDppRowShl1>(none, v));
    v = op(v, row_or<kDppRowShl2>(none, v));
    v = op(v, row_or<kDppRowShl4>(none, v));
    return op(v, row_or<kDppRowShl8>(none, v));
}

template <int FROM, int TO, class F>
__device__ __forceinline__ void unrolled(const F f)  // f(FROM), .., f(TO - 1)
{
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>());
        unrolled<FROM + 1, TO>(f);
    }
}

// (sum(d) + max(d)) >> shift of a chain stays below, and with it every M(j) and U(i,j); kRowTop stands for no M.  32 bits
// take all but the last two values, so nothing may be added to the top: chains of 64 unrounded layers of up to 256 MiB need
// 2^31 to 2^32, and took doubles while 32 bits ended at 2^30 (65,536 of them 62 us, now 45; aligned ones 44 both ways).  A
// wave's own form (linear_wave.h) does with 2^30: 997 chains of 1,001 aligned layers took 61.2 us this way, 60.4 so, and
// unrounded batches of its size gained nothing.
template <class S> constexpr uint64_t kRowBeyond = (uint64_t)kBeyond<S>;
template <> constexpr uint64_t kRowBeyond<uint32_t> = UINT32_MAX - 1;
template <class S> constexpr S kRowTop = (S)kRowBeyond<S>;
template <> constexpr uint32_t kRowTop<uint32_t> = UINT32_MAX;
// M(j) from B(j) and d_j, no less than the top where the weight is the top.  (32 bits: an addition that saturates.)
template <class S> __device__ inline S settled_M(S B, S weight) { return B + weight; }
__device__ inline uint32_t settled_M(uint32_t B, uint32_t weight)
{
    const uint32_t M = B + weight;
    return M < B ? UINT32_MAX : M;
}
// The -T(j) of no entry: its U, the largest size + T(i) - T(j), is more than any M, or, in 32 bits, than those of most
// chains: 2^31 and what of the block lies above i.  (It only says when to stop looking.)
template <class S> __device__ inline S row_no_T(S) { return kRowTop<S>; }
__device__ inline uint32_t row_no_T(uint32_t base) { return 0x80000000u - base; }
constexpr int kRowsQueueBytes = 2048;
__host__ __device__ inline size_t rows_lds_bytes(int n) { return kRowsQueueBytes + (size_t)kRowsOfWave * ((size_t)n + 1) * 2; }

// Sizes come from `load` (scaled; of the lane's own chain, of n layers), the chosen steps go to the row's nxt.
// Returns M(0), or (S)-1 if the row's queue was too short.  Rows of several lengths start together, each
// with its last block; one that has come to its first position runs along on sizes that no lane takes.
template <class S, class Load>
__device__ __forceinline__ S rows_steps(const Load load, const int n, unsigned char *lds, uint16_t *nxt)
{
    constexpr S kTop = kRowTop<S>;
    struct alignas(16) Entry { S M, minus_T, G; int32_t back; };
    static_assert(sizeof(Entry) * kWave <= kRowsQueueBytes, "the queue's place in LDS");
    const int lane = threadIdx.x % kWave, l = lane % kRow;
    Entry *const queue = (Entry *)lds + (lane - l);
    const auto top2 = [](S a, S b) { return a > b ? a : b; };
    const auto least2 = [](S a, S b) { return a < b ? a : b; };
    const auto sum2 = [](S a, S b) { return a + b; };

    // the queue: lane p of the row its entry p from the head, M(j), -T(j), G = the largest size from the block's end to
    // j - 1, hi - j; beyond the entries an M that is no minimum, with a U that ends the search
    const S last = load(n);
    S qM = l == 0 ? last : kTop, q_minus_T = l == 0 ? (S)0 : row_no_T(last), qG = 0;
    int q_back = -1;
    S base = last;  // T(hi)
    S result = -1;
    bool full = false;
    S rows = load(n - 1 - l);
    for (int hi = n - 1;; hi = hi > -kRow ? hi - kRow : hi) {
        const bool is = l <= hi;
        const S d = is ? rows : (S)0;
        rows = load(hi - kRow - l);  // (positions below 0 repeat position 0 and are not used)
        const S sums = row_up_to(d, (S)0, sum2), front = row_up_to(d, (S)0, top2);
        const S T = base + sums - d, minus_T = -T;

        S B = kTop - 1;
        int back = 0;  // hi - j of the choice
        const auto entries = [&](auto first) {  // four of them; false if none after them can matter
            S u;
            unrolled<0, 4>([&](auto k) {
                constexpr int p = decltype(first)::value + decltype(k)::value;
                u = top_of(front, row_value<p>(qG)) + T + row_value<p>(q_minus_T);
                const S v = top_of(u, row_value<p>(qM));
                const int b = row_value<p>(q_back);
                back = v < B ? b : back;  // ties go to the lower index
                B = least_of(v, B);
            });
            return __builtin_amdgcn_ballot_w64(u < B) != 0;
        };
        if (entries(std::integral_constant<int, 0>()) && entries(std::integral_constant<int, 4>()) &&
            entries(std::integral_constant<int, 8>()))
            (void)entries(std::integral_constant<int, 12>());

        // U(i,j) of the block, lanes above m
        S table[kRow];
        S R = 0;
        unrolled<0, kRow>([&](auto k) {
            constexpr int m = kRow - 1 - decltype(k)::value;
            table[m] = R + T + row_value<m>(minus_T);
            const S joined = top_of(R, row_value<m>(d));  // (in every lane: the operand's lane must be on)
            R = l == m ? d : joined;
        });
        // the block, from its highest position down
        const S weight = is ? d : kTop;
        unrolled<0, kRow>([&](auto k) {
            constexpr int m = decltype(k)::value;
            const S v = top_of(table[m], row_value<m>(settled_M(B, weight)));
            back = v <= B ? m : back;
            B = least_of(v, B);
        });
        const S M = settled_M(B, weight);
        if (is) nxt[hi - l] = (uint16_t)(hi - back);
        if (__builtin_amdgcn_ballot_w64(hi >= 0 && hi < kRow) != 0) {
            const S first = __shfl(M, lane - l + (hi & (kRow - 1)), kWave);
            result = hi >= 0 && hi < kRow && !full ? first : result;
        }
        if (__builtin_amdgcn_ballot_w64(hi >= kRow && !full) == 0) return result;

        // the queue seen from the next block
        const S below = row_or<kDppRowShl1>((S)0, row_from(d, (S)0, top2));
        const S next = row_or<kDppRowShl1>(kTop, row_from(M, kTop, least2));
        const S Tlow = row_value<kRow - 1>(T);
        const int shift = lane - l;
        const auto of_row = [&](bool b) { return (uint32_t)(__builtin_amdgcn_ballot_w64(b) >> shift) & 0xffffu; };
        uint32_t fresh = of_row(M < next);
        const uint32_t fresh_sat = of_row(below + (Tlow - T) >= M) & fresh;
        const S least = row_value<0>(least2(M, next));
        qG = top2(qG, row_value<kRow - 1>(front));
        uint32_t old = of_row(qM < least);
        const uint32_t old_sat = of_row(qG + Tlow + q_minus_T >= qM) & old;
        fresh &= fresh_sat ? ~0u << (31 - __clz((int)fresh_sat)) : ~0u;
        old &= fresh_sat ? 0u : old_sat ^ (old_sat - 1);  // (all of them if none is)
        const int ahead = __popc(fresh), entries_now = ahead + __popc(old);
        full |= hi >= kRow && entries_now > kRow;
        if ((fresh >> l) & 1) queue[__popc(fresh >> (l + 1))] = Entry{M, minus_T, below, l - kRow};
        const int at = ahead + __popc(old & ((1u << l) - 1));
        if (((old >> l) & 1) && at < kRow) queue[at] = Entry{qM, q_minus_T, qG, q_back - kRow};
        __syncthreads();
        const Entry e = queue[l];
        __syncthreads();
        base += row_value<kRow - 1>(sums);
        const bool live = l < entries_now;
        qM = live ? e.M : kTop;
        q_minus_T = live ? e.minus_T : row_no_T(base);
        qG = live ? e.G : (S)0;
        q_back = e.back;
    }
}

}  // namespace
}  // namespace ckpt
