// ckpt_solve_cubic as a search over the budgets (Section 3.2: Equation (T), Algorithm 4).
//
// The answer is min over the budgets s of s + c_s, and the smallest s that attains it.  c_s, the
// least checkpoint memory whose segments all fit in s, does not grow with s, and it is defined for
// every integer s >= 0, budget or not (it changes at budgets only, so the smallest s that attains
// the minimum over the integers is a budget).  So a few evaluated points settle whole intervals:
// with c known at the right end b of (a, b], every s in between costs at least s + c_b, and only
// those with s + c_b <= UB, the best cost seen so far, can be optimal.  (Ties survive the test,
// so the smallest optimal budget is found.)  A chain of 64 layers is settled after about 130
// evaluations of its 2,017 budgets, one of 4,096 layers after about 3,000 of 8.4 million.
//
//   1. Points on a geometric grid over [0, sum of the interior layers].
//   2. The intervals between them that may still hold the optimum are kept.
//   3. When few budgets lie in them (each is the difference of two prefix sums: found by bisection,
//      the starts across the lanes) those are evaluated, and that is the end; else the
//      intervals are cut into smaller ones at new points, and so on.
#include <limits>
#include <type_traits>

#include "ckpt_internal.h"

namespace ckpt {
namespace {

extern __shared__ __align__(16) unsigned char search_lds[];

// ---------------------------------------------------------------------------
// short chains: one wave per chain, one lane per point
// ---------------------------------------------------------------------------

// F_s(j) = d_j + min of F_s over the window [l, j-1] of the predecessors within s.  All lanes walk j
// together, every lane with its own s and hence its own l.  The window minimum needs no queue:
// positions are taken in blocks of kBlk, and two arrays per lane hold suffix minima,
//   L1[p]  min F over p .. the end of p's block (of its part that has been filled)
//   L2[q]  min F over the full blocks q, q+1, ..
// so that the minimum over [l, j-1] is that of L1[l], L2[block(l) + 1] and the running minimum of the
// block under way.  Filling position p writes L1[p] and lowers the earlier entries of its block
// (LDS minima without return), a full block lowers L2.  Which entries are written does not depend
// on the lane, so nothing diverges, however far apart the lanes' budgets are.
// What bounds it: the latency of about 45 instructions a cell with one or two waves on a SIMD, which is what the
// LDS space leaves (20 KB a wave at 64 layers in 32 bits): 310 cycles a cell of 64 points alone, 390 with two
// waves.  The loads a cell depends on are issued a cell ahead (the predecessor j-1 always lies in the window
// and is joined from its register), those that the window's start depends on two.
// Batches below rows_from(): 4,096 chains of 64 layers of unrounded sizes 124 us, one chain of 152 layers 88 us (129 us with
// a queue per lane for every budget); 65,536 of 64 layers took 1.28 ms so (31.2), and 0.66 with rows.
//
// Arithmetic.  UB, the cost of a feasible set, bounds the optimum, so a value of F above UB may
// be cut off at any number above UB: with UB < 2^31 (sizes divided by their common power of two) 32
// bits are enough whatever the sizes add up to.  The prefix sums are then kept modulo 2^32: a
// window's sum is at most s plus one size, and the lookahead sees at most three sizes past a window; where
// both stay below 2^31 the differences that are looked at are exact as signed values.  Other chains take
// 64 bits.
constexpr int kBlk = 8;
constexpr int kStack = 64;      // intervals kept, at most one per lane
constexpr int kLookahead = 4;   // prefix sums read ahead of a window's start

__host__ __device__ inline int blocks_of(int n) { return (n + kBlk - 1) / kBlk; }
// Elements of the prefix sums with the padding that the reads past n see.
__host__ __device__ inline int sums_len(int n) { return (n + 1 + kBlk + 1 + kLookahead + 3) / 4 * 4; }
constexpr int kLists = 3 * kStack + kWave;  // elements of the stack (three values an interval) and of the list of points
// LDS of one chain in arithmetic of `width` bytes.
__host__ __device__ inline size_t search_lds_bytes(int n, int width)
{
    return ((size_t)sums_len(n) + kLists + ((size_t)blocks_of(n) * kBlk + blocks_of(n) + 2) * kWave) *
           (size_t)width;
}

template <typename U>  // uint32_t or uint64_t
struct SearchLds {
    typedef std::make_signed_t<U> I;
    U *P;      // [sums_len(n)] P[k] = d_0 + .. + d_k (modulo 2^32 for 32 bits), padded with P[n]
    I *lo;     // [kStack] the intervals' lower ends (exclusive) ...
    I *hi;     // [kStack] ... upper ends ...
    U *c;      // [kStack] ... and c at or beyond the upper end
    I *list;   // [kWave] points
    U *L1;     // [blocks * kBlk][kWave]
    U *L2;     // [blocks + 2][kWave]
    __device__ SearchLds(unsigned char *base, int n)
    {
        P = (U *)base;
        lo = (I *)(P + sums_len(n));
        hi = lo + kStack;
        c = (U *)(hi + kStack);
        list = (I *)(c + kStack);
        L1 = (U *)lo + kLists;
        L2 = L1 + (size_t)blocks_of(n) * kBlk * kWave;
    }
};

template <typename U>
__device__ inline void lds_min(U *p, U v)
{
    (void)__hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// F_s(n) for the lane's s, 0 <= s <= UB; in 32 bits values above 2^31 are cut to that.  FLAT: the prefix sums are
// those in full, so that they are compared with x - s as they are, not by their differences from x (three instructions
// less a cell: 65,536 unrounded chains of 64 layers 1.37 ms, 1.31 with this).
template <bool FLAT, typename U>
__device__ __forceinline__ U lane_cost(const SearchLds<U> &m, const int n, const U s)
{
    typedef std::make_signed_t<U> I;
    constexpr U kMax = std::numeric_limits<U>::max();
    constexpr U kCap = (U)1 << (8 * sizeof(U) - 1);
    const int lane = threadIdx.x;
    const int nb = blocks_of(n);
    U *const L1 = m.L1 + lane, *const L2 = m.L2 + lane;
    const U *const P = m.P;
    for (int q = 0; q < nb * kBlk; ++q) L1[q * kWave] = kMax;
    for (int q = 0; q < nb + 2; ++q) L2[q * kWave] = kMax;
    U p0 = P[0], p1 = P[1], p2 = P[2], p3 = P[3];  // P[l ..] of the last window start found
    // the start of the window of the next cell, whose sums end in x: it moves on while x - P[l] > s (at the latest
    // until x itself: the differences beyond are negative)
    auto advance = [&](int l, const U x) -> int {
        const I w = (I)s;
        const U edge = x > s ? x - s : 0;
        const auto out = [&](const U p) { return FLAT ? p < edge : (I)(x - p) > w; };
        l += (int)out(p0) + (int)out(p1) + (int)out(p2);
        bool far = out(p3);
        l += (int)far;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
            do {
                const U q0 = P[l], q1 = P[l + 1], q2 = P[l + 2], q3 = P[l + 3];
                l += far ? (int)out(q0) + (int)out(q1) + (int)out(q2) + (int)out(q3) : 0;
                far = far && out(q3);
            } while (__builtin_amdgcn_ballot_w64(far) != 0);
        }
        return l;
    };
    // Turn p fills in F(p) and forms F(p + 1); at its start l1 and l2 are the window starts of cells p + 1 and
    // p + 2, and a, c are L1 and L2 of l1 as of the position before p.  (The turns of the last block go on
    // past n: a branch per cell costs more than seven cells of padding.)
    U f = P[0], a = kMax, c = kMax, result = 0;
    int l1 = 0, l2 = advance(0, P[1]);
    p0 = P[l2]; p1 = P[l2 + 1]; p2 = P[l2 + 2]; p3 = P[l2 + 3];
    U x0 = P[0], x1 = P[1];          // P[p], P[p + 1]
    for (int b = 0; b < nb; ++b) {
        U Pb[kBlk];                  // P[p + 2] of the block's turns
#pragma unroll
        for (int u = 0; u < kBlk; ++u) Pb[u] = P[b * kBlk + u + 2];
        U *const row = L1 + b * kBlk * kWave;
        U cur = kMax;                // minimum of the block under way, without the position being added
#pragma unroll
        for (int u = 0; u < kBlk; ++u) {
            const int p = b * kBlk + u;
#pragma unroll
            for (int k = 0; k <= u; ++k) lds_min(row + k * kWave, f);
            if (u == kBlk - 1) {
                const U whole = cur < f ? cur : f;
                for (int q = 0; q <= b; ++q) lds_min(L2 + q * kWave, whole);
            }
            const U an = L1[l2 * kWave], cn = L2[(((unsigned)l2 / kBlk) + 1) * kWave];
            U g = f;
            if (u > 0) {
                const U seen = l1 < b * kBlk ? cur : kMax;
                g = seen < f ? seen : f;
                cur = cur < f ? cur : f;
            } else {
                cur = f;
            }
            U w = a < c ? a : c;
            w = w < g ? w : g;
            f = (x1 - x0) + w;
            if (sizeof(U) == 4) f = f < kCap ? f : kCap;
            result = p + 1 == n ? f : result;
            a = an;
            c = cn;
            x0 = x1;
            x1 = Pb[u];
            l1 = l2;
            l2 = advance(l2, x1);
            p0 = P[l2]; p1 = P[l2 + 1]; p2 = P[l2 + 2]; p3 = P[l2 + 3];
        }
    }
    return result;
}

// The smallest x in [lo, hi] with P[x] - from > bound (hi if there is none below hi).
template <typename U>
__device__ inline int first_above(const U *P, int lo, int hi, U from, U bound, int steps)
{
    for (int k = 0; k < steps; ++k) {
        const int mid = (lo + hi) >> 1;
        const bool up = lo < hi && P[mid] - from <= bound;
        hi = (lo < hi && !up) ? mid : hi;
        lo = up ? mid + 1 : lo;
    }
    return lo;
}

// lane `src`'s value, src the same in every lane
__device__ inline int32_t uniform_lane(int32_t v, int src) { return __builtin_amdgcn_readlane(v, src); }
__device__ inline int64_t uniform_lane(int64_t v, int src)
{
    const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(uint64_t)v, src);
    const uint32_t h = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), src);
    return (int64_t)(((uint64_t)h << 32) | l);
}

template <typename U>
__device__ inline U uniform_lane_u(U v, int src) { return (U)uniform_lane((std::make_signed_t<U>)v, src); }

// min over the wave of (a, b), lexicographic; every lane gets the result
__device__ inline void wave_best(uint32_t &a, uint32_t &b)
{
    const uint64_t m = wave_min_u64(((uint64_t)a << 32) | b);
    a = (uint32_t)(m >> 32);
    b = (uint32_t)m;
}
__device__ inline void wave_best(uint64_t &a, uint64_t &b)
{
    int64_t x = (int64_t)a, y = (int64_t)b;  // (below 2^63, or the largest value of the type: see the caller)
    wave_min_pair(x, y);
    a = (uint64_t)x;
    b = (uint64_t)y;
}

constexpr int kSearchPer = kSearchMaxLayers / kWave + 1;  // positions per lane

// The least s + c_s and the smallest s that attains it.  `total`: the sum of all sizes; `bound`: the cost of a
// feasible set; `span`: no s beyond it can be optimal; `ends[q]`: the first x > r with P[x] - P[r] > span, r = q * 64
// + lane (n if there is none below n); `all`: the sum of the interior layers; `heavy`: a layer that outweighs the
// others, within the span, or 0.
template <typename U>
__device__ __forceinline__ void search_chain(const SearchLds<U> &m, const int n, const uint64_t total, const U bound, const U span,
                                             const int (&ends)[kSearchPer], const int steps, const float all,
                                             const U heavy, U &best_cost, U &best_s)
{
    typedef typename SearchLds<U>::I I;
    const int lane = threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    // s = 0 makes every layer a checkpoint: `total`, optimal only if no set costs less
    best_cost = total <= bound ? (U)total : std::numeric_limits<U>::max();
    best_s = 0;
    const bool flat = total <= std::numeric_limits<U>::max();
    U ub = bound;   // the best cost known
    // the first points cut (0, span] evenly
    I prev = (I)(span >> 6) * lane + (I)(((span & 63) * (U)lane) >> 6);
    I s = (I)(span >> 6) * (lane + 1) + (I)(((span & 63) * (U)(lane + 1)) >> 6);
    if (heavy != 0) {
        // One of them moves to the heavy layer's size: its cost settles nearly all the budgets without that layer, which
        // the even cuts leave in one interval if it outweighs them enough (to be cut 64-fold a round).  A chain of 100
        // layers, one 10^15, the others up to 10^6: 85 to 89 us, without this cut 150 to 246 (every budget evaluated: 86).
        const int below_it = (int)__popcll((unsigned long long)__builtin_amdgcn_ballot_w64((U)s < heavy));
        const int moved = below_it < kWave - 1 ? below_it + 1 : kWave - 1;
        prev = lane == moved ? (I)heavy : prev;
        s = lane + 1 == moved ? (I)heavy : s;
    }
    bool on = s > prev;
    int count = 0;  // intervals on the stack
    enum { kCut, kListed, kEveryBudget } step = kCut;
    int a = 0, x0 = 1;  // kEveryBudget: the start and the first end to come
    for (;;) {
        const U c = sizeof(U) == 8 || flat ? lane_cost<true>(m, n, (U)s) : lane_cost<false>(m, n, (U)s);
        {
            // (a point that is no budget may cost more than the optimum's type holds: it wraps nowhere
            // below 2^63 or 2^32, and what is above the bound is no candidate)
            const U cost = (U)s + c;
            U bc = on && cost <= ub ? cost : (U)std::numeric_limits<I>::max(), bs = (U)s;
            wave_best(bc, bs);
            if (bc <= ub && (bc < best_cost || (bc == best_cost && bs < best_s))) {
                best_cost = bc;
                best_s = bs;
                ub = bc;
            }
        }
        if (step == kListed) break;
        if (step == kCut) {
            // what the points leave of their intervals
            const I room = (I)(ub - c);
            const I top = s - 1 < room ? s - 1 : room;
            const bool live = on && c <= ub && top > prev;
            const uint64_t lives = __builtin_amdgcn_ballot_w64(live);
            const int many = (int)__popcll(lives);
            if (count + many > kStack) {
                step = kEveryBudget;  // more near-optimal intervals than the stack holds (a plateau of ties)
            } else {
                __syncthreads();
                if (live) {
                    const int at = count + (int)__popcll(lives & below);
                    m.lo[at] = prev;
                    m.hi[at] = top;
                    m.c[at] = c;
                }
                count += many;
                __syncthreads();
                // the intervals under the best cost of now
                I lo = 0, hi = 0;
                if (lane < count) {
                    lo = m.lo[lane];
                    hi = m.hi[lane];
                    const U ic = m.c[lane];
                    const I r = ic <= ub ? (I)(ub - ic) : (I)-1;
                    hi = hi < r ? hi : r;
                }
                const uint64_t open = __builtin_amdgcn_ballot_w64(hi > lo);
                if (open == 0) break;
                // About n budgets lie in a width of one mean layer.  When that puts few of them in the
                // intervals: collect them (from every start the ends between the lowest and the highest
                // interval), and if they fit the lanes, evaluate them and be done.  A table of the values seen
                // last (in the room of L1) keeps most repeated ones out: networks repeat their layers.
                float width = hi > lo ? (float)(hi - lo) : 0.0f;
#pragma unroll
                for (int k = kWave / 2; k >= 1; k >>= 1) width += __shfl_xor(width, k, kWave);
                if (width * (float)n * (float)n <= 3.0f * (float)kWave * all) {
                    constexpr unsigned kSeen = kBlk * kWave;
#pragma unroll
                    for (unsigned k = 0; k < kSeen; k += kWave) m.L1[k + lane] = 0;
                    U lowest = hi > lo ? (U)lo : std::numeric_limits<U>::max();
                    U highest = hi > lo ? ~(U)hi : std::numeric_limits<U>::max();
                    if constexpr (sizeof(U) == 4) {
                        lowest = wave_min_u32(lowest);
                        highest = ~wave_min_u32(highest);
                    } else {
                        lowest = wave_min_u64(lowest);
                        highest = ~wave_min_u64(highest);
                    }
                    int found = 0;
                    bool fits = true;
#pragma unroll
                    for (int q = 0; q < kSearchPer; ++q) {
                        if (q * kWave >= n - 1 || !fits) break;
                        const int r = q * kWave + lane;
                        const U pr = m.P[r < n ? r : n];
                        int x = first_above(m.P, r + 1 < n ? r + 1 : n, ends[q], pr, lowest, steps);
                        for (;;) {
                            const U sv = m.P[x] - pr;
                            const bool walks = r < n - 1 && x < ends[q] && sv <= highest;
                            if (__builtin_amdgcn_ballot_w64(walks) == 0) break;
                            bool in = false;
                            for (uint64_t todo = open; todo != 0; todo &= todo - 1) {
                                const int iv = __ffsll((unsigned long long)todo) - 1;
                                const U ilo = (U)uniform_lane(lo, iv), ihi = (U)uniform_lane(hi, iv);
                                in |= sv > ilo && sv <= ihi;
                            }
                            in = in && walks;
                            if (in) {
                                const unsigned at = ((uint32_t)sv * 2654435761u) >> 23;
                                static_assert(kSeen == 512, "nine bits of the product");
                                in = __hip_atomic_exchange(m.L1 + at, sv, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_WORKGROUP) != sv;
                            }
                            const uint64_t ins = __builtin_amdgcn_ballot_w64(in);
                            const int more = (int)__popcll(ins);
                            if (found + more > kWave) {
                                fits = false;
                                break;
                            }
                            if (in) m.list[found + (int)__popcll(ins & below)] = (I)sv;
                            found += more;
                            x += walks ? 1 : 0;
                        }
                    }
                    __syncthreads();
                    if (fits) {
                        if (found == 0) break;
                        on = lane < found;
                        s = m.list[on ? lane : 0];
                        step = kListed;
                        continue;
                    }
                }
                // else the last eight (four, two, one) of them, each cut at as many points as there are lanes for it
                const int lg = count >= 8 ? 3 : count >= 4 ? 2 : count >= 2 ? 1 : 0;
                const int per_lg = 6 - lg;
                const int from = count - (1 << lg) + (lane >> per_lg), k = lane & ((1 << per_lg) - 1);
                const I ilo = (I)__shfl(lo, from, kWave), ihi = (I)__shfl(hi, from, kWave);
                const I wide = ihi > ilo ? ihi - ilo : 0;
                const I part = wide >> per_lg, odd = wide & (I)((1 << per_lg) - 1);
                prev = ilo + part * (I)k + ((odd * (I)k) >> per_lg);
                s = ilo + part * (I)(k + 1) + ((odd * (I)(k + 1)) >> per_lg);
                on = s > prev;
                count -= 1 << lg;
                continue;
            }
        }
        // kEveryBudget: start after start, 64 ends at a time (0 is known)
        while (a < n - 1 && x0 >= n) {
            ++a;
            x0 = a + 1;
        }
        if (a >= n - 1) break;
        const int x = x0 + lane;
        const U sv = m.P[x < n ? x : n - 1] - m.P[a];
        s = (I)(sv <= span ? sv : 0);
        on = true;
        x0 += kWave;
    }
}

// ---------------------------------------------------------------------------
// one wave, one budget
// ---------------------------------------------------------------------------

// mask ? on : off per lane, the mask in scalar registers
__device__ inline uint32_t select_lanes(uint32_t off, uint32_t on, uint64_t mask)
{
    uint32_t r;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"(off), "v"(on), "s"(mask));
    return r;
}
__device__ inline uint64_t select_lanes(uint64_t off, uint64_t on, uint64_t mask)
{
    return ((uint64_t)select_lanes((uint32_t)(off >> 32), (uint32_t)(on >> 32), mask) << 32) |
           select_lanes((uint32_t)off, (uint32_t)on, mask);
}

// F_s(n) by a whole wave, head by head.  While the head h stays in the window, F(j) = d_j + F(h) and h is a
// minimal predecessor of j, for all those j at once; when it leaves (cell e), the new head is an
// index with minimal F in the window of e: what enters later is larger than the minimum, and what lies
// before it is larger or gone.  Of several such indices the last one is taken, which stays longest: networks repeat
// their layers, and a chain of 1,001 of theirs has 64 heads in its slowest pass so, 575 if the first one is taken.
// (The canonical set wants the first one: see first_pred.)  The lanes hold three neighbouring slices of 64 positions
// in registers and slide along the chain: Z, the positions before, A, where the next cells are, and B, whose prefix
// sums are under way; a window that reaches back beyond Z is finished from two older slices and from the values
// parked in F (whose sums come from memory: 64 layers a segment are usual in a chain of 4,096).
// What bounds it is the chain of dependent instructions of a head (about 45, half of them scalar, eight to nine
// cycles each; a loop of its own for the heads of a slice takes three jumps a head out of it); a
// form that kept the values in LDS took 1,190 cycles a head, most of it four LDS round trips. P: prefix sums, P[n]
// below 2^31 or 2^63; F (and head): room for n + 1 + kWave values; RECORD: head[j], a minimal predecessor of j, is
// written for j = 1..n, F(j) for j < n, and *ties says whether any was one of several.  stop(F(h)) is asked once per
// slice; when it says so the pass ends with F(h), which F_s(n) is not below.  The pass ends whatever the sums are: a
// new head keeps the cell it was chosen for, seen or not (on sums that ascend it always sees it; a test for an empty
// window took 5 % of a call), and a slice past the last cell ends the pass with the largest value of the type.
struct NeverStop {
    template <typename U>
    __device__ bool operator()(U) const { return false; }
};
constexpr int kOlder = 2;
template <typename U, bool RECORD, typename H, class Stop = NeverStop>
__device__ __forceinline__ U wave_cost(const U *P, const int n, const U s, U *F, H *head, Stop stop = Stop(),
                                       bool *ties = nullptr)
{
    constexpr U kMax = std::numeric_limits<U>::max();
    const int lane = threadIdx.x % kWave;
    // P at position k, and P[k - 1], what cell k compares (past n: larger than anything, so the cell ends the head)
    auto at = [&](int k) -> U { return P[k < n ? k : n]; };
    auto before = [&](int k) -> U { return k > n ? kMax : P[k > 0 ? k - 1 : 0]; };
    int base = 0;                          // A holds the positions base + lane
    // per position: P + s (a window of sums ending in x begins where this reaches x), the size, P before, F
    U SZ = 0, FZ = kMax, PA = at(lane), QA = before(lane), PB = at(kWave + lane), QB = before(kWave + lane);
    U SA = PA + s, DA = PA - QA;
    U SY[kOlder] = {}, FY[kOlder] = {};    // the slices before Z
    U FA = PA;                             // (F(0) = P[0] in lane 0)
    int HA = 0;
    int h = 0, most = 1;                   // most: of equal values among which a head was chosen
    uint64_t from = ~1ull, test = ~1ull;   // the lanes of the head's cells, and of those that may end it
    U fh = uniform_lane_u(PA, 0), Sh = fh + s;
    for (;;) {
        uint64_t out;
        for (;;) {
            // as if h stayed for all of its cells (a later head overwrites them)
            FA = select_lanes(FA, DA + fh, from);
            if (RECORD) HA = (int)select_lanes((uint32_t)HA, (uint32_t)h, from);
            out = __builtin_amdgcn_ballot_w64(QA > Sh) & test;
            if (out == 0) break;
            const int e = __builtin_ctzll((unsigned long long)out);  // the first cell that does not see h
            if (__builtin_expect(base + e > n, 0)) break;
            // The window of e: P[i] + s >= P[e - 1], i < e; h and what lies before it are out by themselves.  (Before
            // the first slide Z holds no positions: its values are the largest there are.)
            const U Pe = uniform_lane_u(QA, e);
            from = ~0ull << e;
            test = from << 1;
            const uint64_t wa = __builtin_amdgcn_ballot_w64(SA >= Pe) & ~from;
            const uint64_t wz = __builtin_amdgcn_ballot_w64(SZ >= Pe);
            const U va = select_lanes(kMax, FA, wa), vz = select_lanes(kMax, FZ, wz);
            if constexpr (sizeof(U) == 4) fh = wave_min_u32(va < vz ? va : vz); else fh = wave_min_u64(va < vz ? va : vz);
            const uint64_t ea = __builtin_amdgcn_ballot_w64(FA == fh) & wa;
            const uint64_t ez = __builtin_amdgcn_ballot_w64(FZ == fh) & wz;
            // (on sums that do not ascend both may be 0: any lane will do)
            const bool in_a = ea != 0;
            const int last = 63 - __builtin_clzll((unsigned long long)((in_a ? ea : ez) | 1ull));
            const U pa = uniform_lane_u(SA, last), pz = uniform_lane_u(SZ, last);
            if (RECORD) {
                h = (in_a ? base : base - kWave) + last;
                const int equal = (int)__popcll((unsigned long long)ea) + (int)__popcll((unsigned long long)ez);
                most = equal > most ? equal : most;
            }
            Sh = in_a ? pa : pz;
            if (__builtin_expect((wz & 1ull) != 0, 0)) {
                // The whole of Z lies in the window: the slices before it, the last two from registers, then the parked
                // values, if there are any (other lanes stored them: the fence keeps the compiler from moving the loads
                // up; it costs no instruction).
                // 64 positions, lane by lane downwards from `top` or upwards to it: true if all of them are in
                auto join = [&](const U si, const U fi, const int top, const bool downwards) -> bool {
                    const uint64_t in = __builtin_amdgcn_ballot_w64(si >= Pe);
                    const U v = select_lanes(kMax, fi, in);
                    U m;
                    if constexpr (sizeof(U) == 4) m = wave_min_u32(v); else m = wave_min_u64(v);
                    const uint64_t equal = __builtin_amdgcn_ballot_w64(fi == m) & in;
                    if (in != 0 && m < fh) {
                        fh = m;
                        // (some lane holds the minimum, if a value of the type is left for it)
                        const int at_lane = downwards ? __builtin_ctzll((unsigned long long)(equal | 1ull << 63))
                                                      : 63 - __builtin_clzll((unsigned long long)(equal | 1ull));
                        h = downwards ? top - at_lane : top - kWave + 1 + at_lane;
                        Sh = uniform_lane_u(si, at_lane);
                        if (RECORD) most = (equal & (equal - 1)) != 0 ? 2 : most;
                    } else if (RECORD && in != 0 && m == fh) {
                        most = 2;
                    }
                    return in == ~0ull;
                };
                int top = base - kWave - 1;        // (63 or more, or -1)
                bool on = top >= 0;
#pragma unroll
                for (int k = 0; k < kOlder; ++k, top -= kWave)
                    if (on) on = join(SY[k], FY[k], top, false) && top >= kWave;
                if (on) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    for (; top >= 0; top -= kWave)
                        if (!join(P[top - lane] + s, F[top - lane], top, true)) break;
                }
            }
        }
        if (out != 0) {
            // cell n sees h
            if (RECORD) {
                F[base + lane] = FA;               // (base <= n + 1; what lies past n is not looked at)
                if (base + lane <= n) head[base + lane] = (H)HA;
                if (ties) *ties = most > 1;
            }
            // (no cell in A yet and cell n the last of the slice before: its value is in Z)
            return n >= base ? uniform_lane_u(FA, n - base) : uniform_lane_u(FZ, kWave - 1);
        }
        // h outlasts A: slide
        if (stop(fh)) return fh;
        F[base + lane] = FA;
        if (RECORD) head[base + lane] = (H)HA;
        base += kWave;
        if (__builtin_expect(base > n + 1, 0)) return kMax;
        from = test = ~0ull;
#pragma unroll
        for (int k = kOlder - 1; k > 0; --k) {
            SY[k] = SY[k - 1]; FY[k] = FY[k - 1];
        }
        SY[0] = SZ; FY[0] = FZ;
        SZ = SA; FZ = FA;
        PA = PB; QA = QB;
        SA = PA + s; DA = PA - QA;
        PB = at(base + kWave + lane);
        QB = before(base + kWave + lane);
    }
}

// The first minimal predecessor of j, given one of them, from the sums and F as wave_cost leaves it: the canonical set
// takes that one.  The positions before h that hold F(h) and lie in the window of j, 64 at a time.
template <typename U>
__device__ __forceinline__ int first_pred(const U *P, const U *F, const U s, const int j, const int h)
{
    const int lane = threadIdx.x % kWave;
    const U v = F[h], Pj = P[j - 1];
    int first = h;
    for (int top = h - 1; top >= 0; top -= kWave) {
        const int i = top - lane, at = i > 0 ? i : 0;
        const U si = P[at] + s, fi = F[at];
        const uint64_t in = __builtin_amdgcn_ballot_w64(i >= 0 && si >= Pj);
        const uint64_t equal = __builtin_amdgcn_ballot_w64(fi == v) & in;
        if (equal != 0) first = top - (63 - __clzll((unsigned long long)equal));
        if (in != ~0ull) break;
    }
    return first;
}

template <typename U>
__device__ __forceinline__ void solve_short(const uint64_t (&sum)[kSearchPer], const int n, const int shift,
                                            const uint64_t total, const uint64_t bound, const uint64_t span,
                                            const float all, const uint64_t heavy, int64_t &cost,
                                            int64_t &budget, uint32_t &bits)
{
    const SearchLds<U> m(search_lds, n);
    const int lane = threadIdx.x;
    // where the budgets of every start pass the span, from the prefix sums in full (in the room of L1)
    uint64_t *const full = (uint64_t *)m.L1;
    int steps = 1, ends[kSearchPer];
    while ((1 << steps) <= n) ++steps;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        const int k = q * kWave + lane;
        if (k <= n) {
            full[k] = sum[q] >> shift;
            m.P[k] = (U)(sum[q] >> shift);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        const int r = q * kWave + lane;
        ends[q] = n;
        if (q * kWave < n) ends[q] = first_above(full, r + 1 < n ? r + 1 : n, n, sum[q] >> shift, span, steps);
    }
    const U last = m.P[n];
    for (int k = n + 1 + lane; k < sums_len(n); k += kWave) m.P[k] = last;
    __syncthreads();
    U bc, bs;
    search_chain<U>(m, n, total, (U)bound, (U)span, ends, steps, all, (U)heavy, bc, bs);
    // The canonical set for the budget bs: the heads of one pass over the prefix sums in full (in the room of L1
    // again; in 32 bits where they are), then the walk back from n.
    __syncthreads();
    bits = 0;
    static_assert(kSearchMaxLayers <= 256, "a head's position is a byte");
    const auto walk = [&](const auto *P, auto *F) {
        typedef std::remove_pointer_t<decltype(F)> V;
        uint8_t *const head = (uint8_t *)(F + n + 1 + kWave);
        bool ties = false;
        (void)wave_cost<V, true>(P, n, (V)bs, F, head, NeverStop(), &ties);
        __syncthreads();
        for (int j = n;;) {  // (downwards: on sums that ascend a head lies below its cell)
            if ((j & (kWave - 1)) == lane) bits |= 1u << (j / kWave);
            if (j == 0) break;
            const int h = __builtin_amdgcn_readfirstlane(head[j]);
            j = ties ? first_pred(P, F, (V)bs, j, h) : h;
        }
    };
    if (sizeof(U) == 4 && total < (1ull << 31)) {
        walk((const uint32_t *)m.P, (uint32_t *)m.L1);
    } else {
#pragma unroll
        for (int q = 0; q < kSearchPer; ++q) {
            const int k = q * kWave + lane;
            if (k <= n) full[k] = sum[q] >> shift;
        }
        __syncthreads();
        walk(full, full + n + 1);
    }
    cost = (int64_t)((uint64_t)bc << shift);
    budget = (int64_t)((uint64_t)bs << shift);
}

// Inclusive sum over the wave (row shifts inside the rows of 16 lanes, then the rows' last lanes).
template <int CTRL, int ROW_MASK>
__device__ inline uint64_t dpp_sum_step_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROW_MASK, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROW_MASK, 0xf, false);
    return v + (((uint64_t)hi << 32) | lo);
}
__device__ inline uint64_t wave_scan_u64(uint64_t v)
{
    v = dpp_sum_step_u64<kDppRowShr1, 0xf>(v);
    v = dpp_sum_step_u64<kDppRowShr2, 0xf>(v);
    v = dpp_sum_step_u64<kDppRowShr4, 0xf>(v);
    v = dpp_sum_step_u64<kDppRowShr8, 0xf>(v);
    v = dpp_sum_step_u64<kDppRowBcast15, 0xa>(v);
    v = dpp_sum_step_u64<kDppRowBcast31, 0xc>(v);
    return v;
}
__device__ inline uint64_t lane63_u64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

// The cost of a feasible set, by the lane of the best of 64 greedy walks: a lane has a segment limit of
// its own, on a geometric grid over the last eight octaves below the sum of the interior layers, and
// makes a checkpoint of every layer that would take its segment beyond the limit.  In floats, whose
// errors (n + 1 roundings of 2^-24) the result is raised by.
__device__ inline uint64_t greedy_bound(const float *size, const int n, const float all)
{
    const int lane = threadIdx.x;
    const float limit = all * exp2f((float)(lane - (kWave - 1)) * (8.0f / (kWave - 1)));
    float kept = size[0] + size[n], seg = 0.0f, longest = 0.0f;
    auto layer = [&](const float x) {
        const float to = seg + x;
        const bool fits = to <= limit;
        kept += fits ? 0.0f : x;
        seg = fits ? to : 0.0f;
        longest = fmaxf(longest, seg);
    };
    int k = 1;
    for (; k + 3 < n; k += 4) {
        const float x0 = size[k], x1 = size[k + 1], x2 = size[k + 2], x3 = size[k + 3];
        layer(x0); layer(x1); layer(x2); layer(x3);
    }
    for (; k < n; ++k) layer(size[k]);
    const float cost = (kept + longest) * (1.0f + 1.0f / 4096.0f);
    // (positive floats order as their bits)
    return (uint64_t)(double)__uint_as_float(wave_min_u32(__float_as_uint(cost))) + 1;
}

// One chain of n <= kSearchMaxLayers layers: size k at dp[k * pstride], mask byte k to mp[k * mstride].
// NARROW, WIDE: which arithmetic the launch has LDS for.  A chain that needs the 64-bit one in a launch
// without it makes the function return false, with nothing written.
template <bool NARROW, bool WIDE>
__device__ __forceinline__ bool search_one(const int64_t *__restrict__ dp, const int64_t pstride, const int n,
                                           uint8_t *__restrict__ mp, const int64_t mstride,
                                           int64_t *__restrict__ peak_out, int64_t *__restrict__ budget_out,
                                           int32_t *__restrict__ status_out, const unsigned lds)
{
    const int lane = threadIdx.x;
    uint64_t sum[kSearchPer];  // the sizes, then P[q * 64 + lane]
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        const int k = q * kWave + lane;
        sum[q] = k <= n ? (uint64_t)dp[(int64_t)k * pstride] : 0;
    }
    uint64_t base = 0, bits = 0, high = 0;
    uint64_t mx = 0;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        if (q * kWave > n) break;
        bad |= q * kWave + lane <= n && (int64_t)sum[q] <= 0;
        bits |= sum[q];
        mx = sum[q] > mx ? sum[q] : mx;
        high += sum[q] >> 32;
    }
    high = lane63_u64(wave_scan_u64(high));
    mx = ~wave_min_u64(~mx);
#pragma unroll
    for (int k = kWave / 2; k >= 1; k >>= 1) bits |= (uint64_t)__shfl_xor((long long)bits, k, kWave);
    const int shift = bits ? __ffsll((unsigned long long)bits) - 1 : 0;
    float *const size = (float *)search_lds;  // the scaled sizes, for the greedy walks
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        if (q * kWave > n) break;
        if (q * kWave + lane <= n) size[q * kWave + lane] = (float)(sum[q] >> shift);
        sum[q] = wave_scan_u64(sum[q]) + base;
        base = lane63_u64(sum[q]);
    }
    __syncthreads();
    const int32_t status = __any(bad) ? CKPT_ERR_SIZE : chain_overflows(base, high, mx) ? CKPT_ERR_OVERFLOW : CKPT_OK;
    int64_t cost = -1, budget = -1;
    uint32_t on = 0;
    if (status == CKPT_OK) {
        const uint64_t d0 = (uint64_t)lane63_u64(wave_scan_u64(lane == 0 ? sum[0] : 0)) >> shift;
        const uint64_t total = base >> shift;
        uint64_t before_last = 0;  // P[n - 1]
#pragma unroll
        for (int q = 0; q < kSearchPer; ++q)
            if (q * kWave + lane == n - 1) before_last = sum[q];
        before_last = lane63_u64(wave_scan_u64(before_last)) >> shift;
        const uint64_t all = before_last - d0;  // every interior layer: the largest budget
        const uint64_t ends = total - all;
        uint64_t bound = greedy_bound(size, n, (float)all);
        bound = bound < total ? bound : total;
        bound = bound > ends ? bound : ends;
        const uint64_t span = all < bound - ends ? all : bound - ends;
        const uint64_t largest = mx >> shift;
        // (it may be one at the ends: any cut will do)
        const uint64_t heavy = largest > all / 4 && largest <= span ? largest : 0;
        const bool narrow = bound < (1ull << 31) - 1 && span + largest < (1ull << 31) &&
                            (kLookahead - 1) * largest < (1ull << 31);
        if (narrow ? !NARROW : !WIDE || search_lds_bytes(n, 8) > lds) return false;
        if (NARROW && narrow)
            solve_short<uint32_t>(sum, n, shift, total, bound, span, (float)all, heavy, cost, budget, on);
        else if (WIDE)
            solve_short<uint64_t>(sum, n, shift, total, bound, span, (float)all, heavy, cost, budget, on);
    }
    for (int k = lane, q = 0; k <= n; k += kWave, ++q) mp[(int64_t)k * mstride] = (on >> q) & 1u;
    if (lane == 0) {
        *peak_out = cost;
        if (budget_out) *budget_out = budget;
        if (status_out) *status_out = status;
    }
    return true;
}

// Chains whose launch has no LDS for 64-bit arithmetic and that need it.
struct SearchWs {
    int32_t *count;  // [1] (first 256 bytes)
    int32_t *list;   // [batch]
};

__global__ void cubic_search_reset_kernel(SearchWs w) { w.count[threadIdx.x] = 0; }

// ---------------------------------------------------------------------------
// many short chains: a row of lanes per chain
// ---------------------------------------------------------------------------

// A search needs few evaluations if each round knows the last one's: a chain of 64 unrounded layers is settled by 29 with
// eight points a round (4.5 rounds), by 85 with 64 (2.4 rounds).  Where there are chains enough to fill the chip, a wave
// therefore takes kWave / G of them, G lanes each, and the rounds of all run side by side.
//   What an evaluation tells.  A pass for s finds the window start of every cell, and with it the largest budget up to s
// (c is the same there) and the smallest one above it: the sums that just fit a window and those that just do not.  So a
// point costs what its budget costs, an interval without a budget in it is closed without a look, and every round closes
// at least one budget of every open interval at its upper end.
//   The state of a chain is one open interval for each of its lanes: the one below the lane's point.  G points in m open
// intervals, at least one in each, one of them at its upper end, leave at most G: nothing is ever put aside.
//   The pass.  As in lane_cost the window minimum is that of suffix minima, but positions are taken in blocks of four,
// whose values stay in registers: what of the block under way lies in the window is joined by comparing the sums, and L1
// and L2 are written once a block has been filled, so that nothing has to be cleared or lowered cell by cell.  L2 is lowered
// from the first block that any lane still reads.  The window starts of a block do not depend on values.  They come from a
// table over the range of the prefix sums, slots of one width: the first position at or above the slot's lower end, then
// three sums tested at once.  (Moving a start on from that of the cell before takes as many turns as the lane that moves
// farthest: 2.8 instead of 1.3 at eight unrounded chains a wave.)  Table, sums and minima are read a block ahead each.
// What bounds it: issue, about 145 vector and 24 LDS instructions a block of four cells, and the two waves on a SIMD that
// the LDS space leaves (20 KB a wave at 64 layers); the rounds of a wave are those of its slowest chain (5.3 and 6.4 of 4.5
// and 5.0).  65,536 chains of 64 layers, unrounded 0.66 ms (a wave a chain: 1.28), aligned 0.54 (1.10).
constexpr int kRowBlk = 4;
constexpr int kRowSlots = 4;   // slots of the table per layer
constexpr int kRowsMaxLayers = 256;  // (a position is a byte of the table)
static_assert(kRowsMaxLayers == kSearchMaxLayers, "every chain of the search has rows that fit it");
constexpr int kRowsOf8Layers = 72, kRowsOf16Layers = 128;

__host__ __device__ inline int row_blocks(int n) { return (n + kRowBlk - 1) / kRowBlk; }
// Prefix sums from position -1 on, with the padding that what is read ahead sees.
__host__ __device__ inline int row_sums(int n) { return (row_blocks(n) + 4) * kRowBlk + 2; }
// The slots of a chain, four more so that those of the chains of a wave lie in banks of their own.
__host__ __device__ inline int row_slots(int n) { return n * kRowSlots + 4 * kRowSlots; }
// Positions whose minima a lane keeps: those of all windows, and of longer chains those of nearly all of most kinds (the windows
// up to the best cost reach over 37 layers in one of a hundred chains of 64 unrounded layers, over 50 of 128; over 60 in one of
// ten networks of 128; where the layers in front outweigh the rest, over nearly all: see RowsLeft::kFar).  What it saves is
// waves in flight: 65,536 aligned chains of 64 layers 756 us with a ring of 64, 541 with 40; 128 layers with 72, 60, 48: aligned
// 2.0, 1.7, 1.5 ms (5.1 with a wave a chain), networks, of which 60 leave one in ten and fewer leave more, 2.2 with 60 (4.1).
__host__ __device__ inline int row_ring(int n)
{
    const int most = row_blocks(n) * kRowBlk, a = 32 + n / 8, b = 12 + 3 * n / 8;
    const int some = ((a > b ? a : b) + kRowBlk - 1) / kRowBlk * kRowBlk;
    return most < some ? most : some;
}
__host__ __device__ inline size_t rows_lds_bytes(int n, int chains, int ring)
{
    const size_t per_lane = ring + ring / kRowBlk, per_chain = (size_t)row_sums(n) + row_blocks(n) * kRowBlk;
    return ((per_lane + 1) * kWave + per_chain * chains) * 4 + (size_t)row_slots(n) * chains;
}

template <int G>
struct RowsLds {
    static constexpr int kChains = kWave / G;
    int ring;
    uint32_t *L2;  // [ring / kRowBlk][kWave] minimum of the full blocks behind one
    uint32_t *L1;  // [ring][kWave] minimum from a position to the end of its block
    uint32_t *P;   // [row_sums(n)][kChains] d_1 + .. + d_k + span + 1 from k = -1 on (0 there), padded with the last
    uint32_t *F;   // [blocks * kRowBlk][kChains] the values of the last pass
    int *slot;     // [kWave]
    uint8_t *T;    // [kChains][row_slots(n)] the first position at or above a slot's lower end
    __device__ RowsLds(unsigned char *base, int n, int ring) : ring(ring)
    {
        L2 = (uint32_t *)base;
        L1 = L2 + ring / kRowBlk * kWave;
        P = L1 + ring * kWave;
        F = P + (size_t)row_sums(n) * kChains;
        slot = (int *)(F + (size_t)row_blocks(n) * kRowBlk * kChains);
        T = (uint8_t *)(slot + kWave);
    }
};

// ---- across the G lanes of a row ----

constexpr int kDppSwap1 = 0xb1, kDppSwap2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL>
__device__ inline uint32_t dpp_of(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false); }
template <int CTRL>
__device__ inline uint64_t dpp_of(uint64_t v)
{
    return ((uint64_t)dpp_of<CTRL>((uint32_t)(v >> 32)) << 32) | dpp_of<CTRL>((uint32_t)v);
}
template <int CTRL>
__device__ inline float dpp_of(float v) { return __uint_as_float(dpp_of<CTRL>(__float_as_uint(v))); }

// v joined over the row, for all of its lanes (the mirrors stand for swaps by 4 and 8: what they exchange is the same in
// all lanes of a quad, of half a row)
template <int G, typename V, typename Join>
__device__ inline V row_all(V v, Join join)
{
    static_assert(G == 8 || G == 16 || G == 64, "rows that the operations across lanes have");
    v = join(v, dpp_of<kDppSwap1>(v));
    v = join(v, dpp_of<kDppSwap2>(v));
    v = join(v, dpp_of<kDppHalfMirror>(v));
    if constexpr (G > 8) v = join(v, dpp_of<kDppMirror>(v));
    if constexpr (G > 16) {
        v = join(v, __shfl_xor(v, 16, kWave));
        v = join(v, __shfl_xor(v, 32, kWave));
    }
    return v;
}
template <int G, typename V>
__device__ inline V row_min(V v) { return row_all<G>(v, [](V a, V b) { return a < b ? a : b; }); }
template <int G, typename V>
__device__ inline V row_sum(V v) { return row_all<G>(v, [](V a, V b) { return a + b; }); }

// v joined with those of the lanes before, where 0 changes nothing
template <int CTRL, int ROW_MASK>
__device__ inline uint32_t dpp_or_0(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false); }
template <int CTRL, int ROW_MASK>
__device__ inline uint64_t dpp_or_0(uint64_t v)
{
    return ((uint64_t)dpp_or_0<CTRL, ROW_MASK>((uint32_t)(v >> 32)) << 32) | dpp_or_0<CTRL, ROW_MASK>((uint32_t)v);
}
template <int G, typename V, typename Join>
__device__ inline V row_scan(V v, Join join)
{
    const int i = threadIdx.x % G;
    const auto step = [&](V from, int k) { v = join(v, G >= 16 || i >= k ? from : (V)0); };
    step(dpp_or_0<kDppRowShr1, 0xf>(v), 1);
    step(dpp_or_0<kDppRowShr2, 0xf>(v), 2);
    step(dpp_or_0<kDppRowShr4, 0xf>(v), 4);
    if constexpr (G > 8) step(dpp_or_0<kDppRowShr8, 0xf>(v), 8);
    if constexpr (G > 16) {
        step(dpp_or_0<kDppRowBcast15, 0xa>(v), 16);
        step(dpp_or_0<kDppRowBcast31, 0xc>(v), 32);
    }
    return v;
}

// F_s(n) without the size at the end.  FLAT: the prefix sums are those in full; else they are modulo 2^32, and values are cut
// to 2^31.  `record`: the values go to m.F.  `over`: no difference of sums that is not negative is larger, and every negative
// one is as a number without a sign.  `slack`: how far the largest budget up to s lies below it; `gap`: minus how far the next
// one lies above (not above `over` if there is none).  `cut`: a window reached back beyond the ring and was cut off there, so
// that the result is what F_s(n) does not exceed.
template <bool FLAT, int G>
__device__ __forceinline__ uint32_t rows_pass(const RowsLds<G> &m, const bool record, const int n, const uint32_t first,
                                              const uint32_t s, const uint32_t over, const int shift, uint32_t &slack, uint32_t &gap,
                                              bool &cut)
{
    typedef uint32_t U;
    constexpr int C = kWave / G;
    constexpr U kMax = ~0u, kCap = 1u << 31;
    const int lane = threadIdx.x, row = lane / G, nb = row_blocks(n);
    const int ring = m.ring, ring_blocks = ring / kRowBlk;
    const U *const P = m.P + row;   // P[(k + 1) * C]: the sum at position k
    const uint8_t *const T = m.T + row * row_slots(n);
    U least = kMax, most = 0, far = 0;
    U p[kRowBlk][4];
    // three sums from a window's start on against where the window may begin
    const auto test = [&](int &l, const U e, const U p0, const U p1, const U p2) {
        U t0, t1, t2;
        if constexpr (FLAT) {  // (the difference and the comparison are one instruction)
            l += __builtin_sub_overflow(p0, e, &t0) ? 1 : 0;
            l += __builtin_sub_overflow(p1, e, &t1) ? 1 : 0;
            l += __builtin_sub_overflow(p2, e, &t2) ? 1 : 0;
        } else {
            t0 = p0 - e; t1 = p1 - e; t2 = p2 - e;
            l += (int)(t0 > over) + (int)(t1 > over) + (int)(t2 > over);
        }
        far = t2 > far ? t2 : far;
        U a = t0 < t1 ? t0 : t1, z = t0 > t1 ? t0 : t1;
        a = a < t2 ? a : t2;
        z = z > t2 ? z : t2;
        least = a < least ? a : least;
        most = z > most ? z : most;
    };
    const auto sums = [&](const int (&l)[kRowBlk]) {
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) {
            const U *const at = P + l[u] * C;
            p[u][0] = at[0]; p[u][1] = at[C]; p[u][2] = at[2 * C]; p[u][3] = at[3 * C];
        }
    };
    const auto move_on = [&](const U (&e)[kRowBlk], int (&l)[kRowBlk]) {
        far = 0;
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) {
            const U tm = p[u][0] - e[u];
            most = tm > most ? tm : most;
            test(l[u], e[u], p[u][1], p[u][2], p[u][3]);
        }
        while (__builtin_expect(__builtin_amdgcn_ballot_w64(far > over) != 0, 0)) {
            far = 0;
            sums(l);
#pragma unroll
            for (int u = 0; u < kRowBlk; ++u) test(l[u], e[u], p[u][1], p[u][2], p[u][3]);
        }
    };
    // the window of the cell behind the sum x, which begins at e = x - s, holds the position with this sum (no more than four
    // sizes below x, or out)
    const auto holds = [&](U sum, U e, U x) { return FLAT ? sum >= e : x - sum <= s; };
    // the sums that block b's positions end in, and where the windows of the cells behind them may begin
    const auto load = [&](U (&x)[kRowBlk], int b) {
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) x[u] = P[(b * kRowBlk + u + 1) * C];
    };
    // (modulo 2^32 the sums wrap now and then as they ascend; the table is that of the sums in full)
    U wraps = 0, latest = 0;
    const auto table = [&](const U (&x)[kRowBlk], U (&e)[kRowBlk], int (&l)[kRowBlk]) {
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) {
            e[u] = x[u] - s;
            if constexpr (FLAT) {
                l[u] = T[(uint32_t)(e[u] >> shift)];
            } else {
                wraps += x[u] < latest ? 1 : 0;
                latest = x[u];
                l[u] = T[(uint32_t)((((uint64_t)wraps << 32 | x[u]) - s) >> shift)];
            }
        }
    };
    // In turn b: the sums x that block b's positions end in and those of the two blocks behind it, where the windows of the
    // cells behind each may begin (e), their starts l, for the next block what the table says of them.  Block b has slot b %
    // kTurns of each: the turns are written out, so that nothing is moved from one to the next.
    constexpr int kTurns = 4;
    int l[kTurns][kRowBlk] = {};
    U x[kTurns][kRowBlk], e[kTurns][kRowBlk];
    load(x[0], 0);
    load(x[1], 1);
    load(x[2], 2);
    table(x[0], e[0], l[0]);
    table(x[1], e[1], l[1]);
    sums(l[0]);
    move_on(e[0], l[0]);
    U f[kRowBlk + 1], edge = e[0][0] - 1;  // edge: the sum at the last position before the block (before the first: out)
    f[kRowBlk] = first;
    int low = 0;                           // the first block that holds a window's start
    int turn = 0;                          // the last multiple of `ring`
    cut = false;
    U *const L1 = m.L1 + lane, *const L2 = m.L2 + lane;
    const auto block = [&](const int b, auto r) {
        constexpr int r0 = decltype(r)::value, r1 = (r0 + 1) % kTurns, r2 = (r0 + 2) % kTurns, r3 = (r0 + 3) % kTurns;
        f[0] = f[kRowBlk];
        const int back = (b - ring_blocks) * kRowBlk;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(l[r0][0] < back) != 0, 0)) {
            cut |= l[r0][0] < back;
#pragma unroll
            for (int u = 0; u < kRowBlk; ++u) l[r0][u] = l[r0][u] > back ? l[r0][u] : back;
        }
        U la[kRowBlk], lc[kRowBlk];
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) {
            // (a position before the turn's beginning: below 0, so the larger one as a number without a sign)
            const unsigned near = (unsigned)(l[r0][u] - turn), far_end = near + (unsigned)ring, at = near < far_end ? near : far_end;
            la[u] = L1[at * kWave];
            lc[u] = L2[at / kRowBlk * kWave];
        }
        sums(l[r1]);
        table(x[r2], e[r2], l[r2]);
        load(x[r3], b + 3);  // (past the last block: the padding)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kRowBlk; ++u) {
            const U from = e[r0][u];
            U w = la[u] < lc[u] ? la[u] : lc[u];
            w = f[u] < w ? f[u] : w;
            w = holds(edge, from, x[r0][u]) ? w : f[u];
#pragma unroll
            for (int k = 0; k < u; ++k) {
                const U v = holds(x[r0][k], from, x[r0][u]) ? f[k] : kMax;
                w = v < w ? v : w;
            }
            f[u + 1] = ((u + 1 < kRowBlk ? x[r0][(u + 1) % kRowBlk] : x[r1][0]) - x[r0][u]) + w;
            if (!FLAT) f[u + 1] = f[u + 1] < kCap ? f[u + 1] : kCap;
        }
        if (record) {
#pragma unroll
            for (int u = 0; u < kRowBlk; ++u) m.F[(b * kRowBlk + u) * C + row] = f[u];
        }
        U whole = f[kRowBlk - 1];
        const int spot = b - turn / kRowBlk;
        U *const here = L1 + spot * kRowBlk * kWave;
        here[(kRowBlk - 1) * kWave] = whole;
#pragma unroll
        for (int u = kRowBlk - 2; u >= 0; --u) {
            whole = f[u] < whole ? f[u] : whole;
            here[u * kWave] = whole;
        }
        move_on(e[r1], l[r1]);
        // (cell after cell a start only moves on)
        if (__builtin_amdgcn_ballot_w64(l[r1][0] < (low + 1) * kRowBlk) == 0) ++low;
        low = low > b + 1 - ring_blocks ? low : b + 1 - ring_blocks;
        for (int q = b - 1, at = spot; q >= low; --q) {
            at = at > 0 ? at - 1 : ring_blocks - 1;
            lds_min(L2 + at * kWave, whole);
        }
        L2[spot * kWave] = kMax;
        turn += spot + 1 == ring_blocks ? ring : 0;
        edge = x[r0][kRowBlk - 1];
    };
    for (int b = 0;; b += kTurns) {
        block(b, std::integral_constant<int, 0>());
        if (b + 1 >= nb) break;
        block(b + 1, std::integral_constant<int, 1>());
        if (b + 2 >= nb) break;
        block(b + 2, std::integral_constant<int, 2>());
        if (b + 3 >= nb) break;
        block(b + 3, std::integral_constant<int, 3>());
        if (b + 4 >= nb) break;
    }
    slack = least;
    gap = most;
    const int last = (n - 1) % kRowBlk;
    return last == 0 ? f[1] : last == 1 ? f[2] : last == 2 ? f[3] : f[4];
}

// The cost of a feasible set without the sizes at the ends, by the lane of the best of G greedy walks (see greedy_bound), half
// an octave to an octave between their limits.
template <int G>
__device__ inline uint64_t rows_bound(const float *size, const int n, const float all)
{
    constexpr int C = kWave / G;
    const int i = threadIdx.x % G;
    const float limit = all * exp2f(-0.5f - (float)i * (5.6f / G));
    const float *const d = size + threadIdx.x / G;
    float kept = 0.0f, seg = 0.0f, longest = 0.0f;
    const auto layer = [&](const float x) {
        const float to = seg + x;
        const bool fits = to <= limit;
        kept += fits ? 0.0f : x;
        seg = fits ? to : 0.0f;
        longest = fmaxf(longest, seg);
    };
    constexpr int kAtOnce = 8;
    int k = 1;
    for (; k + kAtOnce <= n; k += kAtOnce) {
        float x[kAtOnce];
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j) x[j] = d[(k + j) * C];
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j) layer(x[j]);
    }
    for (; k < n; ++k) layer(d[k * C]);
    const float cost = (kept + longest) * (1.0f + 1.0f / 4096.0f);
    return (uint64_t)(double)__uint_as_float(row_min<G>(__float_as_uint(cost))) + 1;
}

// A chain is expected to be far, one whose windows reach beyond the ring, if a window that does holds no more than this share
// of the span: the best cost lies at 0.3 to 0.4 of it for unrounded sizes, 0.7 to 0.8 for networks, 0.95 for sizes that fall from
// layer to layer.  (Taken so, of 64 layers, 0 to 2 % of aligned and unrounded chains and networks, 74 % of networks whose
// pictures are all halved in the first third; 0, 0 and 74 % are.)
constexpr float kFarShare = 0.75f;

// What a row knows of its chain before the search.
template <int G, int MOST>
struct RowChain {
    static constexpr int PER = MOST / G + 1;
    int per, k0;                // the lane's sizes: how many, and the first one's position
    uint64_t own[PER], before;  // ... and the sum of those before
    int32_t status;
    int shift;
    uint64_t d0, dn, total, all, largest;  // scaled: the sizes at the ends, all sizes, the interior ones, the largest
    uint64_t span;                         // no budget beyond it can be optimal
    // (n <= MOST; size: LDS for a float a layer and chain)
    __device__ __forceinline__ RowChain(const int64_t *__restrict__ dp, const int n, const int64_t pstride, float *const size)
    {
        constexpr int C = kWave / G;
        const int row = threadIdx.x / G, i = threadIdx.x % G;
        per = (n + G) / G;
        k0 = i * per;
        uint64_t sum = 0, bits = 0, high = 0, mx = 0;
        bool bad = false;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            own[q] = 0;
            if (q < per) own[q] = k0 + q <= n ? (uint64_t)dp[(int64_t)(k0 + q) * pstride] : 0;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const uint64_t x = own[q];
            bad |= q < per && k0 + q <= n && (int64_t)x <= 0;
            bits |= x;
            high += x >> 32;
            sum += x;
            mx = x > mx ? x : mx;
        }
        const uint64_t d_first = (uint64_t)dp[0], d_last = (uint64_t)dp[(int64_t)n * pstride];
        before = row_scan<G>(sum, [](uint64_t a, uint64_t b) { return a + b; }) - sum;
        sum = row_sum<G>(sum);
        high = row_sum<G>(high);
        bits = row_all<G>(bits, [](uint64_t a, uint64_t b) { return a | b; });
        mx = ~row_min<G>(~mx);
        bad = row_min<G>((uint32_t)!bad) == 0;
        status = bad ? CKPT_ERR_SIZE : chain_overflows(sum, high, mx) ? CKPT_ERR_OVERFLOW : CKPT_OK;
        shift = bits ? __ffsll((unsigned long long)bits) - 1 : 0;
        total = sum >> shift;
        d0 = d_first >> shift;
        dn = d_last >> shift;
        all = status == CKPT_OK ? total - d0 - dn : 0;
        largest = mx >> shift;
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (q < per && k0 + q <= n) size[(k0 + q) * C + row] = (float)(own[q] >> shift);
        __syncthreads();
        span = rows_bound<G>(size, n, (float)all);
        span = span < all ? span : all;
    }
    // Is it expected to be far?  (sums: as size)
    __device__ __forceinline__ bool far(const int n, const int ring, float *const sums) const
    {
        constexpr int C = kWave / G;
        const int row = threadIdx.x / G, i = threadIdx.x % G;
        uint64_t run = before;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            run += own[q];
            if (q < per && k0 + q <= n) sums[(k0 + q) * C + row] = (float)(run >> shift);
        }
        __syncthreads();
        // the least sum that a window beyond the ring has, one that ends in a block's first position
        float least = std::numeric_limits<float>::max();
        for (int b = ring / kRowBlk + 1 + i; b < row_blocks(n); b += G)
            least = fminf(least, sums[b * kRowBlk * C + row] - sums[(b * kRowBlk - ring - 1) * C + row]);
        least = row_all<G>(least, [](float a, float b) { return fminf(a, b); });
        return status == CKPT_OK && least <= kFarShare * (float)span;
    }
};

// Why a row leaves its chain, with nothing written: the ring does not hold its windows, or 32 bits its values.
enum class RowsLeft { kNone, kFar, kWide };

// Chain c of each row where `valid`, n <= MOST.
template <int G, int MOST>
__device__ __forceinline__ RowsLeft search_rows(const int64_t *__restrict__ d, const int64_t c, const bool valid, const int n,
                                                const int64_t cstride, const int64_t pstride, uint8_t *__restrict__ mask_out,
                                                int64_t *__restrict__ peak_out, int64_t *__restrict__ budget_out,
                                                int32_t *__restrict__ status_out, const int ring)
{
    typedef uint32_t U;
    typedef int32_t I;
    constexpr int C = kWave / G, PER = RowChain<G, MOST>::PER;
    const RowsLds<G> m(search_lds, n, ring);
    const int lane = threadIdx.x, row = lane / G, i = lane % G;
    const RowChain<G, MOST> chain(d + c * cstride, n, pstride, (float *)m.L1);
    const int per = chain.per, k0 = chain.k0, shift = chain.shift;
    const auto &own = chain.own;
    const int32_t status = chain.status;
    const uint64_t before = chain.before, d0 = chain.d0, dn = chain.dn, total = chain.total, all = chain.all, largest = chain.largest;
    uint64_t span = chain.span;
    const uint64_t bound = d0 + dn + span;
    // What is looked at of differences from where a window may begin, modulo 2^32: up to a window, or the size at its start, and
    // two sizes more; down to a slot, which is no wider than the largest size, and a size below 0.  (Every chain that the form
    // of a wave takes in 32 bits fits.  65,536 chains of 16 layers, one of some 650 MB, others of up to 8, all odd, 95 us; with
    // four sizes below 0 they were left for 64 bits: 626.)
    const uint64_t reach = (span > largest ? span : largest) + 2 * largest;
    const bool narrow = bound < (1ull << 31) - 1 && reach + 2 * largest < (1ull << 32);
    bool solved = valid && status == CKPT_OK && narrow, beyond = false;  // beyond: windows reach back beyond the ring
    const bool flat = !solved || total + span + 1 < (1ull << 32);
    if (!solved) span = 0;
    if (__builtin_amdgcn_ballot_w64(solved) == 0 && __builtin_amdgcn_ballot_w64(valid && status != CKPT_OK) == 0)
        return valid ? RowsLeft::kWide : RowsLeft::kNone;
    // The prefix sums, of a chain that is left out 1 everywhere, and the table: position k is the first one of the slots
    // behind that of the one before, up to its own; bytes up to a word's beginning, words, bytes.
    __syncthreads();
    const uint64_t end = solved ? all + span + 1 : 1;
    int slot_shift = 0;
    while ((end >> slot_shift) >= (uint64_t)(n * kRowSlots)) ++slot_shift;
    {
        uint8_t *const T = m.T + row * row_slots(n);
        uint64_t run = before;
        int at = i == 0 ? 0 : solved && k0 < n ? (int)(((run >> shift) - d0 + span + 1) >> slot_shift) + 1 : 2;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = k0 + q;
            run += own[q];
            const uint64_t here = solved ? (run >> shift) - d0 + span + 1 : 1;
            int to = -1;
            if (q < per && k < n) {
                m.P[(k + 1) * C + row] = (U)here;
                to = (int)(here >> slot_shift);
            }
            const int words = (at + 3) & ~3, rest = (to + 1) & ~3;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (at + j <= to && at + j < words) T[at + j] = (uint8_t)k;
                if (rest + j <= to && rest + j >= at) T[rest + j] = (uint8_t)k;
            }
            for (int word = words; word + 3 <= to; word += 4) *(uint32_t *)(T + word) = (uint32_t)k * 0x01010101u;
            at = to + 1;
        }
    }
    for (int k = n + i; k < row_sums(n) - 1; k += G) m.P[(k + 1) * C + row] = (U)end;
    if (i == 0) m.P[row] = 0;
    const bool all_flat = __builtin_amdgcn_ballot_w64(!flat) == 0;
    __syncthreads();
    const U first = solved ? (U)d0 : 0, tail = solved ? (U)dn : 0, over = solved ? (U)reach : 0;
    // s = 0 makes every layer a checkpoint
    U ub = (U)bound, best_cost = total <= bound ? (U)total : std::numeric_limits<U>::max(), best_s = 0;
    // a point, what its interval begins above, and whether that is what the neighbour's point leaves
    const auto split = [](U lo, U wide, int k, int of) {
        const U part = (U)((float)wide * (float)k / (float)of);
        return k >= of || part > wide ? lo + wide : lo + part;
    };
    U s = split(0, (U)span, i + 1, G), lo = 0;
    bool leftmost = i == 0;
    bool settled = false, cut;
    U value;
    for (int round = 0;; ++round) {
        U slack, gap;
        if (all_flat) value = rows_pass<true>(m, settled, n, first, s, over, slot_shift, slack, gap, cut);
        else value = rows_pass<false>(m, settled, n, first, s, over, slot_shift, slack, gap, cut);
        if (settled) break;
        const U at = s - slack, least = value + tail, cost = at + least;
        const U low_cost = row_min<G>(cost), low_at = row_min<G>(cost == low_cost ? at : std::numeric_limits<U>::max());
        if (low_cost <= ub && (low_cost < best_cost || (low_cost == best_cost && low_at < best_s))) {
            best_cost = low_cost;
            best_s = low_at;
            ub = low_cost;
        }
        // what is left below the point: above what the neighbour's says of its next budget, and up to where the best cost is
        // reached
        const U above = gap > over ? s - gap - 1 : std::numeric_limits<I>::max();
        const U left = (U)__shfl_up(above < (U)std::numeric_limits<I>::max() ? above : (U)std::numeric_limits<I>::max(), 1, kWave);
        const I from = (I)(leftmost ? lo : left);
        // (a point whose windows were cut says nothing of itself and those below it.  The first round may have such, for its
        // bound is a rough one; where a later one has, the best cost allows them, and the chain is left to a wave of its own)
        const U floor = cut ? first + tail : least;
        const I room = floor > ub ? -1 : (I)(ub - floor), last = cut ? (I)at : (I)at - 1, top = last < room ? last : room;
        const uint64_t cuts = __builtin_amdgcn_ballot_w64(cut && round > 0 && at + first + tail <= ub);
        beyond |= ((cuts >> (row * G)) & (~0ull >> (kWave - G))) != 0;
        solved &= !beyond;
        const bool open = solved && top > from;
        const uint64_t opens = __builtin_amdgcn_ballot_w64(open);
        if (opens == 0) {  // one more pass, for the canonical set: the values for the best budget
            settled = true;
            s = best_s;
            continue;
        }
        // the next points: one for each interval, the others by width; what is left over goes to the last one
        const float wide = open ? (float)(top - from) : 0.0f;
        const float whole = row_sum<G>(wide);
        const int many = row_sum<G>((uint32_t)open);
        const int mine = open ? 1 + (int)(wide / whole * (float)(G - many) * 0.9999f) : 0;
        const int upto_here = (int)row_scan<G>((uint32_t)mine, [](uint32_t a, uint32_t b) { return a + b; });
        m.slot[lane] = 0;
        __syncthreads();
        if (open) m.slot[row * G + upto_here - mine] = i;
        __syncthreads();
        const int owner = (int)row_scan<G>((uint32_t)m.slot[lane], [](uint32_t a, uint32_t b) { return a > b ? a : b; });
        // (a chain without an open interval goes on with its best point, closed)
        const int src = row * G + owner;
        const U o_lo = (U)__shfl(from, src, kWave), o_top = (U)__shfl(top, src, kWave);
        const int o_end = __shfl(upto_here, src, kWave), o_many = __shfl(mine, src, kWave);
        const int k = i - (o_end - o_many);
        const int all_points = (int)row_sum<G>((uint32_t)mine);
        const int of = o_end == all_points ? G - (o_end - o_many) : o_many;
        leftmost = many == 0 || k == 0;
        lo = many == 0 ? best_s : o_lo;
        s = many == 0 ? best_s : split(o_lo, o_top - o_lo, k + 1, of);
        __syncthreads();
    }
    beyond |= cut;
    __syncthreads();
    // from n the first minimal predecessor in the window
    uint64_t mine = 0;
    const U *const P = m.P + row, *const F = m.F + row;
    constexpr int kLook = G == 8 ? 2 : 1;  // positions a lane looks at together: a window holds some ten
    for (int j = n;;) {                    // (value: the least F in the window of j, which is F of its predecessor)
        if (j % G == i) mine |= 1ull << (j / G);
        if (__builtin_amdgcn_ballot_w64(j > 0) == 0) break;
        const U e = P[(j > 0 ? j : 1) * C] - best_s;
        int pred = n, top = j - 1;
        for (bool more = j > 0;;) {
            int first_here = n;
            for (int k = 0; k < kLook; ++k) {
                const int h = top - k * G - i, at = h > 0 ? h : 0;
                const U sum = P[(at + 1) * C], fh = F[at * C];
                // (up to the first that is not in the window: farther sums may be beyond what a difference tells)
                const uint64_t ins = __builtin_amdgcn_ballot_w64(more && h >= 0 && sum - e <= over);
                const uint64_t outs = ~(ins >> (row * G)) & (~0ull >> (kWave - G));
                more = outs == 0;
                const int many = more ? G : __ffsll((unsigned long long)outs) - 1;
                first_here = i < many && fh == value ? h : first_here;
            }
            const int found = (int)row_min<G>((uint32_t)first_here);
            pred = found < pred ? found : pred;
            top -= kLook * G;
            if (__builtin_amdgcn_ballot_w64(more) == 0) break;
        }
        if (j > 0) {
            j = pred < j ? pred : j - 1;  // (there is one)
            value -= j > 0 ? P[(j + 1) * C] - P[j * C] : 0;
        }
    }
    if (!valid) return RowsLeft::kNone;
    if (status == CKPT_OK && (!narrow || beyond)) return narrow ? RowsLeft::kFar : RowsLeft::kWide;
    if (status != CKPT_OK) mine = 0;
    uint8_t *const mp = mask_out + c * cstride;
    for (int k = i, q = 0; k <= n; k += G, ++q) mp[(int64_t)k * pstride] = (uint8_t)((mine >> q) & 1);
    if (i == 0) {
        peak_out[c] = status == CKPT_OK ? (int64_t)((uint64_t)best_cost << shift) : -1;
        if (budget_out) budget_out[c] = status == CKPT_OK ? (int64_t)((uint64_t)best_s << shift) : -1;
        if (status_out) status_out[c] = status;
    }
    return RowsLeft::kNone;
}

// Where the rows may leave chains for their windows (a ring for some of the positions), the call is
//   cubic_rows_sample_kernel  how many of some chains are expected to be far;
//   cubic_rows_kernel         if those are few: the rows, with what they leave done by the same wave or on lists; else nothing;
//   cubic_search_far_kernel   a wave a chain, in 32 bits: the listed far chains if they are many, or all chains;
//   cubic_search_wide_kernel  ... in 64 bits: those that need them, and the listed far chains if they are few.
// Far chains cost the rows their rounds and a wave its search, so a batch of many is better left to waves altogether: 65,536
// chains of 64 layers that fall from one to the next 1.13 ms, 2.8 with rows first and then 64-bit arithmetic for the far ones;
// 4,096 of 256 layers 1.29 (4.1).
// Words of SearchWs::count; its list is followed by one of the far chains, [batch] too.
constexpr int kCountWide = 0, kCountFar = 1, kHeads = 16, kSampled = 32;
constexpr int kSamples = 128;  // workgroups, with a byte each from word kSampled on
constexpr int kXcds = 8;

// Are `from` or more of the sampled chains expected to be far?
__device__ inline bool mostly_far(const SearchWs w, const int from)
{
    static_assert(kSamples / 4 * 2 == kWave, "a wave reads every word twice");
    uint32_t v = (uint32_t)w.count[kSampled + threadIdx.x % (kSamples / 4)];
    v = (v & 0xff00ffu) + ((v >> 8) & 0xff00ffu);
    v = (v & 0xffffu) + (v >> 16);
    return (int)(row_sum<kWave>(v) / 2) >= from;
}

// The chains of one wave of every kSamples-th of the batch, anywhere in it (so that no period of the chains matters).  The
// other words are cleared, which other calls have a launch for.
template <int G, int MOST>
__global__ __launch_bounds__(kWave) void cubic_rows_sample_kernel(const int64_t *__restrict__ d, int64_t batch, int n, int64_t cstride,
                                                                  int64_t pstride, int ring, SearchWs w)
{
    constexpr int C = kWave / G;
    const int64_t waves = (batch + C - 1) / C, any = waves * (int64_t)((blockIdx.x * 2654435761u) >> 16) >> 16;
    const int64_t c = (waves * blockIdx.x + any) / kSamples * C + threadIdx.x / G;
    const bool valid = c < batch;
    const RowChain<G, MOST> chain(d + (valid ? c : batch - 1) * cstride, n, pstride, (float *)search_lds);
    const uint64_t far = __builtin_amdgcn_ballot_w64(chain.far(n, ring, (float *)search_lds) && valid && threadIdx.x % G == 0);
    if (threadIdx.x == 0) ((uint8_t *)(w.count + kSampled))[blockIdx.x] = (uint8_t)__popcll((unsigned long long)far);
    if (blockIdx.x == 0 && threadIdx.x < kSampled) w.count[threadIdx.x] = 0;
}

// IN_WAVE: a wave goes on with its far chains, one after the other; else they go on their list.
template <int G, int MOST, bool IN_WAVE>
__global__ __launch_bounds__(kWave) void cubic_rows_kernel(const int64_t *__restrict__ d, int64_t batch, int n, int64_t cstride,
                                                           int64_t pstride, int ring, int far_from, uint8_t *__restrict__ mask_out,
                                                           int64_t *__restrict__ peak_out, int64_t *__restrict__ budget_out,
                                                           int32_t *__restrict__ status_out, SearchWs w)
{
    if (ring < row_blocks(n) * kRowBlk && mostly_far(w, far_from)) return;
    const int64_t c = (int64_t)xcd_blocked(blockIdx.x, gridDim.x) * (kWave / G) + threadIdx.x / G;
    const bool valid = c < batch;
    const RowsLeft left = search_rows<G, MOST>(d, valid ? c : batch - 1, valid, n, cstride, pstride, mask_out, peak_out,
                                               budget_out, status_out, ring);
    const bool leads = threadIdx.x % G == 0;
    if (leads && left == RowsLeft::kWide) w.list[atomicAdd(w.count + kCountWide, 1)] = (int32_t)c;
    if constexpr (!IN_WAVE) {
        if (leads && left == RowsLeft::kFar) w.list[batch + atomicAdd(w.count + kCountFar, 1)] = (int32_t)c;
    } else {
        for (uint64_t far = __builtin_amdgcn_ballot_w64(leads && left == RowsLeft::kFar); far != 0; far &= far - 1) {
            const int64_t f = c - threadIdx.x / G + __builtin_ctzll((unsigned long long)far) / G;
            __syncthreads();
            const bool done = search_one<true, false>(d + f * cstride, pstride, n, mask_out + f * cstride, pstride, peak_out + f,
                                                      budget_out ? budget_out + f : nullptr, status_out ? status_out + f : nullptr, ~0u);
            if (!done && threadIdx.x == 0) w.list[atomicAdd(w.count + kCountWide, 1)] = (int32_t)f;
        }
    }
}

// EACH: a workgroup for every chain of the batch, with or without one to solve.  Else the waves that the chip holds: of an
// XCD's share, whose neighbours in memory it reads together, they take half one after the other and the rest as they get
// free.  (All of it as they get free: 8,192 chains of 64 layers 188 us instead of 169, all of it one after the other 201.)
template <bool EACH>
__global__ __launch_bounds__(kWave) void cubic_search_far_kernel(const int64_t *__restrict__ d, int64_t batch, int n, int64_t cstride,
                                                                 int64_t pstride, int far_from, int few, uint8_t *__restrict__ mask_out,
                                                                 int64_t *__restrict__ peak_out, int64_t *__restrict__ budget_out,
                                                                 int32_t *__restrict__ status_out, SearchWs w)
{
    const bool every = mostly_far(w, far_from);
    const int count = every ? (int)batch : w.count[kCountFar];
    if (!every && count <= few) return;
    const auto solve = [&](const int at) {
        const int64_t c = every ? at : w.list[batch + at];
        const bool done = search_one<true, false>(d + c * cstride, pstride, n, mask_out + c * cstride, pstride, peak_out + c,
                                                  budget_out ? budget_out + c : nullptr, status_out ? status_out + c : nullptr, ~0u);
        if (!done && threadIdx.x == 0) w.list[atomicAdd(w.count + kCountWide, 1)] = (int32_t)c;
    };
    if constexpr (EACH) {
        const int at = (int)xcd_blocked(blockIdx.x, gridDim.x);
        if (at < count) solve(at);
    } else {
        const int xcd = blockIdx.x % kXcds, share = (count + kXcds - 1) / kXcds, first = share * xcd;
        const int waves = gridDim.x / kXcds, fixed = share / waves / 2;
        for (int turn = 0;; ++turn) {
            int at = turn * waves + blockIdx.x / kXcds;
            if (turn >= fixed) {
                if (threadIdx.x == 0) at = fixed * waves + atomicAdd(w.count + kHeads + xcd, 1);
                at = __builtin_amdgcn_readfirstlane(at);
            }
            if (at >= share || first + at >= count) break;
            solve(first + at);
            __syncthreads();
        }
    }
}

// Every chain of the batch; WIDE false: those that need 64 bits go on the list.
template <bool WIDE>
__global__ __launch_bounds__(kWave) void cubic_search_kernel(const int64_t *__restrict__ d, int n, int64_t cstride,
                                                             int64_t pstride, uint8_t *__restrict__ mask_out,
                                                             int64_t *__restrict__ peak_out,
                                                             int64_t *__restrict__ budget_out,
                                                             int32_t *__restrict__ status_out, SearchWs w)
{
    const int64_t c = xcd_blocked(blockIdx.x, gridDim.x);
    const bool done = search_one<true, WIDE>(d + c * cstride, pstride, n, mask_out + c * cstride, pstride,
                                             peak_out + c, budget_out ? budget_out + c : nullptr,
                                             status_out ? status_out + c : nullptr, ~0u);
    if (!WIDE && !done && threadIdx.x == 0) w.list[atomicAdd(w.count, 1)] = (int32_t)c;
}

// The listed ones, and the far chains if they are no more than `few`.
__global__ __launch_bounds__(kWave) void cubic_search_wide_kernel(const int64_t *__restrict__ d, int64_t batch, int n, int few,
                                                                  int64_t cstride, int64_t pstride,
                                                                  uint8_t *__restrict__ mask_out,
                                                                  int64_t *__restrict__ peak_out,
                                                                  int64_t *__restrict__ budget_out,
                                                                  int32_t *__restrict__ status_out, SearchWs w)
{
    const int wide = w.count[kCountWide], far = few > 0 ? w.count[kCountFar] : 0, count = wide + (far <= few ? far : 0);
    for (int item = blockIdx.x; item < count; item += gridDim.x) {
        const int64_t c = w.list[item < wide ? item : batch + (item - wide)];
        (void)search_one<true, true>(d + c * cstride, pstride, n, mask_out + c * cstride, pstride, peak_out + c,
                                      budget_out ? budget_out + c : nullptr, status_out ? status_out + c : nullptr, ~0u);
        __syncthreads();
    }
}

// `chains` chains of a ragged batch from number `first` on, each where it lies in the flat array, class after class, a
// grid of `chains` workgroups for each (`classes`: four bits a class, the first in the lowest).  lds: the launch's;
// chains that need 64 bits and more of it go on the list.
__global__ __launch_bounds__(kWave) void cubic_search_ragged_kernel(const int64_t *__restrict__ d,
                                                                    const int64_t *__restrict__ off, int64_t first,
                                                                    unsigned chains, unsigned classes, unsigned lds,
                                                                    uint8_t *__restrict__ mask_out,
                                                                    int64_t *__restrict__ peak_out,
                                                                    int64_t *__restrict__ budget_out,
                                                                    int32_t *__restrict__ status_out, SearchWs w)
{
    const unsigned down = blockIdx.x / chains;
    const int k = (int)(classes >> (4 * down)) & 15;
    const int64_t c = first + (blockIdx.x - down * chains), o = off[c], n = off[c + 1] - o - 1;
    if (n > search_class_limit(k) || (k > 0 && n <= search_class_limit(k - 1))) return;
    const bool done = search_one<true, true>(d + o, 1, (int)n, mask_out + o, 1, peak_out + c,
                                             budget_out ? budget_out + c : nullptr,
                                             status_out ? status_out + c : nullptr, lds);
    if (!done && threadIdx.x == 0) w.list[atomicAdd(w.count, 1)] = (int32_t)c;
}

__global__ __launch_bounds__(kWave) void cubic_search_ragged_wide_kernel(const int64_t *__restrict__ d,
                                                                         const int64_t *__restrict__ off,
                                                                         uint8_t *__restrict__ mask_out,
                                                                         int64_t *__restrict__ peak_out,
                                                                         int64_t *__restrict__ budget_out,
                                                                         int32_t *__restrict__ status_out, SearchWs w)
{
    const int count = *w.count;
    for (int item = blockIdx.x; item < count; item += gridDim.x) {
        const int64_t c = w.list[item], o = off[c], n = off[c + 1] - o - 1;
        (void)search_one<false, true>(d + o, 1, (int)n, mask_out + o, 1, peak_out + c,
                                      budget_out ? budget_out + c : nullptr, status_out ? status_out + c : nullptr, ~0u);
        __syncthreads();
    }
}

std::atomic<bool> search_lds_raised[kMaxDevices];

// (the longest of these chains need more than the default)
hipError_t raise_search_lds_limit()
{
    return raise_lds_limit(search_lds_raised,
                           {(const void *)cubic_search_kernel<true>, (const void *)cubic_search_kernel<false>,
                            (const void *)cubic_search_wide_kernel, (const void *)cubic_search_ragged_kernel,
                            (const void *)cubic_search_ragged_wide_kernel, (const void *)cubic_search_far_kernel<true>,
                            (const void *)cubic_search_far_kernel<false>, (const void *)cubic_rows_kernel<16, kRowsMaxLayers, false>},
                           search_lds_bytes(kSearchMaxLayers, 8));
}

// From this many chains on the launch has LDS for 32-bit arithmetic only, twice the waves on a CU, and the
// chains that need 64 bits follow in a second one; fewer chains do not fill the chip either way.
constexpr int64_t kSearchSplitFrom = 1024;
constexpr int kSearchWideBlocks = 1024;
// A row of lanes per chain from here on: 8,192 chains of 16, 64 and 128 layers, unrounded 45, 150 and 472 us (a wave a chain:
// 50, 199, 839), aligned 39, 115, 346 (49, 172, 702); at 4,096 chains the longer ones only, 39, 156, 341 (34, 121, 459), and
// where a wave a chain leaves a CU three or two waves, beyond 128 layers, at 2,048: of 152 and 256 layers unrounded 460 and
// 1,221 (598, 1,542), aligned 227 and 413 (331, 846), networks 293 and 479 (331, 759).
// Eight lanes rather than sixteen where that leaves waves enough, up to 72 layers (a CU holds eight of those waves up to 68,
// then seven): 65,536 aligned chains of 64 layers 541 us (646), of 72 layers 666 and unrounded 836 (760, 1,025), 16,384 of those
// 264 and 326 (239, 371); 65,536 aligned of 90 1,030 (907); 8,192 of 64 153 (115).
constexpr int64_t kRowsOf8From = 16384;
inline int64_t rows_from(int n) { return n > 128 ? 2048 : n > 96 ? 4096 : 8192; }
// The share of a batch's chains that are expected to be far from which on waves take them all.  Far chains among others add a
// launch's time to that of the rows, a wave's search at least: 65,536 unrounded chains of 64 layers with one in ten of layers in
// front that outweigh the rest 0.95 ms (1.27 with a wave a chain), with one in two 1.19 (1.20; 1.6 as rows and waves); 8,192 of
// them with one in ten 253 us as rows and waves, 200 as waves.
// A workgroup for every chain up to this many (see there): 2,048 chains of 152 layers 291 us (340 with the waves that the chip
// holds), 8,192 of 48 layers 134 (148).  Where there is nothing to do that costs 8,192 chains 1 us.
constexpr int64_t kFarEachMost = 8192;
// (a launch has fewer than 2^32 threads)
constexpr int64_t kMostWavesOfALaunch = 1 << 25;
// Waves of this much LDS that the chip holds (LDS is handed out in units of 1,280 bytes).
inline int64_t at_once(size_t lds) { return 256 * ((160 << 10) / (int64_t)align_up(lds, 1280)); }
// The share of a batch's chains that are expected to be far from which on waves take them all.  Far chains among others add to
// the rows' time a wave's search, a quarter of what all of them take with four turns of waves; with one in ten of layers in
// front that outweigh the rest, unrounded others and a share of 1/4, 8,192 chains of 64 layers 280 us, 2,048 of 130 487 (so 201
// and 366; without rows 198 and 360), 65,536 of 64 1.0 ms (1.27 without rows).
inline float far_share(int64_t batch, int n)
{
    return (n <= kRowsOf8Layers ? batch < kRowsOf8From : batch <= 4 * at_once(search_lds_bytes(n, 4))) ? 1.0f / 16 : 1.0f / 4;
}
// A ragged batch goes in one launch up to this many turns of it, with the longest chain's LDS for all: the classes one
// after the other each wait for their slowest wave.  1,000 chains of 2 to 152 layers 114 us (four launches 247), 4,096
// 194 (335), 8,192 373 (387), 16,384 668 (567); of 2 to 256 layers 4,096 427 (519), 8,192 785 (798), 16,384 1,546
// (1,309).  But a launch lasts as long as its slowest wave, and as all its chains together take the waves that the chip
// holds with its LDS; where that says more than the launches of the classes would take (8 us more for each), the short
// chains are too many for the long ones' LDS: 16,383 chains of 24 layers and one of 64 149 us (127 in two launches), 5,900
// of 64 and 100 of 152 310 us (259).
constexpr int64_t kOneLaunchTurns = 8;
inline float launch_us(int longest, float us, int width) { return std::max(search_us(longest), us / (float)at_once(search_lds_bytes(longest, width))); }
// ... with LDS for 64 bits up to one turn of that, for a second launch for the chains that need them costs as much as a
// second turn: 512 chains of 15, 24 and 152 unrounded layers 219 us with two turns, 155 in 32 bits with a second launch.
// More than 192 layers of unrounded sizes mostly need them, and a chain of those in the second launch is what the call
// waits for: there up to twice the longest chain's time, 1,000 chains of 2 to 256 unrounded layers 400 us (627), 1,007 of
// 24 and 16 of 256 339 (663); aligned ones 239 (244) and 209 (211).  700 of 224 to 256 layers are beyond: 573 (377) aligned.
inline bool wide_first(int64_t batch, int longest, float us)
{
    const int64_t turn = at_once(search_lds_bytes(longest, 8));
    return longest > 192 ? batch < kSearchSplitFrom && us <= 2.0f * search_us(longest) * (float)turn : batch <= turn;
}

}  // namespace

hipError_t launch_cubic_search(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                               int64_t *peak_out, int64_t *budget_out, int32_t *status_out, void *ws,
                               hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    if (search_lds_bytes(n, 8) > kDefaultLdsLimit) {
        const hipError_t e = raise_search_lds_limit();
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)batch), block(kWave);
    const SearchWs w{(int32_t *)ws, (int32_t *)((char *)ws + 256)};
    if (batch >= rows_from(n)) {
        // (far chains that are less than a turn of the wide ones' waves go with those: a launch lasts as long as a chain)
        const int few = (int)at_once(search_lds_bytes(n, 8));
        const auto rows = [&](auto lanes, auto most) {
            constexpr int G = decltype(lanes)::value, MOST = decltype(most)::value, C = kWave / G;
            constexpr bool kInWave = MOST <= kRowsOf16Layers;
            const int positions = row_blocks(n) * kRowBlk;
            const int64_t waves = (batch + C - 1) / C;
            const size_t one = search_lds_bytes(n, 4);
            int ring = row_ring(n);
            size_t lds = rows_lds_bytes(n, C, ring);
            // A wave goes on with its far chains where the LDS for that leaves as many waves, and a longer ring what of it there
            // is: 65,536 unrounded chains of 64 layers 665 us (697 with the far ones in a launch), 8,192 150 (180).  Beyond 128
            // layers that gains nothing: 2,048 networks of 152 302 (292).
            const bool in_wave = kInWave && ring < positions && (at_once(one) >= at_once(lds) || waves <= at_once(one));
            if (in_wave) {
                while (ring < positions && rows_lds_bytes(n, C, ring + kRowBlk) <= one) ring += kRowBlk;
                lds = std::max(one, rows_lds_bytes(n, C, ring));
            }
            const bool whole = ring == positions;  // (no chain is far)
            if (whole)
                hipLaunchKernelGGL(cubic_search_reset_kernel, dim3(1), dim3(kSampled), 0, stream, w);
            else
                hipLaunchKernelGGL((cubic_rows_sample_kernel<G, MOST>), dim3(kSamples), block, (size_t)(n + 1) * C * 4, stream, d, batch,
                                   n, st.chain, st.pos, ring, w);
            const int far_from = (int)(far_share(batch, n) * (float)(kSamples * C));
            hipLaunchKernelGGL((in_wave ? cubic_rows_kernel<G, MOST, kInWave> : cubic_rows_kernel<G, MOST, false>), dim3((unsigned)waves), block,
                               lds, stream, d, batch, n, st.chain, st.pos, ring, far_from, mask_out, peak_out, budget_out, status_out, w);
            if (whole) return;
            const bool each = batch <= kFarEachMost;
            hipLaunchKernelGGL(each ? cubic_search_far_kernel<true> : cubic_search_far_kernel<false>,
                               dim3((unsigned)(each ? batch : at_once(one))), block, one, stream, d, batch, n, st.chain, st.pos, far_from, few,
                               mask_out, peak_out, budget_out, status_out, w);
        };
        if (batch >= kRowsOf8From && n <= kRowsOf8Layers) rows(std::integral_constant<int, 8>(), std::integral_constant<int, kRowsOf8Layers>());
        else if (n <= kRowsOf16Layers) rows(std::integral_constant<int, 16>(), std::integral_constant<int, kRowsOf16Layers>());
        else rows(std::integral_constant<int, 16>(), std::integral_constant<int, kRowsMaxLayers>());
        hipLaunchKernelGGL(cubic_search_wide_kernel, dim3(kSearchWideBlocks), block, search_lds_bytes(n, 8), stream, d,
                           batch, n, few, st.chain, st.pos, mask_out, peak_out, budget_out, status_out, w);
    } else if (batch < kSearchSplitFrom) {
        hipLaunchKernelGGL(cubic_search_kernel<true>, grid, block, search_lds_bytes(n, 8), stream, d, n, st.chain, st.pos,
                           mask_out, peak_out, budget_out, status_out, w);
    } else {
        hipLaunchKernelGGL(cubic_search_reset_kernel, dim3(1), dim3(1), 0, stream, w);
        hipLaunchKernelGGL(cubic_search_kernel<false>, grid, block, search_lds_bytes(n, 4), stream, d, n, st.chain,
                           st.pos, mask_out, peak_out, budget_out, status_out, w);
        hipLaunchKernelGGL(cubic_search_wide_kernel, dim3(kSearchWideBlocks), block, search_lds_bytes(n, 8), stream, d,
                           batch, n, 0, st.chain, st.pos, mask_out, peak_out, budget_out, status_out, w);
    }
    return hipGetLastError();
}

hipError_t launch_cubic_search_ragged(const int64_t *d, const int64_t *offsets_dev, int64_t batch,
                                      const SearchClass (&class_of)[kSearchClasses], uint8_t *mask_out, int64_t *peak_out,
                                      int64_t *budget_out, int32_t *status_out, int32_t *count, int32_t *list, hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    const hipError_t e = raise_search_lds_limit();
    if (e != hipSuccess) return e;
    const dim3 block(kWave);
    const SearchWs w{count, list};
    int top = kSearchClasses - 1;
    while (class_of[top].longest == 0) --top;
    const int all = class_of[top].longest;
    float us = 0.0f, several = 0.0f;
    for (const SearchClass &k : class_of)
        if (k.longest != 0) {
            us += k.us;
            several += launch_us(k.longest, k.us, 4) + 8.0f;
        }
    const bool one_launch = batch <= kOneLaunchTurns * at_once(search_lds_bytes(all, 4)) && launch_us(all, us, 4) <= 1.1f * several;
    // all of the arithmetic in the first launch (the longest chains' LDS says whether the rest needs a second one)
    const bool wide = one_launch ? wide_first(batch, all, us) : batch < kSearchSplitFrom;
    const auto lds = [&](int n) { return (unsigned)search_lds_bytes(n, wide ? 8 : 4); };
    if (!wide) hipLaunchKernelGGL(cubic_search_reset_kernel, dim3(1), dim3(1), 0, stream, w);
    if (one_launch) {
        unsigned classes = 0, many = 0;
        for (int k = top; k >= 0; --k)  // the longest chains first
            if (class_of[k].longest != 0) classes |= (unsigned)k << (4 * many++);
        hipLaunchKernelGGL(cubic_search_ragged_kernel, dim3((unsigned)batch * many), block, lds(all), stream, d, offsets_dev,
                           (int64_t)0, (unsigned)batch, classes, lds(all), mask_out, peak_out, budget_out, status_out, w);
    } else {
        for (int k = top; k >= 0; --k) {
            const int n = class_of[k].longest;
            if (n == 0) continue;
            for (int64_t first = 0; first < batch; first += kMostWavesOfALaunch) {
                const unsigned chains = (unsigned)std::min(batch - first, kMostWavesOfALaunch);
                hipLaunchKernelGGL(cubic_search_ragged_kernel, dim3(chains), block, lds(n), stream, d, offsets_dev, first,
                                   chains, (unsigned)k, lds(n), mask_out, peak_out, budget_out, status_out, w);
            }
        }
    }
    if (!wide)
        hipLaunchKernelGGL(cubic_search_ragged_wide_kernel, dim3(kSearchWideBlocks), block, search_lds_bytes(all, 8),
                           stream, d, offsets_dev, mask_out, peak_out, budget_out, status_out, w);
    return hipGetLastError();
}

namespace {

// ---------------------------------------------------------------------------
// long chains: one wave per point, the points of a round on the whole chip
// ---------------------------------------------------------------------------
//
//   table      one workgroup per chain: checks, prefix sums divided by the unit that all sizes are multiples
//              of (their common power of two; their greatest common divisor where that still leaves more
//              than 31 bits: the sizes of a network share its batch size), a first bound
//   round x 2  `points` waves per chain evaluate a point each, cutting the open intervals evenly
//   close x 2  (after each) takes the best cost and lists the intervals that stay open
//   list       a thread per start: the budgets inside the open intervals, each value once (a table of the
//              values seen keeps most repeated ones out); if they are many, a workgroup cuts the intervals further
//   finish     a wave per listed budget, and one for the best point so far; each keeps the set of its best
//   result     the best of the waves, its set spread to bytes
// After a round of 1,024 points a few hundred budgets are left of up to 2,000 layers of one order, and after two one to
// twenty, so `finish` takes one pass; it takes whatever is left.  A call is bound by two or three passes in a row, each
// as long as its slowest wave (a point of many heads).  A point whose F(h) has passed what the best cost seen leaves
// stops: a small s would have a head at every cell. Measured, with every budget evaluated in brackets: one chain of
// 4,096 aligned layers 300 us (1,650), of 1,001 of a network 97 (1,200 to 1,490; 480 while the first of equal
// predecessors was taken and there were always two rounds), of 152 of a network 48 (121 to 137; 90 then); two of 3,115
// aligned layers 396 (2,215); 100 of 1,001 466 (5,260), unrounded 484 (118,000); 1,000 of 300 600 (3,710), unrounded
// 685 (34,000).
constexpr int kOpenMax = 128;       // open intervals kept (more are joined)
constexpr int kMostPoints = 1024;   // of a round, per chain
constexpr int kTableThreads = 1024;
constexpr int kTablePer = (CKPT_CUBIC_MAX_LAYERS + 1 + kTableThreads - 1) / kTableThreads;
constexpr int kBounds = kTableThreads / kWave;

struct LongMeta {
    int32_t status;
    int32_t narrow;      // 1: 32-bit values
    uint64_t unit;       // the sizes were divided by this
    uint64_t ub;         // the best cost known (a bound, then costs); lowered while a round runs
    uint64_t ends;       // d_0 + d_n
    uint64_t all;        // the sizes between them
    uint64_t best_cost;  // of the evaluated points (~0: none)
    uint64_t best_s;
    int32_t open[2];     // intervals before round 0 / 1 ...
    int32_t left;        // ... and after the rounds
    int32_t listed;      // budgets in the list
};
struct Open {
    int64_t lo, hi;      // lo < s <= hi
    uint64_t c;          // F_s(n) is at least this for all of them
    int32_t first;       // number of its first point
    int32_t pad;
};
struct Point {
    int64_t prev, s;
    uint64_t c;          // F_s(n), or with `exact` 0 a value it is not below
    int64_t exact;
};
struct LongWs {
    LongMeta *meta;      // [batch]
    Open *open;          // [batch][3][kOpenMax] before round 0, before round 1, after it
    Point *point;        // [batch][points]
    uint64_t *seen;      // [batch][seen_slots] values listed
    uint64_t *found;     // [batch][finish_waves][2] best cost and its s of a finish wave
    uint64_t *set;       // [batch][finish_waves][n / 64 + 1] and its set, a bit a layer
    uint32_t *list;      // [batch][K] start << 13 | end
    char *P;             // [batch][n + 1] uint64_t (uint32_t in the same bytes when narrow)
};
static_assert(CKPT_CUBIC_MAX_LAYERS < (1 << 13), "a start and an end in 26 bits");

// Points per chain and round: the chip's SIMDs twice over between the chains, within 64 .. 1,024 (512 below 512
// layers, 256 up to 256, which a workspace has room for).
__host__ __device__ inline int long_points(int64_t batch, int n)
{
    const int most = n <= 256 ? kMostPoints / 4 : n < 512 ? kMostPoints / 2 : kMostPoints;
    const int64_t share = batch >= 32 ? 64 : 2048 / batch;
    return (int)(share < most ? share : most) / kWave * kWave;
}
// (up to 1,024: ten bits of a product)
__host__ __device__ inline int seen_slots(int n) { return n <= 256 ? 256 : 1024; }
__host__ __device__ inline int64_t long_budgets(int n) { return (int64_t)n * (n - 1) / 2 + 1; }

// Waves per chain that evaluate what the rounds leave: as many as points, up to 512.
__host__ __device__ inline int finish_waves(int64_t batch, int n)
{
    const int points = long_points(batch, n);
    return n <= 256 ? 64 : points < 512 ? points : n < 512 ? 256 : 512;
}

__host__ size_t carve_long(void *ws, int64_t batch, int n, LongWs *w)
{
    size_t at = 0;
    char *base = (char *)ws;
    const size_t B = (size_t)batch;
    auto take = [&](size_t bytes) { char *here = base + at; at += align_up(bytes); return here; };
    w->meta = (LongMeta *)take(B * sizeof(LongMeta));
    w->open = (Open *)take(B * 3 * kOpenMax * sizeof(Open));
    const size_t points = B * (size_t)long_points(batch, n) * sizeof(Point);
    const size_t sets = B * (size_t)finish_waves(batch, n) * ((size_t)n / kWave + 1) * 8;
    w->point = (Point *)take(points > sets ? points : sets);
    w->set = (uint64_t *)w->point;  // (the rounds are over when the first set is written)
    w->seen = (uint64_t *)take(B * (size_t)seen_slots(n) * 8);
    w->found = (uint64_t *)take(B * (size_t)finish_waves(batch, n) * 16);
    w->list = (uint32_t *)take(B * (size_t)long_budgets(n) * 4);
    w->P = take(B * ((size_t)n + 1) * 8);
    return at;
}

// ---- table ----

// The smallest over the workgroup, for every thread.
__device__ inline uint64_t block_min(uint64_t v, uint64_t *room)
{
    v = wave_min_u64(v);
    __syncthreads();
    if (threadIdx.x % kWave == 0) room[threadIdx.x / kWave] = v;
    __syncthreads();
    v = room[threadIdx.x % (kTableThreads / kWave)];
    static_assert(kTableThreads / kWave <= kWave, "one wave holds the waves' values");
    return wave_min_u64(v);
}

// One workgroup a chain.  What bounds it is issue: sixteen waves on a CU, four to a SIMD, so an instruction of all costs
// sixteen cycles.  Hence waves without sizes do nothing but their segment length, no thread looks at more than its `per`
// sizes, the waves' results are joined in the lanes of a row, and the only division is that by a unit that is no power of
// two.  Networks of 152 and 1,001 layers 4.6 and 12 us; with all of that in every wave 7.8 and 20.
__global__ __launch_bounds__(kTableThreads) void search_table_kernel(const int64_t *__restrict__ d, int n, int64_t cstride,
                                                                     int64_t pstride, int points, int waves, LongWs w)
{
    constexpr int kWaves = kTableThreads / kWave;
    static_assert(kWaves == 16, "a row of lanes holds the waves' values");
    __shared__ uint64_t room[kWaves], part[4][kWaves];
    __shared__ float bound_of[kBounds];
    __shared__ uint64_t ends2[2];
    float *const prefix = (float *)search_lds;  // [n + 1] of the interior sizes
    const int64_t c = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t *dp = d + c * cstride;
    const int per = (n + kTableThreads) / kTableThreads, k0 = tid * per;  // a thread takes `per` sizes in a row
    const bool holds = __builtin_amdgcn_readfirstlane(wave) * kWave * per <= n;
    const auto either = [](uint64_t a, uint64_t b) { return a | b; };
    uint64_t x[kTablePer] = {};
    uint64_t bits = 0, high = 0, sum = 0, mx = 0;
    if (holds) {
#pragma unroll
        for (int q = 0; q < kTablePer; ++q) {
            if (q >= per) break;
            x[q] = k0 + q <= n ? (uint64_t)dp[(int64_t)(k0 + q) * pstride] : 0;
        }
    }
    for (int k = tid; k < seen_slots(n); k += kTableThreads) w.seen[c * seen_slots(n) + k] = 0;
    for (int k = tid; k < 2 * waves; k += kTableThreads) w.found[c * 2 * waves + k] = ~0ull;
    if (holds) {
#pragma unroll
        for (int q = 0; q < kTablePer; ++q) {
            if (q >= per) break;
            bits |= k0 + q > n || (int64_t)x[q] > 0 ? x[q] : 1ull << 63;  // (no size that is positive has that bit)
            high += x[q] >> 32;
            sum += x[q];
            mx = x[q] > mx ? x[q] : mx;
        }
        bits = row_all<kWave>(bits, either);
        high = row_sum<kWave>(high);
        sum = row_sum<kWave>(sum);
        mx = ~wave_min_u64(~mx);
    }
    if (lane == 0) {
        part[0][wave] = bits; part[1][wave] = high; part[2][wave] = sum; part[3][wave] = mx;
    }
    __syncthreads();
    bits = lane63_u64(row_all<kWaves>(part[0][lane % kWaves], either));
    high = lane63_u64(row_sum<kWaves>(part[1][lane % kWaves]));
    sum = lane63_u64(row_sum<kWaves>(part[2][lane % kWaves]));
    mx = ~lane63_u64(row_min<kWaves>(~part[3][lane % kWaves]));
    LongMeta m = {};
    m.status = bits >> 63 ? CKPT_ERR_SIZE : chain_overflows(sum, high, mx) ? CKPT_ERR_OVERFLOW : CKPT_OK;
    if (m.status != CKPT_OK) {
        if (tid == 0) w.meta[c] = m;
        return;
    }
    uint64_t unit = bits & (0 - bits);
    const int shift = __ffsll((unsigned long long)unit) - 1;
    m.narrow = (sum + mx) >> shift < (1ull << 31);
    if (!m.narrow) {
        // Euclid on all sizes at once: the smallest remainder of any size takes the divisor's place until none is left
        uint64_t g = mx;
#pragma unroll
        for (int q = 0; q < kTablePer; ++q) g = x[q] != 0 && x[q] < g ? x[q] : g;
        g = block_min(g, room);
        for (int turn = 0; turn < 12 && g > unit; ++turn) {  // (not settled by then: small divisors do not help)
            uint64_t r = ~0ull;
            if (holds) {
#pragma unroll
                for (int q = 0; q < kTablePer; ++q) {
                    if (q >= per) break;
                    const uint64_t rest = x[q] % g;
                    r = rest != 0 && rest < r ? rest : r;
                }
            }
            r = block_min(r, room);
            if (r == ~0ull) {
                unit = g;
                break;
            }
            g = r;
        }
    }
    m.unit = unit;
    const bool pow2 = (unit & (unit - 1)) == 0;
    if (!pow2) m.narrow = (sum + mx) / unit < (1ull << 31);  // (the largest power of two is the first)
    uint64_t *const P64 = (uint64_t *)w.P + c * (n + 1);
    uint32_t *const P32 = (uint32_t *)P64;
    uint64_t mine = 0, incl = 0;
    if (holds) {
        if (pow2) {
#pragma unroll
            for (int q = 0; q < kTablePer; ++q) x[q] >>= shift;
        } else {
#pragma unroll
            for (int q = 0; q < kTablePer; ++q) {
                if (q >= per) break;
                x[q] /= unit;
            }
        }
#pragma unroll
        for (int q = 0; q < kTablePer; ++q) mine += x[q];
        incl = wave_scan_u64(mine);
    }
    __syncthreads();
    if (lane == kWave - 1) room[wave] = incl;
    if (tid == 0) ends2[0] = x[0];
    __syncthreads();
    const uint64_t of_wave = room[lane % kWaves], total = lane63_u64(row_sum<kWaves>(of_wave));
    if (holds) {
        uint64_t run = incl - mine + lane63_u64(row_sum<kWaves>(lane % kWaves < wave ? of_wave : 0));
#pragma unroll
        for (int q = 0; q < kTablePer; ++q) {
            const int k = k0 + q;
            if (q >= per || k > n) break;
            run += x[q];
            if (m.narrow) P32[k] = (uint32_t)run; else P64[k] = run;
            prefix[k] = bound_prefix(run, ends2[0]);
            if (k == n) ends2[1] = x[q];
        }
    }
    __syncthreads();
    // a bound from 16 segment lengths, one to a wave (see bound_prefix)
    const uint64_t ends = ends2[0] + ends2[1], all = total - ends;
    {
        const float length = fmaxf((float)all * exp2f(-0.5f * (float)(wave + 1)), 1.0f);
        const float inv = 1.0f / length;
        float kept = 0.0f;
        for (int i = 1 + lane; i < n; i += kWave) kept += bound_layer(prefix[i - 1], prefix[i], inv);
#pragma unroll
        for (int k = kWave / 2; k >= 1; k >>= 1) kept += __shfl_xor(kept, k, kWave);
        if (lane == 0) bound_of[wave] = bound_cost(kept, length, all, n);
    }
    __syncthreads();
    if (wave != 0) return;
    const float low = row_min<kBounds>(bound_of[lane % kBounds]);
    if (tid != 0) return;
    uint64_t ub = ends + (uint64_t)(double)low + 1;
    ub = ub < total ? ub : total;
    m.ub = ub;
    m.ends = ends;
    m.all = all;
    m.best_cost = total <= ub ? total : ~0ull;  // s = 0: every layer a checkpoint
    m.best_s = 0;
    const uint64_t span = all < ub - ends ? all : ub - ends;
    m.open[0] = span > 0 ? 1 : 0;
    w.open[c * 3 * kOpenMax] = Open{0, (int64_t)span, 0, 0, 0};
    w.meta[c] = m;
}

// ---- rounds ----

// What a wave reads while others write: past the L1 cache and the XCD's own L2.
template <typename T>
__device__ inline T shared_load(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Point g of a round: the interval that holds it and its place there.
__device__ inline void point_of(const Open *open, int count, int points, int g, int64_t &prev, int64_t &s)
{
    const int lane = threadIdx.x;
    int at = -1;
    for (int k0 = 0; k0 < count; k0 += kWave)
        at += (int)__popcll((unsigned long long)__builtin_amdgcn_ballot_w64(k0 + lane < count && open[k0 + lane].first <= g));
    const Open o = open[at];
    const int next = at + 1 < count ? open[at + 1].first : points;
    const int64_t many = next - o.first, t = g - o.first, wide = o.hi - o.lo;
    const int64_t part = wide / many, rest = wide % many;
    prev = o.lo + part * t + rest * t / many;
    s = o.lo + part * (t + 1) + rest * (t + 1) / many;
}

// A chain's point, evaluated: F_s(n), or less if it stopped (`exact` false then); RECORD, `head`, F: as in wave_cost.
template <typename U, bool RECORD>
__device__ __forceinline__ uint64_t long_cost(const LongWs &w, const LongMeta *meta, const int64_t c, const int n,
                                              const int64_t prev, const int64_t s, bool &exact, uint16_t *head, U *F,
                                              bool *ties = nullptr)
{
    const U *P = (const U *)((const uint64_t *)w.P + c * (n + 1));
    exact = true;
    // No s above prev can be optimal once F(h) is above what the best cost leaves beside it.  (The best cost is read a
    // slice ahead: it comes from memory, past the caches.)
    uint64_t ahead = shared_load(&meta->ub);
    auto stop = [&](U fh) -> bool {
        const uint64_t ub = ahead;
        ahead = shared_load(&meta->ub);
        const bool out = (int64_t)(ub - (uint64_t)fh) <= prev;
        if (out) exact = false;
        return out;
    };
    const U v = wave_cost<U, RECORD>(P, n, (U)s, F, head, stop, ties);
    exact = exact && v != std::numeric_limits<U>::max();
    return (uint64_t)v;
}

__global__ __launch_bounds__(kWave) void search_round_kernel(int n, int points, int round, LongWs w)
{
    const int64_t c = blockIdx.y;
    LongMeta *meta = w.meta + c;
    const int count = meta->open[round];
    if (meta->status != CKPT_OK || count == 0) return;  // (the same for all waves of the chain: nothing to close)
    const int lane = threadIdx.x, g = blockIdx.x;
    int64_t prev, s;
    point_of(w.open + (c * 3 + round) * kOpenMax, count, points, g, prev, s);
    Point p{prev, s, ~0ull, 0};
    if (s > prev) {
        bool exact;
        p.c = meta->narrow ? long_cost<uint32_t, false>(w, meta, c, n, prev, s, exact, nullptr, (uint32_t *)search_lds)
                           : long_cost<uint64_t, false>(w, meta, c, n, prev, s, exact, nullptr, (uint64_t *)search_lds);
        p.exact = exact;
        if (exact && lane == 0) atomicMin((unsigned long long *)&meta->ub, (unsigned long long)(p.c + (uint64_t)s));
    }
    if (lane == 0) w.point[c * points + g] = p;
}

// The end of a round, one wave per chain: the best of the points, and the intervals that stay open under the best
// cost.  (A launch of its own: as the work of the round's last wave it took a device-wide fence in every wave, 36 ns
// of the whole chip each, 2.2 of 2.3 ms for 1,000 chains of 300 layers.)
__global__ __launch_bounds__(kWave) void search_close_kernel(int n, int points, int few_budgets, int round, LongWs w)
{
    const int64_t c = blockIdx.x;
    LongMeta *meta = w.meta + c;
    if (meta->status != CKPT_OK || meta->open[round] == 0) return;
    const int lane = threadIdx.x;
    // (all loads in flight together: read where they are used, this took 12 us)
    const int per = points / kWave;  // consecutive points of a lane
    const Point *pt = w.point + c * points + lane * per;
    Point q[kMostPoints / kWave];
#pragma unroll
    for (int k = 0; k < kMostPoints / kWave; ++k) q[k] = pt[k < per ? k : 0];
    uint64_t cost = ~0ull, at = ~0ull;
#pragma unroll
    for (int k = 0; k < kMostPoints / kWave; ++k) {
        const int64_t prev = q[k].prev, s = q[k].s;
        const uint64_t pc = q[k].c + (uint64_t)s;
        if (k < per && q[k].exact != 0 && s > prev && (pc < cost || (pc == cost && (uint64_t)s < at))) {
            cost = pc;
            at = (uint64_t)s;
        }
    }
    const uint64_t best = wave_min_u64(cost), best_at = wave_min_u64(cost == best ? at : ~0ull);
    uint64_t bc = meta->best_cost, bs = meta->best_s;
    if (best < bc || (best == bc && best_at < bs)) {
        bc = best;
        bs = best_at;
    }
    const uint64_t known = meta->ub, ub = known < bc ? known : bc;
    // the open parts; joined from the kOpenMax-th on
    uint64_t width = 0;
    int many = 0;
#pragma unroll
    for (int k = 0; k < kMostPoints / kWave; ++k) {
        const int64_t prev = q[k].prev, s = q[k].s;
        const uint64_t pc = q[k].c;
        const int64_t last = q[k].exact != 0 ? s - 1 : s;
        const int64_t top = pc > ub ? -1 : last < (int64_t)(ub - pc) ? last : (int64_t)(ub - pc);
        if (k < per && top > prev) {
            width += (uint64_t)(top - prev);
            ++many;
        }
    }
    int incl = many;
#pragma unroll
    for (int k = 1; k < kWave; k <<= 1) {
        const int o = __shfl_up(incl, k, kWave);
        if (lane >= k) incl += o;
    }
    const int count = __builtin_amdgcn_readlane(incl, kWave - 1);
    float whole = (float)width;
#pragma unroll
    for (int k = kWave / 2; k >= 1; k >>= 1) whole += __shfl_xor(whole, k, kWave);
    // About n budgets lie in a width of one mean layer (counted on chains of 152 to 4,096 layers of every kind: within
    // 30 %, repeated values among them).  If few are left, the second round is left out: 1,024 points leave 70 to 350 of a
    // chain of 1,001 layers.
    const bool few = round == 0 && count < kOpenMax && whole * (float)n * (float)n <= (float)few_budgets * (float)meta->all;
    Open *out = w.open + (c * 3 + (few ? 2 : round + 1)) * kOpenMax;
    int slot = incl - many;
    int64_t tail_lo = INT64_MAX, tail_hi = -1;
    uint64_t tail_c = ~0ull;
#pragma unroll
    for (int k = 0; k < kMostPoints / kWave; ++k) {
        const int64_t prev = q[k].prev, s = q[k].s;
        const uint64_t pc = q[k].c;
        const int64_t last = q[k].exact != 0 ? s - 1 : s;
        const int64_t top = pc > ub ? -1 : last < (int64_t)(ub - pc) ? last : (int64_t)(ub - pc);
        if (k >= per || top <= prev) continue;
        if (slot < kOpenMax - 1) {
            out[slot] = Open{prev, top, pc, 0, 0};
        } else {
            tail_lo = prev < tail_lo ? prev : tail_lo;
            tail_hi = top > tail_hi ? top : tail_hi;
            tail_c = pc < tail_c ? pc : tail_c;
        }
        ++slot;
    }
    int kept = count;
    if (count >= kOpenMax) {
        kept = kOpenMax;
        tail_lo = (int64_t)wave_min_u64((uint64_t)tail_lo);
        tail_c = wave_min_u64(tail_c);
        tail_hi = (int64_t)(~wave_min_u64(~(uint64_t)(tail_hi + 1)) - 1);
        if (lane == 0) out[kOpenMax - 1] = Open{tail_lo, tail_hi, tail_c, 0, 0};
    }
    __syncthreads();
    // points for the next round: one each, the others by width
    if (round == 0 && !few && kept > 0) {
        int given = 0;
        const int spare = points > kept ? points - kept : 0;
        for (int k0 = 0; k0 < kept; k0 += kWave) {
            const int k = k0 + lane;
            int mine = 0;
            if (k < kept) {
                const float part = (float)(out[k].hi - out[k].lo) / whole * (float)spare * 0.9999f;
                mine = 1 + (part > 0.0f ? (part < (float)spare ? (int)part : spare) : 0);
            }
            int sum = mine;
#pragma unroll
            for (int j = 1; j < kWave; j <<= 1) {
                const int o = __shfl_up(sum, j, kWave);
                if (lane >= j) sum += o;
            }
            if (k < kept) out[k].first = given + sum - mine;
            given += __builtin_amdgcn_readlane(sum, kWave - 1);
        }
    }
    if (lane == 0) {
        meta->best_cost = bc;
        meta->best_s = bs;
        meta->ub = ub;
        if (round == 0) meta->open[1] = few ? 0 : kept;
        if (round == 1 || few) meta->left = kept;
    }
}

// ---- the budgets that are left ----

// The budgets inside the open intervals are listed, each value once as far as a table of the values seen tells.  Two
// rounds of points that cut the intervals evenly leave few of them where sizes are of one order; where one layer
// outweighs the others 10^8 times, most budgets lie within a single cut (4,096 layers, one of 10^15 among others up to
// 10^6: 935,000 of 8.4 million).  So when there are more than `most`, a workgroup cuts the intervals itself, at budgets
// drawn evenly from those that are left, whatever their scale, and at the largest that is one layer; a wave evaluates
// each, and lists again.  One such chain of 300, 1,001 and 4,096 layers: 105, 258 and 300 us where finishing the list as
// it was took 1.7, 8.2 and 64 ms (every budget evaluated: 0.2, 1.5 and 92 ms).
constexpr int kListMost = 1024;   // threads
constexpr int kListWaves = kListMost / kWave;
constexpr int kListPasses = 32;   // then all that are left are listed (two were the most on any chain tried)
constexpr int kListStarts = 4;    // starts whose bisections a thread runs side by side

// Bytes of F in LDS, before the heads.
__host__ __device__ inline size_t long_f_bytes(int n) { return ((size_t)n + 1 + kWave) * 8; }

// A thread per start, and eight waves where the chip has room for them.
__host__ inline int list_threads(int64_t batch, int n)
{
    const int starts = n < kListMost ? (n + kWave - 1) / kWave * kWave : kListMost;
    return batch <= 512 && starts < 512 ? 512 : starts;
}
// Waves of it that evaluate points: as many as their F leave the chains of a CU room for (the lists themselves take 9
// KB).
__host__ inline int list_waves(int64_t batch, int n)
{
    const size_t room = (size_t)(160 << 10) / (size_t)((batch + 255) / 256), own = 10 << 10;
    const int fit = room > own ? (int)((room - own) / long_f_bytes(n)) : 0, waves = list_threads(batch, n) / kWave;
    return fit < 1 ? 1 : fit < waves ? fit : waves;
}

struct ListLds {
    Open open[2][kOpenMax];
    int64_t drawn[kListWaves], s[kListWaves];  // the budgets drawn, and in ascending order
    uint64_t c[kListWaves];
    int exact[kListWaves];
    unsigned sum[kListWaves];                  // budgets counted by a wave's lanes
    unsigned long long single;                 // the largest that is one layer
    int count;
};

// The first x in [from, n) with P[x] - pa > bound, n if there is none.
template <typename U>
__device__ inline int first_end(const U *P, int from, int n, uint64_t pa, uint64_t bound)
{
    int lo = from, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((uint64_t)P[mid] - pa > bound) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// first_end from a + 1 on for kListStarts starts side by side, none from n - 1 on.
template <typename U>
__device__ __forceinline__ void first_ends(const U *P, const int n, const int (&a)[kListStarts],
                                           const uint64_t (&pa)[kListStarts], const uint64_t bound, int (&x)[kListStarts])
{
    int hi[kListStarts];
#pragma unroll
    for (int j = 0; j < kListStarts; ++j) {
        x[j] = a[j] < n - 1 ? a[j] + 1 : n;
        hi[j] = n;
    }
    for (int step = n; step > 0; step >>= 1) {
#pragma unroll
        for (int j = 0; j < kListStarts; ++j) {
            const int mid = (x[j] + hi[j]) >> 1;
            const bool between = x[j] < hi[j], up = between && (uint64_t)P[mid] - pa[j] <= bound;
            hi[j] = between && !up ? mid : hi[j];
            x[j] = up ? mid + 1 : x[j];
        }
    }
}

// The budgets of start a inside the intervals (which ascend) go on the list until it holds `most`.
template <typename U>
__device__ __forceinline__ void list_start(const LongWs &w, LongMeta *meta, const Open *open, const int count,
                                           const int most, const int64_t c, const int n, const int a)
{
    const U *P = (const U *)((const uint64_t *)w.P + c * (n + 1));
    const int slots = seen_slots(n);
    const uint64_t pa = P[a];
    int x = a + 1;
    for (int k = 0; k < count && x < n; ++k) {
        const uint64_t lo = (uint64_t)open[k].lo, hi = (uint64_t)open[k].hi;
        if ((uint64_t)P[x] - pa <= lo) x = first_end(P, x + 1, n, pa, lo);
        for (; x < n; ++x) {
            const uint64_t sv = (uint64_t)P[x] - pa;
            if (sv > hi) break;
            // (sv > 0: it lies above an interval's lower end; an empty slot is 0)
            unsigned slot = (unsigned)((sv * 0x9E3779B97F4A7C15ull) >> 54) % slots;
            bool fresh = true;
            for (int probe = 0; probe < 8; ++probe, slot = (slot + 1) % slots) {
                const uint64_t was = atomicCAS((unsigned long long *)w.seen + c * slots + slot, 0ull,
                                               (unsigned long long)sv);
                if (was == sv) fresh = false;
                if (was == sv || was == 0) break;
            }
            if (!fresh) continue;
            const int at = atomicAdd(&meta->listed, 1);
            if (at >= most) return;
            w.list[c * long_budgets(n) + at] = (uint32_t)a << 13 | (uint32_t)x;
        }
    }
}

__device__ inline unsigned mixed(unsigned a, unsigned b)
{
    unsigned h = a * 0x9E3779B1u ^ b * 0x85EBCA77u;
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    return h ^ h >> 13;
}

// As many budgets as `points` drawn from those inside the intervals, the first of them the largest that is a single
// layer: where that outweighs the others, it gives the cost that settles all smaller ones.
template <typename U>
__device__ __forceinline__ void draw_budgets(const LongWs &w, ListLds &l, const Open *open, const int count,
                                                 const int64_t c, const int n, const int points, const unsigned pass)
{
    const U *P = (const U *)((const uint64_t *)w.P + c * (n + 1));
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave, threads = blockDim.x;
    // every thread keeps one of its own, each as likely as any other
    unsigned mine = 0;   // (below 2^25 in all)
    int at_a = 0, at_x = 0;
    uint64_t single = 0;
    if (tid == 0) l.single = 0;
    __syncthreads();
    for (int a0 = tid; a0 < n - 1; a0 += kListStarts * threads) {
        int a[kListStarts];
        uint64_t pa[kListStarts];
#pragma unroll
        for (int j = 0; j < kListStarts; ++j) {
            a[j] = min(a0 + j * threads, n);
            pa[j] = P[a[j]];
        }
        for (int k = 0; k < count; ++k) {
            const uint64_t lo = (uint64_t)open[k].lo, hi = (uint64_t)open[k].hi;
            int from[kListStarts], to[kListStarts];
            first_ends(P, n, a, pa, lo, from);
            first_ends(P, n, a, pa, hi, to);
#pragma unroll
            for (int j = 0; j < kListStarts; ++j) {
                const unsigned here = (unsigned)(to[j] - from[j]);
                if (here == 0) continue;
                mine += here;
                const uint64_t one = (uint64_t)P[a[j] + 1] - pa[j];
                if (one > lo && one <= hi && one > single) single = one;
                const unsigned r = mixed((unsigned)a[j] * 131u + (unsigned)k, pass);
                if (r % mine < here) {
                    at_a = a[j];
                    at_x = from[j] + (int)(mixed(r, pass) % here);
                }
            }
        }
    }
    unsigned incl = mine;
#pragma unroll
    for (int k = 1; k < kWave; k <<= 1) {
        const unsigned o = __shfl_up(incl, k, kWave);
        if (lane >= k) incl += o;
    }
    if (lane == kWave - 1) l.sum[wave] = incl;
    single = ~wave_min_u64(~single);
    if (lane == 0) atomicMax(&l.single, (unsigned long long)single);
    if (tid < kListWaves) l.drawn[tid] = -1;
    __syncthreads();
    unsigned before = incl - mine, all = 0;
    for (int k = 0; k < threads / kWave; ++k) {
        before += k < wave ? l.sum[k] : 0;
        all += l.sum[k];
    }
    // point k: the budget of the thread that holds number k * all / points and a bit
    const bool has_single = l.single != 0 && (points > 1 || pass % 2 == 0);
    const unsigned part = all / (unsigned)points;
    for (int k = 0; k < points && mine != 0; ++k) {
        const unsigned r = (unsigned)((uint64_t)all * (unsigned)k / (unsigned)points) +
                           (part ? mixed(pass, (unsigned)k) % part : 0);
        if (k == 0 && has_single) continue;
        if (r >= before && r - before < mine) l.drawn[k] = (int64_t)((uint64_t)P[at_x] - (uint64_t)P[at_a]);
    }
    if (tid == 0 && has_single) l.drawn[0] = (int64_t)l.single;
    __syncthreads();
}

// Cuts the intervals at up to `points` of the budgets that are left.  (By the whole workgroup.)
template <typename U>
__device__ __forceinline__ void cut_at_budgets(const LongWs &w, ListLds &l, LongMeta *meta, const Open *open, Open *out,
                                               const int64_t c, const int n, const int points, const unsigned pass)
{
    const int tid = threadIdx.x, lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), count = l.count;
    draw_budgets<U>(w, l, open, count, c, n, points, pass);
    if (tid < points) {
        const int64_t mine = l.drawn[tid];
        int rank = 0;
        for (int k = 0; k < points; ++k) rank += l.drawn[k] < mine || (l.drawn[k] == mine && k < tid);
        l.s[rank] = mine;
    }
    __syncthreads();
    if (wave < points) {
        // (the same one twice, or none: left out)
        const int64_t s = uniform_lane((int64_t)l.s[wave], 0);
        const int64_t below = wave > 0 ? uniform_lane((int64_t)l.s[wave - 1], 0) : -1;
        uint64_t v = ~0ull;
        bool exact = false;
        if (s > 0 && s != below) {
            int64_t prev = below;
            for (int k = 0; k < count; ++k)
                if (open[k].lo < s && open[k].lo > prev) prev = open[k].lo;
            prev = uniform_lane(prev, 0);
            v = long_cost<U, false>(w, meta, c, n, prev, s, exact, nullptr, (U *)(search_lds + wave * long_f_bytes(n)));
            if (exact && lane == 0) atomicMin((unsigned long long *)&meta->ub, (unsigned long long)(v + (uint64_t)s));
        }
        if (lane == 0) {
            l.c[wave] = v;
            l.exact[wave] = exact ? 1 : 0;
        }
    }
    __syncthreads();
    if (tid == 0) {
        uint64_t bc = meta->best_cost, bs = meta->best_s;
        for (int k = 0; k < points; ++k) {
            const uint64_t cost = l.c[k] + (uint64_t)l.s[k];
            if (l.exact[k] && (cost < bc || (cost == bc && (uint64_t)l.s[k] < bs))) {
                bc = cost;
                bs = (uint64_t)l.s[k];
            }
        }
        meta->best_cost = bc;
        meta->best_s = bs;
        const uint64_t known = shared_load(&meta->ub), ub = known < bc ? known : bc;
        int kept = 0, k = 0;
        auto keep = [&](const int64_t lo, const int64_t last, const uint64_t at_least) {
            if (at_least > ub) return;
            const int64_t hi = last < (int64_t)(ub - at_least) ? last : (int64_t)(ub - at_least);
            if (hi <= lo) return;
            if (kept < kOpenMax) {
                out[kept++] = Open{lo, hi, at_least, 0, 0};
            } else {  // (joined with the last)
                Open &o = out[kOpenMax - 1];
                o.hi = hi;
                o.c = at_least < o.c ? at_least : o.c;
            }
        };
        for (int i = 0; i < count; ++i) {
            int64_t lo = open[i].lo;
            for (; k < points && l.s[k] <= open[i].hi; ++k) {
                if (l.s[k] <= lo || (k > 0 && l.s[k] == l.s[k - 1])) continue;
                keep(lo, l.exact[k] ? l.s[k] - 1 : l.s[k], l.c[k]);
                lo = l.s[k];
            }
            keep(lo, open[i].hi, open[i].c);
        }
        l.count = kept;
        __hip_atomic_store(&meta->listed, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int k = tid; k < seen_slots(n); k += (int)blockDim.x)
        __hip_atomic_store(w.seen + c * seen_slots(n) + k, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
}

// The list, and with CUT what has to be done about one that is too long.  LISTED: an earlier launch has made it.
template <typename U, bool LISTED, bool CUT>
__device__ __forceinline__ void list_budgets(const LongWs &w, ListLds &l, LongMeta *meta, const int64_t c, const int n,
                                             const int points, const int most)
{
    for (unsigned pass = 0;; ++pass) {
        const Open *open = l.open[pass & 1];
        const bool last = pass == kListPasses;
        if (!LISTED || pass > 0)
            for (int a = (int)(blockIdx.x * blockDim.x + threadIdx.x); a < n - 1; a += (int)(gridDim.x * blockDim.x))
                list_start<U>(w, meta, open, l.count, last ? INT32_MAX : most, c, n, a);
        if (!CUT) return;
        __syncthreads();
        if (shared_load(&meta->listed) <= most || last) return;
        cut_at_budgets<U>(w, l, meta, open, l.open[~pass & 1], c, n, points, pass);
    }
}

// Up to kListMost layers one launch does both; longer chains are listed by several workgroups, and a launch of one
// workgroup a chain follows, which has nothing to do as a rule (a workgroup alone lists 4,096 starts 7 us slower).
template <bool LISTED, bool CUT>
__global__ __launch_bounds__(kListMost) void search_list_kernel(int n, int points, int most, LongWs w)
{
    __shared__ ListLds l;
    const int64_t c = blockIdx.y;
    LongMeta *meta = w.meta + c;
    const int count = meta->left;
    if (meta->status != CKPT_OK || count == 0 || (LISTED && meta->listed <= most)) return;
    for (int k = threadIdx.x; k < count; k += (int)blockDim.x) l.open[0][k] = w.open[(c * 3 + 2) * kOpenMax + k];
    if (threadIdx.x == 0) l.count = count;
    __syncthreads();
    if (meta->narrow) list_budgets<uint32_t, LISTED, CUT>(w, l, meta, c, n, points, most);
    else list_budgets<uint64_t, LISTED, CUT>(w, l, meta, c, n, points, most);
}

// A wave per budget, its set recorded on the way (a pass of its own for the set of the best took
// 143 us at 1,001 layers of a network and 85 at 4,096 aligned ones; recording makes a pass 7 to 20 % longer).  The
// last wave of a chain takes the best point of the rounds besides: its set is not known yet.
__global__ __launch_bounds__(kWave) void search_finish_kernel(int n, LongWs w)
{
    const int64_t c = blockIdx.y;
    LongMeta *meta = w.meta + c;
    if (meta->status != CKPT_OK) return;
    const int lane = threadIdx.x, words = n / kWave + 1;
    uint16_t *const head = (uint16_t *)(search_lds + long_f_bytes(n));
    uint64_t *const mine = w.found + (c * gridDim.x + blockIdx.x) * 2;
    uint64_t *const set = w.set + (c * gridDim.x + blockIdx.x) * words;
    uint64_t cost = ~0ull, at = ~0ull;
    const int listed = meta->listed, more = meta->best_cost != ~0ull ? 1 : 0;
    for (int item = blockIdx.x; item < listed + more; item += gridDim.x) {
        uint64_t s = meta->best_s;
        if (item < listed) {
            const uint32_t both = w.list[c * long_budgets(n) + item];
            const int a = (int)(both >> 13), x = (int)(both & 8191u);
            const uint64_t *P64 = (const uint64_t *)w.P + c * (n + 1);
            const uint32_t *P32 = (const uint32_t *)P64;
            s = meta->narrow ? (uint64_t)(P32[x] - P32[a]) : P64[x] - P64[a];
        }
        bool exact, ties = false;
        const int64_t at_s = (int64_t)s;
        const uint64_t v =
            meta->narrow
                ? long_cost<uint32_t, true>(w, meta, c, n, at_s - 1, at_s, exact, head, (uint32_t *)search_lds, &ties)
                : long_cost<uint64_t, true>(w, meta, c, n, at_s - 1, at_s, exact, head, (uint64_t *)search_lds, &ties);
        if (!exact || v + s > cost || (v + s == cost && s > at)) continue;
        uint64_t known = 0;
        if (lane == 0) known = atomicMin((unsigned long long *)&meta->ub, (unsigned long long)(v + s));
        known = uniform_lane_u(known, 0);
        if (v + s > known) continue;
        cost = v + s;
        at = s;
        // The set, from n back to 0, 64 positions at a time: their predecessors in the lanes, one after the other.
        __syncthreads();
        int cur = n;
        for (int word = words - 1; word >= 0; --word) {
            const int b = word * kWave, pred = head[b + lane <= n ? b + lane : n];
            uint64_t bits = 0;
            while (cur >= b) {
                bits |= 1ull << (cur - b);
                const int j = cur;
                cur = cur == 0 ? -1 : __builtin_amdgcn_readlane(pred, cur - b);
                if (ties && cur > 0) {
                    const uint64_t *P64 = (const uint64_t *)w.P + c * (n + 1);
                    cur = meta->narrow
                              ? first_pred((const uint32_t *)P64, (const uint32_t *)search_lds, (uint32_t)s, j, cur)
                              : first_pred(P64, (const uint64_t *)search_lds, s, j, cur);
                }
            }
            if (lane == 0) set[word] = bits;
        }
        if (lane == 0) {
            mine[0] = cost;
            mine[1] = at;
        }
        __syncthreads();
    }
}

// ---- results ----

constexpr int kResultThreads = 256;
__global__ __launch_bounds__(kResultThreads) void search_result_kernel(int n, int waves, int64_t cstride, int64_t pstride,
                                                                     uint8_t *__restrict__ mask_out,
                                                                     int64_t *__restrict__ peak_out,
                                                                     int64_t *__restrict__ budget_out,
                                                                     int32_t *__restrict__ status_out, LongWs w)
{
    const int64_t c = blockIdx.x;
    const int tid = threadIdx.x, lane = tid % kWave;
    const LongMeta m = w.meta[c];
    uint8_t *mp = mask_out + c * cstride;
    // (each wave by itself: the smallest cost, of those the smallest s, and a wave of the finish that found it; what
    // the table left in `found` of a bad chain is not looked at)
    uint64_t cost = ~0ull, at = ~0ull;
    int by = 0;
    for (int k = lane; k < waves; k += kWave) {
        const uint64_t fc = w.found[(c * waves + k) * 2], fs = w.found[(c * waves + k) * 2 + 1];
        if (fc < cost || (fc == cost && fs < at)) {
            cost = fc;
            at = fs;
            by = k;
        }
    }
    const uint64_t best = wave_min_u64(cost), s = wave_min_u64(cost == best ? at : ~0ull);
    by = (int)wave_min_u32(cost == best && at == s ? (uint32_t)by : ~0u);
    // (a checked chain has a best point; if there is none all the same, no set has been written)
    const int32_t status = m.status == CKPT_OK && best == ~0ull ? CKPT_ERR_DEVICE : m.status;
    if (tid == 0 && status_out) status_out[c] = status;
    if (status != CKPT_OK) {
        for (int k = tid; k <= n; k += kResultThreads) mp[(int64_t)k * pstride] = 0;
        if (tid == 0) {
            peak_out[c] = -1;
            if (budget_out) budget_out[c] = -1;
        }
        return;
    }
    const uint64_t *set = w.set + (c * waves + by) * (n / kWave + 1);
    for (int k = tid; k <= n; k += kResultThreads)
        mp[(int64_t)k * pstride] = (uint8_t)((set[k / kWave] >> (k % kWave)) & 1ull);
    if (tid == 0) {
        peak_out[c] = (int64_t)(best * m.unit);
        if (budget_out) budget_out[c] = (int64_t)(s * m.unit);
    }
}

std::atomic<bool> long_lds_raised[kMaxDevices];
constexpr size_t kLongLds = 150 << 10;  // the most that list_waves() takes (F and the heads of the longest chain: 81 KB)

hipError_t raise_long_lds_limit()
{
    return raise_lds_limit(long_lds_raised,
                           {(const void *)search_round_kernel, (const void *)search_list_kernel<false, true>,
                            (const void *)search_list_kernel<true, true>, (const void *)search_finish_kernel},
                           kLongLds);
}

}  // namespace

size_t cubic_search_long_bytes(int64_t batch, int n)
{
    LongWs w;
    return carve_long(nullptr, batch, n, &w);
}

hipError_t launch_cubic_search_long(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                                    int64_t *peak_out, int64_t *budget_out, int32_t *status_out, void *ws,
                                    hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    if (batch > 65535) return hipErrorInvalidConfiguration;
    const int at_once = list_waves(batch, n);
    const size_t f_lds = long_f_bytes(n), set_lds = ((size_t)n + 1 + kWave) * 10, list_lds = at_once * f_lds;
    if (set_lds > kDefaultLdsLimit || list_lds > kDefaultLdsLimit) {
        const hipError_t e = raise_long_lds_limit();
        if (e != hipSuccess) return e;
    }
    LongWs w;
    (void)carve_long(ws, batch, n, &w);
    const int points = long_points(batch, n), waves = finish_waves(batch, n);
    const int most = 2 * waves < seen_slots(n) / 2 ? 2 * waves : seen_slots(n) / 2;
    // Budgets that a second round does not pay for: one for each wave of the finish; half as many where the chains fill the
    // chip, for the round's points take a wave each too, and the finish records sets.  At one and at two budgets a wave
    // instead, 16 unrounded chains of 152 layers 104 and 140 us (87), of 256 105 and 120 (104), 100 of 129 116 and 184 (116);
    // at half, 4 chains of 256 layers of a network 98 (81), one of 256 aligned ones 71 (61).
    const int few_budgets = batch < 8 ? waves : waves / 2;
    const unsigned B = (unsigned)batch;
    hipLaunchKernelGGL(search_table_kernel, dim3(B), dim3(kTableThreads), ((size_t)n + 1) * 4, stream, d, n, st.chain,
                       st.pos, points, waves, w);
    for (int round = 0; round < 2; ++round) {
        hipLaunchKernelGGL(search_round_kernel, dim3((unsigned)points, B), dim3(kWave), f_lds, stream, n, points, round, w);
        hipLaunchKernelGGL(search_close_kernel, dim3(B), dim3(kWave), 0, stream, n, points, few_budgets, round, w);
    }
    const dim3 cutters((unsigned)list_threads(batch, n));
    if (n <= kListMost) {
        hipLaunchKernelGGL((search_list_kernel<false, true>), dim3(1, B), cutters, list_lds, stream, n, at_once, most, w);
    } else {
        hipLaunchKernelGGL((search_list_kernel<false, false>), dim3((unsigned)((n + 255) / 256), B), dim3(256), 0, stream,
                           n, at_once, most, w);
        hipLaunchKernelGGL((search_list_kernel<true, true>), dim3(1, B), cutters, list_lds, stream, n, at_once, most, w);
    }
    hipLaunchKernelGGL(search_finish_kernel, dim3((unsigned)waves, B), dim3(kWave), set_lds, stream, n, w);
    hipLaunchKernelGGL(search_result_kernel, dim3(B), dim3(kResultThreads), 0, stream, n, waves, st.chain, st.pos, mask_out,
                       peak_out, budget_out, status_out, w);
    return hipGetLastError();
}

}  // namespace ckpt
