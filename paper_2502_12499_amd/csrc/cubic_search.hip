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
#include <atomic>
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
// 65,536 chains of 64 layers of unrounded sizes: 1.40 ms, where evaluating all 2,017 budgets of each with
// a queue per lane took 31.2 ms; one chain of 152 layers 88 us (129 us).
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

// F_s(n) for the lane's s, 0 <= s <= UB; in 32 bits values above 2^31 are cut to that.
template <typename U>
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
        l += (int)((I)(x - p0) > w) + (int)((I)(x - p1) > w) + (int)((I)(x - p2) > w);
        bool far = (I)(x - p3) > w;
        l += (int)far;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(far) != 0, 0)) {
            do {
                const U q0 = P[l], q1 = P[l + 1], q2 = P[l + 2], q3 = P[l + 3];
                l += far ? (int)((I)(x - q0) > w) + (int)((I)(x - q1) > w) + (int)((I)(x - q2) > w) +
                               (int)((I)(x - q3) > w)
                         : 0;
                far = far && (I)(x - q3) > w;
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

// The least s + c_s and the smallest s that attains it.  `total`: the sum of all sizes; `bound`: the cost of a feasible set; `span`: no s
// beyond it can be optimal; `ends[q]`: the first x > r with P[x] - P[r] > span, r = q * 64 + lane (n if there is none
// below n); `all`: the sum of the interior layers.
template <typename U>
__device__ __forceinline__ void search_chain(const SearchLds<U> &m, const int n, const uint64_t total, const U bound, const U span,
                                             const int (&ends)[kSearchPer], const int steps, const float all,
                                             U &best_cost, U &best_s)
{
    typedef typename SearchLds<U>::I I;
    const int lane = threadIdx.x;
    const uint64_t below = (1ull << lane) - 1ull;
    // s = 0 makes every layer a checkpoint: `total`, optimal only if no set costs less
    best_cost = total <= bound ? (U)total : std::numeric_limits<U>::max();
    best_s = 0;
    U ub = bound;   // the best cost known
    // the first points cut (0, span] evenly
    I prev = (I)(span >> 6) * lane + (I)(((span & 63) * (U)lane) >> 6);
    I s = (I)(span >> 6) * (lane + 1) + (I)(((span & 63) * (U)(lane + 1)) >> 6);
    bool on = s > prev;
    int count = 0;  // intervals on the stack
    enum { kCut, kListed, kEveryBudget } step = kCut;
    int a = 0, x0 = 1;  // kEveryBudget: the start and the first end to come
    for (;;) {
        const U c = lane_cost<U>(m, n, (U)s);
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

// F_s(n) by a whole wave, head by head.  While the head h stays in the window, F(j) = d_j + F(h) and h is the
// smallest minimal predecessor of j, for all those j at once; when it leaves (cell e), the new head is the
// smallest index with minimal F in the window of e: what enters later is larger than the minimum, and what lies
// before it is larger or gone.  The lanes hold three neighbouring slices of 64 positions in registers and slide
// along the chain: Z, the positions before, A, where the next cells are, and B, whose prefix sums are
// under way; a window that reaches back beyond Z is finished from the values parked in F.
// What bounds it is the chain of dependent instructions of a head (about 50, half of them scalar); a form that
// kept the values in LDS took 1,190 cycles a head, most of it four LDS round trips.
// P: prefix sums, P[n] below 2^31 or 2^63; F: room for n + 1 values; RECORD: head[j], the predecessor of j, is
// written for j = 1..n.
template <typename U, bool RECORD, typename H>
__device__ __forceinline__ U wave_cost(const U *P, const int n, const U s, U *F, H *head)
{
    typedef std::make_signed_t<U> I;
    constexpr U kMax = std::numeric_limits<U>::max();
    const int lane = threadIdx.x % kWave;
    // P at position k, and P[k - 1], what cell k compares (past n: larger than anything, so the cell ends the head)
    auto at = [&](int k) -> U { return P[k < n ? k : n]; };
    auto before = [&](int k) -> U { return k > n ? kMax : P[k > 0 ? k - 1 : 0]; };
    int base = 0;                          // A holds the positions base + lane
    U PZ = 0, FZ = kMax, PA = at(lane), QA = before(lane), PB = at(kWave + lane), QB = before(kWave + lane);
    U FA = PA;                             // (F(0) = P[0] in lane 0)
    int HA = 0;
    int h = 0, t = 1;                      // t: the next cell, relative to base (1..64)
    U fh = uniform_lane_u(PA, 0), Ph = fh;
    for (;;) {
        // the cells from t on, as if h stayed for all of them (a later head overwrites them)
        const uint64_t from = t < kWave ? ~0ull << t : 0ull;
        FA = select_lanes(FA, (PA - QA) + fh, from);
        if (RECORD) HA = (int)select_lanes((uint32_t)HA, (uint32_t)h, from);
        const uint64_t out = __builtin_amdgcn_ballot_w64(QA > Ph + s) & from;
        if (out == 0) {
            // h outlasts A: slide
            F[base + lane] = FA;
            if (RECORD) head[base + lane] = (H)HA;
            base += kWave;
            t = 0;
            PZ = PA; FZ = FA;
            PA = PB; QA = QB;
            PB = at(base + kWave + lane);
            QB = before(base + kWave + lane);
            continue;
        }
        const int e = __ffsll((unsigned long long)out) - 1;  // the first cell that does not see h
        if (base + e > n) {
            if (RECORD && base + lane <= n) head[base + lane] = (H)HA;
            // (t = 0 and cell n the last of the slice before: its value is in Z)
            return n >= base ? uniform_lane_u(FA, n - base) : uniform_lane_u(FZ, kWave - 1);
        }
        // The window of e: P[i] >= P[e - 1] - s, i < e; h and what lies before it are out by themselves.
        const U Pe = uniform_lane_u(QA, e);
        const U low = (I)(Pe - s) > 0 ? Pe - s : 0;
        const uint64_t wa = __builtin_amdgcn_ballot_w64(PA >= low) & ((1ull << e) - 1ull);
        const uint64_t wz = base > 0 ? __builtin_amdgcn_ballot_w64(PZ >= low) : 0ull;
        const U va = select_lanes(kMax, FA, wa), vz = select_lanes(kMax, FZ, wz);
        U mn;
        if constexpr (sizeof(U) == 4) mn = wave_min_u32(va < vz ? va : vz); else mn = wave_min_u64(va < vz ? va : vz);
        const uint64_t ea = __builtin_amdgcn_ballot_w64(FA == mn) & wa;
        const uint64_t ez = __builtin_amdgcn_ballot_w64(FZ == mn) & wz;
        const int sa = __ffsll((unsigned long long)ea) - 1, sz = __ffsll((unsigned long long)ez) - 1;
        const bool in_z = ez != 0;
        const U pa = uniform_lane_u(PA, sa & 63), pz = uniform_lane_u(PZ, sz & 63);
        h = in_z ? base - kWave + sz : base + sa;
        Ph = in_z ? pz : pa;
        fh = mn;
        t = e;
        if ((wz & 1ull) != 0 && base > kWave) {
            // the whole of Z lies in the window: the parked values before it
            for (int top = base - kWave - 1; top >= 0; top -= kWave) {
                const int i = top - lane, ic = i > 0 ? i : 0;
                const U pi = P[ic];
                const uint64_t in = __builtin_amdgcn_ballot_w64(pi >= low) & (top < kWave - 1 ? (2ull << top) - 1ull : ~0ull);
                const U fi = F[ic];
                const U v = select_lanes(kMax, fi, in);
                U m;
                if constexpr (sizeof(U) == 4) m = wave_min_u32(v); else m = wave_min_u64(v);
                if (in != 0 && m <= fh) {
                    fh = m;
                    const int far = 63 - __clzll((unsigned long long)(__builtin_amdgcn_ballot_w64(fi == m) & in));
                    h = top - far;
                    Ph = uniform_lane_u(pi, far);
                }
                if (in != ~0ull) break;
            }
        }
    }
}

template <typename U>
__device__ __forceinline__ void solve_short(const uint64_t (&sum)[kSearchPer], const int n, const int shift,
                                            const uint64_t total, const uint64_t bound, const uint64_t span,
                                            const float all, int64_t &cost,
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
    search_chain<U>(m, n, total, (U)bound, (U)span, ends, steps, all, bc, bs);
    // The canonical set for the budget bs: the heads of one pass over the prefix sums in full (in the room of L1
    // again), then the walk back from n.
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSearchPer; ++q) {
        const int k = q * kWave + lane;
        if (k <= n) full[k] = sum[q] >> shift;
    }
    __syncthreads();
    uint64_t *const F = full + n + 1;
    uint8_t *const head = (uint8_t *)(F + n + kWave);
    static_assert(kSearchMaxLayers <= 256, "a head's position is a byte");
    (void)wave_cost<uint64_t, true>(full, n, (uint64_t)bs, F, head);
    __syncthreads();
    bits = 0;
    for (int j = n;; j = head[j]) {
        if ((j & (kWave - 1)) == lane) bits |= 1u << (j / kWave);
        if (j == 0) break;
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
                                           int32_t *__restrict__ status_out)
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
    // sum(d) + max(d) > INT64_MAX: the high halves alone reach 2^31, or the sum (below 2^64 then) does
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
    const bool ovf = high >= (1ull << 31) || base + mx > (uint64_t)INT64_MAX;
    const int32_t status = __any(bad) ? CKPT_ERR_SIZE : (ovf ? CKPT_ERR_OVERFLOW : CKPT_OK);
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
        const bool narrow = bound < (1ull << 31) - 1 && span + largest < (1ull << 31) &&
                            (kLookahead - 1) * largest < (1ull << 31);
        if (narrow ? !NARROW : !WIDE) return false;
        if (NARROW && narrow)
            solve_short<uint32_t>(sum, n, shift, total, bound, span, (float)all, cost, budget, on);
        else if (WIDE)
            solve_short<uint64_t>(sum, n, shift, total, bound, span, (float)all, cost, budget, on);
    }
    for (int k = lane, q = 0; k <= n; k += kWave, ++q) mp[(int64_t)k * mstride] = (on >> q) & 1u;
    if (lane == 0) {
        *peak_out = cost;
        if (budget_out) *budget_out = budget;
        if (status_out) *status_out = status;
    }
    return true;
}

// Workgroups go to the eight XCDs in turn, and each XCD has its own L2; a wave reads 8 of the 128 bytes of
// a line of a position-major batch.  Within every 512 workgroups the 64 that one XCD receives take
// neighbouring chains.  A bijection on [0, grid).
__device__ inline unsigned xcd_blocked(unsigned b, unsigned grid)
{
    if (b >= grid / 512 * 512) return b;
    return b / 512 * 512 + (b % 8) * 64 + (b / 8) % 64;
}

// Chains whose launch has no LDS for 64-bit arithmetic and that need it.
struct SearchWs {
    int32_t *count;  // [1] (first 256 bytes)
    int32_t *list;   // [batch]
};

__global__ void cubic_search_reset_kernel(SearchWs w) { *w.count = 0; }

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
                                             status_out ? status_out + c : nullptr);
    if (!WIDE && !done && threadIdx.x == 0) w.list[atomicAdd(w.count, 1)] = (int32_t)c;
}

// The listed ones.
__global__ __launch_bounds__(kWave) void cubic_search_wide_kernel(const int64_t *__restrict__ d, int n,
                                                                  int64_t cstride, int64_t pstride,
                                                                  uint8_t *__restrict__ mask_out,
                                                                  int64_t *__restrict__ peak_out,
                                                                  int64_t *__restrict__ budget_out,
                                                                  int32_t *__restrict__ status_out, SearchWs w)
{
    const int count = *w.count;
    for (int item = blockIdx.x; item < count; item += gridDim.x) {
        const int64_t c = w.list[item];
        (void)search_one<false, true>(d + c * cstride, pstride, n, mask_out + c * cstride, pstride, peak_out + c,
                                      budget_out ? budget_out + c : nullptr, status_out ? status_out + c : nullptr);
        __syncthreads();
    }
}

// The chains of a ragged batch that have n_lo .. n_hi layers, each where it lies in the flat array.
template <bool WIDE>
__global__ __launch_bounds__(kWave) void cubic_search_ragged_kernel(const int64_t *__restrict__ d,
                                                                    const int64_t *__restrict__ off, int n_lo, int n_hi,
                                                                    uint8_t *__restrict__ mask_out,
                                                                    int64_t *__restrict__ peak_out,
                                                                    int64_t *__restrict__ budget_out,
                                                                    int32_t *__restrict__ status_out, SearchWs w)
{
    const int64_t c = blockIdx.x, o = off[c], n = off[c + 1] - o - 1;
    if (n < n_lo || n > n_hi) return;
    const bool done = search_one<true, WIDE>(d + o, 1, (int)n, mask_out + o, 1, peak_out + c,
                                             budget_out ? budget_out + c : nullptr,
                                             status_out ? status_out + c : nullptr);
    if (!WIDE && !done && threadIdx.x == 0) w.list[atomicAdd(w.count, 1)] = (int32_t)c;
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
                                      budget_out ? budget_out + c : nullptr, status_out ? status_out + c : nullptr);
        __syncthreads();
    }
}

constexpr int kMaxDevices = 64;
std::atomic<bool> search_lds_raised[kMaxDevices];

// Once per device: the longest of these chains need more dynamic LDS than the default limit.
hipError_t raise_search_lds_limit()
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (search_lds_raised[dev].load(std::memory_order_acquire)) return hipSuccess;
    const int most = (int)search_lds_bytes(kSearchMaxLayers, 8);
    for (const void *f : {(const void *)cubic_search_kernel<true>, (const void *)cubic_search_kernel<false>,
                          (const void *)cubic_search_wide_kernel, (const void *)cubic_search_ragged_kernel<true>,
                          (const void *)cubic_search_ragged_kernel<false>,
                          (const void *)cubic_search_ragged_wide_kernel}) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (e != hipSuccess) return e;
    }
    search_lds_raised[dev].store(true, std::memory_order_release);
    return hipSuccess;
}

// From this many chains on the launch has LDS for 32-bit arithmetic only, twice the waves on a CU, and the
// chains that need 64 bits follow in a second one; fewer chains do not fill the chip either way.
constexpr int64_t kSearchSplitFrom = 1024;
constexpr int kSearchWideBlocks = 1024;

}  // namespace

hipError_t launch_cubic_search(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                               int64_t *peak_out, int64_t *budget_out, int32_t *status_out, void *ws,
                               hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    if (search_lds_bytes(n, 8) > 65536) {
        const hipError_t e = raise_search_lds_limit();
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)batch), block(kWave);
    const SearchWs w{(int32_t *)ws, (int32_t *)((char *)ws + 256)};
    if (batch < kSearchSplitFrom) {
        hipLaunchKernelGGL(cubic_search_kernel<true>, grid, block, search_lds_bytes(n, 8), stream, d, n, st.chain, st.pos,
                           mask_out, peak_out, budget_out, status_out, w);
    } else {
        hipLaunchKernelGGL(cubic_search_reset_kernel, dim3(1), dim3(1), 0, stream, w);
        hipLaunchKernelGGL(cubic_search_kernel<false>, grid, block, search_lds_bytes(n, 4), stream, d, n, st.chain,
                           st.pos, mask_out, peak_out, budget_out, status_out, w);
        hipLaunchKernelGGL(cubic_search_wide_kernel, dim3(kSearchWideBlocks), block, search_lds_bytes(n, 8), stream, d,
                           n, st.chain, st.pos, mask_out, peak_out, budget_out, status_out, w);
    }
    return hipGetLastError();
}

hipError_t launch_cubic_search_ragged(const int64_t *d, const int64_t *offsets_dev, int64_t batch, const int *longest,
                                      uint8_t *mask_out, int64_t *peak_out, int64_t *budget_out, int32_t *status_out,
                                      int32_t *count, int32_t *list, hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    const hipError_t e = raise_search_lds_limit();
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)batch), block(kWave);
    const SearchWs w{count, list};
    const bool wide = batch < kSearchSplitFrom;
    if (!wide) hipLaunchKernelGGL(cubic_search_reset_kernel, dim3(1), dim3(1), 0, stream, w);
    int all = 0;
    for (int k = kSearchClasses - 1; k >= 0; --k) {  // the longest chains first
        const int n = longest[k], below = k > 0 ? search_class_limit(k - 1) + 1 : 1;
        if (n == 0) continue;
        all = all > n ? all : n;
        if (wide)
            hipLaunchKernelGGL(cubic_search_ragged_kernel<true>, grid, block, search_lds_bytes(n, 8), stream, d,
                               offsets_dev, below, n, mask_out, peak_out, budget_out, status_out, w);
        else
            hipLaunchKernelGGL(cubic_search_ragged_kernel<false>, grid, block, search_lds_bytes(n, 4), stream, d,
                               offsets_dev, below, n, mask_out, peak_out, budget_out, status_out, w);
    }
    if (!wide)
        hipLaunchKernelGGL(cubic_search_ragged_wide_kernel, dim3(kSearchWideBlocks), block, search_lds_bytes(all, 8),
                           stream, d, offsets_dev, mask_out, peak_out, budget_out, status_out, w);
    return hipGetLastError();
}

}  // namespace ckpt
