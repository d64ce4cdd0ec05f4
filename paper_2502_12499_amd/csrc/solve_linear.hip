// Linear-time dynamic checkpoint selection (Section 4.2: Equation (TU),
// Lemmas 1-4, Algorithm 6).
//
//   M(n) = d_n,   M(i) = d_i + min_{i<j<=n} max(M(j), U(i,j)),
//   U(i,j) = T(i) - T(j) + R(i,j),  T(k) = sum_{t>k} d_t,  R(i,j) = max_{i<=k<j} d_k.
//
// State per chain while i runs from n-1 down to 0:
//   Q    the monotone queue of Lemma 2 as a stack (pushes and pops happen at
//        the low-index end, the "head"): entries j with M(j) strictly
//        decreasing in j.  An entry keeps M(j) and A(j) = M(j) + T(j), so the
//        crossover test U(i,j) >= M(j) reads T(i) + R(i,j) >= A(j).
//   pt   the crossover entry: the lowest-index entry of Q with U(i,j) >= M(j).
//        U(i,.) increases with j (Lemma 1) and M decreases along Q, so the
//        entries from pt to the far end satisfy the test and the ones between
//        the head and pt do not; since U(i-1,j) > U(i,j) (Lemma 4) pt only
//        moves towards the head, and the entry at pt is never popped because
//        M(i) > U(i,j_pt) >= M(j_pt).  Entries beyond pt are dead.  The
//        minimum of Equation (TU) is at pt (value U(i,j_pt)) or at the entry
//        just before it, the "candidate" (value M); ties go to the lower index.
//   R    the range maximum cannot be undone when j moves left (the paper's
//        "U(i,j') from U(i,j)"), so it is kept exactly in another form: every
//        entry carries G = max of d from its own position up to the next entry
//        towards the far end (fixed when the entry is pushed: the front maximum
//        joined with the G of the entries it replaced), and R(i,j) of an entry
//        is the maximum of d since the head was pushed ("front") joined with
//        the G of the entries above it.  R of the pt entry and of the candidate
//        live in registers (R <- max(R, d_i) each step); the join over the
//        entries above is only taken when pt moves and a new candidate needs
//        its R.  (The general kernel below uses the stack of prefix-maximum
//        records of d_i, d_{i+1}, .. for the same purpose.)
//   nxt  the chosen j for every i; the set is read off by following nxt from 0.
// Every entry enters and leaves each stack once and the pointers move one way
// between pushes, so the work per chain is O(n).
//
// Kernels:
//   ring kernel     one lane per chain, every chain of the batch.  Only the live
//        part of the stack is kept, as a 16-slot ring in LDS laid out
//        [slot][lane].  Values are held as 32-bit multiples of
//        2^sh, sh the number of trailing zero bits common to the sizes read so
//        far (stored values are shifted left when a size with fewer trailing
//        zeros arrives).  nxt(i) - i - 1 is a byte: chains of up to 256 layers
//        keep these bytes in vector registers (the same register for every
//        lane, indexed by the wave-uniform position); longer chains park them in
//        the chain's mask_out slot i.  A final forward sweep turns them into the mask.
//        A lane defers its chain when a ring fills, the values outgrow 30 bits,
//        a step exceeds 255 positions, or a size is not positive: it appends
//        the chain to a list in the workspace, those with large sizes from the list's end if lanes and rows are to
//        share it.
//   rows and waves  few chains, and what the ring kernel leaves of many: four chains to a wave (linear_rows.h) or one
//        (linear_wave.h), in 32-bit integers, doubles or 64-bit integers.  Chains they cannot take either (more than 64
//        entries live) go on a second list.
//   wide kernel     one lane per chain on the first list, where rows do not pay: short and long chains (rows_list_pays),
//        and up to 64 layers those that are many (Deferred): the ring kernel's algorithm in 64-bit arithmetic with plain
//        loops.  What it cannot take goes on the second list, or is done by the wave.
//   list kernel     one wave per chain of the second list (lane 0 works),
//        64-bit values, stacks of full capacity n+1 in LDS (n <= 2047) or in
//        the workspace.  Correct for any input.  (Error statuses are written
//        here and by the form of a wave per chain.)
#include "ckpt_internal.h"
#include "linear_rows.h"
#include "linear_wave.h"

#include <atomic>
#include <type_traits>

namespace ckpt {
namespace {

constexpr int kRing = 16;        // slots per lane in each ring
constexpr int kChunk = 8;        // rows in flight per lane
constexpr int kListBlocks = 1024;

// Whether T(i), or T(i) + d_i + max(d), which bounds M(i) and every U(i,j), is beyond INT64_MAX, T(i+1) and the sizes not
// being so.  (All three together may wrap around 2^64; T + d_i alone does not, and then shows in its top bit.)
__device__ inline bool value_overflows(uint64_t T, int64_t di, int64_t dmax)
{
    const uint64_t two = T + (uint64_t)di, all = two + (uint64_t)dmax;
    return (int64_t)(T | two | all) < 0;
}

constexpr int kLdsStackMaxN = 2047;
constexpr int kWaveMaxLayers = 16383;  // of the wave kernel: 34 KB of LDS

struct LinearWs {
    int32_t *count;   // [3] chains deferred by the ring kernel, without and with a large size (one 64-bit word to a
                      // wave that has both), and chains deferred again by the kernels after it (first 256 bytes)
    int32_t *list;    // [batch] the first; the last from the end backwards
    int32_t *list2;   // [batch] the second
    char *scratch;    // kListBlocks * stack_bytes(n)
    int32_t *list_end;
    bool apart;       // the ring kernel files chains with large sizes from the list's end (where it matters: an atomic for
                      // each end in every wave cost 1,048,576 chains of 4 layers 452 us, 269 without, 64-bit ones 283)
    int lanes_few, lanes_large;  // so many of either kind, and lanes take them
};

// Full-capacity state of one chain: qM, qT, recD (int64), qJ, recK, nxt (int32), padded to 256 bytes.
__host__ __device__ inline size_t stack_bytes(int n) { return (((size_t)n + 1) * 36 + 255) / 256 * 256; }
// In LDS positions are 16-bit, and nxt lies there too: the call that allocates nothing has no room for it elsewhere.
__host__ __device__ inline size_t lds_stack_bytes(int n) { return ((size_t)n + 1) * 30; }

__host__ LinearWs carve_linear(void *ws, int64_t batch, int n)
{
    char *p = (char *)ws;
    LinearWs w;
    w.count = (int32_t *)p; p += 256;
    w.list = (int32_t *)p;  p += align_up((size_t)batch * 4);
    w.list_end = w.list + batch;
    w.apart = false;
    w.lanes_few = w.lanes_large = INT32_MAX;
    w.list2 = (int32_t *)p; p += align_up((size_t)batch * 4);
    w.scratch = p;
    return w;
}

__global__ void linear_reset_kernel(LinearWs w) { w.count[0] = w.count[1] = w.count[2] = 0; }

// The chains that the ring kernel deferred, and the part of them that lanes take and not rows (the limits: lanes_share).
struct Deferred {
    int few, all;       // the first `few` numbers are those without large sizes
    int first, end;     // lanes take these
    const int32_t *list, *list_end;
    __device__ explicit Deferred(const LinearWs &w) : few(w.count[0]), all(few + w.count[1]), list(w.list), list_end(w.list_end)
    {
        const bool these = few >= w.lanes_few, large = all - few >= w.lanes_large;
        first = these ? 0 : few;
        end = large ? all : few;
    }
    __device__ int32_t operator[](int item) const { return item < few ? list[item] : list_end[few - 1 - item]; }
};

// Puts every chain on the first deferred list (layouts the ring kernel does not address).
__global__ void linear_defer_all_kernel(int64_t batch, LinearWs w)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c < batch) w.list[c] = (int32_t)c;
    if (c == 0) w.count[0] = (int32_t)batch;
}

// Largest chain stride (elements) for which 63 strides of 8-byte elements fit a 32-bit offset.
constexpr int64_t kRingMaxChainStride = (int64_t)1 << 22;

// ---------------------------------------------------------------------------
// ring kernel
// ---------------------------------------------------------------------------

// A ring entry is three words, each in a plane of its own laid out [slot][lane]
// (so the 64 lanes of a wave always hit 64 different words of a plane, whatever
// slot each of them is at: no bank conflicts):
//   M    M(j)
//   A    M(j) + T(j)
//   GJ   G << 8 | (j & 255), G = max of d over [j, j'), j' the next entry towards the
//        far end.  A maximum over such words orders by G first, which is all the
//        folds below need; the low byte of j is enough because a step is at most
//        255 positions (checked per chunk), and a byte is what gets stored of it.
constexpr int kPlaneM = 0, kPlaneA = 1, kPlaneGJ = 2, kPlanes = 3;

// LOG_REGS (chains of at most kLogMaxLayers layers): the chosen step of every position is kept as a
// byte in 64 vector registers per lane (two per chunk of eight positions, written and read with a
// wave-uniform register index) instead of being parked in the caller's mask array: nothing but
// the sizes is read and nothing but the mask written.
constexpr int kLogMaxLayers = 256;
typedef uint32_t u32x32 __attribute__((ext_vector_type(32)));

// `block` of `grid`: which 64 chains of the batch the wave takes; `list_base` is added to a
// chain's number when it goes on the deferred list (the place of the batch's first chain among
// all chains of a ragged call, else 0); `ring`: the wave's 12 KB of LDS.
template <bool LOG_REGS>
__device__ __forceinline__ void linear_ring_wave(const int64_t *__restrict__ d, int64_t batch, int n, int64_t cstride,
                                        int64_t pstride, uint8_t *__restrict__ mask_out,
                                        int64_t *__restrict__ peak_out, int32_t *__restrict__ status_out,
                                        const LinearWs &w, const unsigned block, const unsigned grid,
                                        const int64_t list_base, uint32_t (&ring)[kPlanes][kRing][kWave])
{
    // Ring positions are kept pre-multiplied by the byte stride of a slot, so
    // the LDS address of a position is one AND-OR away (the ring is aligned to
    // its own size; the kernel declares it, aligned to 4096 bytes, and hands it in).
    constexpr uint32_t kStep = (uint32_t)(kWave * sizeof(uint32_t));  // bytes from a slot to the next
    constexpr uint32_t kSlotMask = (uint32_t)(kRing - 1) * kStep;
    constexpr uint32_t kPlane = (uint32_t)kRing * kStep;              // bytes from a plane to the next
    constexpr int kA = kPlaneA * (int)(kPlane / 4), kGJ = kPlaneGJ * (int)(kPlane / 4);  // in words
    constexpr uint32_t kNone = 0xffffffffu;  // "no candidate": never passes a test
    static_assert(kPlane == 4096, "plane size and alignment");
    // What the assembly hard-codes: the literal plane offsets 4096 and 8192 of its LDS reads, a
    // ring aligned to a plane so that an address is (position & mask) | lane base, steps and
    // positions that fit the low byte of a GJ word, and lane offsets of the rows that fit 31 bits.
    static_assert(kPlanes == 3 && kRing == 16 && kWave == 64 && kStep == 256, "ring geometry in the assembly");
    static_assert(sizeof(ring) == 3 * 4096 && (kSlotMask & (kStep - 1)) == 0, "ring size and slot mask");
    static_assert(63 * kRingMaxChainStride * 8 < ((int64_t)1 << 31), "32-bit lane offsets");

    const int lane = threadIdx.x;
    const int64_t c0 = (int64_t)xcd_paired_block(block, grid) * kWave;
    const int64_t c = c0 + lane;
    const bool live = c < batch;
    const int64_t cc = live ? c : batch - 1;  // idle lanes shadow the last chain and write nothing
    // Addresses are a wave-uniform base (scalar registers) plus a 32-bit lane offset: the
    // launcher only takes this kernel when 63 chain strides fit 31 bits.
    const char *dbase = (const char *)(d + c0 * cstride);
    uint8_t *mbase = mask_out + c0 * cstride;
    const uint32_t doff = (uint32_t)((cc - c0) * cstride) * 8u;
    const uint32_t moff = (uint32_t)((cc - c0) * cstride);
    // a wave-uniform 64-bit value, moved to scalar registers
    auto scalar = [](uint64_t a) -> uint64_t {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    };
    auto row = [&](int k) -> int64_t {  // k is the same in every lane: the row's base stays scalar
        const int ks = __builtin_amdgcn_readfirstlane(k);
        return *(const int64_t *)(dbase + (int64_t)ks * pstride * 8 + doff);
    };
    uint8_t *mp = mask_out + cc * cstride;
    constexpr uint32_t kLimit = 1u << 30;       // bound on T(i) + d_i + max d, hence on every M(i) and U(i,j)
    constexpr uint32_t kChunkLimit = 1u << 24;  // bound on a single size (it shares a word with a byte of j)

    typedef __attribute__((address_space(3))) uint32_t *LdsPtr;
    const uint32_t lane_base = (uint32_t)(uintptr_t)(LdsPtr)&ring[kPlaneM][0][lane];
    auto entry = [&](uint32_t pos) -> LdsPtr { return (LdsPtr)(uintptr_t)((pos & kSlotMask) | lane_base); };

    const int64_t xn = row(n);
    bool defer = xn <= 0;
    int sh = defer ? 0 : __ffsll((unsigned long long)xn) - 1;
    sh = sh < 31 ? sh : 31;  // so that a size's low word alone says whether it is a multiple of 2^sh
    uint64_t xs = (uint64_t)xn >> sh;
    defer |= xs >= kChunkLimit;

    // Q = {n}: it is the crossover entry (U(i,n) > d_n = M(n) for every i)
    uint32_t hd = 0, pt = 0;                   // ring positions of the head and of the crossover entry
    uint32_t Mhd = (uint32_t)xs, Ghd = 0;      // M and GJ of the head entry
    // (M, GJ) of the three entries under the head, read back after every push so
    // that the steps that follow find them in registers (what lies beyond the
    // crossover entry is never looked at, so it does not matter what they hold there)
    uint32_t M1 = 0, G1 = 0, M2 = 0, G2 = 0, M3 = 0, G3 = 0, M4 = 0, G4 = 0;
    uint32_t Tpt = 0, Jpt = n, Rp = 0;         // crossover entry: T(j), j (only its low byte is kept up), R(i, j)
    uint32_t Jfull = n;                        // its position in full, as of the last chunk check
    uint32_t Mc = kNone, Ac = kNone, Jc = 0, Rc = 0;  // candidate (the entry before pt): M, A, j, R(i, j)
    uint32_t Ti = 0;                           // T(i) / 2^sh
    uint32_t dnext = (uint32_t)xs;             // d_{i+1} / 2^sh
    uint32_t dmax = dnext;                     // a bound on the sizes so far (below twice the largest)
    uint32_t Mi = dnext;
    {
        LdsPtr e = entry(0);
        e[0] = Mhd; e[kA] = Mhd; e[kGJ] = (uint32_t)n & 255u;  // T(n) = 0, nothing beyond n
    }

    // Range and alignment are settled for kChunk rows at a time, before their steps, and a
    // lane that cannot go on is switched off for good (its chain goes on the deferred list):
    // the lanes that run a step hold exact values, which is what ends the loops below and
    // keeps the stack's entries in order.
    // `all` is the OR of the rows (so its trailing zeros are the fewest of theirs and its
    // magnitude bounds each of them; a negative size shows as a huge one), `zero` says that
    // one of them is 0, `ilow` is the lowest position of the chunk.
    auto chunk_check = [&](const uint64_t all, const bool zero, const int ilow) {
        const uint32_t low = (uint32_t)all & ((1u << sh) - 1u);
        if (__builtin_amdgcn_ballot_w64(low != 0) != 0) {
            if (low != 0) {
                // fewer common trailing zeros: rescale everything held so far
                const int tz = __ffs(low) - 1;
                const int k = sh - tz;
                // (and every size held so far, which a G may be, still below 2^24)
                const bool fits = k < 24 && ((Ti + dnext + dmax) >> (30 - k)) == 0 && (dmax >> (24 - k)) == 0;
                defer |= !fits;
                const int kk = fits ? k : 0;
                auto scale_gj = [kk](uint32_t gj) -> uint32_t { return ((gj & ~255u) << kk) | (gj & 255u); };
#pragma unroll
                for (int t = 0; t < kRing; ++t) {
                    LdsPtr e = entry((uint32_t)t * kStep);
                    e[0] <<= kk; e[kA] <<= kk; e[kGJ] = scale_gj(e[kGJ]);
                }
                Mhd <<= kk; Ghd = scale_gj(Ghd); Tpt <<= kk; Rp <<= kk; Rc <<= kk;
                M1 <<= kk; G1 = scale_gj(G1); M2 <<= kk; G2 = scale_gj(G2); M3 <<= kk; G3 = scale_gj(G3);
                M4 <<= kk; G4 = scale_gj(G4);
                Mc = Mc == kNone ? kNone : Mc << kk;
                Ac = Ac == kNone ? kNone : Ac << kk;
                Ti <<= kk; dnext <<= kk; dmax <<= kk;
                sh = tz;
            }
        }
        // sizes positive and below 2^24, T(i) + d + max d below 2^30 now: no sum of this chunk wraps
        const uint64_t scaled = all >> sh;
        defer |= zero | (scaled >= kChunkLimit);
        dmax = (uint32_t)scaled > dmax ? (uint32_t)scaled : dmax;
        defer |= (Ti + dnext + dmax) >= kLimit;
        // The crossover entry's position in full from its low byte: it has not moved up since the
        // last check and lies above the last chunk's lowest position, fewer than 256 places in all.
        // Every step of this chunk is at most j_pt - i - 1 of its lowest position: one byte holds it.
        Jfull -= (Jfull - Jpt) & 255u;
        defer |= (Jfull - (uint32_t)ilow) > 248u;
    };

    uint32_t large = 0;            // the sizes' upper halves together
    u32x32 logA = {}, logB = {};   // LOG_REGS: the steps of chunk k as bytes of logA[k] (u = 0..3) and logB[k] (u = 4..7)
    uint32_t acc0 = 0, acc1 = 0;   // ... of the chunk under way
    // One step of the recurrence for position i = ihi - u, whose size x is already in a register.
    auto step_fn = [&](const int i, const int64_t x, const int u) {
        const uint32_t di = __builtin_amdgcn_alignbit((uint32_t)((uint64_t)x >> 32), (uint32_t)x, (uint32_t)sh);
        const uint32_t di8 = di << 8;  // as a GJ word
        Ti += dnext;
        Rp = di > Rp ? di : Rp;
        Rc = di > Rc ? di : Rc;

        // Move the crossover towards the head while the candidate satisfies
        // U(i,j) >= M(j).  A new candidate's R is the front maximum joined with the
        // G of the entries above it.  Runs while ANY lane has to move; lanes that
        // are done sit out under the exec mask.  (In assembly: the compiler's
        // lowering of this doubly nested divergent loop is several times longer.)
        {
            uint32_t ad, e, t0;
            uint64_t sv, sv2, sv3;
            asm volatile(
                "Lw_%=:\n\t"
                "v_add_u32 %[t0], %[Ti], %[Rc]\n\t"
                "v_cmp_ge_u32 vcc, %[t0], %[Ac]\n\t"
                "s_cbranch_vccz Lw_done_%=\n\t"
                "s_and_saveexec_b64 %[sv], vcc\n\t"
                "v_add_u32 %[pt], %[step], %[pt]\n\t"
                "v_sub_u32 %[Tpt], %[Ac], %[Mc]\n\t"
                "v_mov_b32 %[Jpt], %[Jc]\n\t"
                "v_mov_b32 %[Rp], %[Rc]\n\t"
                "v_mov_b32 %[Ac], -1\n\t"
                "v_mov_b32 %[Mc], -1\n\t"
                "v_cmp_ne_u32 vcc, %[pt], %[hd]\n\t"
                "s_and_saveexec_b64 %[sv2], vcc\n\t"
                // the new candidate, and its R from the G of the entries above it
                // (as GJ words; the shift at the end takes the byte of j off again):
                // the head's and the three under it are in registers
                "s_mov_b64 %[sv3], exec\n\t"
                "v_add_u32 %[e], %[step], %[pt]\n\t"
                "v_and_or_b32 %[ad], %[e], %[mask], %[lo]\n\t"
                "ds_read_b32 %[Mc], %[ad]\n\t"
                "ds_read_b32 %[Ac], %[ad] offset:4096\n\t"
                "ds_read_b32 %[Jc], %[ad] offset:8192\n\t"
                "v_sub_u32 %[t0], %[hd], %[e]\n\t"
                "v_mov_b32 %[Rc], %[di8]\n\t"
                "v_cmp_le_u32 vcc, %[step], %[t0]\n\t"
                "s_and_b64 exec, exec, vcc\n\t"
                "v_max_u32 %[Rc], %[Rc], %[Ghd]\n\t"
                "v_cmp_le_u32 vcc, 2*%[step], %[t0]\n\t"
                "s_and_b64 exec, exec, vcc\n\t"
                "v_max_u32 %[Rc], %[Rc], %[G1]\n\t"
                "v_cmp_le_u32 vcc, 3*%[step], %[t0]\n\t"
                "s_and_b64 exec, exec, vcc\n\t"
                "v_max_u32 %[Rc], %[Rc], %[G2]\n\t"
                "v_cmp_le_u32 vcc, 4*%[step], %[t0]\n\t"
                "s_and_b64 exec, exec, vcc\n\t"
                "v_max_u32 %[Rc], %[Rc], %[G3]\n\t"
                // more than four entries above it (rare: one test for the whole wave): the rest from the ring
                "v_cmp_le_u32 vcc, 5*%[step], %[t0]\n\t"
                "s_cbranch_vccz Lg_done_%=\n\t"
                "v_subrev_u32 %[e], 3*%[step], %[hd]\n\t"
                "Lg_%=:\n\t"
                "v_subrev_u32 %[e], %[step], %[e]\n\t"
                "v_sub_u32 %[t0], %[e], %[pt]\n\t"
                "v_cmp_lt_u32 vcc, %[step], %[t0]\n\t"
                "s_and_b64 exec, exec, vcc\n\t"
                "s_cbranch_execz Lg_done_%=\n\t"
                "v_and_or_b32 %[ad], %[e], %[mask], %[lo]\n\t"
                "ds_read_b32 %[t0], %[ad] offset:8192\n\t"
                "s_waitcnt lgkmcnt(0)\n\t"
                "v_max_u32 %[Rc], %[Rc], %[t0]\n\t"
                "s_branch Lg_%=\n\t"
                "Lg_done_%=:\n\t"
                "s_mov_b64 exec, %[sv3]\n\t"
                "v_lshrrev_b32 %[Rc], 8, %[Rc]\n\t"
                "s_mov_b64 exec, %[sv2]\n\t"
                "s_waitcnt lgkmcnt(0)\n\t"
                "s_mov_b64 exec, %[sv]\n\t"
                "s_branch Lw_%=\n\t"
                "Lw_done_%=:\n\t"
                : [pt] "+v"(pt), [Tpt] "+v"(Tpt), [Jpt] "+v"(Jpt), [Rp] "+v"(Rp), [Mc] "+v"(Mc), [Ac] "+v"(Ac),
                  [Jc] "+v"(Jc), [Rc] "+v"(Rc), [ad] "=&v"(ad), [e] "=&v"(e), [t0] "=&v"(t0), [sv] "=&s"(sv),
                  [sv2] "=&s"(sv2), [sv3] "=&s"(sv3)
                : [Ti] "v"(Ti), [hd] "v"(hd), [di8] "v"(di8), [Ghd] "v"(Ghd), [G1] "v"(G1), [G2] "v"(G2), [G3] "v"(G3),
                  [lo] "v"(lane_base), [mask] "s"(kSlotMask), [step] "i"(kStep)
                : "vcc", "scc", "memory");  // (s_and_saveexec writes SCC)
        }
        const uint32_t Upt = Ti + Rp - Tpt;  // U(i, j_pt)
        const bool take_cand = Mc <= Upt;    // ties go to the lower index; kNone never wins
        const uint32_t best = take_cand ? Mc : Upt;
        const uint32_t nx = take_cand ? Jc : Jpt;
        Mi = di + best;
        const uint32_t step = nx - (uint32_t)i - 1u;
        // Parked with a store the compiler does not count, so that its waits on the
        // rows fetched ahead stay partial (a counted store would make it wait for
        // everything in flight; an uncounted one can only lengthen a wait).
        if constexpr (LOG_REGS) {
            // the step's low byte into byte u % 4 of the chunk's word (u is a literal once unrolled)
            const uint32_t sel = 0x03020100u ^ ((0x04u ^ (uint32_t)(u & 3)) << (8 * (u & 3)));
            if (u < 4)
                acc0 = __builtin_amdgcn_perm(step, acc0, sel);
            else
                acc1 = __builtin_amdgcn_perm(step, acc1, sel);
        } else if (live) {
            const uint64_t rowbase = scalar((uint64_t)(uintptr_t)(mbase + (int64_t)i * pstride));
            // The compiler may form the scalar base with v_readfirstlane right before this
            // statement; a vector memory instruction must not read such a register within five
            // wait states, and the compiler does not look inside the statement: wait here.
            asm volatile("s_nop 4\n\tglobal_store_byte %0, %1, %2" : : "v"(moff), "v"(step), "s"(rowbase) : "memory");
        }

        // Q: drop the entries that M(i) dominates (never the crossover entry),
        // folding their G into the new entry's, then push i
        uint32_t Gacc = di8;  // a GJ word: only its G part is used
        {
            // up to three drops are decided on the mirrors.  The crossover entry is never
            // dropped, M(i) being above its value, and the tests are nested, so what the
            // mirrors hold beyond it is never looked at.
            const bool p0 = Mhd >= Mi;
            const bool p1 = p0 & (M1 >= Mi);
            const bool p2 = p1 & (M2 >= Mi);
            const bool p3 = p2 & (M3 >= Mi);
            Gacc = p0 ? (Ghd > Gacc ? Ghd : Gacc) : Gacc;
            Gacc = p1 ? (G1 > Gacc ? G1 : Gacc) : Gacc;
            Gacc = p2 ? (G2 > Gacc ? G2 : Gacc) : Gacc;
            hd -= p0 ? kStep : 0u;
            hd -= p1 ? kStep : 0u;
            hd -= p2 ? kStep : 0u;
            if (__builtin_amdgcn_ballot_w64(p3) != 0) {
                // more: the third mirror goes too, and the lanes concerned go on with the fourth (the
                // others fail the first test), then from the ring, one at a time, down to the
                // crossover entry at the latest.
                Gacc = p3 ? (G3 > Gacc ? G3 : Gacc) : Gacc;
                hd -= p3 ? kStep : 0u;
                Mhd = p3 ? M4 : 0u;
                Ghd = G4;
                uint32_t ad;
                uint64_t sv;
                asm volatile(
                    "Lq_%=:\n\t"
                    "v_cmp_ge_u32 vcc, %[Mhd], %[Mi]\n\t"
                    "s_cbranch_vccz Lq_done_%=\n\t"
                    "s_and_saveexec_b64 %[sv], vcc\n\t"
                    "v_max_u32 %[G], %[G], %[Ghd]\n\t"
                    "v_subrev_u32 %[hd], %[step], %[hd]\n\t"
                    "v_and_or_b32 %[ad], %[hd], %[mask], %[lo]\n\t"
                    "ds_read_b32 %[Mhd], %[ad]\n\t"
                    "ds_read_b32 %[Ghd], %[ad] offset:8192\n\t"
                    "s_waitcnt lgkmcnt(0)\n\t"
                    "s_mov_b64 exec, %[sv]\n\t"
                    "s_branch Lq_%=\n\t"
                    "Lq_done_%=:\n\t"
                    : [hd] "+v"(hd), [Mhd] "+v"(Mhd), [Ghd] "+v"(Ghd), [G] "+v"(Gacc), [ad] "=&v"(ad), [sv] "=&s"(sv)
                    : [Mi] "v"(Mi), [lo] "v"(lane_base), [mask] "s"(kSlotMask), [step] "i"(kStep)
                    : "vcc", "scc", "memory");  // (s_and_saveexec writes SCC)
            }
        }
        // a ring that is full keeps its entries: the chain is deferred and the new entry
        // takes the head's slot, so that the lane's stack stays in order for the rest of the chunk
        const bool full = (hd - pt) >= (uint32_t)(kRing - 1) * kStep;
        defer |= full;
        hd += full ? 0u : kStep;
        {
            Gacc = (Gacc & ~255u) | ((uint32_t)i & 255u);
            LdsPtr e = entry(hd);
            e[0] = Mi; e[kA] = Mi + Ti; e[kGJ] = Gacc;
        }
        Mhd = Mi;
        Ghd = Gacc;
        {
            LdsPtr e1 = entry(hd - kStep), e2 = entry(hd - 2 * kStep), e3 = entry(hd - 3 * kStep);
            M1 = e1[0]; G1 = e1[kGJ];
            M2 = e2[0]; G2 = e2[kGJ];
            M3 = e3[0]; G3 = e3[kGJ];
            LdsPtr e4 = entry(hd - 4 * kStep);
            M4 = e4[0]; G4 = e4[kGJ];
        }
        const bool fresh = hd == pt + kStep;  // the new entry is the candidate; R(i', i) starts empty
        Mc = fresh ? Mi : Mc;
        Ac = fresh ? Mi + Ti : Ac;
        Jc = fresh ? (uint32_t)i : Jc;
        Rc = fresh ? 0u : Rc;
        dnext = di;
    };

    // Rows are fetched kChunk positions ahead of their use, so that the HBM
    // latency of a row overlaps the work on the rows before it.
    int64_t rows[kChunk], ahead[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) rows[u] = row(max(n - 1 - u, 0));
    int chunk = 0;
    for (int ihi = n - 1; ihi >= 0; ihi -= kChunk, ++chunk) {
#pragma unroll
        for (int u = 0; u < kChunk; ++u)  // rows below 0 re-read row 0 and are not used
            ahead[u] = row(max(ihi - kChunk - u, 0));
        uint64_t all = 0;
        bool zero = false;
#pragma unroll
        for (int u = 0; u < kChunk; ++u) {
            const uint64_t x = (uint64_t)rows[u];  // a row below 0 holds row 0 again: harmless here
            all |= x;
            zero |= x == 0;
        }
        large |= (uint32_t)(all >> 32);
        if (!defer) chunk_check(all, zero, max(ihi - kChunk + 1, 0));
        if (!defer) {
#pragma unroll
            for (int u = 0; u < kChunk; ++u)
                if (ihi - u >= 0) step_fn(ihi - u, rows[u], u);
            if constexpr (LOG_REGS) {
                const int k = __builtin_amdgcn_readfirstlane(chunk);
                logA[k] = acc0;
                logB[k] = acc1;
                acc0 = 0;
                acc1 = 0;
            }
        }
#pragma unroll
        for (int u = 0; u < kChunk; ++u) rows[u] = ahead[u];
    }

    const auto results = [&] {
        peak_out[c] = (int64_t)((uint64_t)Mi << sh);
        if (status_out) status_out[c] = CKPT_OK;
        if constexpr (LOG_REGS) {
            // forward sweep over the steps in the registers: position i = n-1 - (8k + u), ascending.
            // Rows are addressed by a scalar base that moves up one row per position, plus the lane's
            // offset; only the first chunk taken (the last one filled) can reach below position 0.
            int cur = 0;
            auto sweep_chunk = [&](const int ks, const bool guarded) {
                const uint32_t w0 = logA[ks], w1 = logB[ks];
                const int ilow = n - 1 - (kChunk * ks + kChunk - 1);  // the chunk's lowest position (below 0 if guarded)
                uint8_t *rowp = mbase + (int64_t)ilow * pstride;      // wave-uniform; one row up per position
#pragma unroll
                for (int u = kChunk - 1; u >= 0; --u, rowp += pstride) {
                    const int i = ilow + (kChunk - 1 - u);
                    if (guarded && i < 0) continue;
                    const uint32_t step = ((u < 4 ? w0 : w1) >> (8 * (u & 3))) & 255u;
                    const bool on = i == cur;
                    cur = on ? i + 1 + (int)step : cur;
                    rowp[moff] = on ? 1 : 0;
                }
            };
            int k = chunk - 1;
            if (k >= 0) sweep_chunk(__builtin_amdgcn_readfirstlane(k), true);
            for (--k; k >= 0; --k) sweep_chunk(__builtin_amdgcn_readfirstlane(k), false);
            mp[(int64_t)n * pstride] = 1;
            return;
        }
        // forward sweep: replace the parked steps by the mask (once they have all landed)
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        int cur = 0;
        constexpr int kSweep = 32;  // rows in flight per lane in this sweep, which does nothing but wait for them
        for (int k0 = 0; k0 <= n; k0 += kSweep) {
            uint8_t b[kSweep];
#pragma unroll
            for (int u = 0; u < kSweep; ++u) b[u] = (k0 + u) <= n ? mp[(int64_t)(k0 + u) * pstride] : 0;
#pragma unroll
            for (int u = 0; u < kSweep; ++u) {
                const int k = k0 + u;
                const bool on = k == cur;
                if (on) cur = k + 1 + b[u];
                b[u] = on ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < kSweep; ++u)
                if ((k0 + u) <= n) mp[(int64_t)(k0 + u) * pstride] = b[u];
        }
    };
    if (live && !defer) results();
    // (after the results: in front of them they wait for the atomic, 172 us instead of 160 for 1,048,576 chains of 16 layers
    // with one in fifty deferred)
    if (!w.apart) {
        if (live && defer) w.list[atomicAdd(w.count, 1)] = (int32_t)(c + list_base);
    } else if (__builtin_amdgcn_ballot_w64(live && defer) != 0) {
        // (about the size from which on a chain of so many layers needs 64 bits: 2^48 of 17, 2^46 of 64)
        const bool file = live && defer, is_large = large >> (__clz(n + 1) - 11) != 0;
        const uint64_t large_ones = __builtin_amdgcn_ballot_w64(file && is_large);
        const uint64_t others = __builtin_amdgcn_ballot_w64(file && !is_large);
        const int first = __builtin_ctzll((unsigned long long)(large_ones | others));
        const int many_large = (int)__popcll((unsigned long long)large_ones), many = (int)__popcll((unsigned long long)others);
        unsigned long long at = 0;
        if (lane == first) {
            if (many_large == 0) at = (uint32_t)atomicAdd(w.count, many);
            else if (many == 0) at = (unsigned long long)atomicAdd(w.count + 1, many_large) << 32;
            else at = atomicAdd((unsigned long long *)w.count, (unsigned long long)many_large << 32 | (unsigned long long)many);
        }
        const int at_other = __builtin_amdgcn_readlane((int)(uint32_t)at, first);
        const int at_large = __builtin_amdgcn_readlane((int)(uint32_t)(at >> 32), first);
        const uint64_t before = (1ull << lane) - 1;
        if (file && is_large) w.list_end[-1 - at_large - (int)__popcll((unsigned long long)(large_ones & before))] = (int32_t)(c + list_base);
        if (file && !is_large) w.list[at_other + (int)__popcll((unsigned long long)(others & before))] = (int32_t)(c + list_base);
    }
}

template <bool LOG_REGS>
__global__ __launch_bounds__(kWave) void linear_ring_kernel(const int64_t *__restrict__ d, int64_t batch, int n,
                                                            int64_t cstride, int64_t pstride,
                                                            uint8_t *__restrict__ mask_out,
                                                            int64_t *__restrict__ peak_out,
                                                            int32_t *__restrict__ status_out, LinearWs w)
{
    __shared__ __attribute__((aligned(4096))) uint32_t ring[kPlanes][kRing][kWave];
    linear_ring_wave<LOG_REGS>(d, batch, n, cstride, pstride, mask_out, peak_out, status_out, w, blockIdx.x,
                               gridDim.x, 0, ring);
}

// ---------------------------------------------------------------------------
// one chain by one wave
// ---------------------------------------------------------------------------

__device__ inline int uniform_bits(int v) { return __builtin_amdgcn_readfirstlane(v); }

// DOUBLES: for values below 2^52 (997 unrounded chains of 1,001 layers 106 us, 124 in 64-bit integers); not where it only
// takes what rows leave, for it costs those registers.
// One chain, its results included; false (with nothing written) if it is left to the list kernel.
template <bool DOUBLES = false>
__device__ __forceinline__ bool wave_chain(const int64_t *__restrict__ dp, const int n, const int64_t pstride,
                                           uint8_t *__restrict__ mp, int64_t *__restrict__ peak_out,
                                           int32_t *__restrict__ status_out, unsigned char *lds)
{
    const int lane = threadIdx.x % kWave;
    // the chain once over: validity, the trailing zeros its sizes share, their sum and largest
    int64_t bits = 0, sum = 0, mx = 0;
    bool bad = false;
    const auto pass = [&](auto in_flight) {
        constexpr int kRows = decltype(in_flight)::value;
        for (int k0 = 0; k0 <= n; k0 += kRows * kWave) {
            int64_t x[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) x[u] = dp[(int64_t)min(k0 + u * kWave + lane, n) * pstride];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                bad |= x[u] <= 0;
                bits |= x[u];
                sum = (int64_t)((uint64_t)sum + (k0 + u * kWave + lane <= n ? (uint64_t)x[u] : 0));
                mx = larger(mx, x[u]);
            }
        }
    };
    // (the hint only says which pass lies out of line: without it one chain of 152 layers 9.3 us instead of 8.9, 997 of
    // 1,001 57.3 instead of 56.2)
    if (__builtin_expect(n < 4 * kWave, 0)) pass(std::integral_constant<int, 4>());
    else pass(std::integral_constant<int, 16>());
    bits = lane_value(bits_up_to(bits), kWave - 1);
    sum = lane_value(sum_up_to(sum), kWave - 1);
    mx = lane_value(max_up_to(mx), kWave - 1);
    int32_t status = __any(bad) ? CKPT_ERR_SIZE : CKPT_OK;
    static_assert(kWaveMaxLayers + 2 <= 1 << 15, "sizes below 2^48 do not overflow");
    if (status == CKPT_OK && (bits >> 48) != 0) {
        int64_t high = 0;
        for (int k = lane; k <= n; k += kWave) high += dp[(int64_t)k * pstride] >> 32;
        high = lane_value(sum_up_to(high), kWave - 1);
        if (chain_overflows((uint64_t)sum, (uint64_t)high, (uint64_t)mx)) status = CKPT_ERR_OVERFLOW;
    }
    uint16_t *const nxt = (uint16_t *)(lds + kQueueBytes);
    int64_t peak = -1;
    if (status == CKPT_OK) {
        const int sh = uniform_bits(__ffsll((unsigned long long)bits) - 1);
        const auto at = [&](int k) -> uint64_t { return (uint64_t)dp[(int64_t)(k > 0 ? k : 0) * pstride] >> sh; };
        bool done;
        const uint64_t most = (uint64_t)(sum + mx) >> sh;
        if (most < (uint64_t)kBeyond<int32_t>) {
            int32_t m0;
            done = wave_steps<int32_t>([&](int k) { return (int32_t)at(k); }, n, lds, nxt, m0);
            peak = (int64_t)m0 << sh;
        } else if (DOUBLES && most < (uint64_t)kBeyond<double>) {
            double m0;
            done = wave_steps<double>([&](int k) { return (double)at(k); }, n, lds, nxt, m0);
            peak = done ? (int64_t)m0 << sh : -1;
        } else {
            uint64_t m0;
            done = wave_steps<uint64_t>([&](int k) { return at(k); }, n, lds, nxt, m0);
            peak = done ? (int64_t)(m0 << sh) : -1;
        }
        if (!done) return false;
    }
    // The set: 64 positions at a time, their steps in the lanes, and from one checkpoint to the next by reading a lane
    // (an LDS read per checkpoint costs three times as much).
    __syncthreads();
    const int none = n + 2 * kWave;
    int cur = status == CKPT_OK ? 0 : none;
    int steps = nxt[min(lane, n - 1)];
    for (int b = 0; b <= n; b += kWave) {
        const int ahead = nxt[min(b + kWave + lane, n - 1)];
        uint64_t set = 0;
        while (cur < b + kWave) {
            set |= 1ull << (cur - b);
            cur = cur == n ? none : __builtin_amdgcn_readlane(steps, cur - b);
        }
        if (b + lane <= n) mp[(int64_t)(b + lane) * pstride] = (uint8_t)((set >> lane) & 1ull);
        steps = ahead;
    }
    if (lane == 0) {
        *peak_out = peak;
        if (status_out) *status_out = status;
    }
    return true;
}

// ---------------------------------------------------------------------------
// wide kernel: one lane per chain deferred by the ring kernel, 64-bit values
// ---------------------------------------------------------------------------

struct alignas(32) WideEntry {
    int64_t M;   // M(j)
    int64_t G;   // max of d over [j, j'), j' the next entry towards the far end
    uint64_t A;  // M(j) + T(j), both of up to 63 bits
    int32_t J;   // j
    int32_t pad;
};

constexpr int kWideBlocks = 2048;
constexpr int kWideRows = 8;  // rows read together

// The ring kernel's algorithm again, in 64-bit arithmetic and with plain loops,
// for the chains whose values did not fit 32 bits there.  The lanes of a wave
// take listed chains and walk i together.  A chain with a size that is not
// positive, with sums beyond 64 bits, with more than kRing live entries or with
// a step beyond 255 positions goes on to the list kernel.
// Five waves fit a CU (32 KB of LDS each), so latency is what bounds it: the rows come eight at a time, a group ahead,
// the queue's two top entries lie in registers, and the sweep at the end reads eight steps together.  (Row by
// row: 167 us at 65,536 chains of 64 layers and 1,175 at 100,000 of 256, now 138 and 955.  The steps in LDS: fewer
// waves fit, 65,536 chains of 130 layers 462 us instead of 260.  32 chains a wave: 2 % faster there, 18 % slower at
// 262,144 chains.)
// With `groups` (a ragged call) a listed number is a chain's place among all chains: its group
// gives the length, where the chain is staged and where its results go, per lane.
constexpr int kLanesLayers = kWave;
// PART: the deferred chains that rows leave to lanes (of at most kLanesLayers layers), and what is left of those by the
// whole wave, chain by chain; else all that are deferred.
template <bool PART>
__global__ __launch_bounds__(kWave) void linear_wide_kernel(const int64_t *__restrict__ d, int n_all,
                                                            int64_t cstride, int64_t pstride_all,
                                                            uint8_t *__restrict__ mask_out,
                                                            int64_t *__restrict__ peak_out,
                                                            int32_t *__restrict__ status_out, LinearWs w,
                                                            const RaggedGroupDev *__restrict__ groups, int n_groups)
{
    __shared__ WideEntry ring[kRing][kWave];
    const int lane = threadIdx.x;
    const Deferred deferred(w);
    const int count = PART ? deferred.end : deferred.all;
    for (int item0 = (PART ? deferred.first : 0) + blockIdx.x * kWave; item0 < count; item0 += gridDim.x * kWave) {
        const bool live = item0 + lane < count;
        const int64_t c = deferred[live ? item0 + lane : count - 1];  // the number results are filed under
        int n = n_all;
        int64_t pstride = pstride_all;
        const int64_t *dp = d + c * cstride;
        uint8_t *mp = mask_out + c * cstride;
        if (groups) {
            const RaggedGroupDev g = groups[ragged_group_of_place(groups, n_groups, c)];
            n = g.n;
            pstride = g.pitch;
            dp = d + g.stage_off + (c - g.first);
            mp = mask_out + g.stage_off + (c - g.first);
        }
        auto at = [&](int pos) -> WideEntry & { return ring[pos & (kRing - 1)][lane]; };

        const int64_t x = dp[(int64_t)n * pstride];
        int64_t rows[kWideRows], ahead[kWideRows];  // sizes i0, i0 - 1, .. and the ones after them
#pragma unroll
        for (int u = 0; u < kWideRows; ++u) {
            const int k = n - 1 - u;
            rows[u] = dp[(int64_t)(k > 0 ? k : 0) * pstride];
        }
        bool out = x <= 0;  // no longer this kernel's chain
        int64_t dmax = x, dnext = x, Mi = x;
        uint64_t T = 0;
        int hd = 0, pt = 0;
        at(0) = WideEntry{x, 0, (uint64_t)x, n, 0};
        int64_t Tpt = 0, Rp = 0;
        int Jpt = n;
        bool has_c = false;
        int64_t Mc = 0, Rc = 0;
        uint64_t Ac = 0;
        int Jc = 0;
        int64_t Mh = x, Gh = 0, M1 = 0, G1 = 0;  // M and G of the entry at hd and of the one before it

        auto step_to = [&](const int i, const int64_t di) {
            out |= di <= 0;
            dmax = di > dmax ? di : dmax;
            T += (uint64_t)dnext;
            dnext = di;
            out |= value_overflows(T, di, dmax);
            if (out) return;
            const int64_t Ti = (int64_t)T;
            Rp = di > Rp ? di : Rp;
            Rc = di > Rc ? di : Rc;
            // the crossover moves towards the head while the candidate satisfies U(i,j) >= M(j)
            while (has_c && (uint64_t)(Ti + Rc) >= Ac) {
                ++pt;
                Tpt = (int64_t)(Ac - (uint64_t)Mc);
                Jpt = Jc;
                Rp = Rc;
                has_c = pt != hd;
                if (has_c) {
                    const WideEntry e = at(pt + 1);
                    Mc = e.M; Ac = e.A; Jc = e.J;
                    Rc = di;  // joined with the G of the entries above the new candidate
                    for (int q = pt + 2; q <= hd; ++q) {
                        const int64_t g = at(q).G;
                        Rc = g > Rc ? g : Rc;
                    }
                }
            }
            const int64_t Upt = Ti + Rp - Tpt;  // U(i, j_pt)
            const bool take = has_c && Mc <= Upt;  // ties go to the lower index
            Mi = di + (take ? Mc : Upt);
            const int step = (take ? Jc : Jpt) - i - 1;
            out |= step > 255;
            if (live) mp[(int64_t)i * pstride] = (uint8_t)step;
            // Q: drop the entries that M(i) dominates (never the crossover entry), then push i
            int64_t Gacc = di;
            while (hd > pt && Mh >= Mi) {
                Gacc = Gh > Gacc ? Gh : Gacc;
                --hd;
                Mh = M1;
                Gh = G1;
                const WideEntry &e = at(hd - 1);  // (where hd is pt now it is not looked at)
                M1 = e.M;
                G1 = e.G;
            }
            ++hd;
            out |= hd - pt >= kRing;
            at(hd) = WideEntry{Mi, Gacc, (uint64_t)Mi + T, i, 0};
            M1 = Mh;
            G1 = Gh;
            Mh = Mi;
            Gh = Gacc;
            if (hd == pt + 1) {
                has_c = true;
                Mc = Mi; Ac = (uint64_t)Mi + T; Jc = i; Rc = 0;
            }
        };
        for (int i0 = n - 1; i0 >= 0; i0 -= kWideRows) {
#pragma unroll
            for (int u = 0; u < kWideRows; ++u) {
                const int k = i0 - kWideRows - u;
                ahead[u] = dp[(int64_t)(k > 0 ? k : 0) * pstride];
            }
#pragma unroll
            for (int u = 0; u < kWideRows; ++u) {
                if (i0 - u < 0) break;
                step_to(i0 - u, rows[u]);
            }
#pragma unroll
            for (int u = 0; u < kWideRows; ++u) rows[u] = ahead[u];
        }
        if (PART) {
            for (uint64_t left = __builtin_amdgcn_ballot_w64(live && out); left != 0; left &= left - 1) {
                const int of = __builtin_ctzll((unsigned long long)left);
                const int64_t one = __shfl(c, of, kWave);
                const int its_n = __shfl(n, of, kWave);
                const int64_t its_stride = __shfl(pstride, of, kWave), at_d = __shfl((int64_t)(dp - d), of, kWave);
                static_assert(sizeof(ring) >= kQueueBytes + 2 * (kLanesLayers + 1), "the wave's LDS, none of it in use now");
                __syncthreads();
                (void)wave_chain(d + at_d, its_n, its_stride, mask_out + at_d, peak_out + one,
                                 status_out ? status_out + one : nullptr, (unsigned char *)ring);
            }
            __syncthreads();
        }
        if (!live) continue;
        if (out) {
            if (!PART) w.list2[atomicAdd(w.count + 2, 1)] = (int32_t)c;
            continue;
        }
        peak_out[c] = Mi;
        if (status_out) status_out[c] = CKPT_OK;
        // forward sweep: the parked steps to the mask
        int cur = 0;
        __threadfence_block();
        for (int k0 = 0; k0 <= n; k0 += kWideRows) {
            int step[kWideRows];  // (position n has none: what lies there is not used)
#pragma unroll
            for (int u = 0; u < kWideRows; ++u) step[u] = mp[(int64_t)(k0 + u < n ? k0 + u : n) * pstride];
#pragma unroll
            for (int u = 0; u < kWideRows; ++u) {
                if (k0 + u > n) break;
                const bool on = k0 + u == cur;
                cur = on ? cur + 1 + step[u] : cur;
                mp[(int64_t)(k0 + u) * pstride] = on ? 1 : 0;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// list kernel: one wave per deferred chain, full-capacity stacks, 64-bit
// ---------------------------------------------------------------------------

extern __shared__ __align__(16) unsigned char lin_lds[];

// One chain by one lane: the recurrence with stacks of full capacity.  `base`: room for the stacks and the steps
// of a chain of n_room layers.
template <typename Pos>
__device__ void list_chain(const int64_t *__restrict__ dp, const int n, const int64_t pstride, uint8_t *__restrict__ mp,
                           int64_t *__restrict__ peak_out, int32_t *__restrict__ status_out, char *base, const int n_room)
{
    const size_t n1 = (size_t)n_room + 1;
    int64_t *qM = (int64_t *)base;
    int64_t *qT = qM + n1;
    int64_t *recD = qT + n1;
    Pos *qJ = (Pos *)(recD + n1);
    Pos *recK = qJ + n1;
    Pos *nxt = recK + n1;

    int64_t x = dp[(int64_t)n * pstride];
    bool bad_size = x <= 0;
    bool ovf = false;
    int64_t dmax = x;
    qJ[0] = (Pos)n;
    qM[0] = x;
    qT[0] = 0;
    int hd = 0, pt = 0;    // Q occupies slots 0..hd, crossover at pt
    int top = -1, rp = 0;  // records occupy slots 0..top
    uint64_t T = 0;        // T(i)
    int64_t dnext = x;     // d_{i+1}
    int64_t Mi = x;

    for (int i = n - 1; i >= 0; --i) {
        const int64_t di = dp[(int64_t)i * pstride];
        bad_size |= di <= 0;
        dmax = di > dmax ? di : dmax;
        T += (uint64_t)dnext;
        ovf |= T > (uint64_t)INT64_MAX;
        dnext = di;
        if (bad_size | ovf) continue;  // keep scanning for errors, skip the work
        ovf |= value_overflows(T, di, dmax);
        if (ovf) continue;
        const int64_t Ti = (int64_t)T;

        while (top >= 0 && recD[top] <= di) --top;
        ++top;
        recD[top] = di;
        recK[top] = (Pos)i;
        if (rp > top) rp = top;

        while (pt < hd) {
            const int e = pt + 1;
            const int je = qJ[e];
            int r = rp;
            while (recK[r] >= je) ++r;  // the top record has k = i < je
            if (Ti - qT[e] + recD[r] < qM[e]) break;
            pt = e;
            rp = r;
        }
        int64_t best = Ti - qT[pt] + recD[rp];  // U(i, j_pt)
        int nx = qJ[pt];
        if (pt < hd) {
            const int64_t Mp = qM[pt + 1];
            if (Mp <= best) {
                best = Mp;
                nx = qJ[pt + 1];
            }
        }
        Mi = di + best;
        nxt[i] = (Pos)nx;

        while (hd > pt && qM[hd] >= Mi) --hd;
        ++hd;
        qJ[hd] = (Pos)i;
        qM[hd] = Mi;
        qT[hd] = Ti;
    }
    if (!ovf) ovf = value_overflows(T, dnext, dmax);  // sum(d) + max(d)

    int32_t status = CKPT_OK;
    if (bad_size) status = CKPT_ERR_SIZE;
    else if (ovf) status = CKPT_ERR_OVERFLOW;
    if (status_out) *status_out = status;
    *peak_out = status == CKPT_OK ? Mi : -1;
    if (status != CKPT_OK) {
        for (int k = 0; k <= n; ++k) mp[(int64_t)k * pstride] = 0;
        return;
    }
    int cur = 0;
    for (int k = 0; k <= n; ++k) {
        const bool on = k == cur;
        mp[(int64_t)k * pstride] = on ? 1 : 0;
        if (on && k < n) cur = nxt[k];
    }
}

// n_all: the chains' length, or in a ragged call (`groups` or `off`) the longest one, for which the stacks
// are laid out; a listed number is then a chain's place among all chains, as in the wide kernel, or with `off` the chain
// itself, where it lies in the flat arrays (with strides of 0 and 1).
// flagged: 0, or the number of chains of a batch in which the wave kernel marked those left (w.list[c] != 0).
template <bool LDS_STACKS>
__global__ __launch_bounds__(kWave) void linear_list_kernel(const int64_t *__restrict__ d, int n_all,
                                                            int64_t cstride, int64_t pstride_all,
                                                            uint8_t *__restrict__ mask_out,
                                                            int64_t *__restrict__ peak_out,
                                                            int32_t *__restrict__ status_out, LinearWs w,
                                                            const RaggedGroupDev *__restrict__ groups, int n_groups,
                                                            const int64_t *__restrict__ off, int flagged)
{
    if (threadIdx.x != 0) return;
    const int count = flagged ? flagged : w.count[2];
    typedef std::conditional_t<LDS_STACKS, uint16_t, int32_t> Pos;
    static_assert(kLdsStackMaxN < 65536, "positions in LDS");
    char *const base = LDS_STACKS ? (char *)lin_lds : w.scratch + (size_t)blockIdx.x * stack_bytes(n_all);
    for (int item = blockIdx.x; item < count; item += gridDim.x) {
        if (flagged && w.list[item] == 0) continue;
        const int64_t c = flagged ? item : w.list2[item];
        int n = n_all;
        int64_t pstride = pstride_all;
        const int64_t *dp = d + c * cstride;
        uint8_t *mp = mask_out + c * cstride;
        if (groups) {
            const RaggedGroupDev g = groups[ragged_group_of_place(groups, n_groups, c)];
            n = g.n;
            pstride = g.pitch;
            dp = d + g.stage_off + (c - g.first);
            mp = mask_out + g.stage_off + (c - g.first);
        } else if (off) {
            n = (int)(off[c + 1] - off[c] - 1);
            dp = d + off[c];
            mp = mask_out + off[c];
        }
        list_chain<Pos>(dp, n, pstride, mp, peak_out + c, status_out ? status_out + c : nullptr, base, n_all);
    }
}

// ---------------------------------------------------------------------------
// wave kernel: one wave per chain
// ---------------------------------------------------------------------------

// Every group of a ragged call in one launch: a wave looks up the group its 64 chains belong to
// and solves them where that group is staged, with the step log in registers if the group's
// chains have up to kLogMaxLayers layers (a wave-uniform branch: long and short groups run side by
// side on the chip), or, with PER_CHAIN, one chain of the group as the wave kernel does (ragged_wave_per_chain).
// The last groups, the longest chains, start first.  Results go to the chains' places.
template <bool PER_CHAIN>
__global__ __launch_bounds__(kWave) void linear_ring_ragged_kernel(const int64_t *__restrict__ d_stage,
                                                                   const RaggedGroupDev *__restrict__ groups,
                                                                   int n_groups, uint8_t *__restrict__ mask_stage,
                                                                   int64_t *__restrict__ peak_stage,
                                                                   int32_t *__restrict__ status_stage, LinearWs w)
{
    __shared__ __attribute__((aligned(4096))) uint32_t ring[kPlanes][kRing][kWave];
    const unsigned wave = gridDim.x - 1 - blockIdx.x;
    const RaggedGroupDev g = groups[PER_CHAIN ? ragged_group_of_linear_wave(groups, n_groups, wave)
                                              : ragged_group_of_wave(groups, n_groups, wave)];
    const unsigned waves = (unsigned)((g.count + kWave - 1) / kWave);
    const unsigned block = wave - (unsigned)(PER_CHAIN ? g.linear_first : g.wave_first);
    if (PER_CHAIN && ragged_wave_per_chain(g.n, g.count)) {
        static_assert(sizeof(ring) >= kQueueBytes + 2 * (4095 + 1), "the wave's LDS for the longest of these chains");
        const int64_t at = g.stage_off + block, c = g.first + (int64_t)block;
        const bool done = wave_chain(d_stage + at, g.n, g.pitch, mask_stage + at, peak_stage + c, status_stage + c,
                                     (unsigned char *)ring);
        if (!done && threadIdx.x == 0) w.list2[atomicAdd(w.count + 2, 1)] = (int32_t)c;
    } else if (g.n <= kLogMaxLayers)
        linear_ring_wave<true>(d_stage + g.stage_off, g.count, g.n, 1, g.pitch, mask_stage + g.stage_off,
                               peak_stage + g.first, status_stage + g.first, w, block, waves, g.first, ring);
    else
        linear_ring_wave<false>(d_stage + g.stage_off, g.count, g.n, 1, g.pitch, mask_stage + g.stage_off,
                                peak_stage + g.first, status_stage + g.first, w, block, waves, g.first, ring);
}

// Few chains: a wave each.  A lane-per-chain wave alone on its SIMD takes 640 ns a position, this 40 (32 bits): one chain
// of 152 layers 11 us (23 with a ballot per pointer move of Algorithm 6 and 150 ns a position), 997 of 1,001 layers 59 us
// (157).
// OWN_LIST: a chain of more than 64 live entries is done by list_chain in the same LDS at once; else it is
// marked in w.list and left to linear_list_kernel.
template <bool OWN_LIST>
__global__ __launch_bounds__(kWave) void linear_wave_kernel(const int64_t *__restrict__ d, int n, int64_t cstride,
                                                            int64_t pstride, uint8_t *__restrict__ mask_out,
                                                            int64_t *__restrict__ peak_out,
                                                            int32_t *__restrict__ status_out, LinearWs w)
{
    const int64_t c = blockIdx.x;
    const int64_t *dp = d + c * cstride;
    uint8_t *mp = mask_out + c * cstride;
    int32_t *st = status_out ? status_out + c : nullptr;
    const bool done = wave_chain<true>(dp, n, pstride, mp, peak_out + c, st, lin_lds);
    if (threadIdx.x != 0) return;
    if (OWN_LIST) {
        if (!done) list_chain<uint16_t>(dp, n, pstride, mp, peak_out + c, st, (char *)lin_lds, n);
    } else {
        w.list[c] = done ? 0 : 1;
    }
}

// The four chains of a wave, a row of lanes each (what is passed is a lane's own chain's); false in the rows whose
// chain is left to wave_chain (nothing of it is written).  n_most: at least the longest one's length; lds:
// rows_lds_bytes(n_most).
__device__ __forceinline__ bool rows_chains(const int64_t *__restrict__ dp, const bool is_chain, const int n,
                                            const int n_most, const int64_t pstride, uint8_t *__restrict__ mp, int64_t *__restrict__ peak_out,
                                            int32_t *__restrict__ status_out, unsigned char *lds)
{
    const int lane = threadIdx.x % kWave, l = lane % kRow;
    // the chain once over: validity, the trailing zeros its sizes share, their sum and largest
    constexpr int kLoads = 4;
    int64_t bits = 0, mx = 0;
    uint64_t sum = 0;
    for (int k0 = 0; __builtin_amdgcn_ballot_w64(k0 <= n) != 0; k0 += kLoads * kRow) {
        int64_t x[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) x[u] = dp[(int64_t)min(k0 + u * kRow + l, n) * pstride];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            bits |= x[u] > 0 ? x[u] : INT64_MIN;
            sum += k0 + u * kRow + l <= n ? (uint64_t)x[u] : 0;
            mx = larger(mx, x[u]);
        }
    }
    bits = row_value<kRow - 1>(row_up_to(bits, (int64_t)0, [](int64_t a, int64_t b) { return a | b; }));
    const auto add = [](uint64_t a, uint64_t b) { return a + b; };
    sum = row_value<kRow - 1>(row_up_to(sum, (uint64_t)0, add));
    mx = row_value<kRow - 1>(row_up_to(mx, (int64_t)0, [](int64_t a, int64_t b) { return larger(a, b); }));
    static_assert(kWaveMaxLayers + 2 <= 1 << 15, "sums of sizes below 2^48 stay below 2^63");
    bool fits = bits > 0;  // (a size that is not positive sets the top bit)
    if (__builtin_amdgcn_ballot_w64(bits >> 48 > 0) != 0) {
        uint64_t high = 0;
        for (int k0 = 0; __builtin_amdgcn_ballot_w64(k0 <= n) != 0; k0 += kRow)
            high += k0 + l <= n ? (uint64_t)dp[(int64_t)(k0 + l) * pstride] >> 32 : 0;
        high = row_value<kRow - 1>(row_up_to(high, (uint64_t)0, add));
        fits = fits && !chain_overflows(sum, high, (uint64_t)mx);
    }
    const int sh = __ffsll((unsigned long long)bits) - 1;
    const uint64_t most = (sum + (uint64_t)mx) >> sh;
    const auto at = [&](int k) -> uint64_t { return (uint64_t)dp[(int64_t)(k > 0 ? k : 0) * pstride] >> sh; };
    uint16_t *const nxt = (uint16_t *)(lds + kRowsQueueBytes) + (size_t)(lane / kRow) * (n_most + 1);
    int64_t peak = -1;
    if (__builtin_amdgcn_ballot_w64(fits) != 0) {
        if (__builtin_amdgcn_ballot_w64(fits && most >= kRowBeyond<double>) != 0)
            peak = (int64_t)rows_steps<uint64_t>([&](int k) { return at(k); }, n, lds, nxt);
        else if (__builtin_amdgcn_ballot_w64(fits && most >= kRowBeyond<uint32_t>) != 0)
            peak = (int64_t)rows_steps<double>([&](int k) { return (double)(int64_t)at(k); }, n, lds, nxt);
        else {
            const uint32_t m0 = rows_steps<uint32_t>([&](int k) { return (uint32_t)at(k); }, n, lds, nxt);
            peak = m0 == UINT32_MAX ? -1 : (int64_t)m0;
        }
    }
    const bool done = fits && peak >= 0;
    // the set: from one checkpoint to the next, each step marked where it lies
    static_assert(kWaveMaxLayers < 0x8000, "the mark is a step's top bit");
    __syncthreads();
    for (int cur = done ? 0 : n; __builtin_amdgcn_ballot_w64(cur < n) != 0;) {
        const int step = nxt[cur];
        if (cur < n) {
            if (l == 0) nxt[cur] = (uint16_t)(step | 0x8000);
            cur = step;
        }
    }
    __syncthreads();
    if (done && is_chain) {
        for (int k = l; k <= n; k += kRow) mp[(int64_t)k * pstride] = k == n ? 1 : (uint8_t)(nxt[k] >> 15);
        if (l == 0) {
            *peak_out = peak << sh;
            if (status_out) *status_out = CKPT_OK;
        }
    }
    return done;
}

// Batches between: four chains a wave, what does not fit a row by the whole wave afterwards.
template <bool OWN_LIST>
__global__ __launch_bounds__(kWave, 4) void linear_rows_kernel(const int64_t *__restrict__ d, int64_t batch, int n,
                                                            int64_t cstride, int64_t pstride,
                                                            uint8_t *__restrict__ mask_out,
                                                            int64_t *__restrict__ peak_out,
                                                            int32_t *__restrict__ status_out, LinearWs w)
{
    const int lane = threadIdx.x % kWave, row = lane / kRow;
    const int64_t c0 = (int64_t)xcd_blocked(blockIdx.x, gridDim.x) * kRowsOfWave;
    const bool is_chain = c0 + row < batch;
    const int64_t c = is_chain ? c0 + row : batch - 1;
    const bool done = rows_chains(d + c * cstride, is_chain, n, n, pstride, mask_out + c * cstride, peak_out + c,
                                  status_out ? status_out + c : nullptr, lin_lds);
    if (!OWN_LIST && is_chain && lane % kRow == 0) w.list[c] = 0;
    for (uint64_t left = __builtin_amdgcn_ballot_w64(is_chain && !done && lane % kRow == 0); left != 0; left &= left - 1) {
        const int64_t one = c0 + __builtin_ctzll((unsigned long long)left) / kRow;
        const int64_t *dp = d + one * cstride;
        uint8_t *mp = mask_out + one * cstride;
        int32_t *st = status_out ? status_out + one : nullptr;
        __syncthreads();
        const bool by_wave = wave_chain(dp, n, pstride, mp, peak_out + one, st, lin_lds);
        if (by_wave || lane != 0) continue;
        if (OWN_LIST) list_chain<uint16_t>(dp, n, pstride, mp, peak_out + one, st, (char *)lin_lds, n);
        else w.list[one] = 1;
    }
}

// The chains that the ring kernel left, four to a wave, or a wave each if they are few (a handful that outgrew the ring
// would wait for a row's pace and then for the wave's: 65,537 chains of 2,047 aligned layers 1.68 ms so).  With
// `groups` a listed number is a chain's place among all chains.  What does not fit a row, more than n_rows layers among it,
// is done by the whole wave, what that cannot do goes on the second list.
constexpr unsigned kRowsListBlocks = 4096;  // four waves a SIMD
constexpr int kListedAlone = 1024;
__global__ __launch_bounds__(kWave, 4) void linear_rows_list_kernel(const int64_t *__restrict__ d, int n_all,
                                                                    int64_t cstride, int64_t pstride_all,
                                                                    uint8_t *__restrict__ mask_out,
                                                                    int64_t *__restrict__ peak_out,
                                                                    int32_t *__restrict__ status_out, LinearWs w, int n_rows,
                                                                    const RaggedGroupDev *__restrict__ groups, int n_groups)
{
    const int lane = threadIdx.x % kWave;
    const Deferred deferred(w);
    const int lanes_take = deferred.end - deferred.first, count = deferred.all - lanes_take;
    const auto listed = [&](int64_t item) -> int64_t { return deferred[(int)(item < deferred.first ? item : item + lanes_take)]; };
    // (c the same in the lanes that are to have the chain)
    struct Chain { int64_t at, pstride; int n; };
    const auto chain = [&](int64_t c) -> Chain {
        if (!groups) return {c * cstride, pstride_all, n_all};
        const RaggedGroupDev g = groups[ragged_group_of_place(groups, n_groups, c)];
        return {g.stage_off + (c - g.first), g.pitch, g.n};
    };
    const bool alone = count <= kListedAlone;
    const int per = alone ? 1 : kRowsOfWave;
    for (int64_t first = (int64_t)xcd_blocked(blockIdx.x, gridDim.x) * per; first < count; first += (int64_t)gridDim.x * per) {
        uint64_t left = 1;
        if (!alone) {
            const bool is_chain = first + lane / kRow < count;
            const int64_t c = listed(is_chain ? first + lane / kRow : count - 1);
            const Chain its = chain(c);
            const bool is_row = is_chain && its.n <= n_rows;
            const bool done = rows_chains(d + its.at, is_row, min(its.n, n_rows), n_rows, its.pstride, mask_out + its.at,
                                          peak_out + c, status_out ? status_out + c : nullptr, lin_lds);
            left = __builtin_amdgcn_ballot_w64(is_chain && !(is_row && done) && lane % kRow == 0);
        }
        for (; left != 0; left &= left - 1) {
            const int64_t one = listed(first + __builtin_ctzll((unsigned long long)left) / kRow);
            const Chain at = chain(one);
            __syncthreads();
            const bool by_wave = wave_chain(d + at.at, at.n, at.pstride, mask_out + at.at, peak_out + one,
                                            status_out ? status_out + one : nullptr, lin_lds);
            if (!by_wave && lane == 0) w.list2[atomicAdd(w.count + 2, 1)] = (int32_t)one;
        }
        __syncthreads();
    }
}

// The chains of a ragged batch where they lie in the flat arrays, four to a wave or one, in the order of `perm`, which
// ascends in their lengths; the longest start first.  What is left goes on the second list.  With rows, the `longest`
// longest get a wave each all the same: a row takes 72 ns a position, a wave 40, and a few deep chains are what a call
// waits for (65,536 chains of 15 to 257 layers, sixteen of 1,001 among them: 148 us, 139); and the rows' LDS is that of
// the n_rows layers the others have at most (262,143 chains of 257 layers and one of 4,095: 683 us, 1,614 with LDS for
// that one in every row).
template <bool ROWS>
__global__ __launch_bounds__(kWave, 4) void linear_flat_kernel(const int64_t *__restrict__ d, const int64_t *__restrict__ off,
                                                               const int32_t *__restrict__ perm, int64_t batch, int longest,
                                                               int n_rows,
                                                               uint8_t *__restrict__ mask_out,
                                                               int64_t *__restrict__ peak_out,
                                                               int32_t *__restrict__ status_out, LinearWs w)
{
    const int lane = threadIdx.x % kWave;
    const bool alone = !ROWS || blockIdx.x < (unsigned)longest;
    const int64_t p0 = alone ? batch - 1 - blockIdx.x : (int64_t)(gridDim.x - 1 - blockIdx.x) * kRowsOfWave;
    uint64_t left = 1;
    if (!alone) {
        const int64_t many = batch - longest;
        const bool is_chain = p0 + lane / kRow < many;
        const int64_t c = perm[is_chain ? p0 + lane / kRow : many - 1], o = off[c];
        const bool done = rows_chains(d + o, is_chain, (int)(off[c + 1] - o - 1), n_rows, 1, mask_out + o, peak_out + c,
                                      status_out ? status_out + c : nullptr, lin_lds);
        left = __builtin_amdgcn_ballot_w64(is_chain && !done && lane % kRow == 0);
    }
    for (; left != 0; left &= left - 1) {
        const int64_t c = perm[p0 + __builtin_ctzll((unsigned long long)left) / kRow], o = off[c];
        __syncthreads();
        const bool done = wave_chain<!ROWS>(d + o, (int)(off[c + 1] - o - 1), 1, mask_out + o, peak_out + c,
                                            status_out ? status_out + c : nullptr, lin_lds);
        if (!done && lane == 0) w.list2[atomicAdd(w.count + 2, 1)] = (int32_t)c;
    }
}

// A wave per chain up to 1,024 chains, one for each SIMD of the chip; four chains to a wave up to 65,536, and the ring
// kernel's lanes beyond.  Waves and rows, us: 1,001 layers, 1,024 chains 62 and 79, 2,048 chains 100 and 82, unrounded
// ones 131 and 115, 204 and 121.  Rows and lanes at 65,536 chains: 64 layers 49 and 51 (unrounded, which the lanes try
// in 32 bits first, 55 and 137), 256 layers 154 and 170 (251 and 482), 1,001 layers 610 and 723 (1,004 and 2,950); at
// 131,072 aligned ones 88 and 56 for 64 layers.  The LDS of the steps has to leave a SIMD three waves (four end at 1,023
// layers), or one up to 16,384 chains: 16,384 of 3,000 layers 0.89 ms, 2.0 with lanes, but 65,536 of 2,047 5 % slower than
// those.  Rows take the same time whatever the sizes are; lanes take less where all chains move alike, so 65,536 chains
// whose layers are all of one size are slower by rows: 64 layers 43 us (28 by lanes), 256 138 (84), 1,001 581 (385).
// 16,384 of them are not: 15 (26), 47 (79), 192 (352).
static_assert(kLongest <= 1024, "fewer than the chains of a batch that takes rows");
constexpr int64_t kWaveBatch = 1024, kRowsFewBatch = 16384, kRowsBatch = 65536;
constexpr int kRowsFewMaxLayers = 4095, kRowsMaxLayers = 1279;
inline bool rows_fit(int64_t batch, int n)
{
    return batch > kWaveBatch && (batch <= kRowsFewBatch ? n <= kRowsFewMaxLayers : batch <= kRowsBatch && n <= kRowsMaxLayers);
}
// Rows also take what the ring kernel leaves of larger batches (unrounded sizes: all of it), where that kernel's form
// in 64 bits, a lane per chain, is slower: 131,072 unrounded chains of 64 layers 168 us (267), 262,144 of 1,001 5.6 ms
// (8.8), but of 12 layers 142 us (130) and of 3,000 28.8 ms (27.5).
inline bool rows_list_pays(int64_t batch, int n)
{
    return n > kRow && n <= kRowsFewMaxLayers && (n <= 2047 || batch <= 131072);
}
// A wave per chain where those do not fit.
constexpr int64_t kWaveMaxBatch = 16384;
// LDS for the list's stacks that leaves a CU 16 waves (at 511 layers 134 us for 16,384 chains, 104 without).
constexpr int kRowsOwnListMaxLayers = 320;
constexpr int kOwnListMaxLayers = 2047;  // 60 KB of LDS for the stacks, kept free for a case that hardly happens ...
__host__ inline size_t own_list_lds_bytes(int n) { return std::max(lds_stack_bytes(n), wave_lds_bytes(n)); }
__host__ inline size_t rows_all_lds_bytes(int n, bool own)
{
    return std::max(rows_lds_bytes(n), own ? own_list_lds_bytes(n) : wave_lds_bytes(n));
}
// ... and only where all the waves fit the chip with it (LDS is handed out in units of 1,280 bytes; 997 chains of
// 1,001 layers 59 us, 58 so): in two turns 4,096 chains of 511 layers took 286 us, and take 201 with the list in a
// launch of its own; 2,600 198 and 158.
inline bool own_list(int64_t batch, int n)
{
    const int64_t per_cu = (160 << 10) / (int64_t)align_up(own_list_lds_bytes(n), 1280);
    return n <= kOwnListMaxLayers && batch <= 256 * per_cu;
}

}  // namespace

size_t linear_workspace_bytes(int64_t batch, int n)
{
    return 256 + 2 * align_up((size_t)batch * 4) + (size_t)kListBlocks * stack_bytes(n) + 256;
}

// ---------------------------------------------------------------------------
// the call that allocates nothing: the lists live in an array of the library's own
// ---------------------------------------------------------------------------

// Up to CKPT_NOALLOC_MAX_LAYERS layers the list kernel keeps its stacks in LDS, so the
// scratch is the two counters and the two lists of chain indices only.
constexpr size_t kNoallocScratchBytes = 256 + 2 * ((size_t)CKPT_NOALLOC_MAX_BATCH * 4) + 256;
static_assert(CKPT_NOALLOC_MAX_LAYERS <= kLdsStackMaxN, "the list kernel must not need scratch stacks");

namespace {
// One copy per GPU, at an address of its own on each; held until the process ends.
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

std::atomic<void *> scratch_of_device[kMaxDevices];
}  // namespace

hipError_t launch_solve_linear_noalloc(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                                       int64_t *peak_out, int32_t *status_out, hipStream_t stream)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    // The array's name is a host-side stand-in; its device address is looked up once per
    // device, with that device current (two threads that race here store the same address).
    void *ptr = scratch_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        scratch_of_device[dev].store(ptr, std::memory_order_release);
    }
    return launch_solve_linear(d, batch, n, st, mask_out, peak_out, status_out, ptr, stream);
}

namespace {
void launch_list(const int64_t *d, int n, Strides st, uint8_t *mask_out, int64_t *peak_out, int32_t *status_out,
                 const LinearWs &w, int64_t batch, const RaggedGroupDev *groups, int n_groups, const int64_t *off,
                 int flagged, hipStream_t stream)
{
    const unsigned grid = (unsigned)(batch < kListBlocks ? batch : kListBlocks);
    const bool in_lds = n <= kLdsStackMaxN;
    hipLaunchKernelGGL(in_lds ? linear_list_kernel<true> : linear_list_kernel<false>, dim3(grid), dim3(kWave),
                       in_lds ? lds_stack_bytes(n) : 0, stream, d, n, st.chain, st.pos, mask_out, peak_out, status_out, w,
                       groups, n_groups, off, flagged);
}
// Lanes take part of what the ring kernel deferred, of chains of `mean` layers and of `longest` at most: up to kLanesLayers
// layers those with large sizes, which need 64 bits, up to kLanesFewLayers the others, where there are enough of them.
// Lanes take 1.8 us a position whatever their number, up to 80,000; rows take time in proportion and start better.  Rows
// and lanes, us: 65,537 chains in 64 bits, 17 layers 70 and 50, 24 71 and 63, 32 74 and 79; 131,072 of 32 137 and 122, of
// 48 183 and 171; 1,048,576 of 48 1,357 and 1,310; in doubles 65,537 of 17 60 and 49, of 24 64 and 62, 131,072 of 24 115
// and 114; but one chain in fifty in 64 bits, 65,537 of 24 layers 41 and 65.  In a ragged batch a row takes 16 positions for
// any fewer, and lanes the longest's time: unrounded chains of 2 to 24 layers, 500,000 427 and 379; of 2 to 40, 262,145
// 303 and 329, 1,500,000 1,311 and 1,151; of 2 to 64, 262,145 346 and 465, 700,000 748 and 794, 1,500,000 1,556 and 1,457.
constexpr int kLanesFewLayers = 23, kLanesPerLayer = 1984, kLanesPerLayerMore = 15000;
void lanes_share(LinearWs &w, int64_t batch, int longest, int mean)
{
    w.apart = rows_list_pays(batch, longest) && longest <= kLanesLayers;
    if (!w.apart) return;
    if (mean <= kLanesFewLayers) w.lanes_few = kLanesPerLayer * mean + kLanesPerLayerMore * (longest - mean);
    w.lanes_large = kLanesPerLayer * ((mean + longest) / 2);
}
// What the ring kernel deferred, of at most n layers (n_most: the longest chain of all).
void launch_deferred(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out, int64_t *peak_out,
                     int32_t *status_out, const LinearWs &w, int n_rows, int n_most, const RaggedGroupDev *groups,
                     int n_groups, hipStream_t stream)
{
    const bool rows = rows_list_pays(batch, n), part = w.apart;
    if (rows) {
        const unsigned blocks = (unsigned)std::min<int64_t>((batch + kRowsOfWave - 1) / kRowsOfWave, kRowsListBlocks);
        hipLaunchKernelGGL(linear_rows_list_kernel, dim3(blocks), dim3(kWave),
                           std::max(wave_lds_bytes(n), rows_lds_bytes(n_rows)), stream, d, n, st.chain, st.pos, mask_out,
                           peak_out, status_out, w, n_rows, groups, n_groups);
    }
    if (!rows || part) {
        const unsigned blocks = (unsigned)std::min<int64_t>((batch + kWave - 1) / kWave, kWideBlocks);
        hipLaunchKernelGGL(part ? linear_wide_kernel<true> : linear_wide_kernel<false>, dim3(blocks), dim3(kWave), 0, stream, d,
                           n, st.chain, st.pos, mask_out, peak_out, status_out, w, groups, n_groups);
    }
    // (of so few layers the end of a block never has more than 64 entries live: rows put nothing on the second list either,
    // but a ragged batch's longer chains, which get waves, may be on it)
    if (!part || n_most != n)
        launch_list(d, n_most, st, mask_out, peak_out, status_out, w, batch, groups, n_groups, nullptr, 0, stream);
}
}  // namespace

hipError_t launch_solve_linear(const int64_t *d, int64_t batch, int n, Strides st, uint8_t *mask_out,
                               int64_t *peak_out, int32_t *status_out, void *ws, hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    LinearWs w = carve_linear(ws, batch, n);
    if (rows_fit(batch, n)) {
        const bool own = n <= kRowsOwnListMaxLayers;
        const unsigned rgrid = (unsigned)((batch + kRowsOfWave - 1) / kRowsOfWave);
        hipLaunchKernelGGL(own ? linear_rows_kernel<true> : linear_rows_kernel<false>, dim3(rgrid), dim3(kWave),
                           rows_all_lds_bytes(n, own), stream, d, batch, n, st.chain, st.pos, mask_out, peak_out,
                           status_out, w);
        if (!own) launch_list(d, n, st, mask_out, peak_out, status_out, w, batch, nullptr, 0, nullptr, (int)batch, stream);
        return hipGetLastError();
    }
    if (batch <= kWaveMaxBatch && n <= kWaveMaxLayers) {
        if (own_list(batch, n)) {
            hipLaunchKernelGGL(linear_wave_kernel<true>, dim3((unsigned)batch), dim3(kWave), own_list_lds_bytes(n), stream, d,
                               n, st.chain, st.pos, mask_out, peak_out, status_out, w);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(linear_wave_kernel<false>, dim3((unsigned)batch), dim3(kWave), wave_lds_bytes(n), stream, d, n,
                           st.chain, st.pos, mask_out, peak_out, status_out, w);
        launch_list(d, n, st, mask_out, peak_out, status_out, w, batch, nullptr, 0, nullptr, (int)batch, stream);
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)((batch + kWave - 1) / kWave);
    lanes_share(w, batch, n, n);
    hipLaunchKernelGGL(linear_reset_kernel, dim3(1), dim3(1), 0, stream, w);
    if (st.chain <= kRingMaxChainStride)
        if (n <= kLogMaxLayers)
            hipLaunchKernelGGL(linear_ring_kernel<true>, dim3(grid), dim3(kWave), 0, stream, d, batch, n, st.chain,
                               st.pos, mask_out, peak_out, status_out, w);
        else
            hipLaunchKernelGGL(linear_ring_kernel<false>, dim3(grid), dim3(kWave), 0, stream, d, batch, n, st.chain,
                               st.pos, mask_out, peak_out, status_out, w);
    else
        hipLaunchKernelGGL(linear_defer_all_kernel, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0, stream,
                           batch, w);
    launch_deferred(d, batch, n, st, mask_out, peak_out, status_out, w, n, n, nullptr, 0, stream);
    return hipGetLastError();
}

namespace {
// Of a ragged batch the lanes need a staging and wait for the longest chains of every wave, so rows pay longer:
// 131,072 and 262,144 chains of up to 24 layers 110 and 141 us (125 and 143), of up to 1,001 562 and 1,028 (1,141 and
// 1,616), unrounded 661 and 1,228 (1,042 and 1,962), 65,536 of up to 4,000 0.97 ms (2.4).  At 262,144 short ones the
// two meet.
constexpr int64_t kFlatBatch = 262144;
bool flat_rows(int64_t batch, int n) { return batch > kWaveBatch && batch <= kFlatBatch && n <= kRowsFewMaxLayers; }
}  // namespace

bool linear_takes_flat(int64_t batch, int n)
{
    return flat_rows(batch, n) || (batch <= kWaveMaxBatch && n <= kWaveMaxLayers);
}

hipError_t launch_solve_linear_flat(const int64_t *d, const int64_t *off, const int32_t *perm, int64_t batch,
                                    const RaggedTotals &t, uint8_t *mask_out, int64_t *peak_out, int32_t *status_out,
                                    void *ws, hipStream_t stream)
{
    LinearWs w = carve_linear(ws, batch, t.max_layers);
    const bool rows = flat_rows(batch, t.max_layers), deep = t.deep_chains > kLongest && deep_ones_alone(t);
    const int longest = deep ? t.deep_chains : kLongest, n_rows = deep ? std::min(t.rows_longest, kDeepLayers) : t.rows_longest;
    const int64_t waves = rows ? longest + (batch - longest + kRowsOfWave - 1) / kRowsOfWave : batch;
    const size_t lds = std::max(wave_lds_bytes(t.max_layers), rows ? rows_all_lds_bytes(n_rows, false) : 0);
    hipLaunchKernelGGL(rows ? linear_flat_kernel<true> : linear_flat_kernel<false>, dim3((unsigned)waves), dim3(kWave), lds,
                       stream, d, off, perm, batch, longest, n_rows, mask_out, peak_out, status_out, w);
    launch_list(d, t.max_layers, Strides{0, 1}, mask_out, peak_out, status_out, w, batch, nullptr, 0, off, 0, stream);
    return hipGetLastError();
}

hipError_t launch_solve_linear_ragged(const int64_t *d_stage, const RaggedGroupDev *groups, const RaggedTotals &t,
                                      int64_t batch, uint8_t *mask_stage, int64_t *peak_stage, int32_t *status_stage,
                                      void *ws, hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    const int n_groups = t.n_groups;
    const bool per_chain = ragged_waves_pay(t);
    const int longest = per_chain ? t.lane_longest : t.max_layers;  // of the chains that the lanes may defer
    LinearWs w = carve_linear(ws, batch, t.max_layers);
    lanes_share(w, batch, longest, (int)((t.layers - (per_chain ? t.wave_layers : 0)) / batch));
    hipLaunchKernelGGL(linear_reset_kernel, dim3(1), dim3(1), 0, stream, w);
    hipLaunchKernelGGL(per_chain ? linear_ring_ragged_kernel<true> : linear_ring_ragged_kernel<false>,
                       dim3((unsigned)(per_chain ? t.linear_waves : t.waves)), dim3(kWave), 0, stream, d_stage, groups,
                       n_groups, mask_stage, peak_stage, status_stage, w);
    launch_deferred(d_stage, batch, longest, Strides{1, 0}, mask_stage, peak_stage, status_stage, w,
                    deep_ones_alone(t) ? std::min(longest, kDeepLayers) : longest, t.max_layers, groups, n_groups, stream);
    return hipGetLastError();
}

}  // namespace ckpt
