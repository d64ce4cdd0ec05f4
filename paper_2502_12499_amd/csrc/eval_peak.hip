// Peak memory of a given checkpoint set (Equation (cost), Section 3.1, and
// Equation (memory), Section 4), one lane per chain where the batch fills the
// chip, else the rows of 64 chains divided among the waves of a workgroup.
//
// Either is a single streaming pass: per chain it reads 8(n+1) bytes of
// sizes and (n+1) bytes of mask and writes 8 bytes.  With the position-major
// layout the 64 lanes of a wave read 512 contiguous bytes of sizes and 64 of
// mask per position; the loop is unrolled so that several rows are in flight
// per wave.  All state is a handful of 64-bit registers per lane.
#include "ckpt_internal.h"

namespace ckpt {
namespace {

constexpr int kBlock = 64;
constexpr int kPartWaves = 16, kRaggedWaves = 8;
// Ragged calls of up to this many times 64 chains (a group's last 64 may be fewer) take the parts: two waves a SIMD.
constexpr int64_t kRaggedPartsMax = 2048;
// From here on the inputs cannot be in the memory-side cache (256 MiB) from the call that wrote them, and loads past the
// caches are 1 % faster (2.4 GB: 471 us against 476); below, they lose what is there (235 MB: 53 us against 40).
constexpr int64_t kBypassBytes = 1ll << 30;
// In a ragged call they are faster where the waves hold few chains each (the walk of 3,000 chains of 2 to 4,095 layers,
// 1.4 a wave, 1,408 us past the caches, 1,483 through them; of 30,000, 7 a wave, 2,055 and 2,117) and slower where they
// are full (524,288 of 152 and 257 layers: the call 1,008 us past, 985 through).
constexpr int64_t kRaggedBypassChains = 16;

// The evaluation of chain c of a batch laid out by (cstride, pstride).  OBJ = CKPT_OBJ_BOTH keeps
// the running values of both objectives and writes the dynamic peak `second` values after the
// static one.
// BYPASS: the sizes and masks go past the caches.
template <int OBJ, bool BYPASS>
__device__ __forceinline__ void eval_peak_chain(const int64_t *__restrict__ d, const uint8_t *__restrict__ mask,
                                       int64_t batch, int n, int64_t cstride, int64_t pstride,
                                       int64_t *__restrict__ peak_out, int32_t *__restrict__ status_out,
                                       const int64_t c, const int64_t second)
{
    if (c >= batch) return;
    const int64_t *dp = d + c * cstride;
    const uint8_t *mp = mask + c * cstride;

    // Position 0 is the input: always resident, start of the first segment.
    int64_t x0 = dp[0];
    bool bad_size = x0 <= 0;
    bool bad_mask = mp[0] == 0;
    uint64_t total = (uint64_t)x0;
    bool ovf = false;
    int64_t dmax = x0;

    int64_t ckpt_sum = x0;  // sum of checkpoints seen so far
    int64_t seg_sum = 0;    // sum of non-checkpoints since the last checkpoint
    int64_t seg_max = x0;   // max over d_h..d_{k-1}, h the last checkpoint (Equation (memory))
    int64_t best = 0;       // Equation (cost): largest segment, else Equation (memory): largest m(i)
    int64_t best_dyn = 0;   // the latter when both are wanted
    uint8_t last_mask = 1;
    constexpr bool kStatic = OBJ == CKPT_OBJ_STATIC || OBJ == CKPT_OBJ_BOTH;
    constexpr bool kDynamic = OBJ == CKPT_OBJ_DYNAMIC || OBJ == CKPT_OBJ_BOTH;

#pragma unroll 16
    for (int k = 1; k <= n; ++k) {
        const int64_t x = BYPASS ? __builtin_nontemporal_load(dp + (int64_t)k * pstride) : dp[(int64_t)k * pstride];
        const uint8_t m = BYPASS ? __builtin_nontemporal_load(mp + (int64_t)k * pstride) : mp[(int64_t)k * pstride];
        bad_size |= x <= 0;
        total += (uint64_t)x;
        ovf |= total > (uint64_t)INT64_MAX;
        dmax = x > dmax ? x : dmax;
        last_mask = m;
        if (m) {
            ckpt_sum += x;
            if (kStatic) best = seg_sum > best ? seg_sum : best;
            if (kDynamic) {
                const int64_t mi = ckpt_sum + seg_sum + seg_max;
                if (OBJ == CKPT_OBJ_BOTH)
                    best_dyn = mi > best_dyn ? mi : best_dyn;
                else
                    best = mi > best ? mi : best;
                seg_max = x;
            }
            seg_sum = 0;
        } else {
            seg_sum += x;
            if (kDynamic) seg_max = x > seg_max ? x : seg_max;
        }
    }
    bad_mask |= last_mask == 0;
    ovf |= (total + (uint64_t)dmax) > (uint64_t)INT64_MAX;

    int32_t status = CKPT_OK;
    if (bad_size) status = CKPT_ERR_SIZE;
    else if (ovf) status = CKPT_ERR_OVERFLOW;
    else if (bad_mask) status = CKPT_ERR_MASK;

    int64_t peak = kStatic ? ckpt_sum + best : best;
    peak_out[c] = status == CKPT_OK ? peak : -1;
    if (OBJ == CKPT_OBJ_BOTH) peak_out[second + c] = status == CKPT_OK ? best_dyn : -1;
    if (status_out) status_out[c] = status;
}

template <int OBJ, bool BYPASS>
__global__ __launch_bounds__(kBlock) void eval_peak_kernel(const int64_t *__restrict__ d,
                                                           const uint8_t *__restrict__ mask,
                                                           int64_t batch, int n, int64_t cstride,
                                                           int64_t pstride,
                                                           int64_t *__restrict__ peak_out,
                                                           int32_t *__restrict__ status_out)
{
    const int64_t c = (int64_t)xcd_paired_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    eval_peak_chain<OBJ, BYPASS>(d, mask, batch, n, cstride, pstride, peak_out, status_out, c, batch);
}

// The rows of 64 chains are divided among the waves of a workgroup.  A wave sums its part up as if it began with a
// checkpoint of its own; the parts' summaries meet in LDS, and the first wave joins them.
// What bounds it is the latency of a few loads in a row and the launch: a lane per chain waits for n / 16 of them.
// (in LDS: [word][wave - 1][lane], the flags behind; kBest under Equation (cost) only, what follows it not there)
enum { kTotal, kLargest, kCkpt, kHead, kTail, kHeadMax, kTailMax, kFirst, kBestDyn, kDynamicWords, kBest = kDynamicWords };
constexpr int words_of(int objective)
{
    return objective == CKPT_OBJ_STATIC ? kTail + 2 : objective == CKPT_OBJ_DYNAMIC ? (int)kDynamicWords : kDynamicWords + 1;
}
// Waves per 64 chains (1: the walk): two to four a SIMD while a wave has eight rows or more.  256 layers, the walk against
// the rule: 250,000 chains 178 and 149 us, 120,000 144 and 92, 60,000 127 and 49; 500,000 219 and 289 (4 waves).
// 64 layers: 300,000 49 and 52 (4), 100,000 37 and 25.  1,001 layers: 200,000 641 and 502, 20,000 467 and 90, 997 371
// and 47, one 164 and 23.
int parts_of(int64_t groups, int n)
{
    const int most = groups > 4096 || n < 32 || (groups > 2048 && n < 128) ? 1 : groups > 2048 ? 4 : groups > 256 ? 8 : kPartWaves;
    return most < n / 8 ? most : n / 8 > 1 ? n / 8 : 1;
}
size_t parts_lds_bytes(int objective, int waves) { return (size_t)(waves - 1) * kBlock * (words_of(objective) * 8 + 4); }
extern __shared__ __align__(16) uint64_t peak_parts[];
enum : uint32_t { kHas = 1, kBadSize = 2, kOverflow = 4 };

// The chains chain .. of lane 0 .. 63 (the whole workgroup calls it together); the rest as eval_peak_chain.
template <int OBJ>
__device__ __forceinline__ void eval_peak_parts(const int64_t *__restrict__ d, const uint8_t *__restrict__ mask,
                                                int64_t batch, int n, int64_t cstride, int64_t pstride,
                                                int64_t *__restrict__ peak_out, int32_t *__restrict__ status_out,
                                                const int64_t chain, const int64_t second)
{
    constexpr bool kStatic = OBJ == CKPT_OBJ_STATIC || OBJ == CKPT_OBJ_BOTH;
    constexpr bool kDynamic = OBJ == CKPT_OBJ_DYNAMIC || OBJ == CKPT_OBJ_BOTH;
    const int lane = threadIdx.x % kBlock, waves = blockDim.x / kBlock;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock);
    uint32_t *const flags = (uint32_t *)(peak_parts + words_of(OBJ) * (waves - 1) * kBlock) - kBlock;
    auto word = [&](int field, int w) -> uint64_t & {
        const int at = OBJ == CKPT_OBJ_STATIC && field == kBest ? kTail + 1 : field;
        return peak_parts[(at * (waves - 1) + w - 1) * kBlock + lane];
    };
    const int64_t c = chain < batch ? chain : batch - 1;  // (lanes past the batch repeat the last chain, writing nothing)
    const int64_t *dp = d + c * cstride;
    const uint8_t *mp = mask + c * cstride;
    const int per = (n + waves - 1) / waves, first = 1 + wave * per, end = min(first + per, n + 1);

    const int64_t x0 = dp[0];
    uint64_t total = 0, ckpt = 0, head = 0, seg = 0, best = 0, best_dyn = 0;
    int64_t largest = 0, head_max = 0, seg_max = 0, first_x = 0;
    uint32_t f = 0;
#pragma unroll 16
    for (int k = first; k < end; ++k) {
        const int64_t x = dp[(int64_t)k * pstride];
        const uint8_t m = mp[(int64_t)k * pstride];
        f |= x <= 0 ? kBadSize : 0;
        total += (uint64_t)x;
        f |= total > (uint64_t)INT64_MAX ? kOverflow : 0;
        largest = x > largest ? x : largest;
        if (m) {
            ckpt += (uint64_t)x;
            if (!(f & kHas)) {
                head = seg;
                head_max = seg_max;
                first_x = x;
            } else {
                if (kStatic) best = seg > best ? seg : best;
                if (kDynamic) {
                    const uint64_t mi = ckpt + seg + (uint64_t)seg_max;
                    best_dyn = mi > best_dyn ? mi : best_dyn;
                }
            }
            f |= kHas;
            if (kDynamic) seg_max = x;
            seg = 0;
        } else {
            seg += (uint64_t)x;
            if (kDynamic) seg_max = x > seg_max ? x : seg_max;
        }
    }
    if (wave > 0) {
        word(kTotal, wave) = total;
        word(kLargest, wave) = (uint64_t)largest;
        word(kCkpt, wave) = ckpt;
        word(kHead, wave) = head;
        word(kTail, wave) = seg;
        if (kStatic) word(kBest, wave) = best;
        if (kDynamic) {
            word(kHeadMax, wave) = (uint64_t)head_max;
            word(kTailMax, wave) = (uint64_t)seg_max;
            word(kFirst, wave) = (uint64_t)first_x;
            word(kBestDyn, wave) = best_dyn;
        }
        flags[wave * kBlock + lane] = f;
    }
    __syncthreads();
    if (wave > 0 || chain >= batch) return;

    uint64_t all = (uint64_t)x0, below = (uint64_t)x0, run = 0, peak = 0, peak_dyn = 0;
    int64_t run_max = x0;
    uint32_t seen = x0 <= 0 ? kBadSize : 0;
    largest = x0 > largest ? x0 : largest;
    auto add = [&](const uint32_t pf, const uint64_t ptotal, const int64_t plargest, const uint64_t pckpt,
                   const uint64_t phead, const uint64_t ptail, const uint64_t pbest, const int64_t phead_max,
                   const int64_t ptail_max, const int64_t pfirst, const uint64_t pbest_dyn) {
        all += ptotal;
        seen |= (pf & (kBadSize | kOverflow)) | (all > (uint64_t)INT64_MAX ? kOverflow : 0);
        largest = plargest > largest ? plargest : largest;
        if (pf & kHas) {
            const uint64_t whole = run + phead;
            if (kStatic) {
                peak = whole > peak ? whole : peak;
                peak = pbest > peak ? pbest : peak;
            }
            if (kDynamic) {
                const int64_t most = run_max > phead_max ? run_max : phead_max;
                const uint64_t at_first = below + (uint64_t)pfirst + whole + (uint64_t)most;
                peak_dyn = at_first > peak_dyn ? at_first : peak_dyn;
                if (pbest_dyn != 0) peak_dyn = below + pbest_dyn > peak_dyn ? below + pbest_dyn : peak_dyn;
                run_max = ptail_max;
            }
            run = ptail;
        } else {
            run += ptail;
            if (kDynamic) run_max = ptail_max > run_max ? ptail_max : run_max;
        }
        below += pckpt;
    };
    add(f, total, largest, ckpt, head, seg, best, head_max, seg_max, first_x, best_dyn);
    for (int w = 1; w < waves; ++w)
        add(flags[w * kBlock + lane], word(kTotal, w), (int64_t)word(kLargest, w), word(kCkpt, w), word(kHead, w),
            word(kTail, w), kStatic ? word(kBest, w) : 0, kDynamic ? (int64_t)word(kHeadMax, w) : 0,
            kDynamic ? (int64_t)word(kTailMax, w) : 0, kDynamic ? (int64_t)word(kFirst, w) : 0,
            kDynamic ? word(kBestDyn, w) : 0);
    if (all + (uint64_t)largest > (uint64_t)INT64_MAX) seen |= kOverflow;
    const int32_t status = (seen & kBadSize)                                      ? CKPT_ERR_SIZE
                           : (seen & kOverflow)                                   ? CKPT_ERR_OVERFLOW
                           : (mp[0] == 0 || mp[(int64_t)n * pstride] == 0) ? CKPT_ERR_MASK
                                                                                  : CKPT_OK;
    const int64_t of_static = status == CKPT_OK ? (int64_t)(below + peak) : -1;
    const int64_t of_dynamic = status == CKPT_OK ? (int64_t)peak_dyn : -1;
    peak_out[c] = kStatic ? of_static : of_dynamic;
    if (OBJ == CKPT_OBJ_BOTH) peak_out[second + c] = of_dynamic;
    if (status_out) status_out[c] = status;
}

template <int OBJ>
__global__ __launch_bounds__(kBlock *kPartWaves) void eval_peak_parts_kernel(
    const int64_t *__restrict__ d, const uint8_t *__restrict__ mask, int64_t batch, int n, int64_t cstride,
    int64_t pstride, int64_t *__restrict__ peak_out, int32_t *__restrict__ status_out)
{
    const int64_t chain = (int64_t)xcd_paired_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x % kBlock;
    eval_peak_parts<OBJ>(d, mask, batch, n, cstride, pstride, peak_out, status_out, chain, batch);
}

// Every group of a ragged call in one launch: a workgroup looks up the group its 64 chains belong to
// and evaluates them where that group is staged; results go to the chains' places (with both
// objectives the dynamic peaks `batch` values, the number of chains of all groups, further on).
template <int OBJ, bool PARTS, bool BYPASS = false>
__global__ __launch_bounds__(PARTS ? kBlock * kRaggedWaves : kBlock) void eval_peak_ragged_kernel(
    const int64_t *__restrict__ d_stage, const uint8_t *__restrict__ mask_stage,
    const RaggedGroupDev *__restrict__ groups, int n_groups, int64_t batch, int64_t *__restrict__ peak_stage,
    int32_t *__restrict__ status_stage)
{
    const RaggedGroupDev g = groups[ragged_group_of_wave(groups, n_groups, blockIdx.x)];
    const int64_t c = ((int64_t)blockIdx.x - g.wave_first) * kBlock + threadIdx.x % kBlock;
    if constexpr (PARTS)
        eval_peak_parts<OBJ>(d_stage + g.stage_off, mask_stage + g.stage_off, g.count, g.n, 1, g.pitch,
                             peak_stage + g.first, status_stage + g.first, c, batch);
    else
        eval_peak_chain<OBJ, BYPASS>(d_stage + g.stage_off, mask_stage + g.stage_off, g.count, g.n, 1, g.pitch,
                                     peak_stage + g.first, status_stage + g.first, c, batch);
}

std::atomic<bool> parts_lds_raised[kMaxDevices];

}  // namespace

hipError_t launch_eval_peak(const int64_t *d, const uint8_t *mask, int64_t batch, int n, Strides st,
                            int objective, int64_t *peak_out, int32_t *status_out, hipStream_t stream)
{
    if (batch == 0) return hipSuccess;
    const unsigned grid = (unsigned)((batch + kBlock - 1) / kBlock);
    const int waves = parts_of(grid, n);
    auto parts = [&](auto kernel) -> hipError_t {
        const size_t lds = parts_lds_bytes(objective, waves);
        if (lds > kDefaultLdsLimit) {  // (16 waves with the dynamic objective)
            const hipError_t e = raise_lds_limit(parts_lds_raised,
                                                 {(const void *)eval_peak_parts_kernel<CKPT_OBJ_DYNAMIC>,
                                                  (const void *)eval_peak_parts_kernel<CKPT_OBJ_BOTH>},
                                                 parts_lds_bytes(CKPT_OBJ_BOTH, kPartWaves));
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(waves * kBlock), lds, stream, d, mask, batch, n, st.chain,
                           st.pos, peak_out, status_out);
        return hipGetLastError();
    };
    auto walk = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, stream, d, mask, batch, n, st.chain, st.pos, peak_out,
                           status_out);
        return hipGetLastError();
    };
    if (waves > 1)
        return objective == CKPT_OBJ_STATIC    ? parts(eval_peak_parts_kernel<CKPT_OBJ_STATIC>)
               : objective == CKPT_OBJ_DYNAMIC ? parts(eval_peak_parts_kernel<CKPT_OBJ_DYNAMIC>)
                                               : parts(eval_peak_parts_kernel<CKPT_OBJ_BOTH>);
    if (batch * (n + 1) * 9 > kBypassBytes)
        return objective == CKPT_OBJ_STATIC    ? walk(eval_peak_kernel<CKPT_OBJ_STATIC, true>)
               : objective == CKPT_OBJ_DYNAMIC ? walk(eval_peak_kernel<CKPT_OBJ_DYNAMIC, true>)
                                               : walk(eval_peak_kernel<CKPT_OBJ_BOTH, true>);
    return objective == CKPT_OBJ_STATIC    ? walk(eval_peak_kernel<CKPT_OBJ_STATIC, false>)
           : objective == CKPT_OBJ_DYNAMIC ? walk(eval_peak_kernel<CKPT_OBJ_DYNAMIC, false>)
                                           : walk(eval_peak_kernel<CKPT_OBJ_BOTH, false>);
}

hipError_t launch_eval_peak_ragged(const int64_t *d_stage, const uint8_t *mask_stage, const RaggedGroupDev *groups,
                                   const RaggedTotals &t, int64_t batch, int objective, int64_t *peak_stage,
                                   int32_t *status_stage, hipStream_t stream)
{
    const int n_groups = t.n_groups;
    const int64_t waves = t.waves;
    if (waves == 0) return hipSuccess;
    static_assert(kBlock == kWave, "a workgroup takes one of the groups' waves");
    const bool parts = waves <= kRaggedPartsMax;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)waves), dim3(parts ? kBlock * kRaggedWaves : kBlock),
                           parts ? parts_lds_bytes(objective, kRaggedWaves) : 0, stream, d_stage, mask_stage, groups,
                           n_groups, batch, peak_stage, status_stage);
        return hipGetLastError();
    };
    if (parts)
        return objective == CKPT_OBJ_STATIC    ? go(eval_peak_ragged_kernel<CKPT_OBJ_STATIC, true>)
               : objective == CKPT_OBJ_DYNAMIC ? go(eval_peak_ragged_kernel<CKPT_OBJ_DYNAMIC, true>)
                                               : go(eval_peak_ragged_kernel<CKPT_OBJ_BOTH, true>);
    if (batch < kRaggedBypassChains * waves)
        return objective == CKPT_OBJ_STATIC    ? go(eval_peak_ragged_kernel<CKPT_OBJ_STATIC, false, true>)
               : objective == CKPT_OBJ_DYNAMIC ? go(eval_peak_ragged_kernel<CKPT_OBJ_DYNAMIC, false, true>)
                                               : go(eval_peak_ragged_kernel<CKPT_OBJ_BOTH, false, true>);
    return objective == CKPT_OBJ_STATIC    ? go(eval_peak_ragged_kernel<CKPT_OBJ_STATIC, false>)
           : objective == CKPT_OBJ_DYNAMIC ? go(eval_peak_ragged_kernel<CKPT_OBJ_DYNAMIC, false>)
                                           : go(eval_peak_ragged_kernel<CKPT_OBJ_BOTH, false>);
}

}  // namespace ckpt
