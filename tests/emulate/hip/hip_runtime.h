// Stands in for HIP's header when sources under csrc/ are built for the CPU (tests/test_emulated_kernels.py): as much
// of HIP as those use.  A lane is a fiber of its own, and every operation across lanes is a rendezvous of the
// wave (see fibers.cpp): what the lanes of a wave or a workgroup do together has to be reached by all of them that
// have not ended, or the run is stopped.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <functional>

using std::max;
using std::min;

#define __global__
#define __device__
#define __host__
#define __shared__ static  // (one workgroup at a time)
#define __launch_bounds__(...)
#define __forceinline__ inline
#define __align__(x) alignas(x)

typedef int hipError_t;
typedef void *hipStream_t;
enum {
    hipSuccess,
    hipErrorInvalidDevice,
    hipErrorInvalidSymbol,
    hipErrorInvalidConfiguration,
    hipErrorInvalidValue,
    hipFuncAttributeMaxDynamicSharedMemorySize
};
hipError_t hipFuncSetAttribute(const void *kernel, int, int bytes);
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
#define HIP_SYMBOL(x) ((void *)&(x))
inline hipError_t hipGetSymbolAddress(void **p, const void *symbol) { *p = (void *)symbol; return hipSuccess; }
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace emu {
constexpr int kLanes = 64;
enum Kind { kNone, kBallot, kReadLane, kFirstLane, kDpp, kShfl, kMin, kSelect, kBarrier };
extern dim3 thread, block, threads, blocks;
extern unsigned char *dynamic_lds;
// One launch: the grid's workgroups one after the other.  Dynamic LDS ends at a page that cannot be touched, and more
// than 64 KB of it must have been allowed for the kernel (`entry`).
void launch(const char *name, const void *entry, dim3 grid, dim3 block, size_t lds, const std::function<void()> &kernel);
// If set, launches are only checked and handed to this.
extern std::function<void(const char *name, dim3 grid)> instead_of_running;
// Called after every hipFuncSetAttribute: what another thread does at that moment.
extern std::function<void()> meanwhile;
[[noreturn]] void stop(const char *why);
// Device memory of exactly this many bytes, between pages that cannot be touched, full of a pattern.
void *device_memory(size_t bytes);
// A launch whose waves meet more often than this is taken not to end.
extern uint64_t rendezvous_limit;
// The values that the lanes of this wave bring (valid until the lane's next call but one), and which lanes take part.
const uint64_t *meet(uint64_t value, Kind kind);
uint64_t taking_part();
inline int lane() { return (int)(thread.x % kLanes); }

template <class T> uint64_t bits(T v) { uint64_t u = 0; memcpy(&u, &v, sizeof(T)); return u; }
template <class T> T value(uint64_t u) { T v; memcpy(&v, &u, sizeof(T)); return v; }
inline uint64_t ballot(bool b)
{
    const uint64_t *v = meet(b, kBallot);
    uint64_t m = 0;
    for (int l = 0; l < kLanes; ++l)
        if (((taking_part() >> l) & 1) && v[l]) m |= 1ull << l;
    return m;
}
inline int first_lane(int x)
{
    const uint64_t *v = meet((uint32_t)x, kFirstLane);
    return (int)(uint32_t)v[__builtin_ctzll(taking_part())];
}
inline int read_lane(int x, int l) { return (int)(uint32_t)meet((uint32_t)x, kReadLane)[l & 63]; }
inline int dpp(int old, int x, int control, int row_mask)
{
    const uint64_t *v = meet((uint32_t)x, kDpp);
    const int row = lane() / 16;
    int from = -1;
    if (control > 0x110 && control < 0x120) from = lane() - (control - 0x110) >= row * 16 ? lane() - (control - 0x110) : -1;
    if (control > 0x100 && control < 0x110) from = lane() + (control - 0x100) < row * 16 + 16 ? lane() + (control - 0x100) : -1;
    if (control >= 0x150 && control < 0x160) from = row * 16 + (control - 0x150);
    if (control < 0x100) from = lane() / 4 * 4 + ((control >> (2 * (lane() % 4))) & 3);
    if (control == 0x140) from = lane() ^ 15;
    if (control == 0x141) from = lane() ^ 7;
    if (control == 0x142) from = row * 16 - 1;
    if (control == 0x143) from = row > 1 ? 31 : -1;
    return from < 0 || !((row_mask >> row) & 1) ? old : (int)(uint32_t)v[from];
}
inline double dpp(double old, double x, int control, int row_mask)
{
    uint64_t r = 0;
    for (int k = 0; k < 64; k += 32)
        r |= (uint64_t)(uint32_t)dpp((int)(uint32_t)(bits(old) >> k), (int)(uint32_t)(bits(x) >> k), control, row_mask) << k;
    return value<double>(r);
}
inline uint32_t min_u32(uint32_t x)
{
    const uint64_t *v = meet(x, kMin);
    uint32_t m = ~0u;
    for (int l = 0; l < kLanes; ++l)
        if ((taking_part() >> l) & 1) m = std::min(m, (uint32_t)v[l]);
    return m;
}
// The bytes of a (4..7) and b (0..3) that the bytes of sel name.
inline uint32_t permuted(uint32_t a, uint32_t b, uint32_t sel)
{
    uint32_t r = 0;
    for (int k = 0; k < 32; k += 8) r |= (uint32_t)(uint8_t)((((uint64_t)a << 32) | b) >> (8 * ((sel >> k) & 7))) << k;
    return r;
}
template <class T> T exchange(T *p, T v) { const T was = *p; *p = v; return was; }
template <class T> T least(T *p, T v) { const T was = *p; *p = v < was ? v : was; return was; }
}  // namespace emu

#define threadIdx (emu::thread)
#define blockIdx (emu::block)
#define blockDim (emu::threads)
#define gridDim (emu::blocks)
#define hipLaunchKernelGGL(k, grid, block, lds, stream, ...) emu::launch(#k, (const void *)(k), grid, block, lds, [&] { (k)(__VA_ARGS__); })

inline void __syncthreads() { (void)emu::meet(0, emu::kBarrier); }
inline void __threadfence_block() {}
inline bool __any(int b) { return emu::ballot(b != 0) != 0; }
template <class T> T __shfl(T v, int l, int) { return emu::value<T>(emu::meet(emu::bits(v), emu::kShfl)[l & 63]); }
template <class T> T __shfl_xor(T v, int m, int) { return emu::value<T>(emu::meet(emu::bits(v), emu::kShfl)[emu::lane() ^ m]); }
template <class T> T __shfl_up(T v, int d, int)
{
    const uint64_t *all = emu::meet(emu::bits(v), emu::kShfl);
    return emu::value<T>(all[emu::lane() >= d ? emu::lane() - d : emu::lane()]);
}
#define __builtin_amdgcn_ballot_w64(b) emu::ballot(b)
#define __builtin_amdgcn_readlane(v, l) emu::read_lane(v, l)
#define __builtin_amdgcn_readfirstlane(v) emu::first_lane(v)
#define __builtin_nontemporal_load(p) (*(p))
#define __builtin_nontemporal_store(v, p) ((void)(*(p) = (v)))
#define __builtin_amdgcn_update_dpp(old, v, control, rows, banks, bound) emu::dpp(old, v, control, rows)
#define __builtin_amdgcn_mov_dpp(v, control, rows, banks, bound) emu::dpp(0, v, control, rows)
#define __builtin_amdgcn_sched_barrier(...) ((void)0)
#define __builtin_amdgcn_alignbit(hi, lo, shift) ((uint32_t)((((uint64_t)(hi) << 32) | (uint32_t)(lo)) >> ((shift) & 31)))
#define __builtin_amdgcn_perm(a, b, sel) emu::permuted(a, b, sel)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __HIP_MEMORY_SCOPE_AGENT 1
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_store(p, v, ...) ((void)(*(p) = (v)))
#define __hip_atomic_fetch_min(p, v, ...) emu::least(p, v)
#define __hip_atomic_exchange(p, v, ...) emu::exchange(p, v)
template <class T, class V> T atomicAdd(T *p, V v) { return emu::exchange(p, (T)(*p + v)); }
template <class T> T atomicMin(T *p, T v) { return emu::least(p, v); }
template <class T> T atomicMax(T *p, T v) { return emu::exchange(p, *p < v ? v : *p); }
template <class T> T atomicCAS(T *p, T a, T b) { const T was = *p; if (was == a) *p = b; return was; }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline int __ffs(int v) { return __builtin_ffs(v); }
inline int __popc(unsigned v) { return __builtin_popcount(v); }
inline int __clz(int v) { return v ? __builtin_clz((unsigned)v) : 32; }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __clzll(unsigned long long v) { return v ? __builtin_clzll(v) : 64; }
inline uint32_t __float_as_uint(float f) { return (uint32_t)emu::bits(f); }
inline float __uint_as_float(uint32_t u) { return emu::value<float>(u); }
