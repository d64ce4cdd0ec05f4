// The kernels of csrc/cubic_search.hip on the CPU, against the oracle: whole calls of both forms, and the pass of one
// wave on sums that no checked chain has.
#include "cubic_search.cpp"  // (written by the test, see there)

#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

extern "C" void orc_batch_solve_static(const int64_t *, int64_t, int, uint8_t *, int64_t *, int64_t *);

using namespace ckpt;

namespace {
std::mt19937_64 rng(7);
int failures = 0;

typedef std::vector<int64_t> Sizes;
Sizes uniform(int n, int64_t lo, int64_t hi)
{
    Sizes d((size_t)n + 1);
    for (int64_t &x : d) x = lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1));
    return d;
}
Sizes with(Sizes d, int k, int64_t x)
{
    d[(size_t)k] = x;
    return d;
}

enum Form { kLanePerPoint, kWavePerPoint };

// Chains of equal length, chain after chain.
void check(const char *what, const std::vector<Sizes> &chains, Form form)
{
    const int n = (int)chains[0].size() - 1;
    const int64_t batch = (int64_t)chains.size(), n1 = n + 1;
    std::vector<int> want_status;
    Sizes good;
    int64_t *d = (int64_t *)emu::device_memory((size_t)(batch * n1) * 8);
    for (int64_t c = 0; c < batch; ++c) {
        __int128 sum = 0, most = 0;
        bool positive = true;
        for (int k = 0; k <= n; ++k) {
            const int64_t x = d[c * n1 + k] = chains[(size_t)c][(size_t)k];
            sum += x;
            most = x > most ? (__int128)x : most;
            positive &= x > 0;
        }
        want_status.push_back(!positive ? CKPT_ERR_SIZE : sum + most > (__int128)INT64_MAX ? CKPT_ERR_OVERFLOW : CKPT_OK);
        for (int k = 0; k <= n; ++k) good.push_back(want_status.back() == CKPT_OK ? chains[(size_t)c][(size_t)k] : 1);
    }
    std::vector<uint8_t> want_mask((size_t)(batch * n1));
    Sizes want_peak((size_t)batch), want_budget((size_t)batch);
    orc_batch_solve_static(good.data(), batch, n, want_mask.data(), want_peak.data(), want_budget.data());

    uint8_t *mask = (uint8_t *)emu::device_memory((size_t)(batch * n1));
    int64_t *peak = (int64_t *)emu::device_memory((size_t)batch * 8), *budget = (int64_t *)emu::device_memory((size_t)batch * 8);
    int32_t *status = (int32_t *)emu::device_memory((size_t)batch * 4);
    const Strides st{n1, 1};
    const hipError_t e =
        form == kWavePerPoint
            ? launch_cubic_search_long(d, batch, n, st, mask, peak, budget, status,
                                       emu::device_memory(cubic_search_long_bytes(batch, n)), nullptr)
            : launch_cubic_search(d, batch, n, st, mask, peak, budget, status, emu::device_memory(256 + 4 * (size_t)batch), nullptr);
    bool ok = e == hipSuccess;
    for (int64_t c = 0; c < batch && ok; ++c) {
        const bool bad = want_status[(size_t)c] != CKPT_OK;
        ok = status[c] == want_status[(size_t)c] && peak[c] == (bad ? -1 : want_peak[(size_t)c]) &&
             budget[c] == (bad ? -1 : want_budget[(size_t)c]);
        for (int k = 0; k <= n && ok; ++k) ok = mask[c * n1 + k] == (bad ? 0 : want_mask[(size_t)(c * n1 + k)]);
        if (!ok)
            printf("%s, n = %d, chain %d, a %s per point: status %d (%d), peak %lld (%lld), budget %lld (%lld)\n", what, n,
                   (int)c, form == kWavePerPoint ? "wave" : "lane", (int)status[c], want_status[(size_t)c], (long long)peak[c],
                   (long long)want_peak[(size_t)c], (long long)budget[c], (long long)want_budget[(size_t)c]);
    }
    failures += !ok;
}

// A pass over sums that do not ascend ends, whatever it returns.
template <typename U>
__global__ void pass_kernel(const U *P, int n, U s, U *got)
{
    U *const F = (U *)emu::dynamic_lds;
    const U v = wave_cost<U, true>(P, n, s, F, (uint16_t *)(F + n + 1 + kWave));
    if (threadIdx.x == 0) *got = v;
}
template <typename U>
void passes_over_sums_that_wrap(int n, U large)
{
    for (int k : {0, 1, n / 2, n}) {
        U *P = (U *)emu::device_memory(((size_t)n + 1) * sizeof(U)), run = 0, got = 0;
        for (int i = 0; i <= n; ++i) P[i] = run += i == k ? large : (U)(1 + rng() % 1000000);
        for (const U s : {(U)0, (U)1, (U)1000, (U)1000000, (U)100000000, (U)(~(U)0 / 2), (U)~P[1], (U)~P[n / 2], (U)~P[n - 1]})
            hipLaunchKernelGGL(pass_kernel<U>, dim3(1), dim3(64), ((size_t)n + 1 + kWave) * (sizeof(U) + 2), nullptr, P, n, s, &got);
    }
}
}  // namespace

int main()
{
    emu::rendezvous_limit = 100000;  // (a pass of 300 heads: some 10,000)
    for (const int n : {65, 130, 300}) {
        passes_over_sums_that_wrap<uint32_t>(n, ~0u - 5);
        passes_over_sums_that_wrap<uint64_t>(n, ~0ull - 5);
    }
    emu::rendezvous_limit = ~0ull;
    const int64_t top = INT64_MAX;
    for (const int n : {1, 2, 8, 9, 63, 64, 65, 127, 130}) {
        std::vector<Sizes> chains = {uniform(n, 1, 1000000), uniform(n, 1, 3), uniform(n, 1, top / (2 * n + 4)), with(uniform(n, 1, 9), n / 2, 0)};
        for (const int k : {0, n}) {
            chains.push_back(with(uniform(n, 100, 100), k, 1ll << 40));
            for (const int64_t x : {top, top - 0x80000000l, (top - n) / 2}) chains.push_back(with(uniform(n, 1, 1), k, x));
        }
        check("kinds of sizes", chains, kLanePerPoint);
        if (n > 128) check("kinds of sizes", chains, kWavePerPoint);
    }
    // repeated layers: a predecessor is one of many equal ones, next to each other and far apart
    for (const int n : {130, 257, 300}) {
        Sizes blocks = uniform(n, 5, 5), late = blocks;
        for (int k = 0; k <= n; ++k) {
            blocks[(size_t)k] = k % 3 == 2 ? 16 : 4;
            late[(size_t)k] = k % 97 == 40 ? 1 : 1000;
        }
        check("repeated layers", {uniform(n, 5, 5), blocks, late, with(blocks, n / 2, 900)}, kWavePerPoint);
        if (n <= 256) check("repeated layers", {uniform(n, 5, 5), blocks, late, with(blocks, n / 2, 900)}, kLanePerPoint);
    }
    check("large sizes in front", {with(uniform(257, 1, 1000000), 0, 1ll << 43), with(uniform(257, 1, 1000000), 0, top)}, kWavePerPoint);
    // sizes of very different orders: more budgets are left after the rounds than are listed
    for (const int n : {142, 300}) {
        Sizes d = with(uniform(n, 1, 1000000), n / 3, 1000000000000000);
        check("one large layer", {d}, kWavePerPoint);
        check("two large layers", {with(d, n - 1, 1000000000012345)}, kWavePerPoint);
    }
    // ragged batches, by lengths and numbers of chains: the launches they go in (the last of them may be that for the chains
    // that need 64 bits)
    const auto launches_of = [](int64_t batch, std::vector<std::pair<int, int64_t>> lengths, int64_t &waves, bool &second) {
        SearchClass classes[kSearchClasses];
        for (const auto &[n, many] : lengths) {
            int k = 0;
            while (n > search_class_limit(k)) ++k;
            classes[k].longest = n;
            classes[k].us += (float)many * search_us(n);
        }
        int launches = 0;
        waves = 0;
        second = false;
        emu::instead_of_running = [&](const char *name, dim3 grid) {
            second |= strstr(name, "ragged_wide_kernel") != nullptr;
            if (strstr(name, "ragged_kernel")) ++launches, waves += grid.x;
        };
        launch_cubic_search_ragged(nullptr, nullptr, batch, classes, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
        emu::instead_of_running = nullptr;
        return launches;
    };
    int64_t waves;
    bool second;
    // the largest: every chain once for each class of lengths, in launches that there can be
    for (const int64_t batch : {(int64_t)1000, (int64_t)1 << 25, ((int64_t)1 << 26) + 1, (int64_t)INT32_MAX}) {
        launches_of(batch, {{20, batch - 2}, {100, 1}, {256, 1}}, waves, second);
        failures += waves != 3 * batch;
    }
    // a few long chains among short ones: not with LDS for the long ones where the short ones wait for it, and with LDS for
    // 64 bits where a second launch would cost more
    failures += launches_of(16384, {{24, 16383}, {64, 1}}, waves, second) != 2;
    failures += launches_of(4096, {{24, 4095}, {64, 1}}, waves, second) != 1;
    failures += launches_of(1023, {{24, 1007}, {256, 16}}, waves, second) != 1 || second;
    failures += launches_of(700, {{240, 700}}, waves, second) != 1 || !second;
    printf(failures ? "search_driver: %d failed\n" : "search_driver ok\n", failures);
    return failures != 0;
}
