// The kernels of csrc/cubic_search.hip that give a chain a row of lanes, on the CPU, against the oracle.
#include "cubic_search.cpp"  // (written by the test, see there)

#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

extern "C" void orc_batch_solve_static(const int64_t *, int64_t, int, uint8_t *, int64_t *, int64_t *);

using namespace ckpt;

namespace {
std::mt19937_64 rng(11);
int failures = 0;

typedef std::vector<int64_t> Sizes;
Sizes uniform(int n, int64_t lo, int64_t hi)
{
    Sizes d((size_t)n + 1);
    for (int64_t &x : d) x = lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1));
    return d;
}
Sizes spread(int n, double bits)  // unrounded, over so many octaves
{
    Sizes d((size_t)n + 1);
    for (int64_t &x : d) x = (int64_t)exp2(bits * (double)(rng() % 100000) / 100000.0 + 3);
    return d;
}
Sizes network(int n)  // stages of layers w, w, 4w, the picture halved and the width doubled from one to the next
{
    const int64_t batch = 8 + (int64_t)(rng() % 200), width = 16 << (rng() % 3), pixels = 8 * (7 + (int64_t)(rng() % 22));
    int ends[3];
    for (int &e : ends) e = 2 + (int)(rng() % (uint64_t)(n > 4 ? n - 3 : 2));
    Sizes d((size_t)n + 1);
    for (int k = 0; k <= n; ++k) {
        int stage = 0;
        for (const int e : ends) stage += k >= e;
        const int64_t w = width << stage, side = std::max<int64_t>(pixels >> stage, 1);
        d[(size_t)k] = batch * 4 * (k % 3 == 1 ? 4 * w : w) * side * side;
    }
    d[0] = batch * 12 * 4 * pixels * pixels;
    d[(size_t)n] = batch * 4000;
    return d;
}
Sizes with(Sizes d, int k, int64_t x)
{
    d[(size_t)k] = x;
    return d;
}

// Position-major.
template <int G>
void check(const char *what, const std::vector<Sizes> &chains, int ring = 0)
{
    const int n = (int)chains[0].size() - 1;
    if (ring == 0) ring = row_ring(n);
    if (rows_lds_bytes(n, kWave / G, ring) > kDefaultLdsLimit) return;
    const int64_t batch = (int64_t)chains.size(), n1 = n + 1;
    Sizes good;
    std::vector<int> want_status;
    int64_t *d = (int64_t *)emu::device_memory((size_t)(batch * n1) * 8);
    for (int64_t c = 0; c < batch; ++c) {
        __int128 sum = 0, most = 0;
        bool positive = true;
        for (int k = 0; k <= n; ++k) {
            const int64_t x = d[k * batch + c] = chains[(size_t)c][(size_t)k];
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
    constexpr int C = kWave / G;
    const SearchWs w{(int32_t *)emu::device_memory(4), (int32_t *)emu::device_memory((size_t)batch * 4)};
    *w.count = 0;
    const auto kernel = n <= kRowsOf8Layers ? cubic_rows_kernel<G, kRowsOf8Layers> : cubic_rows_kernel<G, kRowsMaxLayers>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((batch + C - 1) / C)), dim3(64), rows_lds_bytes(n, C, ring), nullptr, d,
                       batch, n, (int64_t)1, batch, ring, mask, peak, budget, status, w);
    if (search_lds_bytes(n, 8) > kDefaultLdsLimit && raise_search_lds_limit() != hipSuccess) ++failures;
    hipLaunchKernelGGL(cubic_search_wide_kernel, dim3(2), dim3(64), search_lds_bytes(n, 8), nullptr, d, n, (int64_t)1, batch, mask,
                       peak, budget, status, w);
    bool ok = true;
    for (int64_t c = 0; c < batch && ok; ++c) {
        const bool bad = want_status[(size_t)c] != CKPT_OK;
        ok = status[c] == want_status[(size_t)c] && peak[c] == (bad ? -1 : want_peak[(size_t)c]) &&
             budget[c] == (bad ? -1 : want_budget[(size_t)c]);
        for (int k = 0; k <= n && ok; ++k) ok = mask[k * batch + c] == (bad ? 0 : want_mask[(size_t)(c * n1 + k)]);
        if (!ok)
            printf("%s, n = %d, chain %d, %d lanes: status %d (%d), peak %lld (%lld), budget %lld (%lld)\n", what, n, (int)c, G,
                   (int)status[c], want_status[(size_t)c], (long long)peak[c], (long long)want_peak[(size_t)c],
                   (long long)budget[c], (long long)want_budget[(size_t)c]);
    }
    failures += !ok;
}

template <int G>
void all_kinds()
{
    const int64_t top = INT64_MAX;
    for (const int n : {1, 2, 3, 4, 5, 8, 9, 24, 63, 64, 65, 100, 128, 129, 256}) {
        std::vector<Sizes> chains = {uniform(n, 1, 1000000), uniform(n, 1, 3), spread(n, 12), spread(n, 22), uniform(n, 7, 7), with(uniform(n, 1, 9), n / 2, 0)};
        for (const int k : {0, n}) {
            chains.push_back(with(uniform(n, 100, 100), k, 1ll << 29));
            chains.push_back(with(uniform(n, 1, 1), k, top));
        }
        for (const int k : {n / 2, n - 1}) chains.push_back(with(spread(n, 9), k, 1 << 26));
        check<G>("kinds of sizes", chains);
        // (with less room than most windows take, and for all)
        for (const int ring : {8, 32, row_blocks(n) * kRowBlk}) check<G>("kinds of sizes", chains, std::min(ring, row_blocks(n) * kRowBlk));
        // more than 2^32 in all, and more than 32 bits hold
        check<G>("large sums", {spread(n, 25), uniform(n, 1 << 27, 1 << 28), with(uniform(n, 1, 1000), n / 2, 1ll << 40), uniform(n, 1, top / (2 * n + 4)), spread(n, 12)});
        std::vector<Sizes> large;
        for (int k = 0; k < 24; ++k) large.push_back(with(uniform(n, 1ll << (19 + k % 8), 1ll << 27), n / 2, (1ll << 26) + 1));
        check<G>("sums around 2^32", large);
        std::vector<Sizes> networks;
        for (int k = 0; k < 16; ++k) networks.push_back(network(n));
        check<G>("networks", networks);
        Sizes blocks = uniform(n, 5, 5);
        for (int k = 0; k <= n; ++k) blocks[(size_t)k] = k % 3 == 2 ? 16 : 4;
        check<G>("repeated layers", {blocks, with(blocks, n / 2, 900), uniform(n, 1 << 20, 1 << 20)});
    }
    // every number of chains that a wave has rows for, and one more
    std::vector<Sizes> chains;
    for (int k = 0; k <= kWave / G; ++k) {
        chains.push_back(spread(40, 12));
        check<G>("numbers of chains", chains);
    }
}
}  // namespace

int main()
{
    emu::rendezvous_limit = 3000000;
    all_kinds<8>();
    all_kinds<16>();
    printf(failures ? "rows_driver: %d failed\n" : "rows_driver ok\n", failures);
    return failures != 0;
}
