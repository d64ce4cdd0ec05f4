// The kernels of csrc/cubic_search.hip that give a chain a row of lanes, on the CPU, against the oracle.
#include "cubic_search.cpp"  // (written by the test, see there)

#include <math.h>
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

Sizes pyramid(int n)  // the picture halved four times in the first third, the width doubled twice
{
    const int64_t first = (8 + (int64_t)(rng() % 200)) << 14;
    Sizes d((size_t)n + 1);
    for (int k = 0; k <= n; ++k) d[(size_t)k] = (first << (k % 3 == 1)) >> std::min(8, 2 * (12 * k / std::max(n, 1)));
    return d;
}
Sizes falling(int n)
{
    Sizes d((size_t)n + 1);
    for (int k = 0; k <= n; ++k) d[(size_t)k] = 1 + (int64_t)((1 << 27) * pow(0.9, k) * (0.7 + 0.6 * (double)(rng() % 1000) / 1000.0));
    return d;
}

// Which chains the rows may leave for their windows' reach.
enum Far { kNone, kSome, kAll, kAny };

// Position-major.  Twice: what is left by a row again, and by a wave.
template <int G, int MOST>
void check(const char *what, const std::vector<Sizes> &chains, Far far, int ring = 0)
{
    const int n = (int)chains[0].size() - 1;
    if (ring == 0) ring = row_ring(n);
    const int whole = row_blocks(n) * kRowBlk;
    const int64_t batch = (int64_t)chains.size(), n1 = n + 1;
    Sizes good;
    std::vector<int> want_status, shift;
    std::vector<bool> fits, large;  // certainly 32 bits, certainly more
    int64_t *d = (int64_t *)emu::device_memory((size_t)(batch * n1) * 8);
    for (int64_t c = 0; c < batch; ++c) {
        __int128 sum = 0, most = 0;
        uint64_t bits = 0;
        bool positive = true;
        for (int k = 0; k <= n; ++k) {
            const int64_t x = d[k * batch + c] = chains[(size_t)c][(size_t)k];
            sum += x;
            bits |= (uint64_t)x;
            most = x > most ? (__int128)x : most;
            positive &= x > 0;
        }
        want_status.push_back(!positive ? CKPT_ERR_SIZE : sum + most > (__int128)INT64_MAX ? CKPT_ERR_OVERFLOW : CKPT_OK);
        for (int k = 0; k <= n; ++k) good.push_back(want_status.back() == CKPT_OK ? chains[(size_t)c][(size_t)k] : 1);
        shift.push_back(__builtin_ctzll(bits));
        fits.push_back((sum + most) >> shift.back() < INT32_MAX && 3 * most >> shift.back() < (1ll << 31));
        large.push_back(most >> shift.back() >= (1ll << 31));
    }
    std::vector<uint8_t> want_mask((size_t)(batch * n1));
    Sizes want_peak((size_t)batch), want_budget((size_t)batch);
    orc_batch_solve_static(good.data(), batch, n, want_mask.data(), want_peak.data(), want_budget.data());

    constexpr int C = kWave / G;
    const dim3 grid((unsigned)((batch + C - 1) / C)), block(kWave);
    const auto failed = [&](const char *how, int c) {
        printf("%s, n = %d, chain %d, %d lanes, ring %d: %s\n", what, n, c, G, ring, how);
        ++failures;
    };
    // the rows with a list of what they leave, everything by a wave a chain (of some lengths with a workgroup for each chain),
    // what the rows leave in the same wave
    for (const int turn : {0, 1, 2}) {
        const int far_from = turn == 1 ? 0 : INT32_MAX;
        const bool each = (n + turn) % 2 == 0, in_wave = turn == 2;
        if (in_wave && MOST > kRowsOf16Layers) break;
        uint8_t *mask = (uint8_t *)emu::device_memory((size_t)(batch * n1));
        int64_t *peak = (int64_t *)emu::device_memory((size_t)batch * 8), *budget = (int64_t *)emu::device_memory((size_t)batch * 8);
        int32_t *status = (int32_t *)emu::device_memory((size_t)batch * 4);
        const int32_t unwritten = status[0];
        const SearchWs w{(int32_t *)emu::device_memory(256), (int32_t *)emu::device_memory((size_t)batch * 8)};
        hipLaunchKernelGGL((cubic_rows_sample_kernel<G, MOST>), dim3(kSamples), block, (size_t)n1 * C * 4, nullptr, d, batch, n, (int64_t)1,
                           batch, ring, w);
        int sampled = 0;
        for (int k = 0; k < kSamples; ++k) sampled += ((const uint8_t *)(w.count + kSampled))[k];
        if (ring == row_ring(n) && (far == kAll ? sampled < kSamples : far == kNone && sampled != 0)) failed("not as expected of the sample", -1);
        const size_t lds = std::max(rows_lds_bytes(n, C, ring), in_wave ? search_lds_bytes(n, 4) : 0);
        const auto kernel = in_wave ? cubic_rows_kernel<G, MOST, MOST <= kRowsOf16Layers> : cubic_rows_kernel<G, MOST, false>;
        hipLaunchKernelGGL(kernel, grid, block, lds, nullptr, d, batch, n, (int64_t)1, batch, ring, far_from, mask, peak, budget, status, w);
        // what is left is on one list or the other, and nothing of it written; the rest is solved
        const bool none = far_from == 0 && ring < whole;
        std::vector<int> left((size_t)batch);
        const int wide = w.count[kCountWide], beyond = w.count[kCountFar];
        if (wide < 0 || beyond < 0 || wide + beyond > (none ? 0 : batch)) return failed("lists longer than the batch", -1);
        for (int k = 0; k < wide; ++k) left[(size_t)w.list[k]] += 1;
        for (int k = 0; k < beyond; ++k) left[(size_t)w.list[batch + k]] += 2;
        int64_t rest = 0;  // chains that a ring may be too short for
        for (int64_t c = 0; c < batch; ++c) {
            const int how = none ? 2 : left[(size_t)c];
            if (how > 2) failed("left twice", (int)c);
            if (status[c] != (how ? unwritten : want_status[(size_t)c])) failed(how ? "left and written" : "neither solved nor left", (int)c);
            if (none) continue;
            if (how && want_status[(size_t)c] != CKPT_OK) failed("a bad chain is left", (int)c);
            if (how == 1 && fits[(size_t)c]) failed("left for 64 bits", (int)c);
            const bool needs_64 = want_status[(size_t)c] == CKPT_OK && (large[(size_t)c] || want_peak[(size_t)c] >> shift[(size_t)c] >= (1ll << 31));
            if (needs_64 && how == 0) failed("not left for 64 bits", (int)c);
            rest += want_status[(size_t)c] == CKPT_OK && how != 1;
        }
        if (in_wave && beyond != 0) failed("listed", -1);
        if (!none && !in_wave && ((far == kNone || ring == whole) ? beyond != 0 : far == kSome ? beyond == 0 || beyond >= rest : far == kAll && beyond != rest)) {
            printf("%d of %d chains are beyond the ring\n", beyond, (int)rest);
            failed("wrong number", -1);
        }
        if (ring < whole)
            hipLaunchKernelGGL(each ? cubic_search_far_kernel<true> : cubic_search_far_kernel<false>, dim3(each ? (unsigned)batch : 2 * kXcds), block, search_lds_bytes(n, 4), nullptr, d, batch, n, (int64_t)1, batch, far_from, 3,
                               mask, peak, budget, status, w);
        for (int64_t c = 0; c < batch; ++c)
            if (beyond > 3 && left[(size_t)c] == 2 && status[c] != CKPT_OK && fits[(size_t)c]) failed("not solved in 32 bits", (int)c);
        hipLaunchKernelGGL(cubic_search_wide_kernel, dim3(2), block, search_lds_bytes(n, 8), nullptr, d, batch, n, 3, (int64_t)1, batch, mask, peak, budget,
                           status, w);
        for (int64_t c = 0; c < batch; ++c) {
            const bool bad = want_status[(size_t)c] != CKPT_OK;
            bool ok = status[c] == want_status[(size_t)c] && peak[c] == (bad ? -1 : want_peak[(size_t)c]) &&
                      budget[c] == (bad ? -1 : want_budget[(size_t)c]);
            for (int k = 0; k <= n && ok; ++k) ok = mask[k * batch + c] == (bad ? 0 : want_mask[(size_t)(c * n1 + k)]);
            if (!ok) {
                printf("status %d (%d), peak %lld (%lld), budget %lld (%lld)\n", (int)status[c], want_status[(size_t)c], (long long)peak[c],
                       (long long)want_peak[(size_t)c], (long long)budget[c], (long long)want_budget[(size_t)c]);
                return failed("wrong", (int)c);
            }
        }
    }
}

template <int G, int MOST>
void all_kinds(const std::vector<int> &lengths)
{
    const int64_t top = INT64_MAX;
    for (const int n : lengths) {
        const int whole = row_blocks(n) * kRowBlk;
        std::vector<Sizes> chains = {uniform(n, 1, 1000000), uniform(n, 1, 3), spread(n, 12), uniform(n, 7, 7), with(uniform(n, 1, 9), n / 2, 0)};
        for (const int k : {0, n}) {
            chains.push_back(with(uniform(n, 100, 100), k, 1ll << 29));
            chains.push_back(with(uniform(n, 1, 1), k, top));
        }
        check<G, MOST>("even sizes", std::vector<Sizes>(chains.begin(), chains.begin() + 2), kNone);
        check<G, MOST>("kinds of sizes", chains, kAny);
        chains.push_back(spread(n, 22));
        for (const int k : {n / 2, n - 1}) chains.push_back(with(spread(n, 9), k, 1 << 26));
        // (with less room than most windows take, and for all)
        check<G, MOST>("kinds of sizes", chains, kAny);
        for (const int ring : {8, 32, whole}) check<G, MOST>("kinds of sizes", chains, n > 60 && ring == 8 ? kAll : kAny, std::min(ring, whole));
        // more than 2^32 in all, and more than 32 bits hold
        check<G, MOST>("large sums", {spread(n, 25), uniform(n, 1 << 27, 1 << 28), with(uniform(n, 1, 1000), n / 2, 1ll << 40), uniform(n, 1, top / (2 * n + 4)), spread(n, 12)}, kAny);
        std::vector<Sizes> large;
        for (int k = 0; k < 24; ++k) large.push_back(with(uniform(n, 1ll << (19 + k % 8), 1ll << 27), n / 2, (1ll << 26) + 1));
        check<G, MOST>("sums around 2^32", large, kAny);
        std::vector<Sizes> heavy;  // one size that a few of add up to 2^32, before or among ones that add up to more or less
        for (int k = 0; k < 16; ++k) {
            const int at[] = {0, 1, n / 2, n};
            const int64_t x = (600000001 + (int64_t)(rng() % 115000000)) | 1;
            heavy.push_back(with(k < 8 ? uniform(n, 1, 1 << 20) : k < 12 ? uniform(n, 1 << 20, 1 << 22) : uniform(n, 1 << 24, 1 << 26), at[k % 4], x));
        }
        check<G, MOST>("one large size", heavy, kAny);
        std::vector<Sizes> networks;
        for (int k = 0; k < 16; ++k) networks.push_back(network(n));
        check<G, MOST>("networks", networks, kAny);
        Sizes blocks = uniform(n, 5, 5);
        for (int k = 0; k <= n; ++k) blocks[(size_t)k] = k % 3 == 2 ? 16 : 4;
        check<G, MOST>("repeated layers", {blocks, with(blocks, n / 2, 900), uniform(n, 1 << 20, 1 << 20)}, kAny);
        // layers in front that outweigh the rest: windows that reach farther than the ring, of all chains or of some
        std::vector<Sizes> front;
        for (int k = 0; k < 9; ++k) front.push_back(falling(n));
        check<G, MOST>("falling sizes", front, n > 60 ? kAll : n < 30 ? kNone : kAny);
        for (int k = 0; k < 9; ++k) front.push_back(k % 2 ? pyramid(n) : k % 4 ? with(uniform(n, 1, 3), n / 3, 0) : uniform(n, 1 << 20, 1 << 25));
        check<G, MOST>("pyramids and others", front, n > 60 ? kSome : n < 30 ? kNone : kAny);
    }
    // every number of chains that a wave has rows for, and one more
    std::vector<Sizes> chains;
    for (int k = 0; k <= kWave / G; ++k) {
        chains.push_back(spread(40, 12));
        check<G, MOST>("numbers of chains", chains, kNone);
    }
}
}  // namespace

int main()
{
    emu::rendezvous_limit = 3000000;
    if (raise_search_lds_limit() != hipSuccess) return 1;
    // (the forms that launch_cubic_search takes, by their lengths)
    all_kinds<8, kRowsOf8Layers>({1, 2, 3, 4, 5, 8, 9, 24, 63, 64, 65, kRowsOf8Layers});
    all_kinds<16, kRowsOf16Layers>({1, 4, 5, 24, 63, 64, 65, 100, kRowsOf16Layers});
    all_kinds<16, kRowsMaxLayers>({129, 200, 256});
    printf(failures ? "rows_driver: %d failed\n" : "rows_driver ok\n", failures);
    return failures != 0;
}
