// The kernels of csrc/solve_linear.hip on the CPU, against the oracle, each form launched by itself whatever the batch.
#include "solve_linear.cpp"  // (written by the test, see there)

#include <stdio.h>
#include <stdlib.h>

#include <numeric>
#include <random>
#include <vector>

extern "C" void orc_ragged_solve_dynamic(const int64_t *d, const int64_t *offsets, int64_t batch, uint8_t *mask, int64_t *peak);

using namespace ckpt;

namespace {
std::mt19937_64 rng(11);
int failures = 0;

typedef std::vector<int64_t> Sizes;
int64_t between(int64_t lo, int64_t hi) { return lo + (int64_t)(rng() % (uint64_t)(hi - lo + 1)); }
Sizes uniform(int n, int64_t lo, int64_t hi)
{
    Sizes d((size_t)n + 1);
    for (int64_t &x : d) x = between(lo, hi);
    return d;
}
Sizes with(Sizes d, int k, int64_t x)
{
    d[(size_t)k] = x;
    return d;
}
// A large layer at the far end and ever smaller ones before it: every position stays in the queue.
Sizes live_entries(int n)
{
    Sizes d((size_t)n + 1, 1);
    for (int k = 1; k < n; ++k) d[(size_t)k] = n - k;
    if (n > 1) d[(size_t)n - 1] = 1ll << 40;
    return d;
}
// sum(d) + max(d) is `most`, or one less, by the size at k.
Sizes up_to(int n, int k, int64_t most)
{
    Sizes d = with(uniform(n, 1, std::max<int64_t>(1, most / (4 * n + 4))), k, 0);
    const int64_t rest = std::accumulate(d.begin(), d.end(), (int64_t)0);
    return with(d, k, (most - rest) / 2);
}

enum Form { kLanes, kWideLanes, kWaves, kRows, kListedRows, kRowsAndLanes, kFlatWaves, kFlatRows, kFlatFewRows, kStaged };
const char *const kNames[] = {"a lane per chain", "a lane per chain in 64 bits", "a wave per chain", "a row per chain",
                              "a row per listed chain", "a row or a lane per listed chain", "a wave per chain of a ragged batch", "a row per chain of a ragged batch",
                              "a wave per long chain of a ragged batch", "a staged ragged batch"};

void launch_form(Form form, const int64_t *d, const int64_t *off, const int32_t *perm, int64_t batch, int n, Strides st,
                 uint8_t *mask, int64_t *peak, int32_t *status)
{
    char *const ws = (char *)emu::device_memory(linear_workspace_bytes(batch, n));
    LinearWs w = carve_linear(ws, batch, n);
    w.apart = form == kRowsAndLanes;
    if (form == kRowsAndLanes) w.lanes_few = w.lanes_large = kLanesPerLayer * n;
    const unsigned lanes = (unsigned)((batch + kWave - 1) / kWave), rows = (unsigned)((batch + kRowsOfWave - 1) / kRowsOfWave);
    hipLaunchKernelGGL(linear_reset_kernel, dim3(1), dim3(1), 0, nullptr, w);
    switch (form) {
    case kLanes:
    case kWideLanes:
    case kListedRows:
    case kRowsAndLanes:
        if (form == kLanes || form == kRowsAndLanes)
            hipLaunchKernelGGL(n <= kLogMaxLayers ? linear_ring_kernel<true> : linear_ring_kernel<false>, dim3(lanes),
                               dim3(kWave), 0, nullptr, d, batch, n, st.chain, st.pos, mask, peak, status, w);
        else
            hipLaunchKernelGGL(linear_defer_all_kernel, dim3((unsigned)((batch + 255) / 256)), dim3(256), 0, nullptr, batch, w);
        if (form == kListedRows || form == kRowsAndLanes)
            hipLaunchKernelGGL(linear_rows_list_kernel, dim3(rows), dim3(kWave), rows_all_lds_bytes(n, false), nullptr, d, n,
                               st.chain, st.pos, mask, peak, status, w, n, (const RaggedGroupDev *)nullptr, 0);
        if (form == kRowsAndLanes)
            hipLaunchKernelGGL(linear_wide_kernel<true>, dim3(lanes), dim3(kWave), 0, nullptr, d, n, st.chain, st.pos, mask, peak,
                               status, w, (const RaggedGroupDev *)nullptr, 0);
        else if (form != kListedRows)
            hipLaunchKernelGGL(linear_wide_kernel<false>, dim3(lanes), dim3(kWave), 0, nullptr, d, n, st.chain, st.pos, mask, peak,
                               status, w, (const RaggedGroupDev *)nullptr, 0);
        if (form != kRowsAndLanes) launch_list(d, n, st, mask, peak, status, w, batch, nullptr, 0, nullptr, 0, nullptr);
        break;
    case kWaves:
        launch_solve_linear(d, batch, n, st, mask, peak, status, ws, nullptr);  // (as few as these get a wave each)
        break;
    case kRows: {
        const bool own = n <= kRowsOwnListMaxLayers;
        hipLaunchKernelGGL(own ? linear_rows_kernel<true> : linear_rows_kernel<false>, dim3(rows), dim3(kWave),
                           rows_all_lds_bytes(n, own), nullptr, d, batch, n, st.chain, st.pos, mask, peak, status, w);
        if (!own) launch_list(d, n, st, mask, peak, status, w, batch, nullptr, 0, nullptr, (int)batch, nullptr);
        break;
    }
    case kFlatWaves: {
        RaggedTotals t = {};
        t.max_layers = n;
        launch_solve_linear_flat(d, off, perm, batch, t, mask, peak, status, ws, nullptr);
        break;
    }
    case kFlatRows:
    case kFlatFewRows: {  // (as many by a wave each as are longer than the others' rows; more than those that always are)
        int longest = kLongest;
        if (form == kFlatFewRows) longest += ((int)batch - longest) / 2;
        const int32_t last = perm[batch - longest - 1];
        const int n_rows = (int)(off[last + 1] - off[last] - 1);
        hipLaunchKernelGGL(linear_flat_kernel<true>, dim3(longest + (unsigned)((batch - longest + kRowsOfWave - 1) / kRowsOfWave)),
                           dim3(kWave), std::max(rows_all_lds_bytes(n_rows, false), wave_lds_bytes(n)), nullptr, d, off, perm,
                           batch, longest, n_rows, mask, peak, status, w);
        launch_list(d, n, Strides{0, 1}, mask, peak, status, w, batch, nullptr, 0, off, 0, nullptr);
        break;
    }
    case kStaged: {
        RaggedTotals t = {};
        RaggedGroupDev *const groups = (RaggedGroupDev *)emu::device_memory((size_t)n * sizeof(RaggedGroupDev));
        const auto length = [&](int64_t p) { return (int)(off[perm[p] + 1] - off[perm[p]] - 1); };
        for (int64_t p = 0, q; p < batch; p = q) {
            for (q = p; q < batch && length(q) == length(p); ++q) {}
            int64_t tile;
            const int k = t.n_groups;
            groups[k] = ragged_next_group(t, length(p), q - p, &tile);
        }
        const auto place = [&](const RaggedGroupDev &g, int64_t p, int k) { return (size_t)(g.stage_off + k * g.pitch + (p - g.first)); };
        int64_t *const staged = (int64_t *)emu::device_memory((size_t)t.staged * 8), *const peaks = (int64_t *)emu::device_memory((size_t)batch * 8);
        uint8_t *const masks = (uint8_t *)emu::device_memory((size_t)t.staged);
        int32_t *const codes = (int32_t *)emu::device_memory((size_t)batch * 4);
        for (int g = 0; g < t.n_groups; ++g)
            for (int64_t p = groups[g].first; p < groups[g].first + groups[g].count; ++p)
                for (int k = 0; k <= groups[g].n; ++k) staged[place(groups[g], p, k)] = d[off[perm[p]] + k];
        launch_solve_linear_ragged(staged, groups, t, batch, masks, peaks, codes, ws, nullptr);
        for (int g = 0; g < t.n_groups; ++g)
            for (int64_t p = groups[g].first; p < groups[g].first + groups[g].count; ++p) {
                for (int k = 0; k <= groups[g].n; ++k) mask[off[perm[p]] + k] = masks[place(groups[g], p, k)];
                peak[perm[p]] = peaks[p];
                status[perm[p]] = codes[p];
            }
        break;
    }
    }
}

// Chains by each of the forms: of one length where the form asks for that.
void check(const char *what, const std::vector<Sizes> &chains, std::initializer_list<Form> forms)
{
    const int64_t batch = (int64_t)chains.size();
    std::vector<int64_t> off = {0};
    std::vector<int> want_status;
    Sizes good;
    int n = 0;
    for (const Sizes &chain : chains) {
        __int128 sum = 0, most = 0;
        bool positive = true;
        for (const int64_t x : chain) {
            sum += x;
            most = x > most ? (__int128)x : most;
            positive &= x > 0;
        }
        want_status.push_back(!positive ? CKPT_ERR_SIZE : sum + most > (__int128)INT64_MAX ? CKPT_ERR_OVERFLOW : CKPT_OK);
        for (const int64_t x : chain) good.push_back(want_status.back() == CKPT_OK ? x : 1);
        off.push_back(off.back() + (int64_t)chain.size());
        n = std::max(n, (int)chain.size() - 1);
    }
    const size_t many = (size_t)off.back();
    std::vector<uint8_t> want_mask(many);
    Sizes want_peak((size_t)batch);
    orc_ragged_solve_dynamic(good.data(), off.data(), batch, want_mask.data(), want_peak.data());

    int64_t *const offsets = (int64_t *)emu::device_memory((size_t)(batch + 1) * 8);
    int32_t *const perm = (int32_t *)emu::device_memory((size_t)batch * 4);
    std::copy(off.begin(), off.end(), offsets);
    std::iota(perm, perm + batch, 0);
    std::stable_sort(perm, perm + batch, [&](int a, int b) { return chains[(size_t)a].size() < chains[(size_t)b].size(); });
    for (const Form form : forms) {
        for (int layout = 0; layout < (form >= kFlatWaves ? 1 : 2); ++layout) {  // chain after chain, position after position
            const Strides st = layout == 0 ? Strides{n + 1, 1} : Strides{1, batch};
            const auto place = [&](int64_t c, int64_t k) { return (size_t)(form >= kFlatWaves ? off[(size_t)c] + k : c * st.chain + k * st.pos); };
            int64_t *const d = (int64_t *)emu::device_memory(many * 8);
            uint8_t *const mask = (uint8_t *)emu::device_memory(many);
            int64_t *const peak = (int64_t *)emu::device_memory((size_t)batch * 8);
            int32_t *const status = (int32_t *)emu::device_memory((size_t)batch * 4);
            for (int64_t c = 0; c < batch; ++c)
                for (size_t k = 0; k < chains[(size_t)c].size(); ++k) d[place(c, (int64_t)k)] = chains[(size_t)c][k];
            launch_form(form, d, offsets, perm, batch, n, st, mask, peak, status);
            bool ok = true;
            for (int64_t c = 0; c < batch && ok; ++c) {
                const bool bad = want_status[(size_t)c] != CKPT_OK;
                ok = status[c] == want_status[(size_t)c] && peak[c] == (bad ? -1 : want_peak[(size_t)c]);
                for (size_t k = 0; k < chains[(size_t)c].size() && ok; ++k)
                    ok = mask[place(c, (int64_t)k)] == (bad ? 0 : want_mask[(size_t)off[(size_t)c] + k]);
                if (!ok)
                    printf("%s, n = %d, chain %d, %s: status %d (%d), peak %lld (%lld)\n", what, (int)chains[(size_t)c].size() - 1,
                           (int)c, kNames[form], (int)status[c], want_status[(size_t)c], (long long)peak[c],
                           (long long)want_peak[(size_t)c]);
            }
            failures += !ok;
        }
    }
}

const auto kEqualLengths = {kLanes, kWideLanes, kWaves, kRows, kListedRows};

std::vector<Sizes> kinds(int n)
{
    const int64_t top = INT64_MAX;
    std::vector<Sizes> chains = {uniform(n, 1, 1000000), uniform(n, 1, 3), uniform(n, 7, 7), uniform(n, 256, 32768), uniform(n, 1, top / (2 * n + 4)),
                                 with(uniform(n, 1, 9), n / 2, 0), with(uniform(n, 1, 9), n, -5), with(uniform(n, 1, 9), 0, top),
                                 with(uniform(n, 1, top / (n + 3)), n / 2, top / 2), live_entries(n)};
    for (int64_t &x : chains[3]) x *= 4096;
    Sizes up = chains[1], down = up, powers = up;
    for (int k = 0; k <= n; ++k) {
        up[(size_t)k] = k + 1;
        down[(size_t)k] = n + 1 - k;
        powers[(size_t)k] = 1ll << between(0, 40);
    }
    chains.insert(chains.end(), {up, down, powers});
    for (const int64_t most : {(int64_t)1 << 30, (int64_t)1 << 52, (int64_t)1 << 62, top})
        for (const int k : {0, n / 2, n})
            if (n > 2)
                for (int less = 0; less < 2; ++less) chains.push_back(up_to(n, k, most - less));
    return chains;
}
}  // namespace

int main()
{
    for (const int n : {1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 100, 130, 257, 330}) check("kinds of sizes", kinds(n), kEqualLengths);
    // sum(d) + max(d) in the upper half of 32 bits, and on both sides of what they take
    std::vector<Sizes> all;
    for (const int n : {3, 15, 16, 17, 47, 64, 65, 100}) {
        std::vector<Sizes> chains;
        for (const int k : {0, 1, n / 2, n - 1, n})
            for (int less = 0; less < 5; ++less) {
                chains.push_back(up_to(n, k, (1ll << 32) - less));
                chains.push_back(with(uniform(n, 1, ((1ll << 32) - 8) / (n + 2)), k, (1ll << 32) / (n + 2) - less));
            }
        check("the upper half of 32 bits", chains, kEqualLengths);
        all.insert(all.end(), chains.begin(), chains.end());
    }
    check("the upper half of 32 bits, ragged", all, {kFlatWaves, kFlatRows, kFlatFewRows, kStaged});
    // ever fewer trailing zeros towards the front, with sizes up to the lanes' limit of 2^24 before and after each of them
    for (const int n : {9, 12, 17, 24}) {
        std::vector<Sizes> chains;
        for (int c = 0; c < 400; ++c) {
            Sizes d = uniform(n, 1, 1 << 22);
            for (int k = 0; k <= n; ++k) {
                if (rng() % 4 == 0) d[(size_t)k] = between(1 << 22, (1 << 24) + (1 << 23));
                d[(size_t)k] = std::max<int64_t>(1, d[(size_t)k] >> (k / 3)) << (k / 3);
            }
            chains.push_back(d);
        }
        check("fewer trailing zeros", chains, {kLanes});
    }
    // what the lanes defer, on both sides of the numbers from which on the lanes of the next kernel take it
    for (const int few : {2 * kLanesPerLayer - 1, 2 * kLanesPerLayer})
        for (const int large : {2 * kLanesPerLayer - 1, 2 * kLanesPerLayer}) {
            std::vector<Sizes> chains;
            for (int c = 0; c < few; ++c) chains.push_back(with(uniform(2, 1ll << 31, 1ll << 34), 1, c % 500 ? (1ll << 32) + 1 : -c));
            for (int c = 0; c < large; ++c) chains.push_back(with(uniform(2, 1ll << 60, INT64_MAX / 5), 0, c % 500 ? (1ll << 59) + 1 : INT64_MAX));
            std::shuffle(chains.begin(), chains.end(), rng);
            check("deferred chains", chains, {kRowsAndLanes});
        }
    for (const int longest : {5, 40, 200}) {
        std::vector<Sizes> chains;
        while (chains.size() < 90)
            for (const Sizes &d : kinds((int)between(1, longest))) chains.push_back(d);
        check("ragged", chains, {kFlatWaves, kFlatRows, kFlatFewRows, kStaged});
    }
    // many short chains and a few deep ones: what the lanes leave of them goes to rows with LDS for the short ones, more
    // than so many that each gets a wave
    for (const int longest : {40, kDeepLayers + 20}) {
        std::vector<Sizes> chains;
        for (int c = 0; c < kListedAlone + 100; ++c) {
            const int n = (int)between(17, 24);
            chains.push_back(c % 300 == 0 ? with(uniform(n, 1, 9), n / 2, c % 600 ? -1 : INT64_MAX)
                                          : uniform(n, 1ll << 31, c % 3 ? 1ll << 40 : INT64_MAX / 32));
        }
        for (int c = 0; c < 2; ++c) chains.push_back(uniform(longest - c, 1ll << 31, 1ll << (c ? 34 : 50)));
        for (const int n : {130, 257, 300}) chains.push_back(live_entries(std::min(n, longest)));
        std::shuffle(chains.begin(), chains.end(), rng);
        check("ragged, deep chains", chains, {kStaged, kFlatRows});
    }
    printf(failures ? "linear_driver: %d failed\n" : "linear_driver ok\n", failures);
    return failures != 0;
}
