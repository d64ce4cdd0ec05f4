// The kernels of csrc/eval_peak.hip and csrc/eval_timeline.hip on the CPU, against the oracle, and what two host threads
// do to each other between the LDS limit of a kernel and its launch.
#include "ckpt_internal.h"

#include <stdio.h>

#include <random>
#include <vector>

extern "C" void orc_batch_peak(const int64_t *, const uint8_t *, int64_t, int, int, int64_t *);
extern "C" void orc_batch_timeline(const int64_t *, const uint8_t *, int64_t, int, int, int64_t *);

using namespace ckpt;

namespace {
std::mt19937_64 rng(3);
int failures = 0;

template <class T>
T *memory(int64_t count) { return (T *)emu::device_memory((size_t)count * sizeof(T)); }

struct Batch {
    int64_t chains, n1;
    int64_t *d;
    uint8_t *mask;
    Batch(int64_t batch, int n) : chains(batch), n1(n + 1), d(memory<int64_t>(batch * n1)), mask(memory<uint8_t>(batch * n1))
    {
        for (int64_t k = 0; k < batch * n1; ++k) {
            d[k] = 1 + (int64_t)(rng() % 1000000);
            mask[k] = k % n1 == 0 || k % n1 == n || rng() % 4 == 0;
        }
    }
};

void peak(int64_t batch, int n, int objective)
{
    const Batch b(batch, n);
    const int values = objective == CKPT_OBJ_BOTH ? 2 : 1;
    int64_t *got = memory<int64_t>(batch * values);
    int32_t *status = memory<int32_t>(batch);
    bool ok = launch_eval_peak(b.d, b.mask, batch, n, Strides{b.n1, 1}, objective, got, status, nullptr) == hipSuccess;
    for (int v = 0; v < values; ++v) {
        std::vector<int64_t> want((size_t)batch);
        orc_batch_peak(b.d, b.mask, batch, n, objective == CKPT_OBJ_BOTH ? v : objective, want.data());
        for (int64_t c = 0; c < batch; ++c) ok &= got[v * batch + c] == want[(size_t)c] && status[c] == CKPT_OK;
    }
    if (!ok) printf("peak, %d chains of %d layers, objective %d\n", (int)batch, n, objective);
    failures += !ok;
}

void timeline(int64_t batch, int n, int objective)
{
    const Batch b(batch, n);
    int64_t *got = memory<int64_t>(batch * 2 * b.n1);
    int32_t *status = memory<int32_t>(batch);
    std::vector<int64_t> want((size_t)(batch * 2 * b.n1));
    orc_batch_timeline(b.d, b.mask, batch, n, objective, want.data());
    bool ok = launch_eval_timeline(b.d, b.mask, batch, n, Strides{b.n1, 1}, objective, got, Strides{2 * b.n1, 1}, status,
                                   nullptr) == hipSuccess;
    for (int64_t k = 0; k < batch * 2 * b.n1; ++k) ok &= got[k] == want[(size_t)k];
    if (!ok) printf("timeline, %d chains of %d layers, objective %d\n", (int)batch, n, objective);
    failures += !ok;
}
}  // namespace

int main()
{
    // a call with less LDS comes between another one's limit and its launch
    emu::meanwhile = [] { timeline(1, 560, CKPT_OBJ_STATIC); };
    timeline(1, 1024, CKPT_OBJ_STATIC);
    emu::meanwhile = [] { timeline(1, 560, CKPT_OBJ_DYNAMIC); };
    timeline(1, 1024, CKPT_OBJ_DYNAMIC);
    emu::meanwhile = nullptr;
    for (const int objective : {CKPT_OBJ_STATIC, CKPT_OBJ_DYNAMIC}) {
        for (const int n : {1, 7, 32, 33, 512, 513, 600, 1024, 1025}) timeline(n == 33 ? 65 : 3, n, objective);
    }
    for (const int objective : {CKPT_OBJ_STATIC, CKPT_OBJ_DYNAMIC, CKPT_OBJ_BOTH}) {
        for (const int n : {1, 16, 31, 32, 127, 128, 129, 640}) peak(n == 32 ? 65 : 3, n, objective);  // 1 to 16 waves
    }
    printf(failures ? "eval_driver: %d failed\n" : "eval_driver ok\n", failures);
    return failures != 0;
}
