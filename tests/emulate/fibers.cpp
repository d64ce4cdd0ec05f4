// The lanes of a workgroup as fibers (x86-64): each runs until it meets the others of its wave, or of the workgroup.
#include "hip/hip_runtime.h"

#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>

#include <map>

namespace emu {

dim3 thread, block, threads, blocks;
unsigned char *dynamic_lds;
uint64_t rendezvous_limit = ~0ull;
std::function<void()> meanwhile;
std::function<void(const char *, dim3)> instead_of_running;

namespace {
constexpr unsigned kMostLanes = 1024;
constexpr size_t kStack = 128 << 10, kPage = 4096;
constexpr size_t kLdsOfACu = 160 << 10, kLdsLimit = 64 << 10;

struct Lane {
    void *sp;
    Kind waits;  // kNone: runs
    int turn;
    bool ended;
};
struct Wave {
    uint64_t brought[2][kLanes];  // (a lane is at most one meeting ahead of another)
    uint64_t part;
};
Lane lanes[kMostLanes];
Wave waves[kMostLanes / kLanes];
Lane *now;
char *stacks;
void *scheduler;
const std::function<void()> *kernel;
const char *kernel_name;
uint64_t meetings;
std::map<const void *, size_t> lds_limit;

extern "C" void emu_switch(void **save, void *to);
asm(".text\n.globl emu_switch\nemu_switch:\n"
    "push %rbp\npush %rbx\npush %r12\npush %r13\npush %r14\npush %r15\n"
    "mov %rsp, (%rdi)\nmov %rsi, %rsp\n"
    "pop %r15\npop %r14\npop %r13\npop %r12\npop %rbx\npop %rbp\nret\n");

void lane_entry()
{
    (*kernel)();
    now->ended = true;
    emu_switch(&now->sp, scheduler);
    abort();
}

void resume(unsigned t)
{
    now = &lanes[t];
    now->waits = kNone;
    thread = dim3(t);
    emu_switch(&scheduler, now->sp);
}

// Lets the wave go on as long as all its lanes meet in the same operation; false once none of them can.
bool run_wave(unsigned w, unsigned count)
{
    const unsigned first = w * kLanes, end = std::min(count, first + kLanes);
    bool moved = false;
    for (;;) {
        Kind kind = kNone;
        uint64_t part = 0;
        for (unsigned t = first; t < end; ++t) {
            if (lanes[t].ended) continue;
            if (kind != kNone && lanes[t].waits != kind) stop("the lanes of a wave are apart");
            kind = lanes[t].waits;
            part |= 1ull << (t - first);
        }
        if (kind == kNone || kind == kBarrier) return moved;
        if (++meetings > rendezvous_limit) stop("does not end");
        waves[w].part = part;
        for (unsigned t = first; t < end; ++t)
            if (!lanes[t].ended) resume(t);
        moved = true;
    }
}
}  // namespace

void stop(const char *why)
{
    printf("%s: %s\n", kernel_name, why);
    exit(1);
}

const uint64_t *meet(uint64_t value, Kind kind)
{
    Wave &w = waves[thread.x / kLanes];
    Lane *me = now;
    uint64_t *brought = w.brought[me->turn];
    me->turn ^= 1;
    brought[lane()] = value;
    me->waits = kind;
    emu_switch(&me->sp, scheduler);
    return brought;
}

uint64_t taking_part() { return waves[thread.x / kLanes].part; }

void *device_memory(size_t bytes)
{
    const size_t body = (bytes + 15) / 16 * 16, pages = (body + kPage - 1) / kPage * kPage;
    char *p = (char *)mmap(nullptr, pages + 2 * kPage, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (p == MAP_FAILED || mprotect(p + kPage, pages, PROT_READ | PROT_WRITE) != 0) abort();
    memset(p + kPage, 0xcd, pages);
    return p + kPage + pages - body;
}

void launch(const char *name, const void *entry, dim3 grid, dim3 group, size_t lds, const std::function<void()> &f)
{
    kernel_name = name;
    kernel = &f;
    meetings = 0;
    if (group.x > kMostLanes || (uint64_t)grid.x * group.x > UINT32_MAX || lds > kLdsOfACu) stop("no such launch");
    if (lds > kLdsLimit && (!lds_limit.count(entry) || lds > lds_limit[entry])) stop("more LDS than is allowed");
    if (instead_of_running) {
        instead_of_running(name, grid);
        return;
    }
    if (!stacks)
        stacks = (char *)mmap(nullptr, kMostLanes * kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    blocks = grid;
    threads = group;
    dynamic_lds = (unsigned char *)device_memory(lds + 1);
    for (unsigned y = 0; y < grid.y; ++y) {
        for (unsigned x = 0; x < grid.x; ++x) {
            block = dim3(x, y, 0);
            for (unsigned t = 0; t < group.x; ++t) {
                void **sp = (void **)(stacks + (t + 1) * kStack);
                *--sp = nullptr;
                *--sp = (void *)lane_entry;
                for (int k = 0; k < 6; ++k) *--sp = nullptr;
                lanes[t] = Lane{sp, kNone, 0, false};
            }
            for (unsigned t = 0; t < group.x; ++t) resume(t);
            for (;;) {
                bool moved = false, waits = false;
                for (unsigned w = 0; w * kLanes < group.x; ++w) moved |= run_wave(w, group.x);
                if (moved) continue;
                for (unsigned t = 0; t < group.x; ++t) {
                    if (lanes[t].ended) continue;
                    waits = true;
                    resume(t);
                }
                if (!waits) break;
            }
        }
    }
    const size_t pages = (lds + 1 + 15) / 16 * 16;
    munmap((void *)((uintptr_t)dynamic_lds / kPage * kPage - kPage), (pages + kPage - 1) / kPage * kPage + 2 * kPage);
}

}  // namespace emu

hipError_t hipFuncSetAttribute(const void *kernel, int, int bytes)
{
    emu::lds_limit[kernel] = (size_t)bytes;
    std::function<void()> other;
    std::swap(other, emu::meanwhile);  // (once)
    if (other) other();
    return hipSuccess;
}
