// Drives csrc/host_copy.hpp over a runtime of its own: device memory is host memory, work
// is queued and done only when its stream or an event on it is waited for (so that a result
// read too early is wrong), and pinned memory or events can be refused.  Prints the number
// of failures.
#include <cstdio>
#include <deque>
#include <functional>
#include <random>

#include "paper_1407_5140_amd/csrc/host_copy.hpp"

using namespace rewl;

static std::deque<std::function<void()>> g_queue;
static long g_marks_done = 0, g_marks = 0, g_live = 0, g_launches = 0, g_misaligned = 0, g_slots = 0;
static int g_refuse_pinned = 0, g_refuse_events = 0, g_fail_copy = 0;
static hipError_t g_last = hipSuccess;
static const int k_collect = 0;                      // its address names the kernel

static hipError_t report(hipError_t e) { return g_last = e; }
static void drain(const std::function<bool()>& enough)
{
    while (!g_queue.empty() && !enough()) {
        g_queue.front()();
        g_queue.pop_front();
    }
}

extern "C" {
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (g_refuse_pinned) return report(hipErrorOutOfMemory);
    ++g_live;
    ++g_slots;
    *p = malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    --g_live;
    free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned)
{
    if (g_refuse_events) return report(hipErrorOutOfMemory);
    ++g_live;
    *e = (hipEvent_t) new long(0);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    --g_live;
    delete (long*)e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    *(long*)e = ++g_marks;
    g_queue.push_back([] { ++g_marks_done; });
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    const long mark = *(long*)e;
    drain([=] { return g_marks_done >= mark; });
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t)
{
    drain([] { return false; });
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (g_fail_copy && --g_fail_copy == 0) return report(hipErrorUnknown);
    g_queue.push_back([=] { memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t)
{
    if (f != &k_collect) return report(hipErrorInvalidDeviceFunction);
    const Collect c = *(const Collect*)args[0];      // arguments are taken at the launch
    char* out = *(char**)args[1];
    ++g_launches;
    if ((int)grid.x != c.n || c.n < 1 || c.n > kCollect) return report(hipErrorInvalidConfiguration);
    for (int i = 0; i < c.n; ++i) g_misaligned += ((uintptr_t)c.src[i] | c.off[i]) & 15 ? 1 : 0;
    g_queue.push_back([=] {
        for (int i = 0; i < c.n; ++i) memcpy(out + c.off[i], c.src[i], c.bytes[i]);
    });
    return hipSuccess;
}
}

static int g_fails = 0;
static void check(bool ok, const char* what, const char* name)
{
    if (ok) return;
    ++g_fails;
    std::printf("FAIL %s: %s\n", name, what);
}

// pieces of the given sizes, each behind the last at a multiple of 256, copied and compared
static hipError_t pass(const char* name, const std::vector<size_t>& sizes, bool with_stage, bool expect = true)
{
    size_t total = 0, out = 0;
    for (size_t s : sizes) {
        total += (s + 255) & ~size_t(255);
        out += s;
    }
    char* dev = (char*)aligned_alloc(256, total + 256);
    std::mt19937 rng(1);
    for (size_t i = 0; i < total; i += 4) {
        const uint32_t v = rng();
        memcpy(dev + i, &v, 4);
    }
    std::vector<char> host(out + 1, 0x5a), stage(with_stage ? kStageBytes : 0);
    std::vector<Piece> p;
    size_t at = 0, to = 0;
    for (size_t s : sizes) {
        p.push_back({host.data() + to, dev + at, s});
        at += (s + 255) & ~size_t(255);
        to += s;
    }
    g_launches = g_misaligned = g_slots = 0;
    const hipError_t e = copy_pieces(nullptr, with_stage ? stage.data() : nullptr, &k_collect, p);
    if (expect) {
        bool same = e == hipSuccess;
        for (const Piece& q : p) same = same && memcmp(q.dst, q.src, q.bytes) == 0;
        check(same, "bytes", name);
        check(host[out] == 0x5a, "written beyond the end", name);
        check(g_queue.empty(), "work left in the queue", name);
        check(g_last == hipSuccess, "an error left for the next call", name);
    }
    check(g_misaligned == 0, "a collected piece not at a multiple of 16", name);
    check(g_live == 0, "pinned memory or events not released", name);
    drain([] { return false; });
    free(dev);
    return e;
}

int main()
{
    const size_t M = size_t(1) << 20;
    std::vector<size_t> few = {16, 40, 1, 15, 17, 0, 65535, 65536, 8};
    std::vector<size_t> many, full, mixed;
    for (int i = 0; i < 200; ++i) many.push_back((size_t)(i * 37 % 300));
    for (int i = 0; i < 40; ++i) full.push_back(65536 - (i % 3) * 7);
    for (int i = 0; i < 70; ++i) {
        mixed.push_back((size_t)(i * 1013 % 60000));
        if (i % 9 == 0) mixed.push_back(kPieceBytes + 1 + i);
        if (i % 23 == 5) mixed.push_back(2 * kSlotBytes + (i == 5 ? 0 : M / 3 + i));
    }
    mixed.push_back(2 * kSlotBytes - 1);
    mixed.push_back(5 * kSlotBytes);
    for (int pinned = 0; pinned < 2; ++pinned)
        for (int events = 0; events < 2; ++events)
            for (bool stage : {true, false}) {
                g_refuse_pinned = pinned;
                g_refuse_events = events;
                pass("few", few, stage);
                pass("many", many, stage);
                check(!stage || g_launches == 4, "200 pieces (some empty) are four launches", "many");
                pass("full", full, stage);
                pass("mixed", mixed, stage);
                check((g_slots > 0) == !pinned, "large pieces through the slots", "mixed");
            }
    g_refuse_pinned = g_refuse_events = 0;
    for (int k : {1, 3, 6}) {                        // a copy that fails is reported, and nothing is left behind
        g_fail_copy = k;
        check(pass("failing", {2 * kSlotBytes + 5, 64, 3 * kSlotBytes}, true, false) == hipErrorUnknown, "status", "failing");
        g_fail_copy = 0;
        g_last = hipSuccess;
    }
    std::printf("copies checked, %d failures\n", g_fails);
    return g_fails;
}
