// host_copy.hpp -- device memory on its way to the host.  Host code alone, over the
// runtime's C entry points.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <algorithm>
#include <cstring>
#include <vector>

namespace rewl {

// Large copies into pageable memory go through two pinned slots in turn, the host
// copying one out while the other fills (50 MB: 2.9 -> 2.3 ms).  Where pinned memory
// cannot be had, the copy is a pageable one.
constexpr size_t kSlotBytes = size_t(4) << 20;
inline hipError_t copy_out(hipStream_t st, void* dst, const void* src, size_t bytes)
{
    if (bytes < 2 * kSlotBytes) return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
    struct Slots {
        char* p = nullptr;
        hipEvent_t done[2] = {nullptr, nullptr};
        ~Slots()
        {
            for (hipEvent_t e : done)
                if (e) (void)hipEventDestroy(e);
            if (p) (void)hipHostFree(p);
        }
    } s;
    hipError_t e = hipHostMalloc((void**)&s.p, 2 * kSlotBytes, hipHostMallocDefault);
    for (int i = 0; i < 2 && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&s.done[i], hipEventDisableTiming);
    if (e != hipSuccess) {
        (void)hipGetLastError();                     // not to be taken for a later call's
        return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
    }
    const size_t n = (bytes + kSlotBytes - 1) / kSlotBytes;
    auto size_of = [&](size_t k) { return std::min(kSlotBytes, bytes - k * kSlotBytes); };
    for (size_t k = 0; k <= n && e == hipSuccess; ++k) {
        if (k < n) {
            e = hipMemcpyAsync(s.p + (k & 1) * kSlotBytes, (const char*)src + k * kSlotBytes, size_of(k), hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(s.done[k & 1], st);
        }
        if (k > 0 && e == hipSuccess && (e = hipEventSynchronize(s.done[(k - 1) & 1])) == hipSuccess)
            std::memcpy((char*)dst + (k - 1) * kSlotBytes, s.p + ((k - 1) & 1) * kSlotBytes, size_of(k - 1));
    }
    if (e != hipSuccess) (void)hipStreamSynchronize(st);      // nothing may still write the slots
    return e;
}

// A copy into pageable memory costs 10 to 15 us whatever its size, and a state has 9 to
// 15 pieces per instance: pieces up to kPieceBytes are therefore written into a pinned
// stage by k_collect, up to kCollect of them per launch, and copied out after one wait
// (4-walker Ising L = 8 instance: state 156 -> 32 us, checkpoint 217 -> 15 us).
constexpr size_t kStageBytes = size_t(1) << 20, kPieceBytes = size_t(1) << 16;
constexpr int kCollect = 64;
struct Collect {
    const char* src[kCollect];                       // multiples of 16
    uint32_t off[kCollect], bytes[kCollect];         // off: a multiple of 16
    int32_t n;
};

struct Piece {
    void* dst;
    const void* src;
    size_t bytes;
};

// The pieces, in host memory when it returns.  stage: kStageBytes of pinned memory, or null
// (each piece is then copied by itself); kernel: k_collect.
inline hipError_t copy_pieces(hipStream_t st, char* stage, const void* kernel, const std::vector<Piece>& pieces)
{
    size_t i = 0;
    while (i < pieces.size()) {
        Collect c{};
        std::vector<const Piece*> staged;
        size_t used = 0;
        hipError_t e = hipSuccess;
        auto collect = [&]() {
            void* args[] = {&c, &stage};
            const hipError_t r = hipLaunchKernel(kernel, dim3(c.n), dim3(256), args, 0, st);
            c.n = 0;
            return r;
        };
        for (; i < pieces.size(); ++i) {               // one stage full
            const Piece& q = pieces[i];
            if (q.bytes == 0) continue;
            if (!stage || q.bytes > kPieceBytes) {
                e = copy_out(st, q.dst, q.src, q.bytes);
                if (e != hipSuccess) break;
                continue;
            }
            const size_t room = (q.bytes + 15) & ~size_t(15);
            if (used + room > kStageBytes) break;
            c.src[c.n] = (const char*)q.src;
            c.off[c.n] = (uint32_t)used;
            c.bytes[c.n] = (uint32_t)q.bytes;
            staged.push_back(&q);
            used += room;
            if (++c.n == kCollect && (e = collect()) != hipSuccess) break;
        }
        if (e == hipSuccess && c.n > 0) e = collect();
        const hipError_t e2 = hipStreamSynchronize(st);
        if (e == hipSuccess) e = e2;
        if (e != hipSuccess) return e;
        size_t off = 0;
        for (const Piece* q : staged) {
            std::memcpy(q->dst, stage + off, q->bytes);
            off += (q->bytes + 15) & ~size_t(15);
        }
    }
    return hipSuccess;
}

}  // namespace rewl
