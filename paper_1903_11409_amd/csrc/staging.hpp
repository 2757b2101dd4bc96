// Pinned host memory that plan creation writes its tables (and the caller's CSR arrays) into, so that
// ONE asynchronous copy brings everything to the device and the call returns at once: copies from
// pageable memory cost 3 to 14 us of host time each and, where the source may be reused, a wait for
// the stream.  The copy is a kernel that reads the pinned memory: a copy engine's transfer takes
// 8 us for 160 KB however small, and the queues wait for each other before and after it (128
// molecules, plan + two products: 36 us a step through the copy engine, 30 us with the kernel).
#pragma once

#include <hip/hip_runtime_api.h>

#include <chrono>
#include <cstddef>
#include <cstdint>
#include <thread>

namespace bspmm {

constexpr size_t kStageBlockMax = (size_t)8 << 20;   // larger plans are copied from pageable memory
constexpr size_t kStagePoolMax = (size_t)32 << 20;   // pinned memory the pool holds at most

// A block of the pool, taken for one copy.  Blocks go back by themselves when the copy has run.
struct StageBlock {
    char* ptr = nullptr;
    void* slot = nullptr;
};

// A block of at least `bytes` on the current device, or {nullptr} (too large, pool exhausted, no
// memory): the caller then copies from pageable memory.  Waits for no copy; making room in a full pool
// frees blocks, which may wait for the device.
StageBlock stage_take(size_t bytes);

// A copy that has been enqueued.
struct StagedCopy {
    const void* slot = nullptr;
    uint32_t mark = 0;
};

// Enqueue the copy of the block's first `bytes` (a multiple of 16) to `dst` and hand the block back:
// it is reused only after the copy has run.
hipError_t stage_copy(StageBlock b, void* dst, size_t bytes, hipStream_t stream, StagedCopy* copy);

// Returns hipSuccess when the copy, which was enqueued on `stream`, has run and what it wrote is visible to
// work enqueued from now on, on any stream; the error when it never will.
hipError_t stage_wait(const StagedCopy& copy, hipStream_t stream);

// The same for a copy from pageable memory, by an event that was recorded behind it.
hipError_t event_wait(hipEvent_t copied);

// The wait itself: until done(), but no longer than state() (what the runtime says of the work waited for)
// is hipErrorNotReady.  state() is asked from the second millisecond on only, ten times a millisecond.
template <typename Done, typename State>
hipError_t wait_until(Done done, State state)
{
    using Clock = std::chrono::steady_clock;
    Clock::time_point ask = Clock::now() + std::chrono::milliseconds(1);
    while (!done()) {
        std::this_thread::yield();
        if (Clock::now() < ask) continue;
        const hipError_t e = state();
        if (e != hipErrorNotReady) return done() ? hipSuccess : e == hipSuccess ? hipErrorUnknown : e;
        std::this_thread::sleep_for(std::chrono::microseconds(100));
    }
    return hipSuccess;
}

// Plans that exist: when the last one goes and none has been made for a second, idle blocks are freed
// (which may wait for the device).
void stage_plan_made();
void stage_plan_gone();

}  // namespace bspmm
