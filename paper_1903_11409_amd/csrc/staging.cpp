// Pool of pinned staging blocks (see staging.hpp).
#include "staging.hpp"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <thread>
#include <vector>

namespace bspmm {

hipError_t launch_stage_copy(const void* from, void* to, size_t bytes, uint32_t* done, uint32_t mark, int grid,
                             hipStream_t stream);

namespace {

using Clock = std::chrono::steady_clock;

// In front of a block's data: a word per workgroup of the copy kernel, which writes the copy's mark
// there when it has read its share (an event instead costs 1 us of host time per plan).
constexpr size_t kMarks = 64, kHeader = 256;

struct Slot {
    char* base = nullptr;
    size_t size = 0;             // bytes of data
    int device = -1;
    uint32_t mark = 0;           // of the copy under way
    int grid = 0;                // ... and its workgroups
    enum State { kIdle, kTaken, kCopying } state = kIdle;
    char* data() const { return base + kHeader; }
    uint32_t* marks() const { return reinterpret_cast<uint32_t*>(base); }
};

struct Pool {
    std::mutex lock;
    std::vector<std::unique_ptr<Slot>> slots;
    size_t bytes = 0;
    size_t next = 0;             // where the search for an idle block begins: the one longest in use
    int64_t plans = 0;
    Clock::time_point last_plan = Clock::now();
};

// (never destroyed: plans may be released while the process ends)
Pool& pool()
{
    static Pool* p = new Pool;
    return *p;
}

// Allocating and freeing pinned memory is harmless to a stream capture that another thread has open,
// but counts as unsafe there unless the calling thread says so.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { swap(); }
    ~RelaxedCapture() { swap(); }
    void swap()
    {
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) (void)hipGetLastError();
    }
};

bool idle(Slot& s)
{
    if (s.state == Slot::kCopying) {
        for (int i = 0; i < s.grid; ++i)
            if (__atomic_load_n(s.marks() + i, __ATOMIC_ACQUIRE) != s.mark) return false;
        s.state = Slot::kIdle;
    }
    return s.state == Slot::kIdle;
}

// Blocks that have left the pool.  Freeing pinned memory may wait for the device, so it is done after the
// lock has been given up: declared before the lock's guard.
struct Gone {
    std::vector<char*> blocks;
    ~Gone()
    {
        for (char* b : blocks) (void)hipHostFree(b);
    }
};

// Idle blocks go, until at most `keep` bytes are held.
void shrink(Pool& p, size_t keep, Gone& gone)
{
    for (size_t i = 0; i < p.slots.size() && p.bytes > keep;) {
        if (!idle(*p.slots[i])) {
            ++i;
            continue;
        }
        p.bytes -= p.slots[i]->size;
        gone.blocks.push_back(p.slots[i]->base);
        p.slots.erase(p.slots.begin() + (ptrdiff_t)i);
    }
    p.next = 0;
}

}  // namespace

StageBlock stage_take(size_t bytes)
{
    if (bytes == 0 || bytes > kStageBlockMax) return {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return {};
    }
    const RelaxedCapture relaxed;
    Gone gone;
    Pool& p = pool();
    std::lock_guard<std::mutex> g(p.lock);
    for (size_t j = 0; j < p.slots.size(); ++j) {
        const size_t at = (p.next + j) % p.slots.size();
        Slot& s = *p.slots[at];
        if (s.device == dev && s.size >= bytes && s.size <= 16 * bytes + ((size_t)1 << 20) && idle(s)) {
            s.state = Slot::kTaken;
            p.next = at + 1;
            return {s.data(), &s};
        }
    }
    size_t size = (size_t)256 << 10;
    while (size < bytes) size *= 2;
    if (p.bytes + size > kStagePoolMax) shrink(p, kStagePoolMax - size, gone);
    if (p.bytes + size > kStagePoolMax) return {};
    void* q = nullptr;
    if (hipHostMalloc(&q, kHeader + size, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return {};
    }
    auto s = std::make_unique<Slot>();
    s->base = static_cast<char*>(q);
    s->device = dev;
    s->size = size;
    s->state = Slot::kTaken;
    std::memset(s->base, 0, kHeader);
    p.bytes += size;
    p.slots.push_back(std::move(s));
    return {p.slots.back()->data(), p.slots.back().get()};
}

hipError_t stage_copy(StageBlock b, void* dst, size_t bytes, hipStream_t stream, StagedCopy* copy)
{
    Slot& s = *static_cast<Slot*>(b.slot);
    static std::atomic<uint32_t> next_mark{0};
    // (no two copies under way have the same one; a new block's words are zero)
    uint32_t mark = ++next_mark;
    if (mark == 0) mark = ++next_mark;
    // (4 KiB a workgroup: 16 bytes a lane, all of a plan's tables in flight at once)
    const int grid = (int)std::min<size_t>(kMarks, (bytes + 4095) / 4096);
    const hipError_t e = launch_stage_copy(b.ptr, dst, bytes, s.marks(), mark, grid, stream);
    std::lock_guard<std::mutex> g(pool().lock);
    s.mark = mark;
    s.grid = e == hipSuccess ? grid : 0;
    s.state = Slot::kCopying;
    *copy = {&s, mark};
    return e;
}

hipError_t stage_wait(const StagedCopy& copy, hipStream_t stream)
{
    Pool& p = pool();
    auto done = [&] {
        // (a block that has gone, or carries another mark, was idle in between: the copy has run)
        std::lock_guard<std::mutex> g(p.lock);
        for (auto& s : p.slots)
            if (s.get() == copy.slot && s->mark == copy.mark && s->state == Slot::kCopying) return idle(*s);
        return true;
    };
    auto state = [&]() -> hipError_t {
        if (stream == hipStreamPerThread) return hipErrorNotReady;     // (names this thread's stream here)
        const RelaxedCapture relaxed;      // (the caller may be recording a graph on its stream)
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        hipError_t e = hipStreamIsCapturing(stream, &st);
        // (a stream that has begun to record since then, or the null stream while another one records, cannot
        // be asked; what came before still runs)
        if (e == hipSuccess) e = st == hipStreamCaptureStatusNone ? hipStreamQuery(stream) : hipErrorNotReady;
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipErrorStreamCaptureImplicit ? hipErrorNotReady : e;
    };
    return wait_until(done, state);
}

hipError_t event_wait(hipEvent_t copied)
{
    const RelaxedCapture relaxed;
    return hipEventSynchronize(copied);
}

void stage_plan_made()
{
    Pool& p = pool();
    std::lock_guard<std::mutex> g(p.lock);
    ++p.plans;
    p.last_plan = Clock::now();
}

void stage_plan_gone()
{
    const RelaxedCapture relaxed;
    Gone gone;
    Pool& p = pool();
    std::lock_guard<std::mutex> g(p.lock);
    if (--p.plans > 0 || p.slots.empty() || Clock::now() - p.last_plan < std::chrono::seconds(1)) return;
    shrink(p, 0, gone);
}

}  // namespace bspmm
