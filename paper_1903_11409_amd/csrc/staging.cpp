// Pool of pinned staging blocks (see staging.hpp).
#include "staging.hpp"

#include <chrono>
#include <memory>
#include <mutex>
#include <vector>

namespace bspmm {

namespace {

using Clock = std::chrono::steady_clock;

struct Slot {
    char* ptr = nullptr;
    size_t size = 0;
    int device = -1;
    hipEvent_t done = nullptr;
    enum State { kIdle, kTaken, kCopying } state = kIdle;
};

struct Pool {
    std::mutex lock;
    std::vector<std::unique_ptr<Slot>> slots;
    size_t bytes = 0;
    int64_t plans = 0;
    Clock::time_point last_plan = Clock::now();
};

// (never destroyed: plans may be released while the process ends)
Pool& pool()
{
    static Pool* p = new Pool;
    return *p;
}

// Event queries and pinned allocations are harmless to a stream capture that another thread has open,
// but count as unsafe there unless the calling thread says so.
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
        const hipError_t e = hipEventQuery(s.done);
        if (e == hipSuccess)
            s.state = Slot::kIdle;
        else if (e != hipErrorNotReady)
            (void)hipGetLastError();
    }
    return s.state == Slot::kIdle;
}

void free_slot(Slot& s)
{
    if (s.done) (void)hipEventDestroy(s.done);
    if (s.ptr) (void)hipHostFree(s.ptr);
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
    Pool& p = pool();
    std::lock_guard<std::mutex> g(p.lock);
    for (auto& s : p.slots)
        if (s->device == dev && s->size >= bytes && s->size <= 16 * bytes + ((size_t)1 << 20) && idle(*s)) {
            s->state = Slot::kTaken;
            return {s->ptr, s.get()};
        }
    size_t size = (size_t)256 << 10;
    while (size < bytes) size *= 2;
    // room for it: idle blocks (of other sizes, of other devices) go first
    for (size_t i = 0; i < p.slots.size() && p.bytes + size > kStagePoolMax;) {
        if (idle(*p.slots[i])) {
            p.bytes -= p.slots[i]->size;
            free_slot(*p.slots[i]);
            p.slots.erase(p.slots.begin() + (ptrdiff_t)i);
        } else {
            ++i;
        }
    }
    if (p.bytes + size > kStagePoolMax) return {};
    auto s = std::make_unique<Slot>();
    s->device = dev;
    s->size = size;
    void* q = nullptr;
    if (hipHostMalloc(&q, size, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        return {};
    }
    s->ptr = static_cast<char*>(q);
    if (hipEventCreateWithFlags(&s->done, hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        s->done = nullptr;
        free_slot(*s);
        return {};
    }
    s->state = Slot::kTaken;
    p.bytes += size;
    p.slots.push_back(std::move(s));
    return {p.slots.back()->ptr, p.slots.back().get()};
}

hipError_t stage_copy(StageBlock b, void* dst, size_t bytes, hipStream_t stream)
{
    Slot& s = *static_cast<Slot*>(b.slot);
    const bool asked = dst != nullptr && bytes > 0;
    hipError_t e = asked ? hipMemcpyAsync(dst, b.ptr, bytes, hipMemcpyHostToDevice, stream) : hipSuccess;
    bool recorded = false;
    if (asked && e == hipSuccess) {
        e = hipEventRecord(s.done, stream);
        recorded = e == hipSuccess;
        if (!recorded) (void)hipStreamSynchronize(stream);     // (the copy may be in flight: the block is not handed back before it)
    }
    std::lock_guard<std::mutex> g(pool().lock);
    s.state = recorded ? Slot::kCopying : Slot::kIdle;
    return e;
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
    Pool& p = pool();
    std::lock_guard<std::mutex> g(p.lock);
    if (--p.plans > 0 || p.slots.empty() || Clock::now() - p.last_plan < std::chrono::seconds(1)) return;
    const RelaxedCapture relaxed;
    for (size_t i = 0; i < p.slots.size();) {
        if (idle(*p.slots[i])) {
            p.bytes -= p.slots[i]->size;
            free_slot(*p.slots[i]);
            p.slots.erase(p.slots.begin() + (ptrdiff_t)i);
        } else {
            ++i;
        }
    }
}

}  // namespace bspmm
