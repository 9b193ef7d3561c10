#include "signal.hpp"

#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <mutex>

namespace tp {

namespace {

constexpr int kMaxDevices = 64;
constexpr int kSlots = 32;
constexpr int kSpacing = 32;  // words between slots: a memory line each
constexpr auto kLookFor = std::chrono::microseconds(100);

// Every GPU holds its own copy (zero when the library's code is loaded there).
static __device__ uint32_t device_counters[kSlots * kSpacing];

struct Slots {
    std::mutex setup;
    std::atomic<bool> ready{false}, failed{false};
    uint32_t* host = nullptr;  // the page of flags
    uint32_t* view = nullptr;  // as the GPU addresses it
    std::atomic<uint32_t*> counters[kMaxDevices] = {};
    std::atomic<uint32_t> free{~uint32_t{0}};  // bit s: slot s is free
    // of the slot's holder alone:
    uint32_t value[kSlots] = {};
    uint32_t done[kMaxDevices][kSlots] = {};  // workgroups counted so far in that device's counter
};
static_assert(kSlots == 32, "one bit of Slots::free each");

// Never destroyed: calls may still run while the process ends.
Slots& slots() {
    static Slots* s = new Slots;
    return *s;
}

// Allocating and looking up a symbol are no stream work: another thread's stream capture is not to mind them.
class CaptureTolerant {
public:
    CaptureTolerant() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
    ~CaptureTolerant() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }

private:
    hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

bool prepare(Slots& s) {
    std::lock_guard<std::mutex> hold(s.setup);
    if (s.ready.load(std::memory_order_relaxed)) return true;
    if (s.failed.load(std::memory_order_relaxed)) return false;
    CaptureTolerant tolerant;
    void *host = nullptr, *view = nullptr;
    if (hipHostMalloc(&host, kSlots * kSpacing * sizeof(uint32_t), hipHostMallocMapped | hipHostMallocPortable | hipHostMallocCoherent) !=
            hipSuccess ||
        hipHostGetDevicePointer(&view, host, 0) != hipSuccess) {
        (void)hipGetLastError();
        s.failed.store(true, std::memory_order_relaxed);
        return false;
    }
    s.host = static_cast<uint32_t*>(host);
    s.view = static_cast<uint32_t*>(view);
    for (int i = 0; i < kSlots * kSpacing; ++i) s.host[i] = 0;
    s.ready.store(true, std::memory_order_release);
    return true;
}

uint32_t* counters_of(Slots& s, int device) {
    uint32_t* p = s.counters[device].load(std::memory_order_acquire);
    if (p) return p;
    std::lock_guard<std::mutex> hold(s.setup);
    CaptureTolerant tolerant;
    void* address = nullptr;
    if (hipGetSymbolAddress(&address, HIP_SYMBOL(device_counters)) != hipSuccess || !address) {
        (void)hipGetLastError();
        return nullptr;
    }
    p = static_cast<uint32_t*>(address);
    s.counters[device].store(p, std::memory_order_release);
    return p;
}

}  // namespace

bool Signal::take(uint32_t workgroups, hipStream_t stream) {
    Slots& s = slots();
    int device = -1;
    hipDevice_t runs_on = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices ||
        hipStreamGetDevice(stream, &runs_on) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    // A kernel runs on its stream's GPU, whatever the thread's current one is, and the counter has to be that GPU's own.
    if (runs_on != device) return false;
    if (!s.ready.load(std::memory_order_acquire) && !prepare(s)) return false;
    uint32_t* counters = counters_of(s, device);
    if (!counters) return false;
    uint32_t free = s.free.load(std::memory_order_relaxed);
    do {
        if (free == 0) return false;
    } while (!s.free.compare_exchange_weak(free, free & (free - 1), std::memory_order_acquire, std::memory_order_relaxed));
    slot_ = __builtin_ctz(free);
    params_.flag = s.view + slot_ * kSpacing;
    params_.value = ++s.value[slot_];
    if (workgroups > 1) {
        params_.counter = counters + slot_ * kSpacing;
        s.done[device][slot_] += workgroups;
        params_.last = s.done[device][slot_] - 1;
    }
    device_ = device;
    workgroups_ = workgroups;
    return true;
}

void Signal::cancel() {
    if (slot_ < 0) return;
    if (workgroups_ > 1) slots().done[device_][slot_] -= workgroups_;
    sound_ = true;
}

hipError_t Signal::wait(hipStream_t stream) {
    const uint32_t* flag = slots().host + slot_ * kSpacing;
    const auto until = std::chrono::steady_clock::now() + kLookFor;
    do {
        for (int i = 0; i < 64; ++i) {
            if (__atomic_load_n(flag, __ATOMIC_ACQUIRE) == params_.value) {
                sound_ = true;
                return hipSuccess;
            }
            __builtin_ia32_pause();
        }
    } while (std::chrono::steady_clock::now() < until);
    const hipError_t e = hipStreamSynchronize(stream);
    // A launch that has not run (a stream that was being captured) may still write to the slot: it is then never used again.
    sound_ = e == hipSuccess && __atomic_load_n(flag, __ATOMIC_ACQUIRE) == params_.value;
    return e;
}

Signal::~Signal() {
    if (slot_ >= 0 && sound_) slots().free.fetch_or(uint32_t{1} << slot_, std::memory_order_release);
}

}  // namespace tp
