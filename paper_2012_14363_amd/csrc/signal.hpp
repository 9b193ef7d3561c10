// How a synchronous call of a small request waits: on a word of pinned host memory that its kernel writes
// when the last workgroup is done.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

namespace tp {

// What a kernel needs to say that it is done (kernels.hip: signal_done).
struct SignalParams {
    uint32_t* flag = nullptr;     // pinned host memory, as the GPU addresses it
    uint32_t* counter = nullptr;  // device memory: workgroups done so far, over all uses of the slot
    uint32_t value = 0;           // what goes into *flag
    uint32_t last = 0;            // the counter as the launch's last workgroup finds it
};

// A slot (flag word and counter) held by one call for one launch.  hipStreamSynchronize puts a barrier packet
// behind the kernel and waits for that packet's signal, after the kernel's end-of-kernel cache write-back;
// a kernel whose stores all go through to memory (`sc0 sc1`) can say itself that they are there.  Measured
// in a PyTorch process, launch + wait: 512 bytes on one workgroup 11.1 us with hipStreamSynchronize, 6.8
// so; 300 KB on 19 workgroups 12.4 -> 8.4, 1 MiB on 64: 12.4 -> 8.7, 4 MiB on 256: 12.9 -> 10.9; into
// pinned host memory 300 KB 17.1 -> 12.8, 1 MiB 30.1 -> 26.8, but 4 MiB on 256 workgroups 86.5 -> 87.0.
// (A signal attached to the kernel's packet, hipExtLaunchKernel's stop event, measures 8.6 and makes the
// next hipDeviceSynchronize 30 us slower.)
//
// The kSlots slots of a process lie in one page of pinned host memory, allocated by the first call that
// wants one and kept until the process ends, and in an array of the library's device image; a call that
// finds none free waits for the stream instead.  Calls on any threads and streams may overlap.
class Signal {
public:
    Signal() = default;
    ~Signal();
    Signal(const Signal&) = delete;
    Signal& operator=(const Signal&) = delete;

    // Takes a slot for a launch of `workgroups` on `stream`; false if there is none to be had or the stream is of
    // another GPU than the current one (its kernels could not reach this one's counter).
    bool take(uint32_t workgroups, hipStream_t stream);
    const SignalParams& params() const { return params_; }
    // The launch was refused: the slot is as it was before.
    void cancel();
    // Waits until the kernel has signalled: looks at the flag for a while, then waits for the stream.
    hipError_t wait(hipStream_t stream);

private:
    int slot_ = -1, device_ = -1;
    uint32_t workgroups_ = 0;
    bool sound_ = false;  // the kernel is known to be done (or never ran): the slot may serve another call
    SignalParams params_;
};

}  // namespace tp
