// Memory a weight handle keeps between calls: buffers that grow on demand and outlive the graphs that use them.
//
// A call that is captured writes the address of its workspace into the graph, and the graph is replayed any time later.  So a
// buffer that a captured call has used is not freed when a larger call needs more: it is retired - kept, unused by later
// calls - until the handle is destroyed.  At most one buffer is retired per growth that follows a capture.
// Host code only (no HIP types), so that the bookkeeping can be tested without a GPU.
#pragma once
#include <stddef.h>

#include <new>

namespace psb {

struct GrownBuffer {
    void* ptr = nullptr;
    size_t bytes = 0;
    bool recorded = false;      // a captured call uses it
};

enum class Grow { ok, wait_failed, no_memory };

// Device: bool allocate(void** ptr, size_t bytes); void release(void* ptr); bool wait() - the calls made so far are done.
class WorkspaceMemory {
public:
    // At least `bytes` at b.ptr.  The contents do not survive growing.  capturing: the caller's launches are being captured.
    template <class Device>
    Grow reserve(GrownBuffer& b, size_t bytes, bool capturing, Device& device)
    {
        if (b.bytes < bytes) {
            if (b.ptr) {
                if (b.recorded) {
                    Retired* const node = new (std::nothrow) Retired{b.ptr, retired_};
                    if (!node) return Grow::no_memory;
                    retired_ = node;
                } else {
                    if (!device.wait()) return Grow::wait_failed;       // an earlier call may still use it
                    device.release(b.ptr);
                }
                b = GrownBuffer();
            }
            if (!device.allocate(&b.ptr, bytes)) {
                b.ptr = nullptr;
                return Grow::no_memory;
            }
            b.bytes = bytes;
        }
        if (capturing) b.recorded = true;
        return Grow::ok;
    }

    template <class Device>
    void release(GrownBuffer& b, Device& device)
    {
        if (b.ptr) device.release(b.ptr);
        b = GrownBuffer();
    }

    template <class Device>
    void release_retired(Device& device)
    {
        while (retired_) {
            Retired* const node = retired_;
            retired_ = node->next;
            device.release(node->ptr);
            delete node;
        }
    }

private:
    struct Retired {
        void* ptr;
        Retired* next;
    };
    Retired* retired_ = nullptr;
};

}  // namespace psb
