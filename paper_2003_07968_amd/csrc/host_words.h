// Where the calls that wait for the stream read their small results (error
// words, diagnostics): a kernel writes them to page-locked host memory, the
// host reads them after its one wait.  A copy to the caller's pageable memory
// costs a staging copy and a second wait in the runtime (lbm_sync of an idle
// stream: 20 us with the copy, 11.5 us with the words).
//
// One page of kHostSlots slots of kHostWords words for the whole process,
// allocated at the first use (75 to 175 us, so not once per lattice) and kept.
// A call holds a slot from its launch to the end of its wait.  No slot is
// given, and the call uses a copy, where the copy is what works or fails as it
// should: the stream's device is not current, the stream is being captured, no
// page can be allocated, more than kHostSlots calls at once.
//
// A device reset by the host program frees the page.  Each use asks the
// runtime for the page's buffer id (0.25 us): an unknown address or another
// allocation at that address is never written to, and a new page takes over.
// A slot whose wait failed is not used again: a kernel may still write to it.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <mutex>

namespace lbm_host {

constexpr int kHostSlots = 16, kHostWords = 32;

class HostWords {
public:
    unsigned long long *w = nullptr;  // null: no slot

    HostWords() = default;
    HostWords(const HostWords &) = delete;
    HostWords &operator=(const HostWords &) = delete;

    // Take a slot for work on a stream of device `dev`.
    HostWords(int dev, hipStream_t stream)
    {
        int cur = -1;
        // a launch needs the stream's device current, which a copy does not
        if (hipGetDevice(&cur) != hipSuccess || cur != dev) return;
        hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &capturing) != hipSuccess ||
            capturing != hipStreamCaptureStatusNone)
            return;
        Pool &p = pool();
        std::lock_guard<std::mutex> lock(p.mu);
        if (!p.alive() && !p.allocate()) return;
        const uint32_t open = ~p.busy & ((1u << kHostSlots) - 1u);
        if (open == 0) return;
        slot_ = __builtin_ctz(open);
        p.busy |= 1u << slot_;
        generation_ = p.generation;
        w = p.page + (size_t)slot_ * kHostWords;
    }

    // After a successful wait for the work that wrote the slot, or if that
    // work was never enqueued.
    void give_back()
    {
        if (!w) return;
        w = nullptr;
        Pool &p = pool();
        std::lock_guard<std::mutex> lock(p.mu);
        if (generation_ == p.generation) p.busy &= ~(1u << slot_);
    }

private:
    struct Pool {
        std::mutex mu;
        unsigned long long *page = nullptr;  // null: none yet
        uint64_t id = 0;                     // its buffer id
        uint32_t busy = 0;
        unsigned generation = 0;             // of the page: slots of a lost one are dropped

        static bool buffer_id(void *p, uint64_t *id)
        {
            *id = 0;
            if (hipPointerGetAttribute(id, HIP_POINTER_ATTRIBUTE_BUFFER_ID, p) == hipSuccess)
                return true;
            (void)hipGetLastError();
            return false;
        }
        bool alive()
        {
            uint64_t now;
            return page && buffer_id(page, &now) && now == id;
        }
        bool allocate()
        {
            page = nullptr;
            // allocating is allowed while another thread captures a graph in
            // the global mode only with this thread's mode relaxed
            hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
            if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return false;
            void *p = nullptr;
            if (hipHostMalloc(&p, kHostSlots * kHostWords * sizeof(*page),
                              hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
                p = nullptr;
                (void)hipGetLastError();
            }
            (void)hipThreadExchangeStreamCaptureMode(&mode);
            if (!p) return false;
            if (!buffer_id(p, &id)) {
                (void)hipHostFree(p);
                return false;
            }
            page = (unsigned long long *)p;
            busy = 0;
            ++generation;
            return true;
        }
    };
    static Pool &pool()
    {
        static Pool p;
        return p;
    }

    int slot_ = 0;
    unsigned generation_ = 0;
};

}  // namespace lbm_host
