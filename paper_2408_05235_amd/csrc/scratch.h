// Device scratch of the library that is kept from call to call and shared by
// the calls on several streams and threads.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <thread>

namespace tl {

// While another thread captures a stream (in the default, global mode), the
// calls that choose and grow a workspace -- event queries, allocations -- are
// refused on every thread and end that capture.  They belong to no captured
// stream: this thread's mode is relaxed around them.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    RelaxedCapture(const RelaxedCapture&) = delete;
    RelaxedCapture& operator=(const RelaxedCapture&) = delete;
};

// Up to SLOTS arrays on one device, each only replaced by a larger one when a
// larger call comes.  Sizes are powers of two, so calls that grow slowly seldom
// allocate, and a replaced array is kept until the pool is given back: freeing
// it would wait for the device, and together the replaced ones are smaller than
// the one in use.  `done` is recorded on the stream of the last call that
// used the array.  A call takes the array its stream used last, else an idle
// one, else another stream's: SLOTS streams can use the pool without waiting
// for each other.  Every call that takes a used array waits (on the device) for
// its event, its own stream's as well: a stream's handle does not tell streams
// apart (hipStreamPerThread is one handle for a stream in every thread, and a
// new stream may get the handle of a destroyed one), and on the stream that
// recorded the event the wait costs nothing.
template <int SLOTS>
class ScratchPool {
public:
    // Runs launch(ws, ws_bytes) with an array of at least `need` bytes, all of
    // its launches on st (a stream that is not being captured).  In the steady
    // state nothing is allocated, and nothing waits on the host.  Where no
    // memory is left the replaced arrays are freed and exactly `need` bytes
    // asked for; when that fails too launch gets (nullptr, 0).
    template <class Launch>
    hipError_t with(size_t need, hipStream_t st, Launch&& launch) {
        std::lock_guard<std::mutex> lock(mutex_);
        const std::thread::id thread = st == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
        hipError_t e;
        Slot* w = nullptr;
        for (Slot& c : slots_)
            if (c.used && c.stream == st && c.thread == thread) { w = &c; break; }
        if (!w || need > w->bytes) {
            const RelaxedCapture relaxed;
            if (!w) {
                e = choose(&w);
                if (e != hipSuccess) return e;
            }
            if (w->done && need > w->bytes) {
                e = grow(*w, need);
                if (e != hipSuccess) return e;
            }
        }
        if (!w->ptr) return launch((void*)nullptr, (size_t)0);
        if (w->used) {
            e = hipStreamWaitEvent(st, w->done, 0);
            if (e != hipSuccess) return e;
        }
        const hipError_t el = launch(w->ptr, w->bytes);
        // recorded also after a failed launch, whose earlier kernels may have
        // been enqueued on st and use the array
        e = hipEventRecord(w->done, st);
        if (e == hipSuccess) {
            w->stream = st;
            w->thread = thread;
            w->used = true;
        }
        return el != hipSuccess ? el : e;
    }

    // Gives everything back; no call uses the pool any more and the device is
    // idle.
    void release() {
        for (Slot& w : slots_) {
            free_arrays(w);
            if (w.done) (void)hipEventDestroy(w.done);
            w = Slot();
        }
    }

private:
    static constexpr int kMinLog = 16, kMaxReplaced = 48;   // (sizes 2^16, 2^17, ...)
    struct Slot {
        void* ptr = nullptr;
        size_t bytes = 0;
        void* replaced[kMaxReplaced] = {};
        int n_replaced = 0;
        hipEvent_t done = nullptr;
        hipStream_t stream = nullptr;
        std::thread::id thread;   // of hipStreamPerThread
        bool used = false;
    };

    // An idle array's slot, else the next in turn, with an event unless none
    // can be had (its array is empty then).
    hipError_t choose(Slot** out) {
        Slot* w = nullptr;
        for (int i = 0; i < SLOTS && !w; ++i) {
            Slot& c = slots_[i];
            if (!c.used) {
                w = &c;
            } else if (SLOTS > 1) {
                const hipError_t e = hipEventQuery(c.done);
                if (e == hipSuccess) w = &c;
                else if (e != hipErrorNotReady) return e;
                else (void)hipGetLastError();   // not ready: no error of the launches below
            }
        }
        if (!w) {
            w = &slots_[next_];
            next_ = (next_ + 1) % SLOTS;
        }
        if (!w->done && hipEventCreateWithFlags(&w->done, hipEventDisableTiming) != hipSuccess) {
            w->done = nullptr;
            (void)hipGetLastError();
        }
        *out = w;
        return hipSuccess;
    }

    // A larger array for w.  The replaced one's users may still run: the new
    // one's are ordered behind them (w.used stays), so that w.done is the last of
    // them all.
    hipError_t grow(Slot& w, size_t need) {
        int log = kMinLog;
        while (log < 62 && ((size_t)1 << log) < need) ++log;
        void* p = nullptr;
        if (w.n_replaced < kMaxReplaced && hipMalloc(&p, (size_t)1 << log) == hipSuccess) {
            if (w.ptr) w.replaced[w.n_replaced++] = w.ptr;
            w.bytes = (size_t)1 << log;
        } else {
            (void)hipGetLastError();   // clear the allocation error before the launches check theirs
            if (w.used) {
                const hipError_t e = hipEventSynchronize(w.done);
                if (e != hipSuccess) return e;
                w.used = false;
            }
            free_arrays(w);
            if (hipMalloc(&p, need) == hipSuccess) {
                w.bytes = need;
            } else {
                p = nullptr;
                (void)hipGetLastError();
            }
        }
        w.ptr = p;
        return hipSuccess;
    }

    static void free_arrays(Slot& w) {
        if (w.ptr) (void)hipFree(w.ptr);
        for (int i = 0; i < w.n_replaced; ++i) (void)hipFree(w.replaced[i]);
        w.ptr = nullptr;
        w.bytes = 0;
        w.n_replaced = 0;
    }

    std::mutex mutex_;
    Slot slots_[SLOTS];
    int next_ = 0;
};

}  // namespace tl
