// A model of the few runtime calls that scratch.h makes, for tests on the CPU.
// Streams are told apart as the runtime does: a handle names one stream at a
// time (a new one after renew()), hipStreamPerThread another one in every
// thread.  Each operation on a stream has a clock; an event carries the clocks
// its stream had reached, and waiting for it joins them, so that a test can ask
// whether two uses of an array are ordered.
#pragma once

#include <cstddef>
#include <map>
#include <set>
#include <utility>

typedef int hipError_t;
constexpr hipError_t hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotReady = 600, hipErrorStreamCapture = 900;
typedef struct FakeStream* hipStream_t;
#define hipStreamPerThread ((hipStream_t)2)
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
constexpr unsigned hipEventDisableTiming = 2;

namespace fake {
typedef std::pair<std::size_t, int> Stream;    // (handle or thread, generation)
typedef std::map<Stream, int> Clocks;          // how far each stream is known to have come
struct State {
    std::map<hipStream_t, int> generation;
    std::map<Stream, Clocks> at;               // per stream: what its next operation comes after
    Clocks done;                               // what the host knows to be finished
    std::map<void*, std::size_t> live;         // allocations
    std::map<void*, std::pair<Stream, int>> last_use;   // told by the test
    bool idle = false;                         // nothing runs on the device
    bool freed_in_use = false;
    std::size_t free_bytes = (std::size_t)-1;  // left on the device
    int syncs = 0, allocs = 0;
    bool capturing = false;                    // another thread captures in the global mode
    bool refused = false;                      // a call that ends that capture was made
    bool all_done = false;                     // every event has completed
    hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
};
inline State& state() {
    static State s;
    return s;
}
inline Stream stream(hipStream_t s) {
    static std::size_t threads = 0;
    thread_local const std::size_t own = ++threads;   // (a thread's id may be a finished one's)
    if (s == hipStreamPerThread) return {own, -1};
    return {(std::size_t)s, state().generation[s]};
}
inline void join(Clocks& a, const Clocks& b) {
    for (const auto& p : b)
        if (a[p.first] < p.second) a[p.first] = p.second;
}
// the stream's next operation: what it comes after, itself included
inline Clocks operation(hipStream_t s) {
    Clocks& c = state().at[stream(s)];
    join(c, state().done);
    ++c[stream(s)];
    return c;
}
inline hipError_t unsafe_call() {
    State& s = state();
    if (!s.capturing || s.mode == hipStreamCaptureModeRelaxed) return hipSuccess;
    s.refused = true;
    return hipErrorStreamCapture;
}
struct Event {
    Clocks reached;
};
}  // namespace fake

typedef fake::Event* hipEvent_t;

inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    std::swap(*m, fake::state().mode);
    return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = new fake::Event();
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
    delete e;
    return hipSuccess;
}
inline hipError_t hipEventQuery(hipEvent_t e) {
    if (hipError_t r = fake::unsafe_call()) return r;
    if (!fake::state().all_done) return hipErrorNotReady;
    fake::join(fake::state().done, e->reached);
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    if (hipError_t r = fake::unsafe_call()) return r;
    ++fake::state().syncs;
    fake::join(fake::state().done, e->reached);
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    e->reached = fake::operation(s);
    return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    fake::join(fake::state().at[fake::stream(s)], e->reached);
    return hipSuccess;
}
template <class T>
hipError_t hipMalloc(T** p, std::size_t n) {
    if (hipError_t r = fake::unsafe_call()) return r;
    fake::State& s = fake::state();
    if (n > s.free_bytes) return hipErrorOutOfMemory;
    if (s.free_bytes != (std::size_t)-1) s.free_bytes -= n;
    ++s.allocs;
    *p = (T*)new char[1];
    s.live[(void*)*p] = n;
    return hipSuccess;
}
// freeing waits for the whole device, which scratch.h does not count on
inline hipError_t hipFree(void* p) {
    if (hipError_t r = fake::unsafe_call()) return r;
    fake::State& s = fake::state();
    ++s.syncs;
    if (s.free_bytes != (std::size_t)-1) s.free_bytes += s.live.at(p);
    s.live.erase(p);
    const auto u = s.last_use.find(p);
    if (u != s.last_use.end()) {
        s.freed_in_use |= !s.idle && s.done[u->second.first] < u->second.second;
        s.last_use.erase(u);
    }
    delete[] (char*)p;
    return hipSuccess;
}
