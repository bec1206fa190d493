// The library's shared scratch (scratch.h) on a model of the runtime: any two
// calls that get the same array must be ordered, by a stream or by an event.
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <thread>
#include <vector>

#include "scratch.h"

namespace {

int checks = 0;
void check(bool ok, const char* what) {
    ++checks;
    if (ok) return;
    std::fprintf(stderr, "failed: %s\n", what);
    std::exit(1);
}

struct Use {
    fake::Stream stream;
    fake::Clocks at;
};

struct Pool {
    tl::ScratchPool<POOL_SLOTS> pool;
    std::map<void*, Use> last;   // of each array
    bool got = false;
    bool ordered = true;
    ~Pool() { pool.release(); }
    hipError_t call(hipStream_t st, size_t need) {
        return pool.with(need, st, [&](void* p, size_t bytes) {
            got = p != nullptr;
            if (!p) return hipSuccess;
            ordered &= bytes >= need && fake::state().live.at(p) >= bytes;
            const fake::Clocks now = fake::operation(st);
            auto it = last.find(p);
            if (it != last.end()) {
                const auto seen = now.find(it->second.stream);
                ordered &= seen != now.end() && seen->second >= it->second.at.at(it->second.stream);
            }
            last[p] = Use{fake::stream(st), now};
            return hipSuccess;
        });
    }
};

void on_thread(const std::function<void()>& f) { std::thread(f).join(); }

hipStream_t handle(int i) { return (hipStream_t)(size_t)(0x1000 + 64 * i); }

void streams_and_threads() {
    fake::state() = fake::State();
    {
        Pool p;
        // one handle, a stream of its own in each of these threads, nothing finished yet
        for (int rep = 0; rep < 3; ++rep)
            for (int t = 0; t < 2; ++t) on_thread([&] { p.call(hipStreamPerThread, 1000); });
        check(p.ordered, "calls of several threads on hipStreamPerThread");
        // more streams than arrays, and handles that come to name new streams
        for (int rep = 0; rep < 4; ++rep) {
            for (int i = 0; i < 7; ++i) p.call(handle(i), 1000 + 10 * i);
            for (int i = 0; i < 7; ++i) ++fake::state().generation[handle(i)];
        }
        check(p.ordered, "a new stream with the handle of a destroyed one");
        fake::state().all_done = true;
        for (int i = 0; i < 9; ++i) p.call(handle(i), 1000);
        check(p.ordered, "idle arrays");
    }
    check(fake::state().live.empty(), "everything is given back");
}

void while_another_thread_captures() {
    fake::state() = fake::State();
    Pool p;
    fake::state().capturing = true;
    for (int i = 0; i < 6; ++i) check(p.call(handle(i), 500 * (i + 1)) == hipSuccess, "a call while a stream is captured");
    check(!fake::state().refused, "no call ends another thread's capture");
    check(fake::state().mode == hipStreamCaptureModeGlobal, "the thread's mode is put back");
    check(p.ordered, "ordered");
    fake::state().capturing = false;
}

void without_memory() {
    fake::state() = fake::State();
    fake::state().free_bytes = 5000;
    Pool p;
    check(p.call(handle(0), 3000) == hipSuccess && p.got, "fits");
    check(p.call(handle(0), 4500) == hipSuccess && p.got, "fits in place of the smaller one");
    check(p.call(handle(0), 6000) == hipSuccess && !p.got, "runs without");
    check(p.call(handle(0), 2000) == hipSuccess && p.got, "and with it again");
    check(p.ordered, "ordered");
}

}  // namespace

int main() {
    streams_and_threads();
    while_another_thread_captures();
    without_memory();
    std::printf("%d checks\n", checks);
    return 0;
}
