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
    ~Pool() {
        check(!fake::state().freed_in_use, "nothing in use is freed");
        fake::state().idle = true;
        pool.release();
    }
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
            fake::state().last_use[p] = {fake::stream(st), now.at(fake::stream(st))};
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
    fake::state().free_bytes = 500000;
    Pool p;
    check(p.call(handle(0), 300000) == hipSuccess && p.got, "fits, its power of two does not");
    check(p.call(handle(0), 450000) == hipSuccess && p.got, "fits in place of the smaller one");
    check(p.call(handle(0), 600000) == hipSuccess && !p.got, "runs without");
    check(p.call(handle(0), 200000) == hipSuccess && p.got, "and with it again");
    check(p.ordered, "ordered");
}

void many_streams_and_little_memory() {
    unsigned x = 1;
    for (int rep = 0; rep < 200; ++rep) {
        fake::state() = fake::State();
        fake::state().free_bytes = 1200000;
        Pool p;
        for (int i = 1; i <= 40; ++i) {
            x = x * 1664525u + 1013904223u;
            check(p.call(handle(x >> 8 & 7), 1000 + (x >> 12) % (20000 * i)) == hipSuccess, "on many streams");
        }
        check(p.ordered, "ordered");
    }
}

// Slowly growing needs: nothing waits for the device, few allocations, and no
// more memory than four times the largest need.
void growing() {
    fake::state() = fake::State();
    {
        Pool p;
        size_t need = 100000;
        for (int i = 0; i < 500; ++i, need += need / 50) p.call(handle(0), need);
        size_t held = 0;
        for (const auto& a : fake::state().live) held += a.second;
        check(p.ordered && p.got, "ordered");
        check(fake::state().syncs == 0, "growing waits for nothing");
        check(fake::state().allocs <= 16, "and seldom allocates");
        check(held <= 4 * need, "and keeps little");
    }
    check(fake::state().live.empty(), "everything is given back");
}

}  // namespace

int main() {
    growing();
    streams_and_threads();
    while_another_thread_captures();
    without_memory();
    many_streams_and_little_memory();
    std::printf("%d checks\n", checks);
    return 0;
}
