// Which leading part of a queue is tried together (project.hip).  No HIP
// headers, so that it also compiles as plain C++.
#pragma once

#include <stdint.h>

#include "record_format.h"

namespace tl {

// A queue of this many chunks of 64 requests is long: after a part of it fits,
// more is tried (2048 boards under arrivals, 140 chunks 5021 -> 4454 us, 38
// chunks 1436 -> 1402; 27 chunks 646 -> 693).
constexpr int32_t kLongQueue = 32;

// Tries of the first `want` of n chunks: all of them; when they do not fit, a
// guess, then half as many, a quarter, ... until some fit; of a long queue 1, 2,
// 4, ... more while they fit.  Each try costs scans of the whole board, so
// their number has to stay logarithmic in n whatever the guess.
struct QueueTries {
    int32_t n, ok, bad, want, step;   // `ok` chunks fit, `bad` do not

    TL_HOST_DEVICE explicit QueueTries(int32_t chunks) : n(chunks), ok(0), bad(chunks + 1), want(chunks), step(0) {}

    // After the first `want` chunks have been tried; guess is looked at only
    // when they were all n and did not fit.  False: done, and the chunks tried
    // last are the first `ok`.
    TL_HOST_DEVICE bool after(bool fits, int32_t guess) {
        if (want == ok) return false;   // what did not fit has been taken out again
        if (fits) {
            ok = want;
            if (bad - ok <= 1 || n < kLongQueue) return false;
            step = step > 0 ? 2 * step : 1;
            want = step < bad - 1 - ok ? ok + step : bad - 1;
            return true;
        }
        const bool all = want == n;
        bad = want;
        want = ok;
        if (ok == 0) want = !all ? bad / 2 : guess < 0 ? 0 : guess < n - 1 ? guess : n - 1;
        return true;
    }
};

}  // namespace tl
