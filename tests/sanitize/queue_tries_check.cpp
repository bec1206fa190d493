// The tries of a queue's leading chunks (queue_tries.h) for every length, every
// part that fits and every kind of guess: few tries, and what was tried last
// is a part that fits.
#include <cstdio>
#include <cstdlib>

#include "queue_tries.h"

int main() {
    int worst = 0;
    for (int n = 2; n <= 300; ++n) {
        int log = 0;
        while ((1 << log) < n) ++log;
        for (int fit = 0; fit <= n; ++fit) {   // the first `fit` chunks fit together, no more
            const int guesses[] = {-1, 0, 1, 2, n / 3, fit - 1, fit, fit + 1, n - 2, n - 1, n + 5};
            for (int guess : guesses) {
                tl::QueueTries t(n);
                int tries = 0, last;
                do {
                    last = t.want;
                    ++tries;
                } while (t.after(last <= fit, guess) && tries < 1000);
                if (tries > worst) worst = tries;
                const bool kept = fit == n ? last == n : last <= fit;
                if (!kept || last != t.ok || tries > log + 4) {
                    std::fprintf(stderr, "failed: %d chunks, %d fit, guess %d: %d tries, %d kept\n", n, fit, guess, tries, last);
                    return 1;
                }
            }
        }
    }
    std::printf("at most %d tries\n", worst);
    return 0;
}
