// The words in LDS through which a workgroup shares its ticket and the outcome
// of its waits, with one wavefront late to read them.  Prints what every
// wavefront got; 0 when they agree.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <string.h>
#include <vector>

#include "persist.hpp"

#define WAVES 4

template <class F>
static void workgroup(F f) {
    std::vector<std::thread> t;
    for (int w = 0; w < WAVES; ++w)
        t.emplace_back([=] {
            threadIdx.x = 64 * w;
            f(w);
        });
    for (auto& x : t) x.join();
}

static int ticket = 5, err = 0, flag = 1, sh = 0;
static int got[WAVES], ok[WAVES];

static bool agree(const char* what, const int* v, int want) {
    bool good = true;
    for (int w = 0; w < WAVES; ++w) good = good && v[w] == want;
    printf("%s: wanted %d, got %d %d %d %d\n", what, want, v[0], v[1], v[2], v[3]);
    return good;
}

int main(int argc, char** argv) {
    pthread_barrier_init(&emu_barrier, nullptr, WAVES);
    emu_late = argc > 1 ? atoi(argv[1]) : -1;
    const Sched s = {&ticket, &err, (int64_t)10000000000, -1};
    bool good = true;
    // a ticket, then at once a wait through the same word
    workgroup([&](int w) {
        got[w] = sched_next(s, 100, &sh);
        ok[w] = sched_wait(s, &flag, 1, &sh);
    });
    good = agree("ticket before a wait", got, 5) && agree("wait", ok, 1) && good;
    // ... and a wait for several counters
    workgroup([&](int w) {
        got[w] = sched_next(s, 100, &sh);
        SchedDeps d;
        d.n = 0;
        deps_add(d, &flag, 1);
        ok[w] = sched_wait_deps(s, d, &sh);
    });
    good = agree("ticket before several waits", got, 6) && agree("waits", ok, 1) && good;
    // two tickets in a row
    workgroup([&](int w) {
        got[w] = sched_next(s, 100, &sh);
        ok[w] = sched_next(s, 8, &sh);
    });
    good = agree("ticket before a ticket", got, 7) && agree("no ticket left", ok, -1) && good;
    // a batch: an error comes up right after the first look at its word, so all go
    // on with the same matrix once more and all leave after that
    workgroup([&](int w) {
        got[w] = 0;
        sched_batch(
            0, 0, 1, &err, &sh,
            [&](int) {
                if (++got[w] == 1 && w == 0) emu_raise = &err;
                return got[w] < 4;
            },
            [](int) { return 1.0f; });
    });
    good = agree("matrices until the error", got, 2) && good;
    return good ? 0 : 1;
}
