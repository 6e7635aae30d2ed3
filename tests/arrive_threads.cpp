// The session kernel's commit hand-off (md_arrive.h) on host threads: each
// launch, every workgroup (a thread) reads the shared counters, arrives, goes
// on, and commits new counters if it was the last to arrive.  Launches follow
// each other as in a stream.  Now and then a workgroup is late by far more
// than the others take.  Exit status 0 when every launch committed once, no
// workgroup read counters that its launch had already changed, and the count
// was zero after every launch.
#include <chrono>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "md_arrive.h"

int main() {
    std::mt19937 rng(5);
    int count = 0;
    int counters[2] = {0, 0};   // what the launches commit: their number, twice
    for (int launch = 0; launch < 400; ++launch) {
        const int n = 1 + (int)(rng() % 12);
        const int late = rng() % 4 == 0 ? (int)(rng() % n) : -1;   // starts after all others are done
        std::vector<int> seen(2 * n, -1), commits(n, 0);
        auto work = [&](int w, unsigned us) {
            std::this_thread::sleep_for(std::chrono::microseconds(us));
            seen[2 * w] = __atomic_load_n(&counters[0], __ATOMIC_RELAXED);
            std::this_thread::yield();
            seen[2 * w + 1] = __atomic_load_n(&counters[1], __ATOMIC_RELAXED);
            const int before = md::arrive(&count);
            std::this_thread::yield();   // the rows
            if (md::arrive_last(&count, before, n)) {
                commits[w] = 1;
                __atomic_store_n(&counters[0], launch + 1, __ATOMIC_RELAXED);
                __atomic_store_n(&counters[1], launch + 1, __ATOMIC_RELAXED);
            }
        };
        std::vector<std::thread> t;
        for (int w = 0; w < n; ++w)
            t.emplace_back(work, w, w == late ? 3000u : (unsigned)(rng() % 50));
        for (auto& x : t) x.join();
        int total = 0;
        for (int w = 0; w < n; ++w) {
            total += commits[w];
            if (seen[2 * w] != launch || seen[2 * w + 1] != launch) {
                std::printf("launch %d: workgroup %d of %d read %d, %d\n", launch, w, n, seen[2 * w], seen[2 * w + 1]);
                return 1;
            }
        }
        if (total != 1 || count != 0 || counters[0] != launch + 1) {
            std::printf("launch %d: %d commits, count %d\n", launch, total, count);
            return 1;
        }
    }
    std::puts("400 launches committed once each");
    return 0;
}
