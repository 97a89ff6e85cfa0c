// host_ranges: every index once, also when no thread is to be had, and what a
// range throws arrives at the caller.
#include <sys/resource.h>

#include <atomic>
#include <cstdio>
#include <new>
#include <stdexcept>

#include "sem_threads.h"

static bool covers(int64_t n) {
    std::vector<std::atomic<int>> hit(n > 0 ? n : 1);
    for (auto &h : hit) h = 0;
    sem::host_ranges(n, [&](int64_t b, int64_t e) {
        for (int64_t q = b; q < e; ++q) hit[q] += 1;
    });
    for (int64_t q = 0; q < n; ++q)
        if (hit[q] != 1) return false;
    return true;
}

int main(int argc, char **) {
    for (int64_t n : {0, 1, 5, 16, 1000})
        if (!covers(n)) return std::printf("range %lld\n", (long long)n), 1;
    for (int64_t at : {0, 999}) {
        try {
            sem::host_ranges(1000, [&](int64_t b, int64_t e) {
                if (b <= at && at < e) throw std::bad_alloc();
            });
            return std::printf("nothing thrown\n"), 2;
        } catch (const std::bad_alloc &) {
        }
    }
    if (argc > 1) {                      // no memory for another thread's stack
        std::vector<std::atomic<int>> warm(4096);
        const rlimit none{1 << 20, 1 << 20};
        if (setrlimit(RLIMIT_AS, &none) != 0) return 3;
        std::atomic<int64_t> sum{0};
        sem::host_ranges(100, [&](int64_t b, int64_t e) { sum += e - b; });
        if (sum != 100) return 4;
    }
    std::printf("ok\n");
    return 0;
}
