// Host loops over several threads.  Plain C++, so that it also builds with a
// host compiler under sanitizers.
#pragma once

#include <algorithm>
#include <cstdint>
#include <exception>
#include <system_error>
#include <thread>
#include <vector>

namespace sem {

// work(begin, end) over [0, n) in up to 16 ranges.  A range for which no thread
// is to be had runs on the caller's; what a range throws is thrown here after
// all of them have ended (an exception that left a thread, or a vector of
// running threads that an exception destroyed, would end the process).
template <typename F>
void host_ranges(int64_t n, F work) {
    const int nth = (int)std::max<unsigned>(1, std::min<unsigned>(16, std::thread::hardware_concurrency()));
    std::vector<std::exception_ptr> thrown(nth);
    std::vector<std::thread> th;
    th.reserve(nth);
    auto run = [&](int t) {
        try {
            work(n * t / nth, n * (t + 1) / nth);
        } catch (...) {
            thrown[t] = std::current_exception();
        }
    };
    for (int t = 1; t < nth; ++t) {
        try {
            th.emplace_back(run, t);
        } catch (const std::system_error &) {
            run(t);
        }
    }
    run(0);
    for (auto &t : th) t.join();
    for (auto &e : thrown)
        if (e) std::rethrow_exception(e);
}

}  // namespace sem
