// Host threads of the packer.
#pragma once
#include <exception>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

namespace amr {

// work() on n threads, the calling one among them, or on as many as can be started.  What work throws is
// thrown again here once every thread has ended (the first of them): left in its thread it would end
// the process.
template <typename F>
void run_threads(int n, F &&work) {
    std::mutex m;
    std::exception_ptr first;
    auto guarded = [&]() {
        try {
            work();
        } catch (...) {
            std::lock_guard<std::mutex> l(m);
            if (!first) first = std::current_exception();
        }
    };
    struct Team {
        std::vector<std::thread> th;
        void join() {
            for (auto &x : th) x.join();
            th.clear();
        }
        ~Team() { join(); }
    } team;
    if (n > 1) team.th.reserve((size_t)n - 1);
    try {
        for (int t = 1; t < n; t++) team.th.emplace_back(guarded);
    } catch (const std::system_error &) {      // the others take the work
    }
    guarded();
    team.join();
    if (first) std::rethrow_exception(first);
}

}  // namespace amr
