// Host threads for set-up work.
#pragma once
#include <algorithm>
#include <atomic>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace mdx {
namespace host {

// Runs f(k) for k in [0, n) on a few host threads (setup only); an exception
// (host memory) ends the call's other work and is passed on.
template <class F>
void parallel_for(int n, F &&f)
{
    const int nt = (int)std::max(1u, std::min({8u, std::thread::hardware_concurrency(), (unsigned)n}));
    std::atomic<int> next{0};
    std::exception_ptr err;
    std::mutex mu;
    auto work = [&]() {
        try {
            for (int k; (k = next.fetch_add(1)) < n;) f(k);
        } catch (...) {
            std::lock_guard<std::mutex> g(mu);
            err = std::current_exception();
            next = n;
        }
    };
    std::vector<std::thread> th;
    try {
        for (int i = 1; i < nt; ++i) th.emplace_back(work);
    } catch (...) {   // no more threads, or no memory for one: those there are do it
    }
    work();
    for (std::thread &t : th) t.join();
    if (err) std::rethrow_exception(err);
}

}  // namespace host
}  // namespace mdx
