// What the host entry points share: worker threads, and exceptions that stop at the C boundary.
#pragma once
#include "../../include/relibra.h"

#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace relibra {

// Runs fn on `workers` threads, the calling one among them; fewer if no more threads are to be had.  fn takes its work
// from a shared counter.  An exception of a worker (std::bad_alloc) is handed to the caller after all threads have
// ended.
template <class Fn> void run_workers(int workers, const Fn &fn)
{
    std::exception_ptr failed;
    std::mutex m;
    auto guarded = [&]() {
        try {
            fn();
        } catch (...) {
            std::lock_guard<std::mutex> lock(m);
            failed = std::current_exception();
        }
    };
    std::vector<std::thread> pool;
    pool.reserve(workers);
    try {
        for (int w = 1; w < workers; ++w) pool.emplace_back(guarded);
    } catch (...) {                            // no thread, or no memory for one: the ones there are share the work
    }
    guarded();
    for (auto &t : pool) t.join();
    if (failed) std::rethrow_exception(failed);
}

// The body of a host entry point.  An exception must not leave a C function: what the standard library throws in these
// bodies is a want of memory.
template <class Fn> auto entry(const Fn &body) -> decltype(body())
{
    try {
        return body();
    } catch (...) {
        return RELIBRA_ENOMEM;
    }
}

}  // namespace relibra
