#include "workers.h"

#include <sched.h>

#include <algorithm>
#include <cstdlib>
#include <system_error>

namespace smat {

Workers::Workers(int64_t entries)
{
    cpu_set_t set;
    CPU_ZERO(&set);
    const int cpus = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) : 1;
    most_ = static_cast<int>(std::clamp<int64_t>(std::min<int64_t>(cpus, entries / kPerThread + 1), 1, 16));
    if (const char* omp = std::getenv("OMP_NUM_THREADS")) {
        const int n = std::atoi(omp);
        if (n > 0) most_ = std::min(most_, n);
    }
}

Workers::~Workers()
{
    {
        std::lock_guard<std::mutex> lock(mutex_);
        quit_ = true;
    }
    wake_.notify_all();
    for (std::thread& t : threads_) t.join();
}

void Workers::start()
{
    started_ = true;
    threads_.reserve(static_cast<size_t>(most_ - 1));
    try {
        for (int t = 1; t < most_; ++t) threads_.emplace_back([this, t] { work(t); });
    } catch (const std::system_error&) {
        // no more threads to be had: go on with those there are
    }
}

void Workers::take_pieces(int thread)
{
    try {
        for (;;) {
            const int64_t first = next_.fetch_add(grain_, std::memory_order_relaxed);
            if (first >= n_) return;
            (*body_)(first, std::min(n_, first + grain_), thread);
        }
    } catch (...) {
        next_.store(n_, std::memory_order_relaxed);      // no new pieces
        std::lock_guard<std::mutex> lock(mutex_);
        if (!failed_) failed_ = std::current_exception();
    }
}

void Workers::work(int thread)
{
    uint64_t seen = 0;
    std::unique_lock<std::mutex> lock(mutex_);
    for (;;) {
        wake_.wait(lock, [&] { return quit_ || job_ != seen; });
        if (quit_) return;
        seen = job_;
        lock.unlock();
        take_pieces(thread);
        lock.lock();
        if (--running_ == 0) done_.notify_one();
    }
}

void Workers::ranges(int64_t n, int64_t grain, const std::function<void(int64_t, int64_t, int)>& body)
{
    if (n <= 0) return;
    grain = std::max<int64_t>(grain, 1);
    if (n <= grain || most_ == 1) {
        body(0, n, 0);
        return;
    }
    if (!started_) start();
    {
        std::lock_guard<std::mutex> lock(mutex_);
        body_ = &body;
        n_ = n;
        grain_ = grain;
        next_.store(0, std::memory_order_relaxed);
        failed_ = nullptr;
        running_ = static_cast<int>(threads_.size());
        ++job_;
    }
    wake_.notify_all();
    take_pieces(0);
    std::unique_lock<std::mutex> lock(mutex_);
    done_.wait(lock, [&] { return running_ == 0; });
    if (failed_) std::rethrow_exception(failed_);
}

}  // namespace smat
