// Threads of one host-side call (smat_preprocess, smat_bind_device) and the arrays they fill.
#pragma once

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

namespace smat {

// A vector whose resize() leaves new elements as they are: arrays of megabytes are filled by several threads, which
// also take the page faults of fresh memory, instead of being zeroed by one first.
template <typename T>
struct Uninitialized : std::allocator<T> {
    template <typename U> struct rebind { using other = Uninitialized<U>; };
    template <typename U> void construct(U* p) noexcept { ::new (static_cast<void*>(p)) U; }
    template <typename U, typename... Args> void construct(U* p, Args&&... args) { ::new (static_cast<void*>(p)) U(std::forward<Args>(args)...); }
};
template <typename T> using Buf = std::vector<T, Uninitialized<T>>;

// Up to sixteen threads (no more than the process may run on, nor than OMP_NUM_THREADS, nor one per kPerThread stored
// entries: starting one takes as long as some ten thousand entries), started by the first loop that is
// worth it and joined by the destructor: an object lives as long as the call that made it.
class Workers {
public:
    static constexpr int64_t kPerThread = 16384;
    explicit Workers(int64_t entries);
    ~Workers();
    Workers(const Workers&) = delete;
    Workers& operator=(const Workers&) = delete;

    // Threads a loop may run on, the calling one included; `thread` below is less than that.
    int most() const { return most_; }

    // body(first, last, thread) for pieces of at most `grain` that cover [0, n), in no order.  Returns when all have run;
    // rethrows the first exception.  A single piece, or a single thread, runs on the calling thread.
    void ranges(int64_t n, int64_t grain, const std::function<void(int64_t, int64_t, int)>& body);

private:
    void start();
    void take_pieces(int thread);
    void work(int thread);

    int most_ = 1;
    std::vector<std::thread> threads_;
    bool started_ = false;
    std::mutex mutex_;
    std::condition_variable wake_, done_;
    uint64_t job_ = 0;                   // counts the loops; a thread runs each once
    int running_ = 0;
    bool quit_ = false;
    // the loop at hand
    const std::function<void(int64_t, int64_t, int)>* body_ = nullptr;
    int64_t n_ = 0, grain_ = 1;
    std::atomic<int64_t> next_{0};
    std::exception_ptr failed_;
};

}  // namespace smat
