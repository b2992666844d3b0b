// Host threads of one call, which share its copies out of pinned staging into
// pageable memory. A call that returns tens of megabytes fills fresh pages,
// and one core takes those faults at 16 GB/s (2 MiB pages; 5 GB/s with 4 KiB
// ones), less than a third of what the host link delivers; eight cores with a
// 2 MiB page each reach 95 GB/s. The threads live for one call: nothing
// outlives it, and calls on different maps have crews of their own.
#pragma once

#include <stdint.h>

#include <atomic>
#include <condition_variable>
#include <deque>
#include <mutex>
#include <thread>
#include <vector>

namespace tsdf {

class Crew {
public:
    // call(arg, part) for part = 0 .. parts - 1; left counts the parts that
    // are not done. call must not throw.
    struct Job {
        void (*call)(void *, int64_t) = nullptr;
        void *arg = nullptr;
        int64_t parts = 0, next = 0;
        std::atomic<int64_t> left{0};
    };

    // `helpers` threads beside the caller; fewer (or none) when the system
    // gives no more
    explicit Crew(int helpers)
    {
        const int cores = (int)std::thread::hardware_concurrency();
        if (cores > 0 && helpers > cores - 1) helpers = cores - 1;
        try {
            for (int k = 0; k < helpers; ++k) threads_.emplace_back([this] { work(); });
        } catch (...) {
        }
    }
    // every posted job is finished first (wait does that in the good case)
    ~Crew()
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            stop_.store(true);
        }
        cv_.notify_all();
        for (std::thread &t : threads_) t.join();
    }
    Crew(const Crew &) = delete;
    Crew &operator=(const Crew &) = delete;

    // Hands the job to the threads; it, and what arg points to, stay until
    // wait(job) returns.
    void post(Job *job)
    {
        job->next = 0;
        job->left.store(job->parts);
        if (job->parts <= 0) return;
        {
            std::lock_guard<std::mutex> lk(mu_);
            jobs_.push_back(job);
            open_.fetch_add(1);
        }
        cv_.notify_all();
    }

    // Until the job is done. (The caller works on jobs itself only where it
    // has no helpers: it has the next copies to start.)
    void wait(Job *job)
    {
        while (job->left.load() != 0)
            if (!threads_.empty() || !one()) std::this_thread::yield();
    }

private:
    bool one()
    {
        Job *j;
        int64_t part;
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (jobs_.empty()) return false;
            j = jobs_.front();
            part = j->next++;
            if (j->next == j->parts) {
                jobs_.pop_front();
                open_.fetch_sub(1);
            }
        }
        j->call(j->arg, part);
        j->left.fetch_sub(1);
        return true;
    }
    void work()
    {
        for (;;) {
            if (one()) continue;
            // a call posts its jobs within a copy's time of each other: look
            // for the next one for a while before sleeping
            for (int k = 0; k < 4000 && open_.load() == 0 && !stop_.load(); ++k) __builtin_ia32_pause();
            std::unique_lock<std::mutex> lk(mu_);
            cv_.wait(lk, [&] { return stop_.load() || !jobs_.empty(); });
            if (jobs_.empty()) return;  // stopped
        }
    }

    std::vector<std::thread> threads_;
    std::mutex mu_;
    std::condition_variable cv_;
    std::deque<Job *> jobs_;
    std::atomic<int> open_{0};
    std::atomic<bool> stop_{false};
};

// The 2 MiB pages of the caller's memory that [dst, dst + n) touches: a part
// per page, so that two threads never wait for the same page fault.
struct PageParts {
    static constexpr uintptr_t kPage = (uintptr_t)2 << 20;
    uintptr_t lo = 0, hi = 0, base = 0;
    PageParts() = default;
    PageParts(const void *dst, uint64_t n) : lo((uintptr_t)dst), hi((uintptr_t)dst + n), base(lo & ~(kPage - 1)) {}
    int64_t count() const { return hi > lo ? (int64_t)((hi - base + kPage - 1) / kPage) : 0; }
    // bytes [first, first + size) of the range in part p
    uint64_t first(int64_t p) const { return p == 0 ? 0 : base + (uintptr_t)p * kPage - lo; }
    uint64_t size(int64_t p) const
    {
        const uintptr_t end = base + (uintptr_t)(p + 1) * kPage;
        return (end < hi ? end : hi) - lo - first(p);
    }
};

}  // namespace tsdf
