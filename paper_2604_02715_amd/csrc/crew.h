// A set of threads that go through several passes together (host code without HIP, so that it can be tested on its own).
#pragma once

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <type_traits>
#include <vector>

namespace fluxmoe {

// take() hands out the numbers 0, 1, .. of the current pass, wait() ends it for everybody, and the last to arrive runs `once`
// before the next one begins.  The caller is one of them; where the system gives fewer threads than asked for, those that there are
// do the work.  What one of them throws ends the work of all, and run() throws it again when the others have stopped.
class Crew {
public:
    explicit Crew(int wanted) {
        threads_.reserve(size_t(wanted - 1));
        for (int t = 1; t < wanted; ++t) {
            try {
                threads_.emplace_back([this, t]() {
                    {
                        std::unique_lock<std::mutex> lock(m_);
                        cv_.wait(lock, [this]() { return work_ != nullptr || closed_; });
                        if (!work_) return;
                    }
                    work_(this, user_, uint32_t(t));
                });
            } catch (const std::system_error&) {
                break;
            } catch (const std::bad_alloc&) {
                break;
            }
        }
    }
    ~Crew() {
        { std::lock_guard<std::mutex> lock(m_); closed_ = true; }
        cv_.notify_all();
        for (auto& t : threads_) t.join();
    }
    uint32_t size() const { return uint32_t(threads_.size()) + 1; }
    template <typename F>
    void run(F&& f) {
        const auto work = [](Crew* crew, void* u, uint32_t me) { crew->share(*static_cast<std::remove_reference_t<F>*>(u), me); };
        {
            std::lock_guard<std::mutex> lock(m_);
            user_ = &f;
            work_ = work;
        }
        cv_.notify_all();
        work(this, &f, 0u);
        for (auto& t : threads_) t.join();
        threads_.clear();
        if (thrown_) std::rethrow_exception(thrown_);
    }
    uint64_t take() { return next_.fetch_add(1, std::memory_order_relaxed); }
    template <typename F>
    void wait(F&& once) {
        std::unique_lock<std::mutex> lock(m_);
        if (stopped_) throw Stop();
        const uint64_t pass = pass_;
        if (++arrived_ == size()) {
            once();
            arrived_ = 0;
            next_.store(0, std::memory_order_relaxed);
            ++pass_;
            cv_.notify_all();
        } else {
            cv_.wait(lock, [&]() { return pass_ != pass || stopped_; });
            if (pass_ == pass) throw Stop();
        }
    }

private:
    struct Stop {};                              // another one has thrown
    template <typename F>
    void share(F& f, uint32_t me) {
        try {
            f(me);
        } catch (...) {
            {
                std::lock_guard<std::mutex> lock(m_);
                if (!stopped_) thrown_ = std::current_exception();
                stopped_ = true;
                next_.store(1ull << 63, std::memory_order_relaxed);      // nothing left to take; no pass ends any more, which would reset it
            }
            cv_.notify_all();
        }
    }

    std::vector<std::thread> threads_;
    std::mutex m_;
    std::condition_variable cv_;
    void (*work_)(Crew*, void*, uint32_t) = nullptr;
    void* user_ = nullptr;
    bool closed_ = false;
    bool stopped_ = false;
    std::exception_ptr thrown_;
    std::atomic<uint64_t> next_{0};
    uint64_t pass_ = 0;
    uint32_t arrived_ = 0;
};

}  // namespace fluxmoe
