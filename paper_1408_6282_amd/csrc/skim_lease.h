// skim_lease.h -- objects lent to threads.
//
// A thread keeps what it is lent until it ends; then the next thread that asks
// gets it.  So there are never more objects than threads held one at once, and
// threads that come and go leave none behind.
#pragma once

#include <mutex>
#include <vector>

namespace skim {

template <class T> class LeasePool {
  public:
    T *take() {
        std::lock_guard<std::mutex> lk(mu_);
        if (free_.empty()) return nullptr;
        T *t = free_.back();
        free_.pop_back();
        return t;
    }
    void give(T *t) {
        std::lock_guard<std::mutex> lk(mu_);
        free_.push_back(t);
    }

  private:
    std::mutex mu_;
    std::vector<T *> free_;
};

// To be used as a thread_local; the pool has to outlive every thread.
template <class T> class Lease {
  public:
    explicit Lease(LeasePool<T> &pool) : pool_(pool) {}
    Lease(const Lease &) = delete;
    Lease &operator=(const Lease &) = delete;
    ~Lease() {
        if (t_) pool_.give(t_);
    }
    template <class Make> T *get(Make make) {
        if (!t_) t_ = pool_.take();
        if (!t_) t_ = make();
        return t_;
    }
    // Not to be lent again (something may still write to it).
    void drop() { t_ = nullptr; }

  private:
    LeasePool<T> &pool_;
    T *t_ = nullptr;
};

}  // namespace skim
