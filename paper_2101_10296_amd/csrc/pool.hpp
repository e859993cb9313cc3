// Helper threads of host planning.
#pragma once

#include <new>
#include <system_error>
#include <thread>
#include <utility>

namespace qaoa {

// Up to 15 threads beside the caller's, joined on every way out (a joinable thread's destructor ends
// the process).
class Pool {
public:
    static constexpr int MOST = 15;
    ~Pool() { join(); }
    template <class... F>
    bool start(F&&... f) {   // false: no thread to be had, or no memory for it
        if (n_ == MOST) return false;
        try {
            t_[n_] = std::thread(std::forward<F>(f)...);
        } catch (const std::system_error&) {
            return false;
        } catch (const std::bad_alloc&) {
            return false;
        }
        ++n_;
        return true;
    }
    void join() {
        while (n_ > 0) t_[--n_].join();
    }

private:
    std::thread t_[MOST];
    int n_ = 0;
};

}  // namespace qaoa
