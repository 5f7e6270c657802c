// Which kernels may use how much dynamic LDS.  Host code on plain values: the kernels' owners share a table, and so do the
// threads that drive caches of their own.
#pragma once

#include <stddef.h>

#include <mutex>

namespace moei {

template <int N>  // kernels that it remembers; others are raised anew at every call
class LdsLimits {
  public:
    // Calls `raise` unless it has been called for this kernel with as many bytes, and returns its result (0: done).  A limit
    // is known only once it has been raised, and one thread raises at a time: a lower one that came later would take the higher one back.
    template <typename F>
    int at_least(const void* kernel, size_t bytes, F raise) {
        std::lock_guard<std::mutex> only(m_);
        int i = 0;
        while (i < n_ && kernel_[i] != kernel) ++i;
        if (i < n_ && bytes_[i] >= bytes) return 0;
        const int rc = raise();
        if (rc != 0 || i == N) return rc;
        kernel_[i] = kernel;
        bytes_[i] = bytes;
        if (i == n_) ++n_;
        return 0;
    }

  private:
    std::mutex m_;
    const void* kernel_[N] = {};
    size_t bytes_[N] = {};
    int n_ = 0;
};

}  // namespace moei
