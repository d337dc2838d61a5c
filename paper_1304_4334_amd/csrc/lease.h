// Host objects lent to one call at a time (plain C++, used by the batched
// driver for its streams and page-locked memory).
#pragma once

#include <stddef.h>

#include <mutex>
#include <vector>

namespace smc {

// Idle objects shared by all host threads of the process, at most `keep` of
// them: a call takes one that fits it, or makes its own, and gives it back at
// its end.  So there are never more objects than calls at a time plus `keep`,
// however many threads have made calls.
template <class T>
class LeaseStore {
 public:
  explicit LeaseStore(size_t keep) : keep_(keep) { idle_.reserve(keep + 1); }

  // The idle object given back last for which fits() holds, or NULL.
  template <class Fits>
  T *take(Fits &&fits) {
    std::lock_guard<std::mutex> lock(mutex_);
    for (size_t i = idle_.size(); i-- > 0;)
      if (fits(*idle_[i])) {
        T *x = idle_[i];
        idle_.erase(idle_.begin() + i);
        return x;
      }
    return nullptr;
  }

  // Gives x back.  Returns the object that now has to go (the one idle
  // longest), which the caller destroys outside the lock, or NULL.
  T *give(T *x) {
    std::lock_guard<std::mutex> lock(mutex_);
    idle_.push_back(x);
    if (idle_.size() <= keep_) return nullptr;
    T *out = idle_.front();
    idle_.erase(idle_.begin());
    return out;
  }

 private:
  const size_t keep_;
  std::mutex mutex_;
  std::vector<T *> idle_;
};

}  // namespace smc
