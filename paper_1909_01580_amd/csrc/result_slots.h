// Slots of one block of host memory for the results of the reductions, handed
// out per call in flight.  Host code only.
#pragma once

#include <stdint.h>

#include <mutex>

namespace hgks {

// kCount slots of kDoubles doubles each.  `Alloc()` gives the block (null: no
// slots), once per process at the first take; it is kept.  A slot belongs to a
// call from take() until give(): a context holds none between its calls, so
// any number of contexts may be alive, and up to kCount calls of as many
// threads have one at a time.
template <double* (*Alloc)()>
class ResultSlots {
 public:
  static constexpr int kCount = 64, kDoubles = 8;

  // Null when no slot is free (or there is no block).
  double* take() {
    std::lock_guard<std::mutex> lock(mu_);
    if (!tried_) {
      tried_ = true;
      block_ = Alloc();
    }
    if (!block_ || !free_) return nullptr;
    const int k = __builtin_ctzll(free_);
    free_ &= free_ - 1;
    return block_ + kDoubles * k;
  }

  void give(double* p) {
    if (!p) return;
    std::lock_guard<std::mutex> lock(mu_);
    free_ |= 1ull << ((p - block_) / kDoubles);
  }

 private:
  std::mutex mu_;
  double* block_ = nullptr;
  bool tried_ = false;
  uint64_t free_ = ~0ull;
};

}  // namespace hgks
