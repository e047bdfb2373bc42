// What a kernel's occupancy query said, by dynamic LDS size (host code only).
#pragma once

#include <stddef.h>

namespace gmc {

// Blocks of one kernel that a CU holds at once.  Callers come with a few sizes
// in turn, so the last kSizes answers are kept and a query costs its driver
// calls once.  Dynamic LDS above 64 KB has to be granted to the kernel first:
// the grant only grows, as another thread may be between its plan and its
// launch with the size that it was granted.  The caller holds a lock.
class KernelRoom {
 public:
  // grant(lds) raises the kernel's limit; ask(lds, &n) queries; both false on
  // failure, which reads as no room.
  template <class Grant, class Ask>
  int blocks(size_t lds, Grant grant, Ask ask) {
    for (int i = 0; i < used_; ++i)
      if (lds_[i] == lds) return blocks_[i];
    int n = 0;
    bool ok = lds <= granted_;
    if (!ok && grant(lds)) {
      granted_ = lds;
      ok = true;
    }
    if (!ok || !ask(lds, &n)) n = 0;
    const int at = used_ < kSizes ? used_++ : next_;
    next_ = (at + 1) % kSizes;
    lds_[at] = lds;
    blocks_[at] = n;
    return n;
  }

 private:
  static constexpr int kSizes = 8;
  size_t lds_[kSizes] = {}, granted_ = 64 * 1024;
  int blocks_[kSizes] = {};
  int used_ = 0, next_ = 0;
};

}  // namespace gmc
