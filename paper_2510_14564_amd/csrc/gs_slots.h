// Pinned host words that queued device work writes and the host reads (no HIP
// in this header: the allocation is passed in).
#pragma once

#include <cstddef>
#include <mutex>
#include <vector>

namespace gs {

// Pairs of 64-bit words, handed out to one call at a time.  As many exist as
// calls ran at once, and at most `keep` of them wait for the next call; the others
// are freed when they come back.  Safe from any thread.
class SlotPool {
 public:
  typedef unsigned long long* (*Alloc)();              // two words, or NULL
  typedef void (*Free)(unsigned long long*);
  SlotPool(Alloc alloc, Free release, size_t keep) : alloc_(alloc), free_(release), keep_(keep) {
    idle_.reserve(keep);   // give() allocates nothing
  }

  unsigned long long* take() {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (!idle_.empty()) {
        unsigned long long* const p = idle_.back();
        idle_.pop_back();
        return p;
      }
    }
    return alloc_();
  }
  void give(unsigned long long* p) {
    {
      std::lock_guard<std::mutex> lock(mu_);
      if (idle_.size() < keep_) {
        idle_.push_back(p);
        return;
      }
    }
    free_(p);
  }

 private:
  std::mutex mu_;
  std::vector<unsigned long long*> idle_;
  const Alloc alloc_;
  const Free free_;
  const size_t keep_;
};

// One call's slot.  It goes back to the pool only once work_done() has said
// that the work which writes it has ended: a call that fails with such work
// queued leaves its slot out of the pool, where that work may still write it.
class Slot {
 public:
  explicit Slot(SlotPool& pool) : pool_(pool), p_(pool.take()) {}
  ~Slot() {
    if (p_ && done_) pool_.give(p_);
  }
  Slot(const Slot&) = delete;
  Slot& operator=(const Slot&) = delete;
  unsigned long long* get() const { return p_; }
  void work_done() { done_ = true; }

 private:
  SlotPool& pool_;
  unsigned long long* const p_;
  bool done_ = false;
};

}  // namespace gs
