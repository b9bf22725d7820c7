// Result slots of the calls that wait for the device: pinned words that
// kernels (or a copy) write and the host reads after its stream
// synchronisation.  A copy to pageable memory instead made the runtime stage
// it and wait twice.  One page, made by the first call that finds it missing
// and kept; a call takes a slot and gives it back, and a call that finds none
// falls back to the workspace and a pageable copy.  Host code alone.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace rsz {

constexpr int kResultHeader = 80;   // bytes of a stream's header

struct ResultSlot {
  uint64_t bytes;
  int32_t status;
  uint8_t header[kResultHeader];
  uint8_t pad[128 - 12 - kResultHeader];
};
static_assert(sizeof(ResultSlot) == 128, "a slot is two cache lines");

class ResultSlots {
 public:
  static constexpr int kSlots = 32;
  // alloc: the page (null: none now; the next call asks again).
  explicit ResultSlots(void *(*alloc)(size_t)) : alloc_(alloc) {}

  ResultSlot *take(int *index) {
    std::lock_guard<std::mutex> lk(mu_);
    if (!page_) page_ = (ResultSlot *)alloc_(kSlots * sizeof(ResultSlot));
    if (!page_ || used_ == ~0u) return nullptr;
    *index = __builtin_ctz(~used_);
    used_ |= 1u << *index;
    return page_ + *index;
  }
  void give(int index) {
    std::lock_guard<std::mutex> lk(mu_);
    used_ &= ~(1u << index);
  }

 private:
  void *(*alloc_)(size_t);
  std::mutex mu_;
  ResultSlot *page_ = nullptr;
  uint32_t used_ = 0;   // bit i: slot i is taken
};

// A call's slot (null: none free), given back when the call returns.
class Result {
 public:
  explicit Result(ResultSlots &slots) : slots_(slots) { slot = slots.take(&index_); }
  ~Result() {
    if (slot) slots_.give(index_);
  }
  // The device may still write the slot (its stream could not be waited for):
  // it stays taken for good.
  void abandon() { slot = nullptr; }
  Result(const Result &) = delete;
  Result &operator=(const Result &) = delete;
  ResultSlot *slot;

 private:
  ResultSlots &slots_;
  int index_ = 0;
};

}  // namespace rsz
