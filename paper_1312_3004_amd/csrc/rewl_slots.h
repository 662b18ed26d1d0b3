// rewl_slots.h -- slots of one block of memory, shared by the handles of a
// process.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace rewl_host {

// 64 slots of 512 bytes.  The block is allocated once and stays until the
// process ends; a handle takes a slot when it first needs one and gives it
// back when it is destroyed.  Safe with several threads.
class SlotBlock {
  public:
    static constexpr int kSlots = 64;
    static constexpr size_t kBytes = 512;

    // Has `alloc(bytes)` allocate the block (null: tried again next time).
    template <class Alloc>
    void reserve(Alloc alloc) {
        std::lock_guard<std::mutex> lock(mu_);
        if (!base_) base_ = (unsigned char *)alloc(kSlots * kBytes);
    }
    // A free slot, or null.
    unsigned char *take() {
        std::lock_guard<std::mutex> lock(mu_);
        if (!base_ || used_ == ~(uint64_t)0) return nullptr;
        const int i = __builtin_ctzll(~used_);
        used_ |= (uint64_t)1 << i;
        return base_ + i * kBytes;
    }
    void give(unsigned char *slot) {
        if (!slot) return;
        std::lock_guard<std::mutex> lock(mu_);
        used_ &= ~((uint64_t)1 << ((slot - base_) / kBytes));
    }

  private:
    std::mutex mu_;
    unsigned char *base_ = nullptr;
    uint64_t used_ = 0;
};

}  // namespace rewl_host
