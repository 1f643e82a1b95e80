// A setting that a kernel needs once on every device of the process (the limit on its dynamic LDS), which several
// threads may come to make.  Host code only.
#pragma once

#include <atomic>
#include <cstdint>

namespace rvn {

class OncePerDevice {
  public:
    // Whether it still has to be made on `device`; making it twice does no harm.  Devices past the last bit: every time.
    bool wanted(int device) const {
        return device < 0 || device >= 64 || !(made_.load(std::memory_order_acquire) >> device & 1u);
    }
    void made(int device) {
        if (device >= 0 && device < 64) made_.fetch_or((uint64_t)1 << device, std::memory_order_release);
    }

  private:
    std::atomic<uint64_t> made_{0};
};

}  // namespace rvn
