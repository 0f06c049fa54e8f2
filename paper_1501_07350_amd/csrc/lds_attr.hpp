// lds_attr.hpp -- a kernel's dynamic LDS limit (host code, plain C++).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace offt {

constexpr size_t kDefaultLds = 64 * 1024;   // dynamic LDS a kernel may use without raising its limit

// Makes sure that a kernel may be launched with `lds` bytes of dynamic LDS on
// device `dev`: its limit is raised once per device, to `limit`, what the
// device has.  Every caller sets the same value, so it does not matter which of
// several threads sets it last.  `done` holds a bit per device; `set` sets the
// limit and returns 0 on success.
template <typename Set>
int raise_lds_limit(std::atomic<uint64_t>& done, int dev, size_t lds, size_t limit, Set set) {
    if (lds <= kDefaultLds) return 0;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;   // 0: set on each launch
    if (done.load(std::memory_order_acquire) & bit) return 0;
    const int rc = set(limit);
    if (rc == 0) done.fetch_or(bit, std::memory_order_release);
    return rc;
}

}  // namespace offt
