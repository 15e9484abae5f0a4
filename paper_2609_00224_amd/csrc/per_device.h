// Values that do not change as long as a process lives, asked for once per
// device: plain C++, no device code.  Internal to the library.
#ifndef QTEA_PER_DEVICE_H_
#define QTEA_PER_DEVICE_H_

#include <algorithm>
#include <atomic>

namespace qtea_detail {

constexpr int kMaxDevices = 64;

// query(dev), which is kept in `known` unless it is 0 (a failure: asked again
// next time).  Threads that ask at once may each run the query.
template <class Query>
int per_device(std::atomic<int> (&known)[kMaxDevices], int dev, Query query) {
  if (dev < 0) return 0;
  if (dev >= kMaxDevices) return query(dev);
  int n = known[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    n = query(dev);
    known[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Most workgroups of a kernel whose workgroups wait for one another, on a
// device that holds `resident` of them: a quarter, so that calls on four
// streams (the hardware queues of a process) are resident together, at most
// `most`; a single workgroup waits for nobody.
inline int waiting_workgroups(int resident, int most) { return std::max(1, std::min(most, resident / 4)); }

}  // namespace qtea_detail

#endif  // QTEA_PER_DEVICE_H_
