// persistent_grid.hpp -- the grid of a persistent launch.  Host code only.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <mutex>
#include <vector>

namespace pulse {

// Largest grid of a ticketed launch.
constexpr uint32_t kMaxGrid = 1u << 16;

// Blocks of `kernel` (launched with `block` threads) that fit on the current
// device at once.  The occupancy query is made once per (device, kernel) and
// remembered: at most the library's persistent kernels times the process's
// devices, sixteen kernels on eight devices among them.
inline int persistent_grid(const void* kernel, int block) {
  struct Entry {
    const void* kernel;
    int dev, block, grid;
  };
  static std::vector<Entry> cache;
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  {
    std::lock_guard<std::mutex> g(mu);
    for (const Entry& e : cache)
      if (e.kernel == kernel && e.dev == dev && e.block == block) return e.grid;
  }
  int cus = 0, per_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess) return 0;
  int grid = cus * (per_cu > 0 ? per_cu : 1);
  if (grid > (int)kMaxGrid) grid = (int)kMaxGrid;
  std::lock_guard<std::mutex> g(mu);
  try {
    cache.push_back(Entry{kernel, dev, block, grid});
  } catch (...) {  // no memory: asked again next time
  }
  return grid;
}

}  // namespace pulse
