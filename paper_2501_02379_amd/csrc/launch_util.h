// Host-side launch helpers shared by the kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <map>
#include <mutex>
#include <utility>

namespace tgrad {

constexpr size_t kLdsLimit = 160 * 1024;

template <typename Kern>
inline bool allow_lds(Kern kern, size_t bytes) {
  if (bytes <= 48 * 1024) return true;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes) == hipSuccess;
}

// Workgroups of `kern` that are resident on one compute unit at a time (registers, LDS), asked of
// the runtime once per kernel, workgroup and LDS size (`most` bounds the answer).  The tile loops are persistent
// (stride = grid size), so the grid is exactly one resident set: more workgroups would run as a ragged second set.
template <typename Kern>
int resident_blocks(Kern kern, int threads, size_t lds, int most = 4) {
  static std::mutex mu;
  static std::map<std::pair<std::pair<const void*, int>, size_t>, int> cache;
  const std::pair<std::pair<const void*, int>, size_t> key({reinterpret_cast<const void*>(kern), threads}, lds);
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second < most ? it->second : most;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, threads, lds) != hipSuccess || nb < 1) nb = 1;
  cache[key] = nb;
  return nb < most ? nb : most;
}

// Compute units of the current device (256 on an MI355X), asked of the runtime once per device.
inline int compute_units() {
  constexpr int kMaxDev = 64;
  static std::atomic<int> cached[kMaxDev];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) dev = 0;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

}  // namespace tgrad
