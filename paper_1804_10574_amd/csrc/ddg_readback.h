// Device -> host copies, large ones through a ring of pinned slots (ddg_readback.cpp). One per module: SLOTS * PIECE
// bytes of pinned memory (8 MiB), allocated at the first large copy and given back with the module. Calls from
// several threads take turns.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <mutex>

namespace ddg {

struct Readback {
  static constexpr int SLOTS = 8;
  static constexpr size_t PIECE = (size_t)1 << 20;
  void* ring = nullptr;
  hipEvent_t ev[SLOTS] = {};
  std::mutex mu;
  // Enqueues on s and returns when `host` holds the data.
  hipError_t copy(void* host, const void* dev, size_t bytes, hipStream_t s);
  void release();
};

}  // namespace ddg
