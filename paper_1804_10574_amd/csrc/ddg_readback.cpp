// Device -> host copies of a module's state (weights, velocity, gradients, stored inputs).
//
// A large copy into fresh pageable memory moves about 10 GB/s here: the runtime stages it in 1 MiB pieces, and its
// one thread takes the page faults of the destination between two pieces. From RING_MIN on pieces land in a
// small ring of pinned slots instead while threads of this process copy earlier pieces out: 102 MB (23
// bottleneck blocks) 9.8 -> 3.5 ms with a transfer a piece; at 1.7 MB the two are even (0.10 ms), below the
// runtime's way is shorter (0.04 MB: 22 against 38 us), and it needs no pinned memory. A transfer costs the queue about 12 us
// beside its bytes (102 MB by 0.5 / 1 / 2 / 4 MiB: 4.8 / 3.4 / 2.8 / 2.6 ms; the link alone 1.85), so two pieces go together.
// A module's first copy allocates the ring, so it is no larger than this. ms, first copy / later ones: 27 MB 1.5 / 0.83, with 16 MiB in
// eight slots 2.0 / 0.82, with a transfer a piece 1.7 / 1.0; 102 MB 3.8 / 2.9, 4.2 / 2.8 and 4.2 / 3.4.
//
// The callers are C functions, so no exception leaves this file: without host memory for the bookkeeping the copy is
// the runtime's, without threads the caller copies the pieces out itself.
#include "ddg_readback.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <memory>
#include <new>
#include <thread>

namespace ddg {

namespace {

constexpr size_t PIECE = Readback::PIECE, RING_MIN = (size_t)8 << 20, TOGETHER = 2;   // pieces of a transfer (the last may have fewer)
constexpr size_t SHARE = (size_t)256 << 10, SHARES = PIECE / SHARE;   // what a thread copies out at a time
constexpr int SLOTS = Readback::SLOTS;
static_assert(SLOTS % TOGETHER == 0, "the slots of a transfer are neighbours");
constexpr int WORKERS = 7;            // beside the calling thread

struct Job {
  char* dst; const char* ring; size_t bytes, pieces, shares;
  std::atomic<size_t> landed{0}, ticket{0};     // pieces, shares
  std::atomic<bool> stop{false};
  std::unique_ptr<std::atomic<int>[]> left;    // shares of a piece not yet copied out; null: no memory for it
  Job(char* d, const char* r, size_t b, size_t n)
      : dst(d), ring(r), bytes(b), pieces(n), shares((b + SHARE - 1) / SHARE), left(new (std::nothrow) std::atomic<int>[n]) {
    if (left) for (size_t i = 0; i < n; ++i) left[i].store((int)std::min(SHARES, shares - i * SHARES), std::memory_order_relaxed);
  }
  void copy_out(size_t share) {
    const size_t piece = share / SHARES;
    memcpy(dst + share * SHARE, ring + (piece % SLOTS) * PIECE + (share % SHARES) * SHARE, std::min(SHARE, bytes - share * SHARE));
    left[piece].fetch_sub(1, std::memory_order_release);
  }
  bool emptied(size_t piece) const { return left[piece].load(std::memory_order_acquire) == 0; }
  void work() {   // until every share has an owner, or stop
    for (;;) {
      const size_t i = ticket.fetch_add(1, std::memory_order_relaxed);
      if (i >= shares) return;
      while (landed.load(std::memory_order_acquire) <= i / SHARES) {
        if (stop.load(std::memory_order_relaxed)) return;
        std::this_thread::yield();
      }
      copy_out(i);
    }
  }
};

// The copy through the ring. With workers, they copy every piece out and the caller only feeds them.
hipError_t through_ring(Readback& rb, char* dst, const char* src, size_t bytes, hipStream_t s) {
  const size_t pieces = (bytes + PIECE - 1) / PIECE;
  Job job(dst, (const char*)rb.ring, bytes, pieces);
  if (!job.left) return hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost);
  std::thread team[WORKERS];
  const unsigned hw = std::thread::hardware_concurrency();
  const size_t want = std::min<size_t>(WORKERS, hw > 1 ? hw - 1 : 0);
  size_t workers = 0;
  try {
    for (; workers < want; ++workers) team[workers] = std::thread([&job] { job.work(); });
  } catch (...) {}   // (system_error, bad_alloc) fewer threads, or none: the caller copies
  hipError_t err = hipSuccess;
  size_t sent = 0, landed = 0;
  auto end_of = [&](size_t first) { return std::min(first + TOGETHER, pieces); };   // of the transfer from piece `first` on
  while (landed < pieces && err == hipSuccess) {
    while (sent < pieces && err == hipSuccess) {
      const size_t end = end_of(sent);
      bool room = true;
      for (size_t i = sent; i < end; ++i) room = room && (i < (size_t)SLOTS || job.emptied(i - SLOTS));
      if (!room) break;
      err = hipMemcpyAsync((char*)rb.ring + (sent % SLOTS) * PIECE, src + sent * PIECE, std::min(end * PIECE, bytes) - sent * PIECE,
                           hipMemcpyDeviceToHost, s);
      if (err == hipSuccess) err = hipEventRecord(rb.ev[(end - 1) % SLOTS], s);
      if (err == hipSuccess) sent = end;
    }
    if (err != hipSuccess) break;
    if (landed == sent) { std::this_thread::yield(); continue; }   // the ring is full of pieces being copied out
    const size_t end = end_of(landed);
    err = hipEventSynchronize(rb.ev[(end - 1) % SLOTS]);
    if (err != hipSuccess) break;
    if (workers == 0)
      for (size_t i = landed * SHARES; i < std::min(end * SHARES, job.shares); ++i) job.copy_out(i);
    landed = end;
    job.landed.store(landed, std::memory_order_release);
  }
  if (err != hipSuccess) { job.stop.store(true); (void)hipStreamSynchronize(s); }
  for (size_t i = 0; i < workers; ++i) team[i].join();
  return err;
}

}  // namespace

hipError_t Readback::copy(void* host, const void* dev, size_t bytes, hipStream_t s) {
  if (bytes < RING_MIN) return hipMemcpy(host, dev, bytes, hipMemcpyDeviceToHost);
  std::lock_guard<std::mutex> hold(mu);
  if (!ring) {
    void* p = nullptr;
    if (hipHostMalloc(&p, SLOTS * PIECE, hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return hipMemcpy(host, dev, bytes, hipMemcpyDeviceToHost);
    }
    for (int i = 0; i < SLOTS; ++i) {
      const hipError_t e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
      if (e == hipSuccess) continue;
      while (i-- > 0) (void)hipEventDestroy(ev[i]);
      (void)hipHostFree(p);
      (void)hipGetLastError();
      return hipMemcpy(host, dev, bytes, hipMemcpyDeviceToHost);
    }
    ring = p;
  }
  return through_ring(*this, (char*)host, (const char*)dev, bytes, s);
}

void Readback::release() {
  if (!ring) return;
  for (int i = 0; i < SLOTS; ++i) (void)hipEventDestroy(ev[i]);
  (void)hipHostFree(ring);
  ring = nullptr;
}

}  // namespace ddg
