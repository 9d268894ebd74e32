"""The read-back through the ring of pinned slots on the host: ddg_readback.cpp linked against stand-ins for the runtime
calls it makes (copies are memcpy). Its callers are C functions, so whatever allocation, thread, event or pinned memory
is not to be had, the copy comes back whole and nothing is thrown."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1804_10574_amd", "csrc")

HARNESS = r"""
#include "ddg_readback.h"
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <new>

static std::atomic<long> left{-1};     // allocations until they fail; -1: they do not
static int events_left = -1; static bool no_pinned = false;
static std::atomic<long> plain{0};     // copies by the runtime's way
void* operator new(size_t n) {
  long l = left.load();
  while (l > 0 && !left.compare_exchange_weak(l, l - 1)) {}
  if (l == 0) throw std::bad_alloc();
  if (void* p = malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
extern "C" {
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { ++plain; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = no_pinned ? nullptr : malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (events_left == 0) return hipErrorOutOfMemory;
  if (events_left > 0) --events_left;
  *e = (hipEvent_t)16; return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

static char *src, *dst;
static bool copies(size_t n) {
  ddg::Readback rb;
  memset(dst, 0, n);
  const bool ok = rb.copy(dst, src, n, nullptr) == hipSuccess && memcmp(dst, src, n) == 0;
  rb.release();
  return ok;
}

int main() {
  const size_t MiB = (size_t)1 << 20, most = 21 * MiB;
  src = (char*)malloc(most); dst = (char*)malloc(most);
  for (size_t i = 0; i < most; ++i) src[i] = (char)(i * 2654435761u >> 13);
  for (size_t n : {8 * MiB, 8 * MiB + 1, 20 * MiB + 77, most}) {
    if (!copies(n) || plain) return printf("%zu bytes: not copied through the ring\n", n), 1;
    for (long k = 0; k < 24; ++k) {
      printf("%zu bytes, %ld allocations succeed\n", n, k); fflush(stdout);
      left = k;
      const bool ok = copies(n);
      left = -1;
      if (!ok) return printf("not copied\n"), 1;
    }
    plain = 0;
    for (int k = 0; k < 8; ++k) {
      events_left = k;
      const bool ok = copies(n);
      events_left = -1;
      if (!ok) return printf("not copied with %d events\n", k), 1;
    }
    no_pinned = true;
    const bool ok = copies(n);
    no_pinned = false;
    if (!ok || plain != 9) return printf("not copied without pinned memory\n"), 1;
    plain = 0;
  }
  printf("all copies whole\n");
  return 0;
}
"""


# the first copy of a module pays for the pinned memory: 8 MiB of it, whatever is copied
PINNED = HARNESS[:HARNESS.index("int main")].replace("*p = no_pinned", "pinned += n; *p = no_pinned").replace("static bool no_pinned", "static size_t pinned = 0; static bool no_pinned") + r"""
int main() {
  const size_t MiB = (size_t)1 << 20, most = 40 * MiB + 5;
  src = (char*)malloc(most); dst = (char*)malloc(most);
  for (size_t i = 0; i < most; ++i) src[i] = (char)(i * 2654435761u >> 13);
  for (size_t n : {8 * MiB, 9 * MiB + 1, 19 * MiB, 26 * MiB + 300000, most}) {
    pinned = 0;
    if (!copies(n) || plain) return printf("%zu bytes: not copied through the ring\n", n), 1;
    if (pinned == 0 || pinned > 8 * MiB) return printf("%zu bytes: %zu pinned\n", n, pinned), 1;
  }
  printf("all copies whole\n");
  return 0;
}
"""


def run(tmp_path, harness):
    gxx = shutil.which("g++")
    inc = "/opt/rocm/include"
    if not gxx or not os.path.isdir(inc):
        pytest.skip("needs g++ and the HIP headers")
    main = tmp_path / "main.cpp"
    main.write_text(harness)
    exe = tmp_path / "readback"
    subprocess.run([gxx, "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", inc, "-I", CSRC, str(main),
                    os.path.join(CSRC, "ddg_readback.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout[-200:], r.stderr[-200:])
    assert "all copies whole" in r.stdout


def test_a_copy_comes_back_whole_whatever_is_missing(tmp_path):
    run(tmp_path, HARNESS)


def test_a_first_copy_pins_no_more_than_8_mib(tmp_path):
    run(tmp_path, PINNED)
