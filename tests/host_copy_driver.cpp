// Runs csrc/host_copy.h on the CPU against stand-ins for the HIP calls that it
// makes (a copy is done when it is enqueued; waiting for the first event takes
// as long as the work enqueued before it).  tests/test_host_copy.py builds and
// runs one case a process.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>
#include <unistd.h>

#include <vector>

#include "host_copy.h"

static int waits = 0;             // event waits so far
static useconds_t first_wait = 0; // length of the first one
static int current = 0;           // the current device
static const void* pinned = nullptr;   // an address that the runtime knows
static int to_pinned = 0;         // copies enqueued to it
struct Event { int device; };
static int device_of(hipStream_t s) { return s ? *(int*)s : current; }   // a stream is its device's number

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event{current}; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {   // an event belongs to the device it was created on
  return ((Event*)e)->device == device_of(s) ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = device_of(s); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
  if (waits++ == 0 && first_wait) usleep(first_wait);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (d == pinned) ++to_pinned;
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  memset(a, 0, sizeof(*a));
  a->type = p == pinned ? hipMemoryTypeHost : hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

static double cpu_seconds() {
  timespec t;
  clock_gettime(CLOCK_PROCESS_CPUTIME_ID, &t);
  return t.tv_sec + 1e-9 * t.tv_nsec;
}

static std::vector<unsigned char> pattern(size_t n) {
  std::vector<unsigned char> v(n);
  unsigned x = 12345u + (unsigned)n;
  for (auto& b : v) b = (unsigned char)((x = x * 1664525u + 1013904223u) >> 24);
  return v;
}

// every byte arrives, at sizes around the chunks and the threads' shares
static int values() {
  dugks::HostCopy hc;
  for (size_t n : {size_t(1), size_t(1000), (size_t(16) << 20) - 1, size_t(16) << 20, (size_t(16) << 20) + 1,
                   (size_t(20) << 20) - 3, (size_t(37) << 20) + 12345}) {
    const std::vector<unsigned char> src = pattern(n);
    std::vector<unsigned char> dst(n, 0);
    if (hc.out(dst.data(), src.data(), n, nullptr) != hipSuccess || dst != src) {
      fprintf(stderr, "%zu bytes differ\n", n);
      return 1;
    }
  }
  return 0;
}

// while the work enqueued before the copy runs, no thread uses the CPU
static int idle() {
  dugks::HostCopy hc;
  const size_t n = size_t(16) << 20;
  const std::vector<unsigned char> src = pattern(n);
  std::vector<unsigned char> dst(n, 0);
  const double t0 = cpu_seconds();
  if (hc.out(dst.data(), src.data(), n, nullptr) != hipSuccess) return 1;
  const double copy = cpu_seconds() - t0;   // the copy itself
  waits = 0;
  first_wait = 800000;
  const double t1 = cpu_seconds();
  if (hc.out(dst.data(), src.data(), n, nullptr) != hipSuccess) return 1;
  const double waited = cpu_seconds() - t1;
  fprintf(stderr, "CPU seconds: %.3f, with 0.8 s to wait %.3f\n", copy, waited);
  return dst == src && waited < copy + 0.4 ? 0 : 1;   // one thread waiting actively would add 0.8
}

// a stream of another device than the current one, then of the current one
static int devices() {
  dugks::HostCopy hc;
  const size_t n = size_t(17) << 20;
  const std::vector<unsigned char> src = pattern(n);
  int dev[3] = {1, 0, 2};
  for (int& d : dev) {
    std::vector<unsigned char> dst(n, 0);
    if (hc.out(dst.data(), src.data(), n, (hipStream_t)&d) != hipSuccess || dst != src || current != 0) {
      fprintf(stderr, "device %d\n", d);
      return 1;
    }
  }
  return 0;
}

// memory that is pinned already is filled by one copy
static int direct() {
  dugks::HostCopy hc;
  const size_t n = size_t(24) << 20;
  const std::vector<unsigned char> src = pattern(n);
  std::vector<unsigned char> dst(n, 0);
  pinned = dst.data();
  return hc.out(dst.data(), src.data(), n, nullptr) == hipSuccess && dst == src && to_pinned == 1 ? 0 : 1;
}

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  if (!strcmp(what, "values")) return values();
  if (!strcmp(what, "idle")) return idle();
  if (!strcmp(what, "devices")) return devices();
  if (!strcmp(what, "direct")) return direct();
  return 2;
}
