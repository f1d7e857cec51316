// A stand-in for the HIP runtime that runs no kernel: the library's host code on a machine without
// a GPU.  "Device" memory is host memory, launches are checked against the runtime's limits and
// logged, allocations and launches can be made to fail, and the few words the host reads back are
// written as the kernels would (the exact scan's total, the head of a localize step).  A stream is
// busy from a launch, copy or fill until it is waited for; work on another stream that depends on
// a fill of the null stream (which a non-blocking stream does not wait for) is reported.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <string>

#include "fpsk_internal.h"

namespace {

std::map<const void*, std::string> g_names;      // host stub of a kernel -> its name
std::map<void*, size_t> g_blocks;
std::set<const void*> g_lists;                   // row lists that tables_kernel has written
std::set<void*> g_busy;                          // streams with unfinished work
std::string g_log, g_faults, g_unordered, g_fail_kernel;
int g_fail_alloc = 0, g_scan_total = 0, g_candidates = 0;
double g_rms = 1.0, g_sigma = 0.0;
hipError_t g_error = hipSuccess;
struct Config {
  dim3 grid, block;
  size_t shmem;
  hipStream_t st;
} g_config;

void* take(size_t n) {
  void* p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (p == MAP_FAILED) return nullptr;
  g_blocks[p] = n;
  return p;
}

hipError_t alloc(void** p, size_t n) {
  if (g_fail_alloc > 0 && --g_fail_alloc == 0) return hipErrorOutOfMemory;
  *p = take(n);
  return *p != nullptr ? hipSuccess : hipErrorOutOfMemory;
}

hipError_t release(void* p) {
  g_busy.clear();                                // frees wait for the device
  auto it = g_blocks.find(p);
  if (it == g_blocks.end()) {
    g_faults += "free of memory that is not allocated; ";
    return hipErrorInvalidValue;
  }
  munmap(p, it->second);
  g_lists.erase(p);
  g_blocks.erase(it);
  return hipSuccess;
}

template <typename T>
const T& arg(void** args, int i) {
  return *static_cast<const T*>(args[i]);
}

// Pointers into allocations that exist (a probe's stream pass: lists, tables, factors).
void check_pointers(const std::string& k, void** args) {
  if (k.find("stream_kernel") == std::string::npos) return;
  const auto& s = arg<fpsk::StreamArgs>(args, 0);
  for (const void* p : {static_cast<const void*>(s.perm), static_cast<const void*>(s.ctab),
                        static_cast<const void*>(s.coff), static_cast<const void*>(s.P),
                        static_cast<const void*>(s.Q), static_cast<const void*>(s.partS),
                        static_cast<const void*>(s.maxpart)}) {
    if (g_blocks.find(const_cast<void*>(p)) == g_blocks.end()) {
      g_faults += k + " got memory that is not allocated; ";
    }
  }
  if (g_lists.count(s.perm) == 0) g_faults += k + " got row lists that no kernel has written; ";
}

// What a kernel would leave for the host or for the kernels after it.
void emulate(const std::string& k, void** args) {
  auto selection = [&](const fpsk::SelArgs& a, bool first) {
    if (first && a.hist[0] != 0) g_faults += k + " found counts of another selection; ";
    a.hist[0] = first ? 1 : 0;
  };
  if (k.find("scan_count_kernel") != std::string::npos) {
    *arg<unsigned long long*>(args, 3) += g_scan_total;
  } else if (k.find("sel_hist1_kernel") != std::string::npos) {
    const auto& a = arg<fpsk::SelArgs>(args, 0);
    selection(a, true);
    if (a.clear != nullptr) *a.clear = 0;
  } else if (k.find("sel_median_kernel") != std::string::npos) {
    selection(arg<fpsk::SelArgs>(args, 0), false);
  } else if (k.find("rms_kernel") != std::string::npos) {
    selection(arg<fpsk::SelArgs>(args, 0), false);
    const auto& u = arg<fpsk::SetupArgs>(args, 1);
    *u.head = fpsk::HostHead{};
    u.head->rms = g_rms;
    u.head->sigma = g_sigma;
    u.head->extra = 1.0;
    u.head->found = u.found != nullptr ? static_cast<uint32_t>(*u.found) : 0;
  } else if (k.find("sel_mad_kernel") != std::string::npos || k.find("sel_small_kernel") != std::string::npos) {
    if (k.find("sel_mad_kernel") != std::string::npos) selection(arg<fpsk::SelArgs>(args, 0), false);
    const auto& r = arg<fpsk::RoundArgs>(args, 1);
    *r.count = g_candidates;
    r.head->sigma = g_sigma;
  } else if (k.find("moments_at_kernel") != std::string::npos) {
    const auto& m = arg<fpsk::MomentsAtArgs>(args, 0);
    if (m.cands != nullptr) m.head->found = g_candidates;
  }
}

hipError_t launch(const void* f, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t st) {
  auto it = g_names.find(f);
  const std::string k = it != g_names.end() ? it->second : "?";
  char line[256];
  std::snprintf(line, sizeof(line), "%s %u %u %u\n", k.c_str(), grid.x, grid.y, grid.z);
  g_log += line;
  const bool fits = grid.x > 0 && grid.y > 0 && grid.z > 0 &&
                    static_cast<uint64_t>(grid.x) * block.x < (uint64_t{1} << 32) &&
                    grid.y < 65536 && grid.z < 65536 && block.x * block.y * block.z <= 1024 &&
                    shmem <= 160 * 1024;
  if (!fits) return g_error = hipErrorInvalidConfiguration;
  if (!g_fail_kernel.empty() && k.find(g_fail_kernel) != std::string::npos) {
    g_fail_kernel.clear();
    return g_error = hipErrorOutOfMemory;
  }
  if (st != nullptr && g_busy.count(nullptr) != 0) {
    g_unordered += k + " does not wait for the null stream's fill; ";
  }
  g_busy.insert(st);
  check_pointers(k, args);
  if (k.find("tables_kernel") != std::string::npos) g_lists.insert(arg<fpsk::TableArgs>(args, 0).perm);
  emulate(k, args);
  return hipSuccess;
}

}  // namespace

extern "C" {

// Controls.
void rt_reset() {
  g_log.clear();
  g_faults.clear();
  g_unordered.clear();
  g_fail_kernel.clear();
  g_fail_alloc = 0;
  g_error = hipSuccess;
}
void rt_fail_alloc(int nth) { g_fail_alloc = nth; }       // the nth allocation from now fails
void rt_fail_kernel(const char* name) { g_fail_kernel = name; }   // its next launch fails
void rt_scan_total(int n) { g_scan_total = n; }
void rt_candidates(int n) { g_candidates = n; }
void rt_noise(double rms, double sigma) { g_rms = rms, g_sigma = sigma; }
int rt_alloc_pending() { return g_fail_alloc; }
int rt_busy() { return static_cast<int>(g_busy.size()); }
int64_t rt_blocks() { return static_cast<int64_t>(g_blocks.size()); }
const char* rt_log() { return g_log.c_str(); }
const char* rt_faults() { return g_faults.c_str(); }
const char* rt_unordered() { return g_unordered.c_str(); }

// The runtime's entry points that the library uses.
void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, uint3*, uint3*, dim3*,
                           dim3*, int*) {
  g_names[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t st) {
  g_config = {grid, block, shmem, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* st) {
  *grid = g_config.grid;
  *block = g_config.block;
  *shmem = g_config.shmem;
  *st = g_config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t st) {
  return launch(f, grid, block, args, shmem, st);
}
hipError_t hipExtLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t shmem, hipStream_t st,
                              hipEvent_t, hipEvent_t, int) {
  return launch(f, grid, block, args, shmem, st);
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return alloc(p, n); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return alloc(p, n); }
hipError_t hipFree(void* p) { return release(p); }
hipError_t hipHostFree(void* p) { return release(p); }
hipError_t hipMemset(void* p, int v, size_t n) {
  if (n <= (size_t{1} << 24)) std::memset(p, v, n);       // (new memory is zero already)
  g_busy.insert(nullptr);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  std::memcpy(d, s, n);
  g_busy.insert(st);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t st) {
  g_busy.erase(st);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  g_busy.clear();
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* s = take(size_t{16} << 20);
  *p = s;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_error;
  g_error = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipEventCreate(hipEvent_t* e) {
  static int made = 0;
  *e = reinterpret_cast<hipEvent_t>(static_cast<intptr_t>(++made));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}
}
