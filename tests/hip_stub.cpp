// A stand-in for the HIP runtime on the CPU: device memory is zeroed host memory,
// copies are memcpy, launches run nothing and are logged by their kernel's name.
// Time is what the launches are set to cost: an event holds the clock as it stood.
#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace {
struct Dim3 {
  unsigned x, y, z;
};
std::map<const void*, std::string> kernels;
std::map<void*, size_t> blocks;
size_t live = 0, limit = ~size_t(0);
int last_error = 0, failures = 0, waits = 0, allocations = 0;
std::string log_text;
std::vector<std::pair<std::string, double>> costs;
double clock_us = 0.0;
struct Watch {
  std::string name;
  int arg;
  uintptr_t bits;
};
std::vector<Watch> watches;
struct Fill {
  std::string name;
  int arg, value, count;
};
std::vector<Fill> fills;
struct Call {
  Dim3 grid, block;
  size_t lds;
  void* stream;
};
std::vector<Call> calls;
std::map<std::string, unsigned> grids;
}  // namespace

extern "C" {
// ---- control ----
size_t stub_live() { return live; }
int stub_failures() { return failures; }
int stub_allocations() { return allocations; }
int stub_waits() { return waits; }  // waits of the host for the device
unsigned stub_grid(const char* what) {  // workgroups of the last launch of the first kernel so named
  for (const auto& g : grids)
    if (g.first.find(what) != std::string::npos) return g.second;
  return 0;
}
void stub_limit(size_t bytes) { limit = bytes; }
const char* stub_log() { return log_text.c_str(); }
void stub_clear() { log_text.clear(); }
void stub_cost(const char* name, double us) { costs.insert(costs.begin(), {name, us}); }
// The low four bits that pointer argument `arg` of kernels with this name has had set.
void stub_watch(const char* name, int arg) { watches.push_back({name, arg, 0}); }
unsigned stub_watched(int k) { return (unsigned)watches[k].bits; }

// Kernels with this name leave `count` ints of `value` at their pointer argument `arg`.
void stub_fill(const char* name, int arg, int value, int count) { fills.push_back({name, arg, value, count}); }

// ---- the runtime ----
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
  calls.push_back({grid, block, lds, stream});
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
  const Call c = calls.back();
  calls.pop_back();
  *grid = c.grid;
  *block = c.block;
  *lds = c.lds;
  *stream = c.stream;
  return 0;
}
int hipLaunchKernel(const void* host, Dim3 grid, Dim3, void** args, size_t, void*) {
  const std::string& name = kernels[host];
  grids[name] = grid.x;
  log_text += name + "\n";
  double us = 1.0;
  for (const auto& c : costs)
    if (name.find(c.first) != std::string::npos) {
      us = c.second;
      break;
    }
  clock_us += us;
  for (Watch& w : watches)
    if (name.find(w.name) != std::string::npos) w.bits |= *static_cast<uintptr_t*>(args[w.arg]) & 15u;
  for (const Fill& f : fills)
    if (name.find(f.name) != std::string::npos)
      std::fill_n(*static_cast<int**>(args[f.arg]), f.count, f.value);
  return 0;
}
int hipMalloc(void** p, size_t n) {
  ++allocations;
  *p = nullptr;
  if (live + n > limit) {
    ++failures;
    return last_error = 2;  // out of memory
  }
  const size_t room = (n + 511) / 256 * 256;
  *p = aligned_alloc(256, room);
  if (!*p) return last_error = 2;
  if (n < (size_t(64) << 20)) memset(*p, 0, room);
  blocks[*p] = n;
  live += n;
  return 0;
}
int hipFree(void* p) {
  if (!p) return 0;
  auto it = blocks.find(p);
  if (it == blocks.end()) return last_error = 1;
  live -= it->second;
  blocks.erase(it);
  free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  if (live + n > limit) return last_error = 2;
  *p = calloc(n, 1);
  return 0;
}
int hipHostFree(void* p) {
  free(p);
  return 0;
}
int hipMemcpyAsync(void* dst, const void* src, size_t n, int, void*) {
  memmove(dst, src, n);
  return 0;
}
int hipMemset(void* p, int v, size_t n) {
  memset(p, v, n);
  return 0;
}
int hipMemsetAsync(void* p, int v, size_t n, void*) { return hipMemset(p, v, n); }
int hipGetLastError() { return std::exchange(last_error, 0); }
const char* hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipGetDevice(int* d) { return *d = 0; }
int hipGetDeviceCount(int* n) {
  *n = 1;
  return 0;
}
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return ++waits, 0; }
int hipStreamSynchronize(void*) { return ++waits, 0; }
int hipEventCreate(void** e) {
  *e = new double(0.0);
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) {
  delete static_cast<double*>(e);
  return 0;
}
int hipEventRecord(void* e, void*) {
  *static_cast<double*>(e) = clock_us;
  return 0;
}
int hipEventSynchronize(void*) {
  log_text += "event_wait\n";
  return 0;
}
int hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = (float)(1e-3 * (*static_cast<double*>(b) - *static_cast<double*>(a)));
  return 0;
}
}
