// A stand-in for the HIP runtime, for tests of the library's host code without a GPU:
// loaded before libspkadd.so, its definitions take the runtime's place.  Device memory is
// host memory up to a limit, kernels do not run (the few whose results the host waits
// for write what the test has set), streams run at once, and every event belongs to the
// device that was current when it was made, as the runtime has it.
//
// A stream handle is 0x1000 * (device + 1) + number; the null stream is the current
// device's.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "internal.h"

namespace {

struct Event {
  int dev;
  hipStream_t stream = nullptr;  // of the last record
  long at = 0;                   // number of the last record in the log
};

int g_dev = 0;
hipError_t g_last = hipSuccess;
size_t g_limit = (size_t)64 << 30, g_used = 0, g_peak = 0;
std::map<void*, size_t> g_mem;
std::map<const void*, std::string> g_kernels;
std::map<const void*, size_t> g_vars;
std::map<const void*, void*> g_var_mem;
std::vector<std::string> g_log;
int g_fail_records = 0;
long g_events = 0, g_events_made = 0, g_foreign_records = 0;
int g_tables = 0, g_stale_tables = 0;  // launches with a copy of the column pointers; with a freed one
std::map<std::string, size_t> g_units;  // blocks launched of each kernel
struct { dim3 g, b; size_t lds; hipStream_t s; } g_call;

hipError_t ret(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}
int dev_of(hipStream_t s) { return s ? (int)((size_t)s / 0x1000) - 1 : g_dev; }
void note(const char* what, hipStream_t s, const void* x = nullptr) {
  char buf[256];
  snprintf(buf, sizeof(buf), "%s %zx %zx", what, (size_t)s, (size_t)x);
  g_log.push_back(buf);
}

}  // namespace

extern "C" {

// ---- what the tests set and read ----
int fake_bins[spk::NBINS];  // bin counts that the binning kernels leave
int fake_windows = 0;       // row windows
long long fake_total = 0;   // result of every scan
void fake_limit(size_t bytes) { g_limit = bytes; }
size_t fake_used() { return g_used; }
size_t fake_peak() { return g_peak; }
void fake_peak_reset() { g_peak = g_used; }
void fake_fail_records(int n) { g_fail_records = n; }
long fake_events() { return g_events; }
long fake_events_made() { return g_events_made; }
long fake_foreign_records() { return g_foreign_records; }
int fake_tables() { return g_tables; }
int fake_stale_tables() { return g_stale_tables; }
int fake_last_error() { return (int)g_last; }
int fake_log_size() { return (int)g_log.size(); }
const char* fake_log(int i) { return g_log[(size_t)i].c_str(); }
void fake_log_clear() { g_log.clear(); }
// blocks launched of the kernels whose names hold `part`
size_t fake_blocks(const char* part) {
  size_t n = 0;
  for (auto& x : g_units) n += x.first.find(part) != std::string::npos ? x.second : 0;
  return n;
}
int fake_bin_g1() { return spk::BIN_G1; }
int fake_bin_g3() { return spk::BIN_G3; }
int fake_bin_win() { return spk::BIN_WIN; }

// ---- the runtime ----
void** __hipRegisterFatBinary(const void*) { return (void**)calloc(1, sizeof(void*)); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_kernels[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { g_vars[var] = size; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_call = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_call.g;
  *b = g_call.b;
  *lds = g_call.lds;
  *s = g_call.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  using spk::PlanSummary;
  const std::string& name = g_kernels[f];
  // fewer than 2^32 work-items along each dimension of a grid
  if (((size_t)g.x * b.x) >> 32 || ((size_t)g.y * b.y) >> 32) {
    note("refused", s, f);
    g_log.push_back(name);
    return ret(hipErrorInvalidConfiguration);
  }
  g_units[name] += (size_t)g.x * g.y;
  auto is = [&](const char* k) { return name.find(k) != std::string::npos; };
  size_t fixed = 0;  // the kernel's own LDS arrays
  for (const char* k : {"k_bitmap_wgILi", "k_hash_wgILi"})
    if (is(k)) {
      const size_t waves = (size_t)atoi(name.c_str() + name.find(k) + strlen(k)) / 64;
      fixed = k[2] == 'b' ? 4 * (2 * waves + 1) : 8 * (waves + 1) + 4;
    }
  if (lds + (fixed + 15) / 16 * 16 > 160 * 1024) return ret(hipErrorInvalidValue);
  if (is("k_bounds") && !is("batch")) (*(PlanSummary**)args[8])->nnz_in = 1;
  if (is("k_bin_scan")) {
    PlanSummary* sum = *(PlanSummary**)args[4];
    for (int b = 0; b < spk::NBINS; ++b) sum->bin_count[b] = fake_bins[b];
  }
  if (is("k_win_scan")) (*(PlanSummary**)args[5])->n_windows = fake_windows;
  if (is("k_scan_small")) **(long long**)args[2] = fake_total;
  if (is("k_scan_apply")) **(long long**)args[5] = fake_total;
  if (is("KArgs") && !is("batch")) {
    const char* t = (const char*)((const spk::KArgs*)args[0])->cpt;
    bool live = false;
    for (auto& x : g_mem) live |= t >= (const char*)x.first && t < (const char*)x.first + x.second;
    if (t) ++g_tables;
    if (t && !live) ++g_stale_tables;
  }
  note(name.c_str(), s);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
  *p = nullptr;
  if (g_used + bytes > g_limit) return ret(hipErrorOutOfMemory);
  *p = calloc(1, bytes ? bytes : 1);
  g_mem[*p] = bytes;
  g_used += bytes;
  if (g_used > g_peak) g_peak = g_used;
  note("malloc", nullptr, (void*)bytes);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  g_used -= g_mem.at(p);
  note("free", nullptr, (void*)g_mem.at(p));
  g_mem.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) { return hipMalloc(p, bytes); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) {
  *p = calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* var) {
  if (!g_var_mem[var]) g_var_mem[var] = calloc(1, g_vars.at(var));
  *p = g_var_mem[var];
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  memcpy(d, s, n);
  note("copy", st);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new Event{g_dev};
  ++g_events;
  ++g_events_made;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (Event*)e;
  --g_events;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (g_fail_records > 0) {
    --g_fail_records;
    return ret(hipErrorInvalidHandle);
  }
  Event* ev = (Event*)e;
  if (ev->dev != dev_of(s)) {
    ++g_foreign_records;
    return ret(hipErrorInvalidHandle);
  }
  ev->stream = s;
  ev->at = (long)g_log.size();
  note("record", s, e);
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  note("wait", s, e);
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  note("sync", s);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  static size_t next = 1;
  *s = (hipStream_t)(0x1000 * (size_t)(g_dev + 1) + ++next);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = g_dev;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  g_dev = d;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof(*p));
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  memset(a, 0, sizeof(*a));
  a->numRegs = 64;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 4;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error of the stand-in runtime"; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *x = nullptr;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

}  // extern "C"
