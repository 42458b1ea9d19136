// A stand-in for the HIP runtime and the kernel launches, for tests of the C
// ABI's host code on the CPU: linked with mps_abi.cpp alone
// (test_host_plan.py).  "Device" memory is zeroed host memory under a settable
// limit, a launch appends a line to a log, and a grid that HIP would refuse
// (2^32 threads or more in a dimension) is refused here too.
#include "../paper_2512_20064_amd/csrc/sweep.h"

#include <sys/mman.h>

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>

namespace {

std::map<char*, size_t> g_live;  // allocation -> bytes
size_t g_limit = size_t(1) << 40, g_now = 0, g_peak = 0;
std::string g_log;
int g_flagged = 0;         // what the flag counter reads after a call
const char* g_host_lo = nullptr;  // site pointers in [lo, hi) are pinned host memory
const char* g_host_hi = nullptr;
hipError_t g_err = hipSuccess;
int g_mallocs = 0;
int g_obj;  // address of every stream, event and graph

hipError_t set(hipError_t e) { return g_err = e; }

void line(const char* fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_log += buf;
  g_log += '\n';
}

hipError_t grid(unsigned long long blocks, unsigned threads) {
  return set(blocks * threads > 0xFFFFFFFFull ? hipErrorInvalidConfiguration : hipSuccess);
}

}  // namespace

extern "C" {

// ---- control of the stand-in ----
void host_reset(size_t limit) {
  g_limit = limit;
  g_peak = g_now;
  g_log.clear();
  g_flagged = 0;
  g_host_lo = g_host_hi = nullptr;
}
void host_clear_log() { g_log.clear(); }
void host_set_flagged(int n) { g_flagged = n; }
void host_set_pinned(const char* lo, const char* hi) {
  g_host_lo = lo;
  g_host_hi = hi;
}
const char* host_log() { return g_log.c_str(); }
size_t host_peak() { return g_peak; }
int host_mallocs() { return g_mallocs; }

// ---- memory ----
hipError_t hipMalloc(void** p, size_t n) {
  if (g_now + n > g_limit) return set(hipErrorOutOfMemory);
  ++g_mallocs;
  void* q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return set(hipErrorOutOfMemory);
  g_live[(char*)q] = n;
  g_now += n;
  g_peak = g_now > g_peak ? g_now : g_peak;
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_live.find((char*)p);
  if (it == g_live.end()) return p ? set(hipErrorInvalidValue) : hipSuccess;
  munmap(p, it->second);
  g_now -= it->second;
  g_live.erase(it);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* room, size_t* all) { return *all = g_limit, *room = g_limit - g_now, hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k == hipMemcpyDeviceToHost && n == sizeof(int)) std::memcpy(dst, &g_flagged, n);  // the flag counter
  else std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  std::memset(a, 0, sizeof *a);
  a->type = (const char*)p >= g_host_lo && (const char*)p < g_host_hi ? hipMemoryTypeHost : hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t*, size_t*, hipDeviceptr_t) { return hipErrorInvalidValue; }
hipError_t hipGetSymbolAddress(void** p, const void* sym) {
  *p = const_cast<void*>(sym);  // the host-side stand-in of the device array
  return hipSuccess;
}

// ---- device, streams, events, graphs ----
hipError_t hipGetDeviceCount(int* n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = g_err;
  g_err = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "stand-in error"; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)&g_obj, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)&g_obj, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)&g_obj, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { return *g = (hipGraph_t)&g_obj, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  return *x = (hipGraphExec_t)&g_obj, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return (void**)&g_obj; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}

}  // extern "C"

// ---- launches ----
namespace mps {

size_t stored_bytes(int kind, int chi_l, int d, int chi_r) {
  const size_t n = (size_t)chi_l * d * chi_r;
  if (kind == 0) return 8 * n;
  if (kind == 1) return 4 * n;
  return (2 * n + 255) / 256 * 256 +
         4 * (size_t)((chi_l + 127) / 128) * (((size_t)d * chi_r + 127) / 128);
}
hipError_t launch_decompress(const DecompressProb&, hipStream_t) { return hipSuccess; }
hipError_t launch_fill_noise(void*, size_t, int, unsigned, hipStream_t) { return hipSuccess; }
hipError_t launch_init(int, const InitProb*, int, const ChunkArgs*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_lp(int, const PackProb*, const int*, int nprob, int blk, hipStream_t) {
  line("pack nprob=%d", nprob);
  return grid(blk, 256);
}
hipError_t launch_colscale(const PackProb*, const int*, int, int cm, hipStream_t) { return grid(cm, 256); }
hipError_t launch_contract_f32(int tile, bool, const ContractProb*, const int*, int nprob, int, const ChunkArgs*,
                               int rows, int group, hipStream_t) {
  line("contract tile=%d nprob=%d rows=%d group=%d", tile, nprob, rows, group);
  return hipSuccess;
}
hipError_t launch_contract_lp(int, int tile, const ContractLpProb*, const int*, int nprob, int, const ChunkArgs*,
                              int rows, int group, hipStream_t) {
  line("contract tile=%d nprob=%d rows=%d group=%d", tile, nprob, rows, group);
  return hipSuccess;
}
hipError_t launch_measure(int, const MeasureProb*, int nprob, const ChunkArgs*, int rows, uint64_t, int*, bool, int, int,
                          hipStream_t) {
  line("measure nprob=%d rows=%d", nprob, rows);
  return hipSuccess;
}
hipError_t launch_sweep_small(const SmallChain*, const int*, int nchain, int items, const ChunkArgs* ch, uint64_t, int*,
                              hipStream_t) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  line("small nchain=%d items=%d rows=%d", nchain, items, ch->rows);
  return grid((unsigned)items, 256);
}
hipError_t launch_sweep_mid(int, int groups, const MidChain*, const int*, int nchain, int items, int, const ChunkArgs* ch,
                            uint64_t, int*, hipStream_t) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  line("mid nchain=%d items=%d rows=%d", nchain, items, ch->rows);
  return grid((unsigned)items, groups <= 4 ? 256 : 512);
}
hipError_t launch_sweep_mid_f32(const MidChain*, const int*, int nchain, int items, int, const ChunkArgs* ch, uint64_t,
                                int*, hipStream_t) {
  if (nchain <= 0 || items <= 0) return hipSuccess;
  line("mid nchain=%d items=%d rows=%d", nchain, items, ch->rows);
  return grid((unsigned)items, 512);
}

}  // namespace mps
