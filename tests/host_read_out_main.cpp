// Read-outs against a HIP runtime that this file stands in for: two devices whose memory is the
// host's, streams that know their device, and kernels that do not run except for the packing of
// particles and records, of which the first reports a live count.  Prints "bad 0" if every check held.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "../include/lcmd.h"
#include "../paper_1307_3711_amd/csrc/lc_internal.h"

namespace {

struct Stream { int device; bool capturing; };
struct Event { int device; };

int g_current = 0;      // current device
int g_state_device = 1; // device of every address asked for
int64_t g_live = 0;     // what the packing kernel reports
int g_packs = 0, g_packs_elsewhere = 0, g_host_mallocs = 0, g_host_frees = 0, g_bad_records = 0;
bool g_global_capture = false;  // the thread captures some other stream, in the strictest mode
hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
std::map<const void*, std::string> g_kernels;
dim3 g_grid, g_block;
size_t g_lds;
hipStream_t g_stream;

int device_of(hipStream_t s) { return s ? ((Stream*)s)->device : g_current; }
bool capturing(hipStream_t s) { return s && ((Stream*)s)->capturing; }

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* d) { *d = g_current; return hipSuccess; }
hipError_t hipSetDevice(int d) { g_current = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  std::memset(a, 0, sizeof *a);
  a->device = g_state_device;
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++g_host_mallocs;
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
  if (g_global_capture && g_mode != hipStreamCaptureModeRelaxed) return hipErrorStreamCaptureUnsupported;
  ++g_host_frees;
  std::free(p);
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* mode) { std::swap(*mode, g_mode); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return capturing(s) ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = capturing(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new Event{g_current}; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (((Event*)e)->device == device_of(s)) return hipSuccess;
  ++g_bad_records;
  return hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotSupported; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return hipSuccess; }
hipError_t hipExtLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) {
  return hipErrorNotSupported;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s) {
  const std::string& name = g_kernels[f];
  if (name.find("k_pack_") == std::string::npos) return hipSuccess;
  ++g_packs;
  if (name.find("k_pack_particles") == std::string::npos) return hipSuccess;
  if (device_of(s) != g_state_device) ++g_packs_elsewhere;
  lc::ClusterDyn* head = *(lc::ClusterDyn**)args[4];  // the read-out's head starts with the cluster's counts
  std::memset(head, 0, sizeof *head + sizeof(int32_t));
  head->n_cur = g_live;
  return hipSuccess;
}

// What hipcc's launch and registration stubs call.
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  g_grid = g; g_block = b; g_lds = lds; g_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_grid; *b = g_block; *lds = g_lds; *s = g_stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { static void* p = nullptr; return &p; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}

}  // extern "C"

namespace {

lc_sim* handle(int64_t capacity, hipStream_t stream, std::vector<char>& mem) {
  lc_config c;
  std::memset(&c, 0, sizeof c);
  c.struct_size = sizeof c;
  c.precision = LC_FP64;
  c.lambda_um = 0.8;
  c.dt = 0.05;
  c.softening_nm = 0.1;
  c.max_splits = 1;
  c.detector_half_angle_deg = 30.0;
  c.box_r0 = 20.0;
  c.t_switch = INFINITY;
  lc_cluster k;
  std::memset(&k, 0, sizeof k);
  k.r0_nm = 2.5;
  k.rw_angstrom = 2.4;
  k.mass_u = 39.948;
  k.ip_ev[0] = 15.76;
  k.intensity_wcm2 = 1e16;
  k.envelope = LC_SIN2;
  k.n_cycles = 10.0;
  k.n_ion = 100;
  k.capacity = capacity;
  k.z_max = 1;
  k.electron_offset_nm = 0.01;
  const size_t bytes = lc_state_bytes(&c, &k, 1);
  mem.assign(bytes + 256, 0);
  void* state = (void*)(((uintptr_t)mem.data() + 255) & ~(uintptr_t)255);
  lc_sim* sim = nullptr;
  return lc_create(&sim, &c, &k, 1, state, bytes, stream) == LC_OK ? sim : nullptr;
}

}  // namespace

int main() {
  int bad = 0;
  auto check = [&](bool ok, const char* what) {
    if (!ok) { ++bad; std::printf("failed: %s\n", what); }
  };
  const int64_t n = 3 * 4096 + 5;  // four packings
  std::vector<double> x(3 * n);
  std::vector<char> mem;
  Stream dev1{1, false};
  for (hipStream_t st : {(hipStream_t)&dev1, (hipStream_t) nullptr}) {
    g_current = 1;
    lc_sim* sim = handle(n, st, mem);
    check(sim != nullptr, "create");
    if (!sim) return 1;
    g_live = n;
    for (int current : {0, 1}) {
      g_current = current;
      g_packs = g_packs_elsewhere = g_bad_records = 0;
      int64_t got = 0;
      check(lc_read_particles(sim, 0, x.data(), nullptr, nullptr, nullptr, nullptr, n, &got) == LC_OK && got == n,
            "particles read with another device current");
      check(g_packs == 4 && g_packs_elsewhere == 0, "every packing runs on the handle's device");
      check(g_bad_records == 0, "the read-out's events are the handle's device's");
      check(g_current == current, "the caller's device stays current");
    }
    g_current = 0;
    lc_destroy(sim);
  }
  // under capture a read-out is refused: nothing recorded into the graph, nothing allocated
  g_current = 1;
  lc_sim* sim = handle(n, (hipStream_t)&dev1, mem);
  if (!sim) return 1;
  g_packs = g_host_mallocs = 0;
  dev1.capturing = true;
  int64_t got = -1;
  int32_t records = -1;
  check(lc_read_particles(sim, 0, x.data(), nullptr, nullptr, nullptr, nullptr, n, &got) == LC_E_HIP && got == -1,
        "particles refused under capture");
  check(lc_read_diagnostics(sim, 0, x.data(), 1, &records) == LC_E_HIP && records == -1, "records refused under capture");
  check(g_packs == 0 && g_host_mallocs == 0, "nothing recorded or allocated under capture");
  dev1.capturing = false;
  check(lc_read_particles(sim, 0, x.data(), nullptr, nullptr, nullptr, nullptr, n, &got) == LC_OK && got == n,
        "particles read after the capture");
  // destroyed while another stream is captured: the pinned buffer is given back all the same
  g_global_capture = true;
  const int frees = g_host_frees;
  lc_destroy(sim);
  check(g_host_frees == frees + 1, "the pinned buffer freed during another stream's capture");
  check(g_mode == hipStreamCaptureModeGlobal, "the thread's capture mode as before");
  std::printf("bad %d\n", bad);
  return bad;
}
