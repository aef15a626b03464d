// A model of the HIP runtime and of the kernel launchers for CPU tests of the
// library's host side (api.cpp): device memory is host memory with a limit,
// streams run their work at once, a captured stream records it, and the
// correlation launches are written to a log instead of running kernels.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "../paper_2310_08770_amd/csrc/common.h"

namespace {

struct Record {
  int ny, nx, count, fused_min, pairs_ok;
};

size_t g_limit = ~(size_t)0, g_live = 0;
int g_asked = 0;           // device allocations asked for
int g_refuse = 0;          // > 0: the allocation that many from now is refused
std::map<void*, size_t> g_size;
hipError_t g_last = hipSuccess;  // kept until it is read, as the runtime does
std::vector<Record> g_log;
std::vector<Record>* g_capture = nullptr;
double g_ms_launch = 1.0, g_ms = 0.0;  // simulated time of a correlation launch, and now
bool g_no_tables = false;  // a window launch without its grid table

hipError_t err(hipError_t e) {
  if (e != hipSuccess) g_last = e;
  return e;
}

void launched(const Record& r) {
  if (g_capture) {
    g_capture->push_back(r);
    return;
  }
  g_log.push_back(r);
  g_ms += g_ms_launch;
}

// What the launchers return: the last error of any call on this thread.
int status() { return hipGetLastError() == hipSuccess ? 0 : -1; }

}  // namespace

extern "C" {

// ---- controls of the tests
void host_limit(size_t bytes) { g_limit = bytes; }
size_t host_live() { return g_live; }
int host_asked() { return g_asked; }
void host_refuse(int k) { g_refuse = k; }
void host_last_error_clear() { g_last = hipSuccess; }
int host_no_tables() { return g_no_tables; }
int host_log(int* out, int cap) {  // (ny, nx, count, fused_min, pairs_ok) each; empties the log
  int n = 0;
  for (const Record& r : g_log)
    if (n < cap) memcpy(out + 5 * n++, &r, sizeof r);
  g_log.clear();
  return n;
}

// ---- runtime
hipError_t hipMalloc(void** p, size_t bytes) {
  ++g_asked;
  if ((g_refuse > 0 && --g_refuse == 0) || bytes > g_limit || g_live > g_limit - bytes) return err(hipErrorOutOfMemory);
  *p = malloc(bytes ? bytes : 1);
  g_size[*p] = bytes;
  g_live += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = g_size.find(p);
  if (it == g_size.end()) return p ? err(hipErrorInvalidValue) : hipSuccess;
  g_live -= it->second;
  g_size.erase(it);
  free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* total) {
  *total = g_limit;
  *f = g_limit > g_live ? g_limit - g_live : 0;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { return (*p = malloc(bytes)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "error"; }

hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t) new double(0.0);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete (double*)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  *(double*)e = g_ms;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(*(double*)b - *(double*)a);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = (hipStream_t) new char;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  delete (char*)s;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_capture = new std::vector<Record>;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t)g_capture;
  g_capture = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *x = (hipGraphExec_t) new std::vector<Record>(*(std::vector<Record>*)g);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete (std::vector<Record>*)g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete (std::vector<Record>*)x;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
  for (const Record& r : *(std::vector<Record>*)x) launched(r);
  return hipSuccess;
}

}  // extern "C"

// ---- launchers
namespace ccpt {

static void* g_scratch = nullptr;
int scratch_setup(int) {
  if (!g_scratch) g_scratch = malloc(kScratchBytes);
  return 0;
}
void* scratch_ptr(int) { return g_scratch; }

int launch_xcorr(int ny, int nx, const GroupParams& g, hipStream_t, const Marker&) {
  launched(Record{ny, nx, g.count, g.fused_min, g.pairs_ok});
  return status();
}
int launch_xcorr64(int n, const GroupParams& g, hipStream_t, const Marker&) {
  launched(Record{n, n, g.count, g.fused_min, g.pairs_ok});
  return status();
}
int launch_window_coef(int, int, const GroupParams&, const WindowTables&, int, hipStream_t) { return status(); }
int launch_window_max(int, int, const GroupParams& g, const WindowTables& t, int, double, hipStream_t) {
  if (!(g.X64 ? (const void*)t.td : (const void*)t.tf)) g_no_tables = true;
  return status();
}
int launch_init_state(FrameState*, int, hipStream_t) { return status(); }
int launch_zero(void* p, size_t bytes, hipStream_t) {
  memset(p, 0, bytes);
  return status();
}
int launch_spectrum(int, int, const void*, int, int, long, int, int, int, float, int, float2*, float2*, const float2*,
                    hipStream_t) { return status(); }
int launch_spectrum64(int, const void*, int, int, long, int, int, double, int, double2*, double2*, const double2*,
                      hipStream_t) { return status(); }
int launch_frame_spectra(int, const FrameDesc*, int, int, int, float, float2*, float2*, const float2*, hipStream_t) {
  return status();
}
int launch_inverse(int, const float2*, int, float, float2*, float*, const float2*, hipStream_t) { return status(); }
int lds_frames(int, int, int, int) { return 0; }
int launch_grad_lds(int, const GradParams&, hipStream_t) { return status(); }
int launch_grad_psi(int, const GradParams&, const float2*, float2*, hipStream_t) { return status(); }
int launch_grad_frames(int, const FrameDesc*, int, int, const float*, const long*, float*, int, float, hipStream_t) {
  return status();
}
int launch_ref_accum(int, float2*, const RefSums&, float2* const*, hipStream_t) { return status(); }
int launch_grad_ref_chain(const float*, const float*, int, int, float, float*, hipStream_t) { return status(); }
int launch_fisher_deriv(int, const float2*, float2*, float2*, hipStream_t) { return status(); }
int launch_fisher_reduce(const float*, const float*, const void*, int, int, int, double*, int, double*, hipStream_t) {
  return status();
}
int launch_align(int, const FrameDesc*, int, int, const ccpt_result*, float2*, unsigned*, hipStream_t) {
  return status();
}
int launch_align_lds(int, const FrameDesc*, int, int, const ccpt_result*, const float2*, float2*, unsigned*,
                     hipStream_t) { return status(); }
int launch_sum_spectra(int, int, const float2*, float2*, hipStream_t) { return status(); }
int launch_scale_by_count(float*, int, float, const unsigned*, hipStream_t) { return status(); }
int launch_rt_update(int, int, int, const RtUpdate&, hipStream_t) { return status(); }
int launch_ref_check(const void*, int, int, int, int, int, double, unsigned*, hipStream_t) { return status(); }
int launch_ref_copy(const void*, int, int, int, int, float*, hipStream_t) { return status(); }

}  // namespace ccpt
