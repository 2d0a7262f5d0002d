// The serving loop's host code (serve.cpp) over a stand-in for the HIP runtime
// and for the plans, for what it does when a step of a request fails or the
// memory is short.  No GPU code runs.  argv[1] names the scenario; prints
// "ok" when every request ended as it has to.
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <atomic>
#include <string>
#include <thread>

#include "fmm_internal.h"

namespace {
std::atomic<bool> hold{false};          // batches stay in flight
std::atomic<int> fail_upload{0};        // upload_job throws so many times
std::atomic<int> fail_wait{0};          // hipStreamWaitEvent fails so many times
std::atomic<int> fail_precision{0};     // fmm_plan_set_precision fails so many times
std::atomic<int> plans{0};              // plans alive
size_t plan_bytes = 50, partial_bytes = 0;
char dummy;
template <typename T>
T handle() {
  return reinterpret_cast<T>(&dummy);
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = handle<hipStream_t>(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hold ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) {
  return fail_wait > 0 && fail_wait-- > 0 ? hipErrorUnknown : hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = handle<hipGraph_t>(); return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = handle<hipGraphExec_t>();
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }

fmm_plan_t fmm_plan_stream(const double*, int64_t n, int h, int order, hipStream_t) {
  fmm_plan_s* p = new fmm_plan_s();
  p->n = n;
  p->height = h;
  p->order = order;
  ++plans;
  return p;
}
int fmm_plan_set_precision(fmm_plan_t p, int mode) {
  if (fail_precision > 0 && fail_precision-- > 0) return FMM_ERR_OOM;
  p->precision = mode;
  fmm::upload_job(p, nullptr);
  return FMM_OK;
}
void fmm_release(fmm_plan_t p) {
  if (p) --plans;
  delete p;
}
const char* fmm_last_error() { return "stand-in plan error"; }
}

// A dense plan of plan_bytes and, where it may split its M2L, partial_bytes.
namespace fmm {
void set_error(const std::string&) {}
void set_error_code(int) {}
int last_error_code() { return FMM_ERR_HIP; }
void upload_job(fmm_plan_s* p, hipStream_t) {
  const bool split = !p->dense_unsplit && partial_bytes > 0;
  if (p->bytes > 0 && fail_upload > 0 && fail_upload-- > 0)
    throw FmmError{FMM_ERR_HIP, "stand-in upload error"};
  p->job_h.ld = 16;
  p->job_h.locx_rows = 1;
  p->job_h.m2l_ranges = partial_bytes > 0 ? 2 : 1;
  p->job_h.m2l_parts = split ? 2 : 1;
  p->bytes = plan_bytes + (split ? partial_bytes : 0);
}
void launch_step(StepKind, int, bool, const JobDev*, const StepTab*, const CallDev*, int,
                 hipStream_t, int, int, int) {}
int p2p_waves(int64_t, int64_t) { return 1; }
int m2l_svd_nt(int, bool, int64_t, int) { return 1; }
int m2l_svd_nmb(int, bool, int) { return 1; }
void* dev_alloc(size_t n) { return calloc(1, n); }
void dev_free(void* p) { free(p); }
}  // namespace fmm
fmm_plan_s::~fmm_plan_s() {}

namespace {
double xs[8];
int64_t submit(fmm_server_t s) {
  return fmm_server_submit(s, xs, xs, 1, 3, 2, FMM_FP64, xs, xs, nullptr);
}
template <typename F>
bool soon(F f) {
  for (int i = 0; i < 400; ++i) {
    if (f()) return true;
    std::this_thread::sleep_for(std::chrono::milliseconds(5));
  }
  return false;
}
[[noreturn]] void end(bool good, const char* what) {
  std::printf("%s %s\n", good ? "ok" : "FAILED", what);
  std::fflush(stdout);
  std::_Exit(good ? 0 : 1);  // a server that lost a request cannot be destroyed
}
// the request ends with an error (or without one) and the next one runs
void ends(fmm_server_t s, bool may_pass) {
  const int64_t t = submit(s);
  fmm_request_stats st{};
  if (!soon([&] { return fmm_server_poll(s, t, &st) == 1; })) end(false, "request lost");
  if (!may_pass && st.status == FMM_OK) end(false, "error not reported");
  if (fmm_server_wait(s, submit(s), &st) != FMM_OK) end(false, "next request");
  fmm_server_destroy(s);
  end(plans == 0, "plans released");
}
}  // namespace

int main(int, char** argv) {
  const std::string what = argv[1];
  if (what == "upload") {  // dropping the partial sums fails
    plan_bytes = 100;
    partial_bytes = 128;
    fail_upload = 1;
    ends(fmm_server_create(150, 4), true);
  } else if (what == "beside") {  // two plans fit the budget without their partial sums
    partial_bytes = 20;
    hold = true;
    fmm_server_t s = fmm_server_create(2 * plan_bytes, 4);
    const int64_t a = submit(s);
    fmm_request_stats st{};
    if (!soon([&] { return fmm_server_poll(s, a, &st) == 0 && st.batch >= 0; }))
      end(false, "first request not launched");
    const int64_t b = submit(s);
    if (!soon([&] { return fmm_server_poll(s, b, &st) == 0 && st.batch >= 0; }))
      end(false, "second request not launched beside the first");
    hold = false;
    const bool good = fmm_server_wait(s, a, &st) == FMM_OK && fmm_server_wait(s, b, &st) == FMM_OK;
    fmm_server_destroy(s);
    end(good && plans == 0, "both done");
  } else if (what == "wait") {
    fail_wait = 1;
    ends(fmm_server_create(150, 4), false);
  } else if (what == "precision") {
    fail_precision = 1;
    ends(fmm_server_create(150, 4), false);
  }
  end(false, "unknown scenario");
}
