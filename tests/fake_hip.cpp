// A HIP runtime without a device, for tests of the library's host side: this
// program defines the runtime's functions, so that libqtn.so calls these.
// Device memory is host memory, kernels are counted and not run, and the
// failures under test are switched on from the scenarios below.  Capture
// follows the runtime's rules: a stream that waits for an event of a capturing
// stream joins its capture, what is queued there does not run, and waiting for
// such a stream fails.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "qtn.h"

struct ihipStream_t {
  int capture = 0;  // 0 no, 1 the library's own, 2 the caller's
};
struct ihipEvent_t {
  int capture = 0;
  float ms = 1.0f;  // of the launch that it ended
};
struct ihipGraph {};
struct hipGraphExec {};

namespace {

struct Counts {
  int mallocs = 0, copies = 0, captured_copies = 0, graphs = 0, launches = 0;
};
Counts n;
constexpr size_t kDeviceBytes = 4ull << 30;
size_t live_bytes = 0, most_bytes = 0;
std::map<void *, size_t> *sizes;
std::set<ihipStream_t *> *joined;  // streams in the caller's capture
bool malloc_fails = false;

// kernels by the address of their host stub (filled while libqtn.so loads)
struct Kernel {
  const void *host;
  const char *name;
};
Kernel kernels[1024];
int n_kernels = 0;
std::map<std::string, int> *launched;  // by kernel name, counted where set
std::map<std::string, float> *ms_of;   // by part of a kernel's name

std::string name_of(const void *f) {
  for (int i = 0; i < n_kernels; i++)
    if (kernels[i].host == f) return kernels[i].name;
  return "";
}
void count_launch(const void *f, ihipStream_t *s) {
  if (s && s->capture) return;
  n.launches++;
  if (launched) (*launched)[name_of(f)]++;
}

}  // namespace

extern "C" {

void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  if (n_kernels < 1024) kernels[n_kernels++] = {host, name};
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
static hipStream_t pushed;
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t s) {
  pushed = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) {
  *g = dim3(1);
  *b = dim3(1);
  *l = 0;
  *s = pushed;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s) {
  count_launch(f, s);
  return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t s,
                              hipEvent_t, hipEvent_t stop, int) {
  count_launch(f, s);
  if (ms_of && stop)
    for (auto &kv : *ms_of)
      if (name_of(f).find(kv.first) != std::string::npos) stop->ms = kv.second;
  return hipSuccess;
}

hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *, int, size_t) {
  *v = 4;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetSymbolAddress(void **p, const void *s) {
  *p = const_cast<void *>(s);
  return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t bytes) {
  n.mallocs++;
  if (malloc_fails) return hipErrorOutOfMemory;
  *p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  if (!sizes) sizes = new std::map<void *, size_t>;
  (*sizes)[*p] = bytes;
  live_bytes += bytes;
  if (live_bytes > most_bytes) most_bytes = live_bytes;
  return hipSuccess;
}
hipError_t hipDeviceTotalMem(size_t *all, hipDevice_t) {
  *all = kDeviceBytes;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (p) {
    live_bytes -= (*sizes)[p];
    sizes->erase(p);
  }
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) {
  *p = std::calloc(1, bytes);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t bytes, hipMemcpyKind, hipStream_t s) {
  if (s && s->capture) {
    n.captured_copies++;
    return hipSuccess;
  }
  std::memcpy(dst, src, bytes);
  n.copies++;
  return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = new ihipStream_t;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  if (joined) joined->erase(s);
  delete s;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (e->capture == 2 && s->capture == 0) {
    s->capture = 2;
    if (!joined) joined = new std::set<ihipStream_t *>;
    joined->insert(s);
  }
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  return s && s->capture ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
  *st = s && s->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  if (s->capture) return hipErrorIllegalState;
  s->capture = 1;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  s->capture = 0;
  *g = new ihipGraph;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  n.graphs++;
  *e = new hipGraphExec;
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) {
  n.launches++;
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete g;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete e;
  return hipSuccess;
}

hipError_t hipEventCreate(hipEvent_t *e) {
  *e = new ihipEvent_t;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  e->capture = s ? s->capture : 0;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t stop) {
  *ms = stop->ms;
  return hipSuccess;
}

}  // extern "C"

namespace {

#define CHECK(x)                                                    \
  do {                                                              \
    if (!(x)) {                                                     \
      std::printf("line %d: %s (%s)\n", __LINE__, #x, qtn_last_error()); \
      std::exit(1);                                                 \
    }                                                               \
  } while (0)

void end_caller_capture(ihipStream_t *s) {
  s->capture = 0;
  if (joined)
    for (auto *j : *joined) j->capture = 0;
  if (joined) joined->clear();
}

// A planned network of a ring of nv vertices with chords, and its workspace.
struct Net {
  qtn_network *h = nullptr;
  size_t bytes = 0;
  void *ws = nullptr;
  int p = 0;
  explicit Net(int nv, int depth, int precision = QTN_C128) : p(depth) {
    std::vector<int32_t> e;
    for (int i = 0; i < nv; i++) {
      e.insert(e.end(), {i, (i + 1) % nv});
      if (i < nv / 2) e.insert(e.end(), {i, i + nv / 2});
    }
    const std::vector<double> g(depth, 0.3), b(depth, 0.2);
    CHECK(qtn_network_build(nv, e.size() / 2, e.data(), depth, g.data(), b.data(), nullptr, &h) == QTN_OK);
    CHECK(qtn_plan(h, nullptr, precision, &bytes) == QTN_OK);
    ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  }
  int contract(ihipStream_t *s) {
    double e;
    return qtn_contract(h, ws, bytes, s, nullptr, nullptr, &e);
  }
  ~Net() {
    qtn_network_free(h);
    std::free(ws);
  }
};

// A call on a capturing stream is refused, and the one after it finds its
// descriptors on the device.
int refused_under_capture() {
  for (int planned_before = 0; planned_before < 2; planned_before++) {
    Net net(10, 2);
    ihipStream_t s;
    if (planned_before) {  // the runtime and a graph exist; a new schedule does not
      CHECK(net.contract(&s) == QTN_OK);
      CHECK(qtn_set_tune_picks(net.h, nullptr, 0) == QTN_OK);
    }
    s.capture = 2;
    CHECK(net.contract(&s) == QTN_EDEVICE);
    CHECK(n.captured_copies == 0);  // nothing of it in the caller's graph
    end_caller_capture(&s);
    const Counts before = n;
    CHECK(net.contract(&s) == QTN_OK);
    CHECK(n.copies == before.copies + 1);  // the descriptors
    CHECK(net.contract(&s) == QTN_OK);
    CHECK(n.copies == before.copies + 1);  // kept
  }
  return 0;
}

// Without memory for the descriptors every call sends them into the workspace,
// which is all that it pays: one failed allocation, one graph.
int no_memory_for_descriptors() {
  Net net(10, 2);
  ihipStream_t s;
  malloc_fails = true;
  for (int k = 0; k < 3; k++) CHECK(net.contract(&s) == QTN_OK);
  CHECK(n.mallocs == 1 && n.graphs == 1 && n.copies == 3);
  malloc_fails = false;
  CHECK(qtn_set_tune_picks(net.h, nullptr, 0) == QTN_OK);  // a new schedule tries again
  for (int k = 0; k < 3; k++) CHECK(net.contract(&s) == QTN_OK);
  CHECK(n.mallocs == 2 && n.graphs == 2 && n.copies == 4);
  return 0;
}

// Batches keep their descriptors on the device until one of their networks
// goes: many different ones stay under a bound together, every one still runs,
// and what they took is given back.
int descriptors_of_many_batches() {
  constexpr size_t kBound = kDeviceBytes / 128;
  Net net(30, 3);
  ihipStream_t s;
  for (int k = 0; n.copies == k && k < 64; k++) {  // a batch without memory of its own sends them twice
    const std::vector<qtn_network *> nets(8 + k, net.h);
    const int count = (int)nets.size();
    std::vector<double> e(count);
    size_t bytes = 0;
    CHECK(qtn_batch_workspace(nets.data(), count, &bytes) == QTN_OK);
    void *ws = std::aligned_alloc(256, bytes);
    for (int r = 0; r < 2; r++)
      CHECK(qtn_contract_batch(nets.data(), count, ws, bytes, &s, nullptr, e.data()) == QTN_OK);
    std::free(ws);
  }
  CHECK(n.copies > n.mallocs);
  CHECK(most_bytes <= kBound && most_bytes > kBound / 2);
  qtn_network_free(net.h);
  net.h = nullptr;
  CHECK(live_bytes == 0);
  return 0;
}

// The autotuner times a small group alone in a workgroup by each mapping that
// it may pick, and once as a segment program (which no pick changes).
int autotuned_small_groups() {
  Net net(12, 2);
  ihipStream_t s;
  qtn_plan_stats st;
  CHECK(qtn_get_plan_stats(net.h, &st) == QTN_OK && st.max_width <= 16);
  launched = new std::map<std::string, int>;
  CHECK(qtn_autotune(net.h, net.ws, net.bytes, &s, nullptr) == QTN_OK);
  int programs = 0, mappings = 0;
  for (auto &kv : *launched) {
    if (kv.first.find("k_programs") != std::string::npos) programs += kv.second;
    if (kv.first.find("k_block_groups") != std::string::npos) mappings += kv.second;
  }
  constexpr int kPasses = 2, kMappings = 4;  // generic, streaming with 1, 2 and 3 lane bits
  CHECK(programs == kPasses * st.n_groups);
  CHECK(mappings >= kPasses * kMappings * st.n_groups);
  return 0;
}

// Groups that are short in launches of their own keep the cell mapping that
// step launches run, although another is shorter there; long ones do not.
int autotuned_steps() {
  for (int is_long = 0; is_long < 2; is_long++) {
    Net net(20, 3);
    ihipStream_t s;
    qtn_plan_stats before, after;
    CHECK(qtn_get_plan_stats(net.h, &before) == QTN_OK && before.n_cell > 0);
    const float ms = is_long ? 1.0f : 0.005f;
    ms_of = new std::map<std::string, float>{
        {"k_wide_cells", 2 * ms}, {"k_wide_stream", 3 * ms}, {"k_wide_generic", ms}, {"k_wide_mfma", 3 * ms}};
    CHECK(qtn_autotune(net.h, net.ws, net.bytes, &s, nullptr) == QTN_OK);
    CHECK(qtn_get_plan_stats(net.h, &after) == QTN_OK);
    CHECK(after.n_cell == (is_long ? 0 : before.n_cell));
  }
  return 0;
}

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "refused_under_capture") return refused_under_capture();
  if (what == "no_memory_for_descriptors") return no_memory_for_descriptors();
  if (what == "descriptors_of_many_batches") return descriptors_of_many_batches();
  if (what == "autotuned_small_groups") return autotuned_small_groups();
  if (what == "autotuned_steps") return autotuned_steps();
  std::printf("no scenario '%s'\n", what.c_str());
  return 2;
}
