// A HIP runtime of host bookkeeping for tests of the library's call sequences without a device.  Every
// entry point libqe.so imports is here; loaded into the global scope before libqe.so, these definitions
// are the ones it binds to.
//
// Kernels do nothing.  A stream is the ordered list of what was put on it (kernels, waits on events), an
// event the place in a stream where it was recorded, and waiting on the host completes a stream up to
// such a place, with everything it waited on.  So "is any kernel still pending" has an answer, and every
// call is in a text log.  Device addresses are numbers, never memory.
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

namespace {

struct Kernel {
  const void *func;
  dim3 grid, block;
  unsigned shmem;
};
struct Stream;
struct Op {
  bool kernel;
  Stream *dep;  // a wait: on this stream ..
  size_t upto;  // .. up to this place
};
struct Stream {
  int id = 0;
  std::vector<Op> ops;
  size_t done = 0;
  struct Graph *capturing = nullptr;
};
struct Event {
  int id = 0;
  Stream *at = nullptr;
  size_t upto = 0;
};
struct Graph {
  std::vector<Kernel> nodes;
};
struct Exec {
  size_t kernels;
};

std::string g_log, g_result;
std::map<const void *, std::string> g_names;
std::map<void *, Stream *> g_streams;  // by handle: the library's own, and the caller's, made on first use
std::vector<Stream *> g_all;
int g_events = 0, g_fail_launch = 0, g_fail_record = 0;
uintptr_t g_next = uintptr_t(1) << 32;

template <typename... A>
void note(const char *fmt, A... a) {
  char line[600];
  snprintf(line, sizeof(line), fmt, a...);
  g_log += line;
  g_log += '\n';
}

Stream *stream_of(hipStream_t h) {
  Stream *&s = g_streams[h];
  if (s == nullptr) {
    s = new Stream;
    s->id = int(g_all.size());
    g_all.push_back(s);
  }
  return s;
}

void complete(Stream *s, size_t upto) {
  for (; s->done < upto; ++s->done)
    if (s->ops[s->done].dep != nullptr) complete(s->ops[s->done].dep, s->ops[s->done].upto);
}

int pending() {
  int n = 0;
  for (Stream *s : g_all)
    for (size_t i = s->done; i < s->ops.size(); ++i) n += s->ops[i].kernel;
  return n;
}

const char *name_of(const void *f) {
  auto it = g_names.find(f);
  return it == g_names.end() ? "?" : it->second.c_str();
}

hipError_t launch(const void *f, dim3 grid, dim3 block, size_t shmem, hipStream_t h) {
  Stream *s = stream_of(h);
  if (g_fail_launch > 0 && --g_fail_launch == 0) {
    note("launch_failed stream=%d %s", s->id, name_of(f));
    return hipErrorLaunchFailure;
  }
  if (s->capturing != nullptr) {
    s->capturing->nodes.push_back({f, grid, block, unsigned(shmem)});
    note("capture stream=%d %s grid=%u", s->id, name_of(f), grid.x);
    return hipSuccess;
  }
  s->ops.push_back({true, nullptr, 0});
  note("launch stream=%d %s grid=%u", s->id, name_of(f), grid.x);
  return hipSuccess;
}

}  // namespace

extern "C" {

// ---- for the tests
const char *fake_log() { return (g_result = g_log).c_str(); }
void fake_clear() { g_log.clear(); }
int fake_pending() { return pending(); }
void fake_fail_launch(int n) { g_fail_launch = n; }  // the n-th kernel launch from now fails
void fake_fail_record(int n) { g_fail_record = n; }  // the n-th event record from now fails
// run everything a kernel put on this stream now would run after
void fake_drain(void *h) {
  Stream *s = stream_of(static_cast<hipStream_t>(h));
  complete(s, s->ops.size());
}

// ---- registration
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) {
  g_names[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipErrorUnknown; }

// ---- device, memory
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  memset(p, 0, sizeof(*p));
  strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes) {
  *p = reinterpret_cast<void *>(g_next);
  g_next += (bytes + 511) / 256 * 256;
  return hipSuccess;
}
hipError_t hipFree(void *) {
  note("free pending=%d", pending());
  return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpy(void *dst, const void *, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyDeviceToHost) memset(dst, 0, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t h) {
  Stream *s = stream_of(h);
  s->ops.push_back({true, nullptr, 0});
  note("copy stream=%d", s->id);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return hipMalloc(p, 16384); }

// ---- streams, events
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  void *h;
  (void)hipMalloc(&h, 1);
  *s = static_cast<hipStream_t>(h);
  note("stream %d", stream_of(*s)->id);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t h) {
  Stream *s = stream_of(h);
  note("sync stream=%d", s->id);
  complete(s, s->ops.size());
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  Event *v = new Event;
  v->id = g_events++;
  *e = reinterpret_cast<hipEvent_t>(v);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.0f, hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t h) {
  Stream *s = stream_of(h);
  Event *v = reinterpret_cast<Event *>(e);
  if (g_fail_record > 0 && --g_fail_record == 0) {
    note("record_failed stream=%d", s->id);
    return hipErrorUnknown;
  }
  v->at = s;
  v->upto = s->ops.size();
  note("record event=%d stream=%d", v->id, s->id);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  Event *v = reinterpret_cast<Event *>(e);
  note("sync event=%d", v->id);
  if (v->at != nullptr) complete(v->at, v->upto);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t h, hipEvent_t e, unsigned) {
  Stream *s = stream_of(h);
  Event *v = reinterpret_cast<Event *>(e);
  if (v->at != nullptr && v->at != s) s->ops.push_back({false, v->at, v->upto});
  note("wait stream=%d event=%d", s->id, v->id);
  return hipSuccess;
}

// ---- launches, graphs
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t m, hipStream_t s) { return launch(f, g, b, m, s); }
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t m, hipStream_t s, hipEvent_t, hipEvent_t,
                              int) {
  return launch(f, g, b, m, s);
}
hipError_t hipStreamBeginCapture(hipStream_t h, hipStreamCaptureMode) {
  stream_of(h)->capturing = new Graph;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t h, hipGraph_t *g) {
  Stream *s = stream_of(h);
  *g = reinterpret_cast<hipGraph_t>(s->capturing);
  s->capturing = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(new Exec{reinterpret_cast<Graph *>(g)->nodes.size()});
  note("instantiate kernels=%zu", reinterpret_cast<Graph *>(g)->nodes.size());
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t h) {
  Stream *s = stream_of(h);
  const size_t n = reinterpret_cast<Exec *>(e)->kernels;
  for (size_t i = 0; i < n; ++i) s->ops.push_back({true, nullptr, 0});
  note("graph_launch stream=%d kernels=%zu", s->id, n);
  return hipSuccess;
}
hipError_t hipGraphExecKernelNodeSetParams(hipGraphExec_t, hipGraphNode_t, const hipKernelNodeParams *) {
  note("set_params pending=%d", pending());
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  note("exec_destroy pending=%d", pending());
  delete reinterpret_cast<Exec *>(e);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<Graph *>(g);
  return hipSuccess;
}
// a node is the address of its kernel; the graphs are chains
static Graph *g_walk;
hipError_t hipGraphGetNodes(hipGraph_t g, hipGraphNode_t *, size_t *n) {
  g_walk = reinterpret_cast<Graph *>(g);
  *n = g_walk->nodes.size();
  return hipSuccess;
}
hipError_t hipGraphGetRootNodes(hipGraph_t g, hipGraphNode_t *out, size_t *n) {
  if (out != nullptr) *out = reinterpret_cast<hipGraphNode_t>(reinterpret_cast<Graph *>(g)->nodes.data());
  *n = 1;
  return hipSuccess;
}
hipError_t hipGraphNodeGetType(hipGraphNode_t, hipGraphNodeType *t) { return *t = hipGraphNodeTypeKernel, hipSuccess; }
hipError_t hipGraphNodeGetDependentNodes(hipGraphNode_t node, hipGraphNode_t *out, size_t *n) {
  Kernel *k = reinterpret_cast<Kernel *>(node);
  *n = k + 1 < g_walk->nodes.data() + g_walk->nodes.size() ? 1 : 0;
  if (out != nullptr && *n == 1) *out = reinterpret_cast<hipGraphNode_t>(k + 1);
  return hipSuccess;
}
hipError_t hipGraphKernelNodeGetParams(hipGraphNode_t node, hipKernelNodeParams *p) {
  const Kernel *k = reinterpret_cast<const Kernel *>(node);
  p->func = const_cast<void *>(k->func);
  p->gridDim = k->grid;
  p->blockDim = k->block;
  p->sharedMemBytes = k->shmem;
  return hipSuccess;
}

}  // extern "C"
