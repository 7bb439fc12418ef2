// A stand-in for the HIP runtime (loaded before it) for tests of the
// library's host code without a GPU: memory is host memory, kernels are not
// run, and work stays pending on its stream until something waits for it.
// It notes what a program must not do: destroy a graph whose replay is
// pending, a stream with pending work, or a stream before an event that was
// recorded on it; run a kernel on moments that the last writer left in the other
// schedules' layout; pull from a wall stash that the step before did not write.
// The k-th launch of a kernel takes 1 + k^2 / 1000 ms of its stream's time.
#define __HIP_PLATFORM_AMD__
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

namespace {

struct Stream {
  long issued = 0, done = 0;  // work handed in, work known to have ended
  double clock = 0.0;
  Stream *capture = nullptr;  // the capture's first stream, while capturing
};
struct Event {
  Stream *stream = nullptr;
  bool captured = false;
  long at = 0;
  double clock = 0.0;
};
struct Exec {
  std::map<Stream *, long> replays;  // the last replay on each stream
  double cost = 0.0;
};
struct Graph {
  double cost = 0.0;
};

Stream null_stream;
std::set<Stream *> streams = {&null_stream};
std::set<Event *> events;
std::map<Stream *, double> captured_cost;
std::map<const void *, std::string> names;
std::map<std::string, long> launches;
std::set<std::string> faults;
std::vector<double> elapsed;
struct Config {
  dim3 g, b;
  size_t shared;
  hipStream_t s;
} config;

// The moments' layout in each aux array (0 populations', 1 compact), and the
// wall stashes that hold the last step's arrivals.
std::map<const void *, int> layout;
std::set<const void *> fresh, used;

void look(const std::string &name, void **args) {
  auto arg = [&](int i) { return *(const void **)args[i]; };
  std::vector<bool> flags;  // the kernel's truth-valued template arguments, in order
  const std::string t = name.substr(0, name.find('('));
  for (size_t i = 0; i < t.size(); ++i) {
    if (t.compare(i, 4, "true") == 0) flags.push_back(true);
    if (t.compare(i, 5, "false") == 0) flags.push_back(false);
  }
  auto reads = [&](const void *aux, int as) {
    if (layout.count(aux) && layout[aux] != as)
      faults.insert(t + " on moments of the other layout");
  };
  if (t.find("k_pull<") != std::string::npos) {
    layout[arg(4)] = flags.back() ? 1 : 0;
    if (arg(7)) fresh.insert(arg(7));
  } else if (t.find("k_cpull<") != std::string::npos) {
    layout[arg(3)] = 1;
    if (arg(5) && !fresh.count(arg(5))) faults.insert(t + " from a stale wall stash");
    used.insert(arg(5));
    fresh.insert(arg(6));
  } else if (t.find("k_fused<") != std::string::npos) {
    reads(arg(2), flags[2] ? 1 : 0);  // WALLS, EXPORT, COMPACT, PLAIN
    for (const void *p : used) fresh.erase(p);
    used.clear();
  } else if (t.find("k_interface<") != std::string::npos) {
    reads(arg(2), 0);
  }
}

Stream *of(hipStream_t s) { return s ? (Stream *)s : &null_stream; }
void work(Stream *s, double cost) {
  if (s->capture) {
    captured_cost[s->capture] += cost;
  } else {
    ++s->issued;
    s->clock += cost;
  }
}

}  // namespace

extern "C" {

int standin_faults(char *buf, int n) {
  std::string all;
  for (const std::string &f : faults) all += f + "\n";
  std::snprintf(buf, (size_t)n, "%s", all.c_str());
  const int k = (int)faults.size();
  faults.clear();
  return k;
}
long standin_launches(const char *part) {
  long k = 0;
  for (const auto &l : launches)
    if (l.first.find(part) != std::string::npos) k += l.second;
  return k;
}
int standin_elapsed(double *out, int n) {
  const int k = (int)elapsed.size();
  for (int i = 0; i < k && i < n; ++i) out[i] = elapsed[(size_t)i];
  elapsed.clear();
  return k;
}

void **__hipRegisterFatBinary(const void *) {
  static void *p;
  return &p;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  char *plain = abi::__cxa_demangle(name, nullptr, nullptr, nullptr);
  names[host] = plain ? plain : name;
  std::free(plain);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t s) {
  config = {g, b, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s) {
  *g = config.g;
  *b = config.b;
  *shared = config.shared;
  *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t s) {
  long &k = launches[names[f]];
  work(of(s), 1.0 + 1e-3 * (double)k * (double)k);
  ++k;
  look(names[f], args);
  return hipSuccess;
}

hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static char room[64];
  return *p = room, hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) { return *p = std::malloc(n ? n : 1), hipSuccess; }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  std::memmove(d, s, n);
  work(of(st), 0.0);
  return hipSuccess;
}

hipError_t hipDeviceSynchronize() {
  for (Stream *s : streams) s->done = s->issued;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  of(s)->done = of(s)->issued;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  Stream *n = new Stream;
  streams.insert(n);
  return *s = (hipStream_t)n, hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  if (of(s)->done < of(s)->issued) faults.insert("stream destroyed with pending work");
  for (Event *e : events)
    if (e->stream == of(s)) faults.insert("stream destroyed before an event recorded on it");
  streams.erase(of(s));
  delete of(s);
  return hipSuccess;
}

hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  Event *n = new Event;
  events.insert(n);
  return *e = (hipEvent_t)n, hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  events.erase((Event *)e);
  delete (Event *)e;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e_, hipStream_t s) {
  Event *e = (Event *)e_;
  work(of(s), 0.0);
  e->stream = of(s);
  e->captured = of(s)->capture != nullptr;
  e->at = of(s)->issued;
  e->clock = of(s)->clock;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e_) {
  Event *e = (Event *)e_;
  if (e->stream && !e->captured && e->stream->done < e->at) e->stream->done = e->at;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(((Event *)b)->clock - ((Event *)a)->clock);
  elapsed.push_back(*ms);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e_, unsigned) {
  Event *e = (Event *)e_;
  if (e->captured) of(s)->capture = e->stream->capture;
  return hipSuccess;
}

hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st) {
  *st = of(s)->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  of(s)->capture = of(s);
  captured_cost[of(s)] = 0.0;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g) {
  Graph *n = new Graph;
  n->cost = captured_cost[of(s)];
  for (Stream *t : streams)
    if (t->capture == of(s)) t->capture = nullptr;
  return *g = (hipGraph_t)n, hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { return delete (Graph *)g, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  Exec *n = new Exec;
  n->cost = ((Graph *)g)->cost;
  return *x = (hipGraphExec_t)n, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  work(of(s), ((Exec *)x)->cost);
  ((Exec *)x)->replays[of(s)] = of(s)->issued;
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  for (const auto &r : ((Exec *)x)->replays)
    if (streams.count(r.first) && r.first->done < r.second)
      faults.insert("graph destroyed with a pending replay");
  return delete (Exec *)x, hipSuccess;
}

}  // extern "C"
