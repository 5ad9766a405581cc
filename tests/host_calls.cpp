// Test infrastructure: the library's host code against a HIP runtime of this
// file's own, which allocates host memory, runs no kernel and records what is
// launched, captured, replayed and allocated.  Built for the host alone
// (hipcc --cuda-host-only) and run without a GPU; the first argument names the
// check.  Exit status 0: all expectations hold.
#include "pn_api.hip"

#include <map>
#include <memory>
#include <set>
#include <string>

#define EXPECT(cond)                                                          \
  do {                                                                        \
    if (!(cond)) {                                                            \
      std::fprintf(stderr, "%s:%d: failed: %s\n", __FILE__, __LINE__, #cond); \
      std::exit(1);                                                           \
    }                                                                         \
  } while (0)

// ------------------------------------------------------------------ the runtime
struct Launch {
  std::string kernel;     // mangled name
  hipStream_t stream;     // where it was launched
  unsigned blocks, threads;
  bool replayed = false;  // from a graph
  pn::StageArgs stage{};  // k_stage's argument
  pn::EpiArgs epi{};      // an epilogue's argument (k_epilogue..., k_stage_head)
};
using Graph = std::vector<Launch>;

struct Counts {
  int device = 0, host = 0, freed = 0;  // allocations, frees
  int captures = 0, replays = 0;
};
Counts count;
std::map<const void*, std::string> names;
std::map<hipStream_t, Graph> capturing;  // streams under capture
std::vector<Launch> executed;
dim3 cfg_grid, cfg_block;
size_t cfg_shmem;
hipStream_t cfg_stream;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* name, const char*, unsigned, void*,
                           void*, void*, void*, int*) {
  names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shmem, hipStream_t s) {
  cfg_grid = g, cfg_block = b, cfg_shmem = shmem, cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shmem, hipStream_t* s) {
  *g = cfg_grid, *b = cfg_block, *shmem = cfg_shmem, *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t,
                           hipStream_t s) {
  Launch l{names.at(f), s, grid.x, block.x};
  if (l.kernel.find("k_stage_head") != std::string::npos ||
      l.kernel.find("k_epilogue_chain") != std::string::npos)
    l.epi = *static_cast<pn::EpiArgs*>(args[0]);
  else if (l.kernel.find("k_stage") != std::string::npos)
    l.stage = *static_cast<pn::StageArgs*>(args[0]);
  const auto c = capturing.find(s);
  if (c == capturing.end()) executed.push_back(l);
  else c->second.push_back(l);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  EXPECT(!capturing.count(s));
  capturing[s];
  ++count.captures;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status) {
  *status = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  EXPECT(capturing.count(s));
  *g = reinterpret_cast<hipGraph_t>(new Graph(capturing[s]));
  capturing.erase(s);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *x = reinterpret_cast<hipGraphExec_t>(new Graph(*reinterpret_cast<Graph*>(g)));
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<Graph*>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  delete reinterpret_cast<Graph*>(x);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t s) {
  EXPECT(!capturing.count(s));
  for (Launch l : *reinterpret_cast<Graph*>(x)) {
    l.stream = s;
    l.replayed = true;
    executed.push_back(l);
  }
  ++count.replays;
  return hipSuccess;
}
static hipError_t allocate(void** p, size_t n) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipMalloc(void** p, size_t n) {
  ++count.device;
  return allocate(p, n);
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++count.host;
  return allocate(p, n);
}
hipError_t hipFree(void* p) {
  ++count.freed;
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* fixed = std::aligned_alloc(256, (size_t)64 << 20);
  *p = fixed;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(dst, src, n);
  return hipSuccess;
}
static void* handle() { return new char; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = static_cast<hipStream_t>(handle());
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = static_cast<hipEvent_t>(handle());
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  EXPECT(!capturing.count(s));
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

// ------------------------------------------------------------------ the checks
constexpr double G = 1.0, C = 30.0, EPS = 1e-3, DT = 1e-4;

struct System {
  int64_t N;
  std::vector<double> pos, vel, mass;
  explicit System(int64_t n) : N(n), pos(3 * n, 0.5), vel(3 * n, 0.25), mass(n, 1.0) {}
  int step(int64_t nsteps, int flags = 0, hipStream_t s = nullptr, int precision = PN_FP64) {
    return pn_step(pos.data(), vel.data(), mass.data(), N, G, C, EPS, DT, nsteps, precision, s,
                   flags);
  }
};

// A graph of one-launch stages is used with the buffers it was captured with: a
// launch shape of another split count moves them within the scratch memory.
void check_stage_shape() {
  System a(100);
  EXPECT(pn_set_stage_kernel(PN_FP64, 2, 1000, 2) == PN_OK);
  for (int splits : {16, 4, 16}) {
    EXPECT(pn_set_shape(-1, 0, 0, 0, 0, 0) == PN_OK);
    EXPECT(pn_set_shape(PN_FP64, 2, 1000, 1, 4, splits) == PN_OK);
    executed.clear();
    EXPECT(a.step(400) == PN_OK);
    int stages = 0;
    std::set<const void*> packets, rows, state;
    for (const Launch& l : executed) {
      if (!l.stage.pk) continue;
      ++stages;
      packets.insert(l.stage.pk);
      rows.insert(l.stage.e.bpart);
      state.insert(l.stage.bhs_in);
    }
    EXPECT(stages == 4 * 400 + 1);
    EXPECT(packets.size() == 2 && rows.size() == 2 && state.size() == 2);
  }
}

// A system whose buffers no other system had (a graph may be cached for those).
System& fresh(int64_t N) {
  static std::vector<std::unique_ptr<System>> all;
  all.push_back(std::make_unique<System>(N));
  return *all.back();
}

// The entry points that step: one-launch and chained stages, Hermite, an ensemble.
using Advance = int (*)(System&, int64_t nsteps, int flags, hipStream_t s);
int hermite(System& a, int64_t nsteps, int flags, hipStream_t s) {
  return pn_step_hermite(a.pos.data(), a.vel.data(), a.mass.data(), a.N, G, C, EPS, DT, nsteps, s,
                         flags);
}
int rk4(System& a, int64_t nsteps, int flags, hipStream_t s) { return a.step(nsteps, flags, s); }
int ensemble(System& a, int64_t nsteps, int flags, hipStream_t s) {
  const int64_t offsets[3] = {0, a.N / 3, a.N};
  const double g[2] = {G, G}, c[2] = {C, C}, eps[2] = {EPS, EPS};
  return pn_step_batched(2, offsets, g, c, eps, a.pos.data(), a.vel.data(), a.mass.data(), DT,
                         nsteps, PN_FP64, s, flags);
}
struct Scheme {
  Advance run;
  int64_t N, replay;  // bodies; steps of a call that can replay a graph
};
const Scheme kSchemes[] = {{rk4, 100, 17}, {rk4, 2500, 17}, {hermite, 150, 16}, {ensemble, 300, 16}};

// A graph is captured by the first call that can replay it, once 256 steps in a
// row were asked for by calls that allow graphs.
void check_graph_count() {
  EXPECT(pn_set_stage_kernel(PN_FP64, 2, 1000, 2) == PN_OK);
  for (const Scheme& k : kSchemes) {
    const auto captures = [&](std::initializer_list<std::pair<int64_t, int>> calls) {
      System &a = fresh(k.N), &other = fresh(k.N);
      EXPECT(k.run(other, 1, 0, nullptr) == PN_OK);  // (ends any count)
      const Counts before = count;
      for (const auto& c : calls) EXPECT(k.run(a, c.first, c.second, nullptr) == PN_OK);
      const int n = count.captures - before.captures;
      EXPECT((n > 0) == (count.replays > before.replays));
      return n;
    };
    EXPECT(captures({{255, 0}}) == 0);
    EXPECT(captures({{256, 0}}) == 1);
    EXPECT(captures({{257, 0}}) == 1);
    EXPECT(captures({{200, 0}, {55, 0}}) == 0);
    EXPECT(captures({{200, 0}, {56, 0}}) == 1);
    EXPECT(captures({{256, 0}, {40, 0}, {40, 0}}) == 1);
    EXPECT(captures({{256, PN_NOGRAPH}, {100, 0}}) == 0);
    EXPECT(captures({{200, 0}, {100, PN_NOGRAPH}, {55, 0}}) == 0);
    EXPECT(captures({{255, 0}, {k.replay - 1, 0}}) == 0);
    EXPECT(captures({{255, 0}, {k.replay, 0}}) == 1);
    // a step per call
    System& a = fresh(k.N);
    const Counts before = count;
    for (int i = 0; i < 300; ++i) EXPECT(k.run(a, 1, 0, nullptr) == PN_OK);
    EXPECT(count.captures - before.captures == 0);
    EXPECT(k.run(a, k.replay, 0, nullptr) == PN_OK);
    EXPECT(count.captures - before.captures == 1 && count.replays - before.replays == 1);
    EXPECT(k.run(a, k.replay + 16 * 9 + 15, 0, nullptr) == PN_OK);  // 16 steps per replay
    EXPECT(count.captures - before.captures == 1 && count.replays - before.replays == 11);
  }
}

// Steps on a stream that the caller captures are launched directly, into the
// caller's graph, however many were asked for before: no replay there, and no
// capture of the library's own meanwhile.
void check_caller_captures() {
  hipStream_t s = static_cast<hipStream_t>(handle());
  EXPECT(pn_set_stage_kernel(PN_FP64, 2, 1000, 2) == PN_OK);
  for (const Scheme& k : kSchemes) {
    for (const int64_t before : {2, 300}) {  // (300: a graph is cached)
      System& a = fresh(k.N);
      EXPECT(k.run(a, before, 0, s) == PN_OK);
      const Counts c = count;
      hipGraph_t g;
      executed.clear();
      EXPECT(hipStreamBeginCapture(s, hipStreamCaptureModeGlobal) == hipSuccess);
      EXPECT(k.run(a, 300, PN_ASYNC, s) == PN_OK);
      EXPECT(k.run(a, 300, PN_ASYNC, s) == PN_OK);
      EXPECT(hipStreamEndCapture(s, &g) == hipSuccess);
      EXPECT(count.captures == c.captures + 1 && count.replays == c.replays);
      EXPECT(executed.empty() && reinterpret_cast<Graph*>(g)->size() >= 4 * 600);
      EXPECT(hipGraphDestroy(g) == hipSuccess);
    }
  }
}

// An ensemble's epilogue workgroups: as many as run side by side on a CU at 126
// registers per lane (sixteen wavefronts) where there are more than one per CU.
void check_ensemble_epilogues() {
  for (const int systems : {1, 128, 129, 256, 257, 1000}) {  // of two workgroups each
    System& a = fresh(101 * (int64_t)systems);
    std::vector<int64_t> offsets;
    for (int k = 0; k <= systems; ++k) offsets.push_back(101 * (int64_t)k);
    const std::vector<double> g(systems, G), c(systems, C), eps(systems, EPS);
    executed.clear();
    EXPECT(pn_step_batched(systems, offsets.data(), g.data(), c.data(), eps.data(), a.pos.data(),
                           a.vel.data(), a.mass.data(), DT, 1, PN_FP64, nullptr, 0) == PN_OK);
    int found = 0;
    for (const Launch& l : executed) {
      if (l.kernel.find("k_epilogue_batched") == std::string::npos) continue;
      ++found;
      EXPECT(l.blocks == 2u * systems);
      EXPECT(l.threads == (systems <= 128 ? 576u : systems <= 256 ? 320u : 256u));
    }
    EXPECT(found == 4);
  }
}

// pn_accel_noalloc allocates and frees nothing once the device is set up, by
// whichever call: the first of all, and the first after pn_release.
void check_noalloc() {
  System a(300);
  std::vector<double> acc(3 * a.N), phi(a.N), acc1(3 * a.N);
  const auto eval = [&](auto* f, int flags) {
    return f(a.pos.data(), a.vel.data(), a.mass.data(), a.N, G, C, EPS, PN_FP64, acc.data(),
             phi.data(), acc1.data(), nullptr, flags);
  };
  for (int round = 0; round < 2; ++round) {
    EXPECT(eval(round ? pn_accel_noalloc : pn_accel, PN_ASYNC) == PN_OK);  // sets the device up
    const Counts before = count;
    for (int flags : {0, PN_ASYNC, 0}) EXPECT(eval(pn_accel_noalloc, flags) == PN_OK);
    EXPECT(count.device == before.device && count.host == before.host &&
           count.freed == before.freed);
    EXPECT(pn_release() == PN_OK);
  }
  EXPECT(count.host == 2);
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> checks = {
      {"caller_captures", check_caller_captures},
      {"ensemble_epilogues", check_ensemble_epilogues},
      {"graph_count", check_graph_count},
      {"noalloc", check_noalloc},
      {"stage_shape", check_stage_shape},
  };
  if (argc != 2 || !checks.count(argv[1])) return 2;
  checks.at(argv[1])();
  std::printf("%s ok\n", argv[1]);
  return 0;
}
