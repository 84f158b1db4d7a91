// The C ABI's host side on a model of the HIP runtime: no GPU, no device code.
//
// Streams, events and host waits carry vector clocks; every launch that works in
// plan-owned memory has to come after all earlier ones in it, and memory is
// freed only when its last use is known to have finished.  hipStreamPerThread is
// another stream in every (model) thread, and a destroyed stream's handle is
// given out again while its work still runs.  Run with a scenario's name.
#include "xeng_api.cpp"

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <string>

namespace model {
using Clock = std::map<int, long>;  // stream -> operations known to be done
void merge(Clock& a, const Clock& b) {
  for (auto& x : b) a[x.first] = std::max(a[x.first], x.second);
}
struct Stream { int id; Clock seen; };
struct Alloc { size_t bytes; int device; Clock uses; };
int device = 0, thread = 0, next_id = 1;
std::map<std::string, Stream> streams;        // by device, handle, thread, generation
std::map<hipStream_t, int> generation, owner; // owner: device of an explicit stream
std::map<hipStream_t, bool> capturing;
bool null_in_capture = false;
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
Clock host;
std::map<uintptr_t, Alloc> memory;
size_t limit = 1ull << 40;
int mallocs = 0, events = 0, waits = 0, work = 0, tiles = 0, direct = 0;
size_t largest = 0;
uintptr_t next_address = 1ull << 32;

[[noreturn]] void fail(const char* what) {
  std::printf("FAILED: %s\n", what);
  std::exit(1);
}
int device_of(hipStream_t s) {
  return s && s != hipStreamPerThread && owner.count(s) ? owner[s] : device;
}
Stream& stream(hipStream_t s) {
  char key[96];
  std::snprintf(key, sizeof key, "%d %p %d %d", device_of(s), (void*)s,
                s == hipStreamPerThread ? thread : 0, generation[s]);
  Stream& r = streams[key];
  if (!r.seen.size()) r.id = next_id++;
  return r;
}
Clock& step(hipStream_t s) {  // one operation queued on s; what is done before it and by it
  Stream& r = stream(s);
  merge(r.seen, host);
  ++r.seen[r.id];
  return r.seen;
}
void use(const void* p, hipStream_t s) {
  auto it = memory.upper_bound((uintptr_t)p);
  if (it == memory.begin()) fail("work in memory that was never allocated");
  Alloc& a = (--it)->second;
  if ((uintptr_t)p >= it->first + a.bytes) fail("work in memory that is not the plan's");
  if (a.device != device_of(s)) fail("memory of one device used on another");
  if (capturing[s]) fail("plan-owned memory used under capture");
  const Clock c = step(s);
  for (auto& u : a.uses) {
    auto k = c.find(u.first);
    if (k == c.end() || k->second < u.second) fail("two calls in the workspace at once");
  }
  a.uses[stream(s).id] = c.at(stream(s).id);
  ++work;
}
bool refused_now() { return mode != hipStreamCaptureModeRelaxed && [] {
    for (auto& c : capturing) if (c.second) return true;
    return false; }(); }
struct Event { Clock at; };
}  // namespace model
using namespace model;

extern "C" {
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = device_of(s); return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (refused_now()) return hipErrorStreamCaptureUnsupported;
  ++mallocs;
  if (n > limit) return hipErrorOutOfMemory;
  largest = std::max(largest, n);
  *p = (void*)next_address;
  memory[next_address] = Alloc{n, device, {}};
  next_address += (n + 4095) / 4096 * 4096;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  auto it = memory.find((uintptr_t)p);
  if (it == memory.end()) fail("freed twice or never allocated");
  for (auto& u : it->second.uses)
    if (host[u.first] < u.second) fail("memory freed while work in it may run");
  memory.erase(it);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t) new Event; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (!s && null_in_capture) return hipErrorStreamCaptureImplicit;
  ++events;
  ((Event*)e)->at = step(s);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { ++waits; merge(host, ((Event*)e)->at); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { ++waits; merge(host, stream(s).seen); return hipSuccess; }
hipError_t hipDeviceSynchronize() {
  ++waits;
  for (auto& s : streams) merge(host, s.second.seen);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  merge(stream(s).seen, ((Event*)e)->at);
  step(s);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  if (!s && null_in_capture) return hipErrorStreamCaptureImplicit;
  *st = capturing[s] ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, mode); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorName(hipError_t) { return ""; }
const char* hipGetErrorString(hipError_t) { return ""; }
// not reached by the scenarios
#define UNUSED(decl) hipError_t decl { fail(__func__); }
UNUSED(hipGraphDestroy(hipGraph_t)) UNUSED(hipGraphExecDestroy(hipGraphExec_t))
UNUSED(hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t))
UNUSED(hipGraphLaunch(hipGraphExec_t, hipStream_t)) UNUSED(hipHostFree(void*))
UNUSED(hipHostMalloc(void**, size_t, unsigned)) UNUSED(hipMemcpy(void*, const void*, size_t, hipMemcpyKind))
UNUSED(hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t))
UNUSED(hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode))
UNUSED(hipStreamCreateWithFlags(hipStream_t*, unsigned)) UNUSED(hipStreamDestroy(hipStream_t))
UNUSED(hipStreamEndCapture(hipStream_t, hipGraph_t*))
}

namespace xeng {
hipError_t launch_chan(const ChanArgs& a, bool, hipStream_t s) {
  if (!a.partial) ++direct;  // writes vis itself
  if (a.partial) use((char*)a.partial + 8LL * a.nslices * a.F * a.N * (a.N + 1) / 2 - 1, s);
  return hipSuccess;
}
hipError_t launch_small(const ChanArgs& a, bool f, hipStream_t s) { return launch_chan(a, f, s); }
int small_columns(int N) { return N <= 16 ? 16 : N <= 32 ? 32 : N <= 64 ? 64 : 128; }
hipError_t launch_chan_reduce(const int32_t* p, int32_t*, long long, int, bool, hipStream_t s) { use(p, s); return hipSuccess; }
hipError_t launch_pack(const PackArgs& a, bool, hipStream_t s) { use(a.packed, s); return hipSuccess; }
hipError_t launch_packed(const PackedArgs& a, hipStream_t s) { use(a.packed, s); return hipSuccess; }
hipError_t launch_tiles(const TileArgs&, int, bool, hipStream_t) { ++tiles; return hipSuccess; }
hipError_t launch_zero(int32_t*, long long, hipStream_t) { return hipSuccess; }
hipError_t launch_zero_tiles(int32_t*, int, int, int, int, int, hipStream_t) { return hipSuccess; }
#undef UNUSED
#define UNUSED(decl) hipError_t decl { fail(__func__); }
UNUSED(launch_batch(const BatchInst*, int, const BatchItem*, int, int*, int, int, bool, hipStream_t))
UNUSED(launch_beams(BeamArgs, int, bool, hipStream_t)) UNUSED(launch_flag_counts(const FlagArgs&, int, hipStream_t))
UNUSED(launch_flag_scan(const FlagArgs&, int, int, hipStream_t)) UNUSED(launch_gated(const GatedArgs&, int, bool, hipStream_t))
UNUSED(launch_noalloc_prep(const NoallocArgs&, hipStream_t))
UNUSED(launch_normalize(const int32_t*, const int32_t*, long long, double, float*, hipStream_t))
UNUSED(launch_shift_copy(const uint8_t*, uint8_t*, int, int, int, const int*, hipStream_t))
UNUSED(launch_wide(const TileArgs&, int, hipStream_t)) UNUSED(noalloc_workspace(unsigned char**, int*))
}  // namespace xeng

namespace {
struct Shape { int N, F, T; };
// sliced small arrays, the sliced channel kernel, the packed path
const Shape kShapes[] = {{40, 3, 8192}, {200, 2, 8192}, {704, 2, 11008}};
hipStream_t handle(int k) { return (hipStream_t)(uintptr_t)(0x1000 * k); }
uint8_t* const frame = (uint8_t*)0x10;
int32_t* const vis = (int32_t*)0x20;
struct Fixture {
  xeng_plan_t p = nullptr;
  Shape s;
  explicit Fixture(Shape shape, unsigned flags = 0) : s(shape) {
    if (xeng_plan(&p, s.N, s.F, s.T, flags) != XENG_OK) fail("plan");
  }
  // T samples on stream st: whether the call worked in plan-owned memory
  bool call(hipStream_t st, int T = 0) {
    const int w = work, t = tiles, d = direct;
    if (xeng_correlate(p, frame, s.N, s.F, T ? T : s.T, vis, st) != XENG_OK) fail("call refused");
    if (work == w && tiles == t && direct == d) fail("nothing launched");
    return work > w;
  }
};
void check(bool ok, const char* what) {
  if (!ok) fail(what);
}

void streams_in_turn(Shape s) {
  Fixture f(s);
  for (int k = 0; k < 3; ++k) check(f.call(nullptr), "workspace path expected");
  check(events == 0, "no events on the null stream");
  for (int k : {1, 2, 1, 0, 2, 2, 0, 1}) check(f.call(handle(k)), "workspace path expected");
  check(waits == 0 && mallocs == 1, "no host wait, one allocation");
}
void per_thread(Shape s) {
  Fixture f(s);
  for (int k = 0; k < 8; ++k) {
    thread = k % 2;
    check(f.call(hipStreamPerThread), "workspace path expected");
  }
  check(waits == 0, "no host wait");
}
void reused_handles(Shape s) {
  Fixture f(s);
  for (int k = 0; k < 4; ++k) {
    check(f.call(handle(1)), "workspace path expected");
    ++generation[handle(1)];
  }
}
void growth(Shape s) {
  for (hipStream_t st : {(hipStream_t) nullptr, handle(1)}) {
    Fixture f(s);
    f.call(st, s.T / 2);
    check(f.call(handle(2), s.T / 2), "workspace path expected");
    check(f.call(st), "workspace path expected");
    check(f.call(handle(3), s.T / 2), "workspace path expected");
  }
}
void refused(Shape s) {
  Fixture f(s);
  check(f.call(nullptr, s.T / 2), "workspace path expected");
  limit = 1;
  const int m = mallocs;
  for (int k = 0; k < 40; ++k) {
    check(!f.call(nullptr), "no memory, no workspace");
    check(f.call(nullptr, s.T / 2), "the plan keeps the workspace it has");
  }
  check(mallocs == m + 1, "a refusal is remembered");
  limit = 1ull << 40;
  bool again = false;
  for (int k = 0; k < 200 && !again; ++k) again = f.call(nullptr);
  check(again, "asked for again");
}
void captured(Shape s) {
  Fixture f(s);
  check(f.call(nullptr), "workspace path expected");
  capturing[handle(1)] = true;
  check(!f.call(handle(1)), "captured calls take no workspace");
  check(f.call(handle(2)), "beside a capture");
  Fixture g(s);
  check(g.call(handle(2)), "first call beside a capture");
  // a capture that includes the null stream: its order cannot be recorded now
  Fixture h(s);
  check(h.call(nullptr), "workspace path expected");
  null_in_capture = true;
  check(!h.call(handle(2)), "no order after the null stream");
  null_in_capture = false;
  check(h.call(handle(2)), "workspace path expected");
}
void two_devices(Shape s) {
  Fixture f(s);
  check(f.call(nullptr), "workspace path expected");
  device = 1;
  check(!f.call(nullptr), "not on another device");
  owner[handle(1)] = 0, owner[handle(2)] = 1;
  check(!f.call(handle(2)), "not on another device's stream");
  check(!f.call(handle(1)), "nor while another device is current");
  device = 0;
  check(f.call(handle(1)) && f.call(nullptr), "workspace path expected");
}
void last_segment(Shape) {
  // frames of several launches whose last one would take more slices than the
  // first, which takes one and no workspace; the plan has one from another call
  for (Shape s : {Shape{32, 438, 524288 + 515342}, Shape{65, 497, 524288 + 490511}}) {
    Fixture f(s);
    xeng_plan_set_tuning(f.p, 64, 0);
    check(f.call(handle(1), 8192), "workspace path expected");
    xeng_plan_set_tuning(f.p, 0, 0);
    f.call(handle(2));
    capturing[handle(2)] = true;
    f.call(handle(2));
    capturing[handle(2)] = false;
  }
}
void bounded_slices(Shape) {
  // a slice count that the plan names does not take memory without bound
  for (Shape s : {Shape{2048, 16, 32768}, Shape{128, 1024, 32768}}) {
    Fixture f(s);
    xeng_plan_set_tuning(f.p, 2, 0);
    check(f.call(nullptr), "workspace path expected");
    const size_t two = largest;
    xeng_plan_set_tuning(f.p, 64, 0);
    check(!f.call(nullptr), "tile kernels expected");
    check(largest == two, "no more memory");
  }
  // the channel kernel, named, and automatic counts as they were
  Fixture c({200, 64, 32768});
  xeng_plan_set_tuning(c.p, 4, 5);
  check(c.call(nullptr), "channel kernel expected");
  for (int N : {641, 769, 1090, 2048, 4096, 8192})
    for (int F : {1, 3, 16}) {
      Fixture f({N, F, 16384});
      largest = 0;
      f.call(nullptr);
      check(largest <= (4ull << 30) + (1ull << 30), "operands and partial blocks");
    }
}
void paths(Shape) {
  // the faster path of frames measured on both (packed: works in plan-owned memory)
  struct { Shape s; bool packed; } const frames[] = {
      {{2048, 16, 32768}, true}, {{1024, 16, 32768}, true}, {{1024, 1, 8192}, true},
      {{1090, 8, 20011}, true},  {{1281, 2, 2600}, true},   {{704, 16, 5504}, true},
      {{512, 16, 32768}, false}, {{768, 1, 8192}, false},   {{1426, 2, 1577}, false},
      {{1152, 25, 1728}, false}, {{976, 41, 2944}, false},  {{1472, 3, 1728}, false}};
  for (auto& c : frames) {
    Fixture f(c.s);
    if (f.call(nullptr) != c.packed) std::printf("N %d F %d T %d: ", c.s.N, c.s.F, c.s.T);
    check((work > 0) == c.packed, "the slower path");
    work = 0;
  }
  // FP8 frames of 129..256 inputs: tiles, or the channel kernel
  const unsigned f8 = XENG_FORM_F8, add = XENG_FORM_F8 | XENG_ACCUMULATE;
  struct { Shape s; unsigned flags; bool tiles; } const mid[] = {
      {{240, 56, 1843}, add, true}, {{208, 8, 273}, add, true},   {{240, 1, 205}, f8, true},
      {{160, 49, 441}, add, true},  {{256, 64, 32768}, f8, false}, {{200, 16, 65536}, f8, false},
      {{200, 8, 273}, XENG_FORM_I8, false}};
  for (auto& c : mid) {
    Fixture f(c.s, c.flags);
    tiles = 0;
    f.call(nullptr);
    if ((tiles > 0) != c.tiles) std::printf("N %d F %d T %d: ", c.s.N, c.s.F, c.s.T);
    check((tiles > 0) == c.tiles, "the slower path");
  }
}
void batches(Shape) {
  // the frames of a batch that run packed
  auto packs = [](std::vector<xeng_instance> b, unsigned flags = 0) {
    xeng_plan_t p = nullptr;
    check(xeng_plan_batch(&p, b.data(), (int)b.size(), flags) == XENG_OK, "batch plan");
    check(!p->rest || p->rest->large.empty(), "the others' own plan packs none");
    check(p->large.empty() || p->large.size() == b.size() || p->rest, "a plan of the others");
    return p->large;
  };
  typedef std::vector<int> L;
  check(packs({{2048, 4, 8192, 0}, {300, 2, 1000, 0}, {1537, 4, 13001, 0}, {128, 3, 129, 0}}) ==
            L{0, 2}, "large frames among small ones");
  check(packs({{64, 2, 300, 0}, {1536, 2, 20000, 0}, {1090, 1, 33000, 0}, {17, 1, 5, 0}}) == L{1},
        "few tiles");
  check(packs({{1537, 4, 13001, 0}}) == L{0}, "all of them");
  check(packs({{1537, 4, 13001, 2}}).empty(), "a named slice count");
  check(packs({{1537, 4, 13001, 0}}, XENG_ACCUMULATE | XENG_SHARED_VIS).empty(), "shared vis");
  // measured: 407 us by the persistent kernel alone, 568 with the first frame packed
  std::vector<xeng_instance> mixed = {{2048, 4, 8192, 0}, {2048, 4, 4096, 0}};
  for (int T : {2048, 2048}) mixed.push_back({1024, 4, T, 0});
  for (int T : {8192, 8192, 8192, 2048, 2048, 2048, 2048, 2048}) mixed.push_back({512, 4, T, 0});
  for (int N : {256, 128})
    for (int T : {8192, 4096}) mixed.push_back({N, 4, T, 0});
  check(packs(mixed).empty(), "frames that fill the chip together");
}
void one_shot(Shape) {
  // a plan that serves one call: no workspace that the call does not gain back
  struct { Shape s; bool workspace; } const calls[] = {
      {{16, 1, 4096}, true},     {{64, 4, 8192}, false},    {{64, 64, 65536}, true},
      {{128, 16, 16384}, false}, {{200, 4, 16384}, false},  {{200, 16, 65536}, true},
      {{1024, 4, 8192}, false},  {{2048, 16, 32768}, true}, {{1024, 1, 8192}, false}};
  for (auto& c : calls) {
    Fixture f(c.s), kept(c.s);
    xeng_plan_once(f.p);
    check(f.call(nullptr) == c.workspace, "one-shot rule");
    check(kept.call(nullptr), "kept plans take the workspace");
  }
}
}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, std::function<void(Shape)>> all = {
      {"streams_in_turn", streams_in_turn}, {"per_thread", per_thread},
      {"reused_handles", reused_handles},   {"growth", growth},
      {"refused", refused},                 {"captured", captured},
      {"two_devices", two_devices},         {"last_segment", last_segment},
      {"bounded_slices", bounded_slices},
      {"one_shot", one_shot},               {"paths", paths},
      {"batches", batches}};
  if (argc != 3 || !all.count(argv[1])) return 2;
  all.at(argv[1])(kShapes[std::atoi(argv[2])]);
  std::printf("ok\n");
  return 0;
}
