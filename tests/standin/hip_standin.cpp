// A CPU stand-in for the HIP runtime calls that the library makes, for tests
// of its host code: which tables, buffers and orderings its kernels meet.
//
// Device memory is host memory.  Work on a stream runs late: nothing that was
// enqueued runs before something waits for it, and then only what the waits
// on that stream and its events ask for, so a call that relies on another
// stream's work without waiting for it meets memory as it was before.
// Memory starts out filled with 0xCB.  A copy from pageable memory takes its
// data when it is enqueued, one from pinned memory when it runs, a captured
// one on every replay, as the HIP runtime does.
//
// The mover kernels are run by their meaning (the rectangles that the tasks
// of a launch name, copied), with every table index, pointer and offset
// checked against the memory that the test or the library allocated; anything
// out of place is reported by standin_faults().
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../../paper_2106_06601_amd/csrc/index_math.hpp"

using namespace costa;

namespace {

using Work = std::function<void()>;

struct Graph {
  std::vector<Work> nodes;
  std::vector<std::pair<void (*)(void*), void*>> objects;
};
struct Stream {
  std::deque<Work> queue;
  uint64_t queued = 0, done = 0;
  Graph* capture = nullptr;
};
struct Event {
  Stream* stream = nullptr;
  uint64_t upto = 0;
  bool captured = false;
};
struct Object {
  void (*destroy)(void*);
  void* data;
};

Stream null_stream;
std::set<Stream*> streams;
std::map<uintptr_t, size_t> memory;  // what kernels may touch: start -> bytes
std::map<uintptr_t, size_t> pinned;
std::map<const void*, std::string> kernels;
std::map<const void*, std::pair<size_t, void*>> symbols;
std::string faults;
hipError_t last = hipSuccess;
bool implicit_refused = false;  // a blocking stream captures: the null stream reports it

hipError_t err(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
void fault(const std::string& what) {
  if (faults.size() < 4000) faults += what + "\n";
}
Stream& at(hipStream_t s) { return s ? *reinterpret_cast<Stream*>(s) : null_stream; }
bool any_capture() {
  for (Stream* s : streams)
    if (s->capture) return true;
  return false;
}
void add(Stream& s, Work w) {
  if (s.capture) {
    s.capture->nodes.push_back(std::move(w));
  } else {
    s.queue.push_back(std::move(w));
    ++s.queued;
  }
}
void run_to(Stream& s, uint64_t upto) {
  while (s.done < upto && !s.queue.empty()) {
    Work w = std::move(s.queue.front());
    s.queue.pop_front();
    ++s.done;
    w();
  }
}
void run_all() {
  run_to(null_stream, null_stream.queued);
  for (Stream* s : streams) run_to(*s, s->queued);
}
bool holds(const std::map<uintptr_t, size_t>& m, const void* p, size_t n) {
  const uintptr_t a = (uintptr_t)p;
  auto it = m.upper_bound(a);
  if (it == m.begin()) return false;
  --it;
  return a >= it->first && a + n <= it->first + it->second;
}
void* fresh(size_t n) {
  void* p = aligned_alloc(256, (n + 255) / 256 * 256);
  std::memset(p, 0xCB, n);
  return p;
}

// One rectangle, by its meaning (copies only).
void move_piece(const Piece& p, const unsigned char* table, size_t nbufs, int es) {
  if (p.src_buf < 0 || p.dst_buf < 0 || (size_t)p.src_buf >= nbufs || (size_t)p.dst_buf >= nbufs || p.nx < 1 || p.ny < 1)
    return fault("a rectangle of no plan: buffers " + std::to_string(p.src_buf) + ", " + std::to_string(p.dst_buf));
  char* bufs[2];
  std::memcpy(&bufs[0], table + (size_t)p.src_buf * sizeof(void*), sizeof(void*));
  std::memcpy(&bufs[1], table + (size_t)p.dst_buf * sizeof(void*), sizeof(void*));
  for (int64_t y = 0; y < p.ny; ++y)
    for (int64_t x = 0; x < p.nx; ++x) {
      const int64_t so = (p.flags & PIECE_TRANSPOSE) ? x * p.src_ld + y : y * p.src_ld + x;
      const char* src = bufs[0] + (p.src_off + so) * es;
      char* dst = bufs[1] + (p.dst_off + y * p.dst_ld + x) * es;
      if (!holds(memory, src, es) || !holds(memory, dst, es)) return fault("an element outside every buffer");
      std::memcpy(dst, src, es);
    }
}

void move_tasks(const std::string& name, const ArgTable& args, const Piece* pieces, const int32_t* tasks, int64_t n,
                const void* device_table, int32_t items_off) {
  const size_t at = name.find("costa_mover") != std::string::npos ? name.find("costa_mover") : name.find("costa_tiles");
  const char* t = name.c_str() + at + 11;  // the template's arguments: I<scalar>Lb<complex>E...
  const int es = (t[1] == 'd' ? 8 : 4) * (t[4] == '1' ? 2 : 1);
  const unsigned char* table = device_table ? static_cast<const unsigned char*>(device_table) : args.bytes;
  if (device_table && !holds(memory, device_table, (size_t)items_off)) return fault("a call table outside every buffer");
  if (!holds(memory, tasks, (size_t)n * sizeof(int32_t))) return fault("a task table outside every buffer");
  std::set<int32_t> moved;
  for (int64_t b = 0; b < n; ++b) {
    int32_t pi = tasks[b];
    if (pi < 0 || !moved.insert(pi).second) continue;
    for (int left = 1; left > 0; --left, ++pi) {
      if (!holds(memory, pieces + pi, sizeof(Piece))) return fault("a task of no rectangle: " + std::to_string(pi));
      const Piece& p = pieces[pi];
      if (p.flags & PIECE_GROUP_NEXT) ++left;
      if ((p.flags & PIECE_STACK) && pi == tasks[b]) left = stack_size_of(p.flags);
      move_piece(p, table, (size_t)items_off / sizeof(void*), es);
    }
  }
}

// The volume kernel: its own count of overlaps, by one lane.
void volume(const VolumeDealtArgs& a) {
  std::vector<unsigned long long> h(a.nhist, 0);
  for (const VolumeAxis& x : a.axis) {
    auto add = [&](int32_t e, unsigned long long n) { h[x.hist0 + e] += n; };
    for (const VolumeSide* q : {&x.fine, &x.coarse})
      if (a.narrow && q->blk != (int64_t)(uint32_t)q->blk) return fault("a block size that its type does not hold");
    if (a.narrow) count_overlaps<uint32_t>(x, 0, 1, add);
    else count_overlaps<uint64_t>(x, 0, 1, add);
  }
  const VolumeAxis *r = &a.axis[0], *c = &a.axis[1];
  const int16_t *ca = a.cls, *cb = a.cls + 2 * a.P;
  for (int32_t s = 0; s < a.P; ++s)
    for (int32_t t = 0; t < a.P; ++t)
      a.V[(size_t)s * a.P + t] = ca[2 * t] < 0 || cb[2 * s] < 0 ? 0
                                 : h[r->hist0 + cb[2 * s] * r->nclass + ca[2 * t]] *
                                       h[c->hist0 + cb[2 * s + 1] * c->nclass + ca[2 * t + 1]];
}

template <typename T>
T arg(void** args, int k) {
  T v;
  std::memcpy(&v, args[k], sizeof v);
  return v;
}

}  // namespace

// ---- what the tests call -----------------------------------------------------
extern "C" {
void* standin_stream() {
  Stream* s = new Stream();
  streams.insert(s);
  return s;
}
void standin_capture(void* s) { static_cast<Stream*>(s)->capture = new Graph(); }
void* standin_end_capture(void* s) {
  Graph* g = static_cast<Stream*>(s)->capture;
  static_cast<Stream*>(s)->capture = nullptr;
  return g;
}
void standin_replay(void* g, void* s) {
  for (const Work& w : static_cast<Graph*>(g)->nodes) add(at((hipStream_t)s), w);
}
int standin_nodes(void* g) { return (int)static_cast<Graph*>(g)->nodes.size(); }
void standin_destroy_graph(void* g) {
  for (auto& o : static_cast<Graph*>(g)->objects) o.first(o.second);
  delete static_cast<Graph*>(g);
}
void standin_run(void* s) { run_to(at((hipStream_t)s), at((hipStream_t)s).queued); }
// memory of the test (earlier buffers that it overlaps are gone)
void standin_buffer(void* p, size_t n) {
  const uintptr_t a = (uintptr_t)p;
  for (auto it = memory.begin(); it != memory.end();)
    it = it->first < a + n && a < it->first + it->second ? memory.erase(it) : std::next(it);
  if (n) memory[a] = n;
}
// Elements that one lane of the volume kernel counts on an axis of n blocks of
// one element each, or -1 where it leaves its range.
int64_t standin_lane_volume(int32_t n, int32_t first, int32_t step) {
  VolumeAxis x{};
  x.n = n;
  x.fine = VolumeSide{0, 1, 1, 0};
  x.coarse = VolumeSide{0, n, 1, 0};
  x.nblocks = n;
  x.nclass = 1;
  int64_t sum = 0, rounds = 0;
  struct Left {};
  try {
    count_overlaps<uint32_t>(x, first, step, [&](int32_t, unsigned long long e) {
      sum += (int64_t)e;
      if (++rounds > n / step + 1) throw Left();
    });
  } catch (const Left&) {
    return -1;
  }
  return sum;
}
// The kernels' index arithmetic (index_math.hpp).
void standin_divmod(int ulps, const int32_t* u, const int32_t* n, int32_t* y, int32_t* x, int64_t count) {
  reciprocal_ulps = ulps;
  for (int64_t i = 0; i < count; ++i) divmod(u[i], n[i], y[i], x[i]);
  reciprocal_ulps = 0;
}
void standin_xcd_order(int32_t n, int32_t run, int32_t* out) {
  for (int32_t b = 0; b < n; ++b) out[b] = xcd_order(b, n, run);
}
void standin_tile_walk(int32_t lanes, int32_t tid, int32_t len, int64_t ld, int32_t ls, int32_t lc, int32_t steps,
                       int64_t* off, int32_t* slot) {
  auto walk = [&](auto w) {
    for (int32_t k = 0; k < steps; ++k, w.next()) {
      off[k] = w.off;
      slot[k] = w.lds;
    }
  };
  if (lanes == kSmallTileLanes) walk(TileWalk<kSmallTileLanes>(tid, len, ld, ls, lc));
  else walk(TileWalk<kThreadsPerTask>(tid, len, ld, ls, lc));
}
void standin_refuse_implicit(int on) { implicit_refused = on != 0; }
const char* standin_faults() {
  static std::string out;
  out.swap(faults);
  faults.clear();
  return out.c_str();
}

// ---- what the library calls --------------------------------------------------
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
const char* hipGetErrorString(hipError_t e) {
  return e == hipErrorStreamCaptureUnsupported ? "not permitted while a stream captures" : "error";
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipMalloc(void** p, size_t n) {
  if (any_capture()) return err(hipErrorStreamCaptureUnsupported);
  *p = fresh(n);
  memory[(uintptr_t)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  run_all();
  memory.erase((uintptr_t)p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (any_capture()) return err(hipErrorStreamCaptureUnsupported);
  *p = fresh(n);
  memory[(uintptr_t)*p] = pinned[(uintptr_t)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  run_all();
  memory.erase((uintptr_t)p);
  pinned.erase((uintptr_t)p);
  free(p);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = (size_t)1 << 38;
  return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
  if (any_capture()) return err(hipErrorStreamCaptureUnsupported);
  run_to(null_stream, null_stream.queued);
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind kind, hipStream_t stream) {
  Stream& s = at(stream);
  if (kind != hipMemcpyHostToDevice || s.capture || holds(pinned, src, n)) {
    add(s, [=] { std::memcpy(dst, src, n); });
  } else {
    std::vector<char> data((const char*)src, (const char*)src + n);
    add(s, [dst, data] { std::memcpy(dst, data.data(), data.size()); });
  }
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  if (any_capture()) return err(hipErrorStreamCaptureUnsupported);
  run_all();
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t stream) {
  if (at(stream).capture) return err(hipErrorStreamCaptureUnsupported);
  standin_run(stream);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t stream, hipStreamCaptureStatus* st) {
  if (!stream && implicit_refused) return err(hipErrorStreamCaptureImplicit);
  *st = at(stream).capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamGetCaptureInfo_v2(hipStream_t stream, hipStreamCaptureStatus* st, unsigned long long* id,
                                      hipGraph_t* graph, const hipGraphNode_t** deps, size_t* ndeps) {
  *st = at(stream).capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  if (id) *id = 1;
  if (graph) *graph = reinterpret_cast<hipGraph_t>(at(stream).capture);
  if (deps) *deps = nullptr;
  if (ndeps) *ndeps = 0;
  return hipSuccess;
}
hipError_t hipUserObjectCreate(hipUserObject_t* o, void* data, hipHostFn_t destroy, unsigned, unsigned) {
  *o = reinterpret_cast<hipUserObject_t>(new Object{destroy, data});
  return hipSuccess;
}
hipError_t hipUserObjectRelease(hipUserObject_t u, unsigned) {
  Object* o = reinterpret_cast<Object*>(u);
  o->destroy(o->data);
  delete o;
  return hipSuccess;
}
hipError_t hipGraphRetainUserObject(hipGraph_t g, hipUserObject_t u, unsigned, unsigned) {
  Object* o = reinterpret_cast<Object*>(u);
  reinterpret_cast<Graph*>(g)->objects.push_back({o->destroy, o->data});
  delete o;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = reinterpret_cast<hipEvent_t>(new Event());
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t ev, hipStream_t stream) {
  Event& e = *reinterpret_cast<Event*>(ev);
  Stream& s = at(stream);
  e.captured = s.capture != nullptr;
  e.stream = &s;
  e.upto = s.queued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t ev) {
  Event& e = *reinterpret_cast<Event*>(ev);
  if (any_capture() || e.captured) return err(hipErrorStreamCaptureUnsupported);
  if (e.stream) run_to(*e.stream, e.upto);
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t stream, hipEvent_t ev, unsigned) {
  const Event e = *reinterpret_cast<Event*>(ev);
  Stream& s = at(stream);
  if (s.capture && !e.captured) return err(hipErrorStreamCaptureIsolation);
  if (!s.capture && e.captured) return err(hipErrorCapturedEvent);
  if (e.stream && !e.captured) add(s, [e] { run_to(*e.stream, e.upto); });
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol) {
  auto& s = symbols[symbol];
  if (!s.second) {
    s.second = fresh(s.first);
    memory[(uintptr_t)s.second] = s.first;
  }
  *p = s.second;
  return hipSuccess;
}

static thread_local struct {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
} config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  config = {grid, block, shmem, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* stream) {
  *grid = config.grid;
  *block = config.block;
  *shmem = config.shmem;
  *stream = config.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, dim3*, dim3*,
                           int*) {
  kernels[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { symbols[var] = {size, nullptr}; }

hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t stream) {
  const std::string name = kernels[f];
  if (name.find("costa_mover") != std::string::npos || name.find("costa_tiles") != std::string::npos) {
    const ArgTable table = arg<ArgTable>(args, 0);
    const Piece* pieces = arg<const Piece*>(args, 1);
    const int32_t* tasks = arg<const int32_t*>(args, 2) + arg<int32_t>(args, 3);
    const void* device_table = arg<const void*>(args, 4);
    const int32_t items_off = arg<int32_t>(args, 5);
    add(at(stream), [=] { move_tasks(name, table, pieces, tasks, (int64_t)grid.x, device_table, items_off); });
  } else if (name.find("costa_store_table") != std::string::npos) {
    const ArgTable table = arg<ArgTable>(args, 0);
    void* dst = arg<void*>(args, 1);
    const size_t n = (size_t)arg<int32_t>(args, 2) * 16;
    add(at(stream), [=] {
      if (n > sizeof table || !holds(memory, dst, n)) return fault("a stored table outside every buffer");
      std::memcpy(dst, table.bytes, n);
    });
  } else if (name.find("costa_volume_dealt") != std::string::npos) {
    const VolumeDealtArgs a = arg<VolumeDealtArgs>(args, 0);
    add(at(stream), [=] { volume(a); });
  } else {
    fault("a kernel that the stand-in does not run: " + name);
  }
  return hipSuccess;
}
}
