// A model of the HIP runtime for tests of libtr.so's host side without a GPU:
// loaded before the library, it answers every runtime call the library makes.
// No kernel runs and nothing enqueued ever ends by itself: work is complete
// only once a call that waits for it has returned.  Device memory is zeroed
// host memory, copies are made at once.  What it checks and counts:
//   - launches of 2^32 work-items and more per dimension, and empty ones, are
//     refused, as the runtime refuses them;
//   - accesses of job tables (k_put_jobs and copies write them, k_render_wave
//     reads them) that nothing orders: no stream, event or wait between them;
//   - per device, work that nothing has waited for, bytes allocated, capacity;
//   - waits on events during a capture, and on events recorded in one.
#include <dlfcn.h>
#include <sys/mman.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <condition_variable>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#define API extern "C" __attribute__((visibility("default")))

namespace {
constexpr int kOk = 0, kInvalid = 1, kOutOfMemory = 2, kBadConfig = 9, kNotReady = 600, kInCapture = 900,
              kCapturedEvent = 907;
struct Dim3 { uint32_t x, y, z; };
typedef std::map<int, long> Clock;  // real stream -> its last operation known to be ordered before

struct Region { size_t size; int dev; };
struct Stream { int dev = 0; Clock at; long n = 0; };
struct Event { bool recorded = false, captured = false; Clock at; };
struct Access { int stream; long id; bool write; };

std::recursive_mutex mu;
std::map<uintptr_t, Region> mem;
size_t used[2], peak[2], capacity[2] = {~(size_t)0, ~(size_t)0};
long mallocs, frees, races, launches, bad_waits, misuse;
std::map<std::pair<uintptr_t, int>, int> real;  // (handle, host thread for the per-thread one)
std::vector<Stream> streams;
std::map<uintptr_t, std::vector<Access>> tables;  // job table -> accesses
std::map<const void *, std::string> names;
std::map<uintptr_t, bool> capturing;
std::vector<std::string> log_;
int fail_sync, fail_new = -1;
int n_threads;
thread_local int device, last_error, tid = -1;
thread_local Clock host;  // what this thread has waited for
thread_local struct { Dim3 g, b; size_t sh; void *st; } cfg;
int hold;  // 1: the next copy is held, 2: one is
std::condition_variable_any held;
long staged_changed;
double radius;

void merge(Clock &a, const Clock &b) { for (auto &k : b) if (a[k.first] < k.second) a[k.first] = k.second; }
bool covers(const Clock &a, int s, long id) { auto i = a.find(s); return i != a.end() && i->second >= id; }
int real_of(void *st) {
  if (tid < 0) tid = n_threads++;
  const uintptr_t h = (uintptr_t)st;
  const auto key = std::make_pair(h, h == 2 ? tid : -1);
  auto it = real.find(key);
  if (it == real.end()) {
    streams.push_back(Stream());
    streams.back().dev = device;
    it = real.emplace(key, (int)streams.size() - 1).first;
  }
  return it->second;
}
long enqueue(void *st, int &s) {
  s = real_of(st);
  Stream &S = streams[s];
  S.dev = device;
  merge(S.at, host);
  return S.at[s] = ++S.n;
}
void touch(uintptr_t table, int s, long id, bool write) {
  for (const Access &a : tables[table])
    if ((a.write || write) && !covers(streams[s].at, a.stream, a.id)) ++races;
  tables[table].push_back(Access{s, id, write});
}
int fail(int e) { return last_error = e; }
}  // namespace

// ---- controls for the tests
API void model_capacity(int dev, size_t bytes) { capacity[dev] = bytes; }
API size_t model_used(int dev) { return used[dev]; }
API long model_races() { return races; }
API long model_launches() { return launches; }
API long model_bad_waits() { return bad_waits; }
API long model_misuse() { return misuse; }
API long model_frees() { return frees; }
API long model_mallocs() { return mallocs; }
API void model_radius(double r) { radius = r; }  // of the scenes built from now on, about the origin
API void model_fail_sync(int on) { fail_sync = on; }
API void model_fail_new(int after) { fail_new = after; }  // the one after so many; -1 none
API int model_failed_new() { return fail_new < 0; }
API void model_capture(void *st, int on) { capturing[(uintptr_t)st] = on != 0; }
API void model_hold_copy() { std::lock_guard<std::recursive_mutex> l(mu); hold = 1; }
API void model_await_held() { std::unique_lock<std::recursive_mutex> l(mu); held.wait(l, [] { return hold == 2; }); }
API void model_release_copy() { std::lock_guard<std::recursive_mutex> l(mu); hold = 0; held.notify_all(); }
API long model_staged_changed() { return staged_changed; }
API long model_pending(int dev) {  // operations of the device that this thread has not waited for
  std::lock_guard<std::recursive_mutex> l(mu);
  long n = 0;
  for (size_t s = 0; s < streams.size(); ++s)
    if (streams[s].dev == dev && !covers(host, (int)s, streams[s].n)) ++n;
  return n;
}
API int model_log(int i, char *out, int cap) {  // the i-th launch as "name grid block", its length or -1
  if (i < 0 || i >= (int)log_.size()) return -1;
  std::snprintf(out, cap, "%s", log_[i].c_str());
  return (int)log_[i].size();
}

void *operator new(size_t n) {
  Dl_info who;  // (only the library's own allocations count and fail)
  if (fail_new >= 0 && dladdr(__builtin_return_address(0), &who) && std::strstr(who.dli_fname, "libtr.so") && fail_new-- == 0)
    throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

// ---- the runtime
API int hipGetDevice(int *d) { *d = device; return kOk; }
API int hipSetDevice(int d) { if (d < 0 || d > 1) return fail(101); device = d; return kOk; }
API int hipGetDevicePropertiesR0600(void *, int) { return kInvalid; }  // (the library's default)
API int hipGetLastError() { const int e = last_error; last_error = kOk; return e; }
API const char *hipGetErrorString(int) { return "error of the runtime model"; }
API const char *hipGetErrorName(int) { return "hipModelError"; }

API int hipMalloc(void **p, size_t n) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (used[device] + n > capacity[device]) return fail(kOutOfMemory);
  void *q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (q == MAP_FAILED) return fail(kOutOfMemory);
  mem[(uintptr_t)q] = Region{n, device};
  used[device] += n;
  ++mallocs;
  *p = q;
  return kOk;
}
API int hipFree(void *p) {
  if (!p) return kOk;
  std::lock_guard<std::recursive_mutex> l(mu);
  auto it = mem.find((uintptr_t)p);
  if (it == mem.end()) { ++misuse; return fail(kInvalid); }
  for (auto &s : streams) if (s.dev == it->second.dev) merge(host, s.at);  // (waits for the device)
  used[it->second.dev] -= it->second.size;
  tables.erase((uintptr_t)p);
  munmap(p, it->second.size);
  mem.erase(it);
  ++frees;
  return kOk;
}
API int hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return *p ? kOk : fail(kOutOfMemory); }
API int hipHostFree(void *p) { std::free(p); return kOk; }

API int hipDeviceSynchronize() {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (fail_sync) return fail(kInCapture);
  for (auto &s : streams) if (s.dev == device) merge(host, s.at);
  return kOk;
}
API int hipStreamCreateWithFlags(void **s, unsigned) { *s = std::malloc(16); return kOk; }
API int hipStreamDestroy(void *) { return kOk; }
API int hipStreamBeginCapture(void *s, int) { capturing[(uintptr_t)s] = true; return kOk; }
API int hipStreamEndCapture(void *s, void **g) { capturing[(uintptr_t)s] = false; *g = (void *)16; return kOk; }
API int hipStreamIsCapturing(void *s, int *c) { *c = capturing[(uintptr_t)s] ? 1 : 0; return kOk; }
API int hipGraphInstantiate(void **e, void *, void *, char *, size_t) { *e = (void *)16; return kOk; }
API int hipGraphDestroy(void *) { return kOk; }
API int hipGraphExecDestroy(void *) { return kOk; }
API int hipGraphLaunch(void *, void *st) { int s; std::lock_guard<std::recursive_mutex> l(mu); enqueue(st, s); return kOk; }
API int hipStreamSynchronize(void *st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  if (capturing[(uintptr_t)st]) { ++bad_waits; return fail(kInCapture); }
  merge(host, streams[real_of(st)].at);
  return kOk;
}

API int hipEventCreateWithFlags(void **e, unsigned) { *e = new Event(); return kOk; }
API int hipEventCreate(void **e) { *e = new Event(); return kOk; }
API int hipEventDestroy(void *e) { delete (Event *)e; return kOk; }
API int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return kOk; }
API int hipEventRecord(void *ev, void *st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  Event &E = *(Event *)ev;
  int s;
  enqueue(st, s);
  E.recorded = true;
  E.captured = capturing[(uintptr_t)st];
  E.at = streams[s].at;
  return kOk;
}
static int wait_ok(const Event &E) {
  for (auto &c : capturing) if (c.second) { ++bad_waits; return fail(kInCapture); }
  if (E.captured) { ++bad_waits; return fail(kCapturedEvent); }
  return kOk;
}
API int hipEventSynchronize(void *ev) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const Event &E = *(Event *)ev;
  const int e = wait_ok(E);
  if (e == kOk) merge(host, E.at);
  return e;
}
API int hipEventQuery(void *ev) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const Event &E = *(Event *)ev;
  const int e = wait_ok(E);
  if (e != kOk) return e;
  for (auto &k : E.at) if (!covers(host, k.first, k.second)) return kNotReady;
  return kOk;
}
API int hipStreamWaitEvent(void *st, void *ev, unsigned) {
  std::lock_guard<std::recursive_mutex> l(mu);
  merge(streams[real_of(st)].at, ((Event *)ev)->at);
  return kOk;
}

API int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *st) {
  std::unique_lock<std::recursive_mutex> l(mu);
  int r;
  const long id = enqueue(st, r);
  if (tables.count((uintptr_t)d)) touch((uintptr_t)d, r, id, true);
  if (hold == 1) {  // this copy waits for its release: its source must not change meanwhile
    hold = 2;
    held.notify_all();
    std::vector<char> before((const char *)s, (const char *)s + n);
    held.wait(l, [] { return hold == 0; });
    if (std::memcmp(before.data(), s, n)) ++staged_changed;
  }
  std::memcpy(d, s, n);
  return kOk;
}
API int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return kOk; }

API int hipLaunchKernel(const void *f, Dim3 g, Dim3 b, void **args, size_t, void *st) {
  std::lock_guard<std::recursive_mutex> l(mu);
  const uint64_t x = (uint64_t)g.x * b.x, y = (uint64_t)g.y * b.y;
  if (!x || !y || x > UINT32_MAX || y > UINT32_MAX || (uint64_t)b.x * b.y * b.z > 1024) return fail(kBadConfig);
  int s;
  const long id = enqueue(st, s);
  ++launches;
  const std::string &n = names[f];
  log_.push_back(n + " " + std::to_string(g.x) + " " + std::to_string(b.x));
  // (what the host reads of a grid build: no references, and the bounding radius)
  if (n.find("k_cell_scan") != std::string::npos) std::memcpy(*(char **)args[8] + 8, &radius, 8);
  if (n.find("k_put_jobs") != std::string::npos) touch(*(uintptr_t *)args[1], s, id, true);
  if (n.find("k_render_wave") != std::string::npos) touch(*(uintptr_t *)args[0], s, id, false);
  if (n.find("k_tga_offsets") != std::string::npos) {
    touch(*(uintptr_t *)args[2], s, id, true);
    **(int64_t **)args[4] = 0;  // (the file's size)
  }
  if (n.find("k_tga_rowsILb1E") != std::string::npos) touch(*(uintptr_t *)args[4], s, id, false);
  if (n.find("k_aa_mean") != std::string::npos) {  // (stands for the renders into the planes too)
    const uintptr_t planes = *(uintptr_t *)args[1];
    auto it = mem.upper_bound(planes);
    if (it == mem.begin() || planes >= std::prev(it)->first + std::prev(it)->second.size) ++misuse;
    touch(planes, s, id, true);
  }
  return kOk;
}
API int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t sh, void *st) { cfg.g = g; cfg.b = b; cfg.sh = sh; cfg.st = st; return kOk; }
API int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *sh, void **st) { *g = cfg.g; *b = cfg.b; *sh = cfg.sh; *st = cfg.st; return kOk; }
API void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
API void __hipUnregisterFatBinary(void **) {}
API void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names[f] = name; }
API void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
API int hipGetSymbolAddress(void **p, const void *) { static char buf[1 << 20]; *p = buf; return kOk; }
