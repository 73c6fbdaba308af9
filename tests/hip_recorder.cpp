// A HIP runtime that runs nothing: the host entry points libhelm.so calls, with a memory budget
// per device, failures on request and a record of what was called, so that the library's
// handling of memory, streams and errors can be tested without a GPU.  Loaded with its symbols
// global before libhelm.so, it answers in place of libamdhip64.  Small copies and fills are
// done (host memory stands for the devices'), large ones and kernels are not.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <sys/mman.h>

namespace {
constexpr int NDEV = 2, OOM = 2, BAD = 400;
constexpr size_t SMALL = 1 << 20;
struct Block { size_t size; int dev; };
std::recursive_mutex mu;
std::map<void*, Block> blocks;
std::set<void*> dead_streams;
size_t room[NDEV] = {(size_t)64 << 30, (size_t)64 << 30};
long fail_launch = -1;        // launches until hipGetLastError reports one failed
long fail_malloc = -1;        // allocations until one fails (the budget apart)
thread_local long fail_new = 0;   // host allocations of this thread that fail from here on
int last_error = 0;
std::string log_text;
bool logging = false;
size_t handles = 0x1000;
long launches = 0;
std::map<void*, long> at_launch;   // kernels launched before an event was recorded
thread_local int cur = 0;
void* captured_stream = nullptr;

void note(const char* what, const void* p, size_t n = 0) {
    if (!logging) return;
    char b[128];
    std::snprintf(b, sizeof b, "%s %zx %zu %d\n", what, (size_t)p, n, cur);
    log_text += b;
}
#define LOCK std::lock_guard<std::recursive_mutex> lk(mu)
void* fresh() { return (void*)(handles += 16); }
}  // namespace

void* operator new(size_t n) {
    if (fail_new > 0) { --fail_new; throw std::bad_alloc(); }
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
// ---- the test's side
void rec_fail_new(long n) { fail_new = n; }
void rec_budget(int dev, size_t bytes) { LOCK; room[dev] = bytes; }
size_t rec_room(int dev) { LOCK; return room[dev]; }
size_t rec_live(int dev) {
    LOCK;
    size_t n = 0;
    for (auto& b : blocks) n += b.second.dev == dev ? b.second.size : 0;
    return n;
}
void rec_kill_stream(void* s) { LOCK; dead_streams.insert(s); }
void rec_capture(void* s) { LOCK; captured_stream = s; }
void rec_fail_launch(long n) { LOCK; fail_launch = n; }
void rec_fail_malloc(long n) { LOCK; fail_malloc = n; }
void rec_log(int on) { LOCK; logging = on != 0; if (on) log_text.clear(); }
size_t rec_log_size() { LOCK; return log_text.size(); }
void rec_log_text(char* out, size_t n) { LOCK; std::memcpy(out, log_text.data(), n); }

// ---- memory
int hipMalloc(void** p, size_t n) {
    LOCK;
    if (fail_malloc == 0 || n > room[cur]) {
        if (fail_malloc == 0) fail_malloc = -1;
        note("nomem", nullptr, n);
        return last_error = OOM;
    }
    if (fail_malloc > 0) --fail_malloc;
    void* q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED) return last_error = OOM;
    room[cur] -= n;
    blocks[q] = Block{n, cur};
    note("malloc", q, n);
    *p = q;
    return 0;
}
int hipFree(void* p) {
    LOCK;
    auto it = blocks.find(p);
    if (it == blocks.end()) return p ? BAD : 0;
    note("free", p, it->second.size);
    room[it->second.dev] += it->second.size;
    munmap(p, it->second.size);
    blocks.erase(it);
    return 0;
}
int hipMemGetInfo(size_t* f, size_t* t) { LOCK; *f = room[cur]; *t = (size_t)288 << 30; return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { if (n <= SMALL) std::memmove(d, s, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) { if (n <= SMALL) std::memmove(d, s, n); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void*) { if (n <= SMALL) std::memset(d, v, n); return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char a[256]; *p = a; return 0; }

// ---- devices, errors
int hipGetDevice(int* d) { *d = cur; return 0; }
int hipSetDevice(int d) {
    if (d < 0 || d >= NDEV) return BAD;
    cur = d;
    return 0;
}
int hipDeviceSynchronize() { LOCK; note("devsync", nullptr); return 0; }
int hipGetLastError() { LOCK; int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int) { return "recorded"; }

// ---- streams, events, graphs
int hipStreamCreateWithFlags(void** s, unsigned) { LOCK; *s = fresh(); note("newstream", *s); return 0; }
int hipStreamDestroy(void* s) { LOCK; note("delstream", s); dead_streams.insert(s); return 0; }
int hipStreamSynchronize(void* s) {
    LOCK;
    if (dead_streams.count(s)) return BAD;
    note("sync", s);
    return 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) { LOCK; note("wait", s, (size_t)e); return 0; }
int hipEventCreate(void** e) { LOCK; *e = fresh(); return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { LOCK; *e = fresh(); return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void* e, void* s) { LOCK; note("record", s, (size_t)e); at_launch[e] = launches; return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* t, void* a, void* b) {    // a millisecond a kernel
    LOCK;
    *t = (float)(at_launch[b] - at_launch[a]);
    return 0;
}
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g) { *g = fresh(); return 0; }
int hipStreamIsCapturing(void* s, int* c) { LOCK; *c = s && s == captured_stream; return 0; }
int hipGraphInstantiate(void** x, void*, void**, char*, size_t) { *x = fresh(); return 0; }
int hipGraphLaunch(void*, void* s) { LOCK; note("launch", s); return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }

// ---- kernels
struct Dim { unsigned x, y, z; };
static thread_local void* launch_stream;
int __hipPushCallConfiguration(Dim, Dim, size_t, void* s) { launch_stream = s; return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* n, void** s) {
    *g = Dim{1, 1, 1};
    *b = Dim{1, 1, 1};
    *n = 0;
    *s = launch_stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim, Dim, void**, size_t, void* s) {
    LOCK;
    note("launch", s, (size_t)f);
    ++launches;
    if (fail_launch == 0) { last_error = BAD; fail_launch = -1; return BAD; }
    if (fail_launch > 0) --fail_launch;
    return 0;
}
void** __hipRegisterFatBinary(const void*) { static void* h[4]; return h; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
}
