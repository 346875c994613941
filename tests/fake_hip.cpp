// A HIP runtime without a device, for CPU tests of the library's host code: device memory is host
// memory, streams and events do nothing, and a kernel launch only writes the kernel's name to a
// log.  Loaded with global symbols before the library, its functions take the place of the
// runtime's.
#include <cstddef>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {
struct Dim3 { unsigned x, y, z; };
std::map<const void *, std::string> &names()
{
    static auto *m = new std::map<const void *, std::string>();
    return *m;
}
struct Config { Dim3 grid, block; size_t lds; void *stream; };
std::vector<Config> &configs()
{
    static thread_local std::vector<Config> v;
    return v;
}
std::string &calls()
{
    static auto *s = new std::string();
    return *s;
}
int fail_mallocs_from = -1;          // hipMalloc fails from this one on (counted down; -1: never)
float (*elapsed_cb)() = nullptr;
void (*launch_cb)(const char *, void **) = nullptr;
std::mutex mu;
void note(const std::string &s)
{
    std::lock_guard<std::mutex> lock(mu);
    calls() += s + "\n";
}
void *block(size_t n) { return std::calloc(1, n ? n : 1); }
constexpr int kOutOfMemory = 2;
}  // namespace

extern "C" {
// the test's side
const char *fake_calls() { return calls().c_str(); }
void fake_clear() { calls().clear(); }
void fake_fail_mallocs_from(int n) { fail_mallocs_from = n; }
void fake_on_elapsed(float (*f)()) { elapsed_cb = f; }
void fake_on_launch(void (*f)(const char *, void **)) { launch_cb = f; }

// registration and launches
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    names()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterManagedVar(void *, void **, void *, const char *, size_t, unsigned) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t lds, void *st)
{
    configs().push_back({g, b, lds, st});
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *lds, void **st)
{
    const Config c = configs().back();
    configs().pop_back();
    *g = c.grid; *b = c.block; *lds = c.lds; *st = c.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 g, Dim3, void **args, size_t, void *)
{
    note("launch " + names()[f] + " grid " + std::to_string(g.x) + " " + std::to_string(g.y) + " " + std::to_string(g.z));
    if (launch_cb) launch_cb(names()[f].c_str(), args);
    return 0;
}

// memory
int hipMalloc(void **p, size_t n)
{
    if (fail_mallocs_from == 0) return kOutOfMemory;
    if (fail_mallocs_from > 0) --fail_mallocs_from;
    note("malloc " + std::to_string(n));
    *p = block(n);
    return 0;
}
int hipFree(void *p) { std::free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { note("hostmalloc " + std::to_string(n)); *p = block(n); return 0; }
int hipHostFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind)
{
    note("memcpy " + std::to_string(n) + " kind " + std::to_string(kind));
    std::memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *) { return hipMemcpy(d, s, n, kind); }
int hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *) { return hipMemset(d, v, n); }
int hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return 0; }

// devices, streams, events, errors
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void *) { note("stream sync"); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = block(1); return 0; }
int hipStreamDestroy(void *s) { std::free(s); return 0; }
int hipEventCreate(void **e) { note("event create"); *e = block(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { std::free(e); return 0; }
int hipEventRecord(void *, void *) { note("event record"); return 0; }
int hipEventSynchronize(void *) { note("event sync"); return 0; }
int hipEventElapsedTime(float *t, void *, void *) { *t = elapsed_cb ? elapsed_cb() : 1.0f; return 0; }
int hipGetLastError() { return 0; }
int hipPeekAtLastError() { return 0; }
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
}
