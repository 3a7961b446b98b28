// A HIP runtime without a GPU for tests of the library's host side: memory is
// host memory, launches and waits are only noted (kernel name, grid and block), and one
// chosen call or launch can be made to fail.  An error stays until
// hipGetLastError takes it, as in the real runtime.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
struct Dim3 { uint32_t x, y, z; };
std::map<const void *, std::string> g_names;
std::string g_log, g_fail;
int g_skip = -1, g_last = 0;   // g_skip: matching calls to let pass before the failing one
Dim3 g_grid, g_block;
size_t g_shm;
void *g_stream;

constexpr int kError = 719;   // hipErrorLaunchFailure
int outcome(const std::string &what) {
    if (g_skip >= 0 && what.find(g_fail) != std::string::npos && g_skip-- == 0) {
        g_last = kError;
        return kError;
    }
    return 0;
}
void *some_pointer() { static char c; return &c; }
}  // namespace

extern "C" {
// the test's side
void fake_fail(const char *what, int skip) { g_fail = what; g_skip = skip; }
void fake_clear() { g_log.clear(); g_skip = -1; g_last = 0; }
const char *fake_log() { return g_log.c_str(); }

void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *,
                           void *, int *) { g_names[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shm, void *s) {
    g_grid = g; g_block = b; g_shm = shm; g_stream = s;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shm, void **s) {
    *g = g_grid; *b = g_block; *shm = g_shm; *s = g_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 g, Dim3 b, void **, size_t, void *) {
    const std::string &name = g_names[f];
    const int e = outcome(name);
    if (g.x == 0 || g.y == 0 || g.z == 0 || b.x * b.y * b.z > 1024) { g_last = kError; return kError; }
    g_log += name + " " + std::to_string(g.x) + " " + std::to_string(b.x) + " " + std::to_string(e) + "\n";
    return e;
}
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipGetSymbolAddress(void **p, const void *) {
    static char array[32 << 20];
    *p = array;
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = some_pointer(); return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) {
    g_log += "hipStreamWaitEvent 0 0 0\n";
    return outcome("hipStreamWaitEvent");
}
int hipStreamBeginCapture(void *, int) { return outcome("hipStreamBeginCapture"); }
int hipStreamEndCapture(void *, void **g) { *g = some_pointer(); return outcome("hipStreamEndCapture"); }
int hipGraphInstantiate(void **x, void *, void **, char *, size_t) {
    *x = some_pointer();
    return outcome("hipGraphInstantiate");
}
int hipGraphLaunch(void *, void *) { return outcome("hipGraphLaunch"); }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) { *e = some_pointer(); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = some_pointer(); return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return outcome("hipEventRecord"); }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.0f; return 0; }
int hipGetLastError() { const int e = g_last; g_last = 0; return e; }
const char *hipGetErrorString(int) { return "error of the test"; }
}
