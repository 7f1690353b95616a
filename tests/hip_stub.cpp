// Stand-in for the HIP runtime calls of libsoftrobot.so, for host tests of its
// bookkeeping: memory calls keep count, launches are checked for the size of
// their grid, every other call succeeds and does
// nothing (no kernel runs).  Loaded with RTLD_GLOBAL before the library, so the
// library's calls bind here.
#include <cstdlib>
#include <cstring>
#include <set>

namespace {
std::set<void *> live;     // device and pinned allocations
int bad_frees = 0;         // frees of an address that is not allocated
int mallocs = 0, streams = 0, captures = 0;
int fail_from = -1, fail_to = -1;  // device allocations (numbered from 0) that fail
bool fail_pinned = false;
int bad_grids = 0;         // launches beyond what a grid holds
int last = 0;              // what hipGetLastError returns next
constexpr int kInvalid = 1, kOutOfMemory = 2;

int note(int e) { return last = e ? e : last, e; }
int release(void *p) {
    if (!p) return 0;
    if (live.erase(p)) return free(p), 0;
    ++bad_frees;
    return note(kInvalid);
}
void *token() {
    static char mem[8];
    return mem;
}
}  // namespace

extern "C" {
void stub_fail(int from, int to) { mallocs = 0, fail_from = from, fail_to = to; }
void stub_fail_pinned(int on) { fail_pinned = on; }
int stub_bad_frees() { return bad_frees; }
int stub_bad_grids() { return bad_grids; }
int stub_live() { return (int)live.size(); }
int stub_mallocs() { return mallocs; }
int stub_streams() { return streams; }
int stub_captures() { return captures; }

int hipMalloc(void **p, size_t) {
    const int n = mallocs++;
    if (n >= fail_from && n < fail_to) return note(kOutOfMemory);
    live.insert(*p = malloc(16));
    return 0;
}
int hipFree(void *p) { return release(p); }
int hipHostMalloc(void **p, size_t bytes, unsigned) {
    if (fail_pinned) return note(kOutOfMemory);
    live.insert(*p = malloc(bytes));
    memset(*p, 0xff, bytes);  // a build's first word: no bad robot
    return 0;
}
int hipHostFree(void *p) { return release(p); }
int hipGetLastError() {
    const int e = last;
    last = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }

int hipGetDevice(int *d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }
int hipGetSymbolAddress(void **p, const void *) { return *p = token(), 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return ++streams, *s = token(), 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamBeginCapture(void *, int) { return ++captures, 0; }
int hipStreamEndCapture(void *, void **g) { return *g = token(), 0; }
int hipGraphInstantiate(void **e, void *, void *, char *, size_t) { return *e = token(), 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) { return *e = token(), 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = token(), 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 1.f, 0; }
struct Dim3 {
    unsigned x, y, z;
};
int hipLaunchKernel(const void *, Dim3, Dim3, void **, size_t, void *) { return 0; }
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t, void *) {
    // a grid holds less than 2^32 threads in x and at most 65535 workgroups in y and z
    if (g.x == 0 || (unsigned long long)g.x * b.x >= 1ull << 32 || g.y > 65535 || g.z > 65535) ++bad_grids;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *m, void **s) {
    *g = *b = Dim3{1, 1, 1};
    return *m = 0, *s = nullptr, 0;
}
void **__hipRegisterFatBinary(const void *) {
    static void *h;
    return &h;
}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
