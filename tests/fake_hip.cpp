// A HIP runtime of host memory for tests of the library's host side without a GPU:
// allocations come from the heap (those above a limit fail, as on a full device),
// copies are memcpy, launches are not run but noted by kernel name.  Loaded with
// RTLD_GLOBAL before libqaia, whose HIP symbols it then provides.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::map<const void *, std::string> names;
std::vector<std::string> launched;
std::map<void *, size_t> live;
size_t limit = SIZE_MAX, in_use = 0;
int sticky = 0;
struct Dim { uint32_t x, y, z; };
Dim cfg_grid, cfg_block;
size_t cfg_shmem;
void *cfg_stream;
constexpr int kOutOfMemory = 2;
}  // namespace

extern "C" {
// ---- what the tests call
void fake_limit(size_t bytes) { limit = bytes; }  // largest allocation that succeeds
size_t fake_in_use() { return in_use; }
int fake_sticky() { return sticky; }
void fake_clear() { launched.clear(); }
const char *fake_kernels(int of_launches) {  // names, one a line: of the launches so far, or of all kernels
    static std::string all;
    all.clear();
    if (of_launches)
        for (const std::string &s : launched) all += s + "\n";
    else
        for (const auto &kv : names) all += kv.second + "\n";
    return all.c_str();
}
int fake_count(const char *part) {  // launches so far of kernels whose (mangled) name holds `part`
    int n = 0;
    for (const std::string &s : launched) n += s.find(part) != std::string::npos;
    return n;
}

// ---- the runtime
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) { names[host] = name; }
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shmem, void *stream) {
    cfg_grid = g, cfg_block = b, cfg_shmem = shmem, cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *shmem, void **stream) {
    *g = cfg_grid, *b = cfg_block, *shmem = cfg_shmem, *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim, Dim, void **, size_t, void *) {
    launched.push_back(names.count(f) ? names[f] : "?");
    return 0;
}
int hipMalloc(void **p, size_t bytes) {
    if (bytes > limit) return sticky = kOutOfMemory;
    *p = calloc(1, bytes ? bytes : 1);
    live[*p] = bytes;
    in_use += bytes;
    return 0;
}
int hipFree(void *p) {
    if (live.count(p)) in_use -= live[p], live.erase(p), free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) { return memcpy(d, s, n), 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { return memcpy(d, s, n), 0; }
int hipMemset(void *d, int v, size_t n) { return memset(d, v, n), 0; }
int hipGetLastError() { const int e = sticky; sticky = 0; return e; }
const char *hipGetErrorString(int) { return "fake"; }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipGetDevice(int *d) { return *d = 0, 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceGetAttribute(int *v, int, int) { return *v = 256, 0; }  // (asked for the number of CUs)
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { return *n = 4, 0; }
int hipGetSymbolAddress(void **p, const void *) { static char mem[64]; return *p = mem, 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return *s = malloc(1), 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipStreamBeginCapture(void *, int) { return 0; }
int hipStreamEndCapture(void *, void **g) { return *g = malloc(1), 0; }
int hipGraphInstantiate(void **e, void *, void **, char *, size_t) { return *e = malloc(1), 0; }
int hipGraphLaunch(void *, void *) { return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) { return *e = malloc(1), 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = malloc(1), 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventQuery(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { return *ms = 1.0f, 0; }
int hipEventDestroy(void *) { return 0; }
int hipModuleLoadData(void **m, const void *) { return *m = malloc(1), 0; }
int hipModuleGetFunction(void **f, void *, const char *) { return *f = malloc(1), 0; }
int hipModuleUnload(void *) { return 0; }
int hipModuleLaunchKernel(void *, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, void *, void **,
                          void **) { return launched.push_back("generated"), 0; }
}
