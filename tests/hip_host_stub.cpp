// A HIP runtime of host memory, for CPU tests of the library's host code: loaded
// with global symbols before libmt.so, its functions take the place of the real
// runtime's.  Device memory is host memory with a limit, copies are memcpy, and a
// launch runs nothing: it is recorded and advances a clock that events read.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;
    unsigned grid, block;
    size_t lds;
    bool tables_live;       // transport kernels: the tables that the argument starts with
};

std::map<char *, size_t> live;
std::map<const void *, std::string> names;
std::vector<Launch> launches;
size_t limit = (size_t)1 << 40, used = 0, peak = 0;
int allocs_left = -1, copies_left = -1;     // successes before the next failure
float clock_ms = 0.f;
std::string cheap;                          // launches of kernels with this name cost 1, others 2

bool is_live(const void *p) {
    auto it = live.upper_bound((char *)p);
    return it != live.begin() && (--it, (char *)p < it->first + it->second);
}

}  // namespace

extern "C" {

void stub_limit(size_t bytes) { limit = bytes; }
void stub_fail_alloc(int after) { allocs_left = after; }
void stub_fail_copy(int after) { copies_left = after; }
size_t stub_used() { return used; }
size_t stub_peak(int reset) {
    if (reset) peak = used;
    return peak;
}
void stub_cheap(const char *name) { cheap = name; }
int stub_launches() { return (int)launches.size(); }
void stub_clear() { launches.clear(); }
const char *stub_launch(int i, unsigned *grid, unsigned *block, size_t *lds, int *tables_live) {
    const Launch &l = launches[i];
    *grid = l.grid;
    *block = l.block;
    *lds = l.lds;
    *tables_live = l.tables_live;
    return l.name.c_str();
}

hipError_t hipMalloc(void **p, size_t n) {
    if (allocs_left == 0 || used + n > limit) {
        allocs_left = -1;
        return hipErrorOutOfMemory;
    }
    if (allocs_left > 0) --allocs_left;
    char *q = (char *)calloc(1, n);
    live[q] = n;
    used += n;
    if (used > peak) peak = used;
    *p = q;
    return hipSuccess;
}

hipError_t hipFree(void *p) {
    auto it = live.find((char *)p);
    if (it == live.end()) return hipErrorInvalidValue;
    used -= it->second;
    live.erase(it);
    free(p);
    return hipSuccess;
}

hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (copies_left == 0) {
        copies_left = -1;
        return hipErrorUnknown;
    }
    if (copies_left > 0) --copies_left;
    memcpy(d, s, n);
    return hipSuccess;
}

hipError_t hipMemGetInfo(size_t *room, size_t *total) {
    *room = limit - used;
    *total = limit;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    p->warpSize = 64;
    p->sharedMemPerBlock = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char scratch[1 << 20];
    return *p = scratch, hipSuccess;
}

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds,
                           hipStream_t) {
    Launch l{names.count(f) ? names[f] : "", grid.x, block.x, lds, true};
    const void *const *t = (const void *const *)args[0];     // image, cdf, guide, alias
    for (const char *k : {"k_plain", "k_pass", "k_variant_waves"})
        if (l.name.find(std::string(k) + "I") != std::string::npos)
            l.tables_live = is_live(t[0]) && is_live(t[1]) && is_live(t[2]) && is_live(t[3]);
    launches.push_back(l);
    clock_ms += !cheap.empty() && l.name.find(cheap) != std::string::npos ? 1.f : 2.f;
    return hipSuccess;
}

static dim3 next_grid, next_block;
static size_t next_lds;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
    next_grid = grid;
    next_block = block;
    next_lds = lds;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = next_grid;
    *block = next_block;
    *lds = next_lds;
    *s = nullptr;
    return hipSuccess;
}

void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
    names[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}

hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t) new float(0.f), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { return *(float *)e = clock_ms, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b) {
    return *ms = *(float *)b - *(float *)a, hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) { return delete (float *)e, hipSuccess; }

}  // extern "C"
