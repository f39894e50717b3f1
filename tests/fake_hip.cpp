// A HIP runtime on host memory, for tests of the library's host code without a GPU: two devices, every
// allocation kept with its device, limits and failures that a test sets, and launches that run nothing
// but what the tests' checks need of them. Loaded with its symbols global before the library, whose calls
// then come here.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>

struct Dim3 {
    uint32_t x, y, z;
};

constexpr size_t kSmall = 256;     // (smaller blocks are not counted: the library waits by freeing one)
enum { kOk = 0, kInvalid = 1, kOutOfMemory = 2, kInvalidDevice = 101, kCapture = 900, kLaunch = 719 };

namespace {

struct Block {
    int device;
    size_t bytes;
};

std::recursive_mutex g_mu;
std::map<void*, Block>* g_blocks = new std::map<void*, Block>();
std::map<const void*, std::string>* g_names = new std::map<const void*, std::string>();
thread_local int t_device = 0;
thread_local int t_last = kOk;
size_t g_limit[2] = {SIZE_MAX, SIZE_MAX}, g_live[2] = {0, 0};
int64_t g_mallocs = 0, g_frees = 0, g_waits = 0, g_dirty = 0;
void* g_uploaded = nullptr;            // destination of the last copy from the host
int g_fail_sync = 0, g_fail_nth = 0;
char g_fail_name[64] = "";
thread_local int t_fail_new = 0;

int set(int e) {
    if (e != kOk) t_last = e;
    return e;
}

bool clear(const void* p, size_t bytes) {
    const char* c = (const char*)p;
    for (size_t i = 0; i < bytes; ++i)
        if (c[i]) return false;
    return true;
}

// What a launch does here: zero fills run; the exact gain's own sets are looked at (they have to be clear
// when a level's sets are gathered), get a bit, and are cleared by the merge.
int launch(const void* f, void** args) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    const auto it = g_names->find(f);
    const std::string name = it == g_names->end() ? "" : it->second;
    if (g_fail_nth > 0 && name.find(g_fail_name) != std::string::npos && --g_fail_nth == 0) return set(kLaunch);
    if (name.find("k_zero_u32") != std::string::npos) {
        uint32_t* p = *(uint32_t**)args[0];
        memset(p, 0, 4 * *(size_t*)args[1]);
    }
    const bool sets = name.find("k_exact_set") != std::string::npos, merge = name.find("k_exact_merge") != std::string::npos;
    if (sets || merge) {
        void* own = *(void**)args[sets ? 6 : 4];
        const auto b = g_blocks->find(own);
        if (b == g_blocks->end()) return set(kInvalid);
        if (sets) {
            g_dirty += clear(own, b->second.bytes) ? 0 : 1;
            *(uint32_t*)own |= 1u;
        } else {
            memset(own, 0, b->second.bytes);
        }
    }
    return kOk;
}

}  // namespace

void* operator new(size_t n) {
    if (t_fail_new > 0 && --t_fail_new == 0) throw std::bad_alloc();
    void* p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {

// ---- what the tests set and read
void fake_limit(int dev, size_t bytes) { g_limit[dev] = bytes; }
size_t fake_live(int dev) { return g_live[dev]; }
int64_t fake_mallocs() { return g_mallocs; }
int64_t fake_frees() { return g_frees; }
int64_t fake_dirty() { return g_dirty; }
int64_t fake_waits() { return g_waits; }                    // waits for a device that succeeded (frees among them)
void* fake_last_block() { return g_uploaded; }
void fake_fail_sync(int on) { g_fail_sync = on; }
void fake_fail_kernel(const char* name, int nth) {
    snprintf(g_fail_name, sizeof(g_fail_name), "%s", name);
    g_fail_nth = nth;
}
void fake_fail_new(int nth) { t_fail_new = nth; }           // this thread's nth next operator new throws
void fake_set_device(int dev) { t_device = dev; }
// bytes held on device `dev` in blocks of at least `least` bytes
size_t fake_held(int dev, size_t least) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    size_t n = 0;
    for (const auto& b : *g_blocks) n += b.second.device == dev && b.second.bytes >= least ? b.second.bytes : 0;
    return n;
}
// the device of the block that holds p, or -1
int fake_device_of(const void* p) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    for (const auto& b : *g_blocks)
        if (p >= b.first && (const char*)p < (const char*)b.first + b.second.bytes) return b.second.device;
    return -1;
}

// ---- memory
int hipMalloc(void** p, size_t bytes) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    *p = nullptr;
    if (bytes > g_limit[t_device] || g_live[t_device] > g_limit[t_device] - bytes) return set(kOutOfMemory);
    const int fail = t_fail_new;
    t_fail_new = 0;
    *p = calloc(bytes ? bytes : 1, 1);
    (*g_blocks)[*p] = Block{t_device, bytes};
    t_fail_new = fail;
    g_live[t_device] += bytes;
    g_mallocs += bytes > kSmall;
    return kOk;
}
int hipFree(void* p) {
    if (!p) return kOk;
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    const auto b = g_blocks->find(p);
    if (b == g_blocks->end()) return set(kInvalid);
    if (g_fail_sync) return set(kCapture);
    g_live[b->second.device] -= b->second.bytes;
    g_frees += b->second.bytes > kSmall;
    ++g_waits;
    g_blocks->erase(b);
    free(p);
    return kOk;
}
int hipHostMalloc(void** p, size_t bytes, unsigned) { *p = calloc(bytes ? bytes : 1, 1); return kOk; }
int hipHostFree(void* p) { free(p); return kOk; }
int hipMemcpy(void* d, const void* s, size_t n, int) { memcpy(d, s, n); return kOk; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void*) {
    memcpy(d, s, n);
    if (kind == 1) g_uploaded = d;
    return kOk;
}
int hipGetSymbolAddress(void** p, const void*) {
    static void* scratch[2] = {};
    if (!scratch[t_device]) scratch[t_device] = calloc(17u << 20, 1);
    *p = scratch[t_device];
    return kOk;
}

// ---- devices
int hipGetDevice(int* d) { *d = t_device; return kOk; }
int hipSetDevice(int d) { if (d < 0 || d > 1) return set(kInvalidDevice); t_device = d; return kOk; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 65536; return kOk; }
int hipDeviceSynchronize() { if (g_fail_sync) return set(kCapture); ++g_waits; return kOk; }
int hipGetLastError() { const int e = t_last; t_last = kOk; return e; }
const char* hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : (e == kOk ? "no error" : "an error"); }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return kOk; }

// ---- streams, events, graphs
int hipStreamCreateWithFlags(void** s, unsigned) { *s = malloc(1); return kOk; }
int hipStreamDestroy(void* s) { free(s); return kOk; }
int hipStreamSynchronize(void*) { return kOk; }
int hipStreamWaitEvent(void*, void*, unsigned) { return kOk; }
int hipEventCreate(void** e) { *e = malloc(1); return kOk; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = malloc(1); return kOk; }
int hipEventDestroy(void* e) { free(e); return kOk; }
int hipEventRecord(void*, void*) { return kOk; }
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* ms, void*, void*) { *ms = 1.f; return kOk; }
int hipStreamBeginCapture(void*, int) { return kOk; }
int hipStreamEndCapture(void*, void** g) { *g = malloc(1); return kOk; }
int hipGraphInstantiate(void** x, void*, void*, char*, size_t) { *x = malloc(1); return kOk; }
int hipGraphLaunch(void*, void*) { return kOk; }
int hipGraphDestroy(void* g) { free(g); return kOk; }
int hipGraphExecDestroy(void* x) { free(x); return kOk; }

// ---- launches
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    (*g_names)[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
thread_local Dim3 t_grid, t_block;
thread_local size_t t_shared;
thread_local void* t_stream;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t sh, void* s) {
    t_grid = g; t_block = b; t_shared = sh; t_stream = s;
    return kOk;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* sh, void** s) {
    *g = t_grid; *b = t_block; *sh = t_shared; *s = t_stream;
    return kOk;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) { return launch(f, args); }
int hipExtLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*, void*, void*, int) { return launch(f, args); }
int hipLaunchCooperativeKernel(const void* f, Dim3, Dim3, void** args, unsigned, void*) { return launch(f, args); }

}  // extern "C"
