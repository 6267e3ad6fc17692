// Host-side checks of the library's device-memory bookkeeping (Arena, the kept
// blocks, Transfers) with the HIP calls it makes replaced by stand-ins over host
// memory: allocations lie one directly after the other, a copy or a fill that
// does not stay inside one allocation is refused, and the device-wide wait can
// be made to fail as it does while a stream is being captured. Links against
// the host side of primitives.hip. Exits non-zero on a failed expectation.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "common.hpp"

static int failures = 0;
#define EXPECT(c)                                                         \
    do {                                                                  \
        if (!(c)) {                                                       \
            std::fprintf(stderr, "failed: %s (line %d)\n", #c, __LINE__); \
            ++failures;                                                   \
        }                                                                 \
    } while (0)

// ------------------------------------------------------------ stand-ins
static std::vector<char> g_mem(size_t(256) << 20);
static size_t g_top = 0;                    // next free byte
static std::map<char *, size_t> g_alloc;    // live allocations
static int g_frees = 0, g_syncs = 0, g_copies = 0, g_fail_copy = 0;
static hipError_t g_device_sync = hipSuccess;

static bool inside_one(const void *p, size_t n) {
    auto it = g_alloc.upper_bound((char *)p);
    if (it == g_alloc.begin()) return false;
    --it;
    return (const char *)p + n <= it->first + it->second;
}

extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (g_top + n > g_mem.size()) return hipErrorOutOfMemory;
    *p = g_mem.data() + g_top;
    g_alloc[(char *)*p] = n;
    g_top += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    ++g_frees;
    g_alloc.erase((char *)p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (++g_copies == g_fail_copy) return hipErrorInvalidValue;
    if (!inside_one(kind == hipMemcpyHostToDevice ? dst : src, n)) return hipErrorInvalidValue;
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    ++g_syncs;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return g_device_sync; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipUnregisterFatBinary(void **) {}
}
namespace fmm {
bool inject_alloc_failure() { return false; }
bool log_enabled() { return false; }
void log_printf(const char *, ...) {}
}  // namespace fmm

using namespace fmm;

// A block goes to the next arena only once nothing on the device uses it: with
// the wait refused it is freed, which waits by itself.
static void check_wait() {
    void *first = nullptr;
    {
        Arena a;
        first = a.take(1000);
    }
    EXPECT(g_frees == 0);
    {
        Arena a;
        EXPECT(a.take(1000) == first);  // kept and handed out again
        g_device_sync = hipErrorStreamCaptureUnsupported;
    }
    g_device_sync = hipSuccess;
    EXPECT(g_frees == 1);
    Arena a;
    EXPECT(a.take(1000) != first);
}

// Pieces and copies stay inside one allocation also where the next one begins
// right behind it.
constexpr size_t MB = size_t(1) << 20;
static void check_give() {
    Arena a;
    char *own = (char *)a.take(MB);  // a block of its own
    char *p = (char *)a.take(256);   // the first piece of the block behind it
    EXPECT(p == own + MB);
    a.give(p, 256);
    a.give(own, MB);  // not the current block's last piece
    EXPECT(inside_one(a.take(MB + MB / 2), MB + MB / 2));
}

static void check_copies() {
    Arena a;
    ArenaScope scope(&a, &a);
    Transfers tr;
    DBuf<char> b[4];
    std::vector<char> v[4] = {std::vector<char>(MB - 256, 'a'), std::vector<char>(256, 'b'),
                              std::vector<char>(300, 'c'), std::vector<char>(200, 'd')};
    for (int k = 0; k < 4; ++k) tr.up(b[k], v[k]);
    EXPECT(b[2].p == b[1].p + 256 && b[3].p == b[2].p + 512);  // b[0], b[1] fill a block
    try {
        tr.flush_up(nullptr);
        for (int k = 0; k < 4; ++k) EXPECT(std::memcmp(b[k].p, v[k].data(), v[k].size()) == 0);
        std::vector<char> h[4];
        for (int k = 0; k < 4; ++k) tr.down(h[k], b[k], v[k].size());
        g_copies = 0;
        tr.flush_down(nullptr);
        EXPECT(g_copies == 2);
        for (int k = 0; k < 4; ++k) EXPECT(h[k] == v[k]);
    } catch (const Error &e) {
        std::fprintf(stderr, "%s\n", e.what());
        EXPECT(!"a copy left its allocation");
    }
}

// A copy that fails leaves no copy before it in flight: the stream is waited for
// before the host buffers go.
static void check_failed_copy() {
    Arena a;
    ArenaScope scope(&a, &a);
    Transfers tr;
    DBuf<char> b[3];
    for (auto &x : b) tr.up(x, std::vector<char>(2 * MB, 'x'));
    g_fail_copy = 3;
    int code = FMM_OK;
    try {
        tr.flush_up(nullptr);
    } catch (const Error &e) {
        code = e.code;
    }
    EXPECT(code == FMM_ERR_DEVICE && g_copies == 3 && g_syncs == 1);
}

int main(int argc, char **argv) {
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "wait")) check_wait();
    else if (!std::strcmp(what, "give")) check_give();
    else if (!std::strcmp(what, "copies")) check_copies();
    else if (!std::strcmp(what, "failed_copy")) check_failed_copy();
    else return 2;
    if (failures) return 1;
    std::printf("memory checks passed: %s\n", what);
    return 0;
}
