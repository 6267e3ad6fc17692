// Shared definitions of the MI355X KIFMM library (host and device).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <memory>
#include <stdexcept>
#include <string>
#include <vector>

#include "fmm.h"

namespace fmm {

constexpr int kMaxLevel = 21;   // finest level of the 63-bit Morton key
constexpr int kNumDirs = 316;   // M2L offsets d in {-3..3}^3 with max|d| >= 2
constexpr int kMaxOrder = 12;
constexpr double kRadIn = 1.05;   // upward-equivalent / downward-check surface radius (box half-widths)
constexpr double kRadOut = 2.95;  // upward-check / downward-equivalent surface radius
constexpr double kPi = 3.14159265358979323846264338327950288;
constexpr double kFourPi = 12.566370614359172953850573533118;

struct Error : std::runtime_error {
    int code;
    Error(int c, const std::string &m) : std::runtime_error(m), code(c) {}
};

#define FMM_HIP(x)                                                                            \
    do {                                                                                      \
        hipError_t e_ = (x);                                                                  \
        if (e_ != hipSuccess)                                                                 \
            throw ::fmm::Error(e_ == hipErrorOutOfMemory ? FMM_ERR_NOMEM : FMM_ERR_DEVICE,    \
                               std::string(#x) + ": " + hipGetErrorString(e_));               \
    } while (0)

#define FMM_REQUIRE(c, msg)                                  \
    do {                                                     \
        if (!(c)) throw ::fmm::Error(FMM_ERR_ARG, (msg));    \
    } while (0)

// Failure injection for tests of the error paths: with the environment
// variable FMM_FAULT_INJECT=alloc:<k> the k-th device allocation counted from
// when the variable took its current value fails as if the device were out
// of memory (FMM_ERR_NOMEM). Returns true for the allocation that must fail.
bool inject_alloc_failure();

// Blocks of device memory between hipMalloc and the arenas below. A block
// given back is kept for the next plan or solve, up to 512 MB a process (0.2%
// of the GPU's memory); it is freed when it has not been taken again by the time
// more than sixteen arenas have ended (a setup and its plan are two, a solve, a
// right-hand side or a force call one), when an allocation fails, or on request
// (fmm_release_memory). hipMalloc and hipFree
// take about 1 us up to 1 MB, but in a program with several streams 40 and
// 230-900 us for the blocks of a plan: 4.5 ms of the 16 ms that setting up,
// applying once and destroying a 500,000-point plan took. Thread-safe;
// block_give requires that no work on the block is left on any stream.
struct Block {
    void *p = nullptr;
    size_t bytes = 0;
    int dev = 0;
};
// hipMalloc; on failure the kept blocks are freed first, then FMM_ERR_NOMEM
void *device_malloc(size_t bytes);
Block block_take(size_t bytes);      // at least `bytes`, on the current device
void block_give(const Block &b);
void block_free(const Block &b);      // past the pool
void block_pool_tick();              // once per arena: ages the kept blocks
void block_pool_release();           // frees the kept blocks

// Device memory handed out from a few blocks: a plan makes some hundred
// buffers and as many temporaries. One thread uses an arena at a time; what is
// taken from it lives at most as long as the arena. Memory given back is only
// handed out again to work queued later on the same stream.
class Arena {
  public:
    Arena() = default;
    Arena(const Arena &) = delete;
    Arena &operator=(const Arena &) = delete;
    ~Arena() {
        if (blocks_.empty()) return;
        // as hipFree would: work on any stream of the blocks' device may still use them
        int dev = blocks_[0].dev, cur = dev;
        (void)hipGetDevice(&cur);
        if (cur != dev) (void)hipSetDevice(dev);
        const bool idle = hipDeviceSynchronize() == hipSuccess;
        if (!idle) (void)hipGetLastError();
        if (cur != dev) (void)hipSetDevice(cur);
        for (const Block &b : blocks_) {
            if (idle)
                block_give(b);
            else
                block_free(b);  // not waited for (a stream is being captured): left to hipFree's own wait
        }
        block_pool_tick();
    }
    void *take(size_t bytes) {
        bytes = round(bytes);
        if (bytes > left_) {
            if (bytes >= next_) return block(bytes).p;  // its own block; the current one stays in use
            const Block b = block(next_);
            begin_ = cur_ = (char *)b.p;
            left_ = b.bytes;
            if (next_ < kMaxBlock) next_ *= 2;
        }
        char *p = cur_;
        cur_ += bytes;
        left_ -= bytes;
        return p;
    }
    // the current block's last piece can be taken again; others wait for the arena's
    // end (another block may end where the current one begins)
    void give(void *p, size_t bytes) {
        if ((char *)p >= begin_ && (char *)p + round(bytes) == cur_) {
            cur_ -= round(bytes);
            left_ += round(bytes);
        }
    }
    // the start of the block that holds p
    const char *block_of(const void *p) const {
        for (const Block &b : blocks_)
            if ((const char *)p >= (const char *)b.p && (const char *)p < (const char *)b.p + b.bytes) return (const char *)b.p;
        return nullptr;
    }

  private:
    static constexpr size_t kMaxBlock = size_t(16) << 20;
    static size_t round(size_t n) { return (n + 255) / 256 * 256; }
    Block block(size_t bytes) {
        blocks_.reserve(blocks_.size() + 1);
        blocks_.push_back(block_take(bytes));
        return blocks_.back();
    }
    std::vector<Block> blocks_;
    char *begin_ = nullptr, *cur_ = nullptr;  // the current block, its free part
    size_t left_ = 0, next_ = size_t(1) << 20;
};

// Where this thread's buffers come from while a scope is alive: `keep` the
// buffers, `temp` those made with Temp{}; NULL: hipMalloc for each.
struct ArenaScope {
    ArenaScope(Arena *keep, Arena *temp) : keep0(keep_slot()), temp0(temp_slot()) {
        keep_slot() = keep;
        temp_slot() = temp;
    }
    ~ArenaScope() {
        keep_slot() = keep0;
        temp_slot() = temp0;
    }
    ArenaScope(const ArenaScope &) = delete;
    ArenaScope &operator=(const ArenaScope &) = delete;
    static Arena *&keep_slot() {
        static thread_local Arena *a = nullptr;
        return a;
    }
    static Arena *&temp_slot() {
        static thread_local Arena *a = nullptr;
        return a;
    }

  private:
    Arena *keep0, *temp0;
};
struct Temp {};

// Owning device buffer, from the thread's arena or hipMalloc'd.
template <class T>
struct DBuf {
    T *p = nullptr;
    size_t n = 0;
    Arena *home = nullptr;  // NULL: hipMalloc'd
    DBuf() = default;
    explicit DBuf(size_t count) { alloc(count); }
    DBuf(size_t count, Temp) { alloc(count, Temp{}); }
    DBuf(const DBuf &) = delete;
    DBuf &operator=(const DBuf &) = delete;
    DBuf(DBuf &&o) noexcept : p(o.p), n(o.n), home(o.home) { o.p = nullptr; o.n = 0; }
    DBuf &operator=(DBuf &&o) noexcept {
        if (this != &o) { release(); p = o.p; n = o.n; home = o.home; o.p = nullptr; o.n = 0; }
        return *this;
    }
    ~DBuf() { release(); }
    void alloc(size_t count) { alloc_in(count, ArenaScope::keep_slot()); }
    void alloc(size_t count, Temp) { alloc_in(count, ArenaScope::temp_slot()); }
    void release() {
        if (p) {
            if (home)
                home->give(p, bytes());
            else
                (void)hipFree(p);
        }
        p = nullptr;
        n = 0;
    }
    T *get() const { return p; }
    size_t bytes() const { return n * sizeof(T); }

  private:
    void alloc_in(size_t count, Arena *a) {
        release();
        if (!count) return;
        // on failure, the work already queued finishes before the buffers the
        // failing call had allocated are released on the way out
        if (inject_alloc_failure()) {
            (void)hipDeviceSynchronize();
            throw Error(FMM_ERR_NOMEM, "device allocation failed (injected by FMM_FAULT_INJECT)");
        }
        home = a;
        if (a) {
            p = (T *)a->take(count * sizeof(T));
        } else {
            p = (T *)device_malloc(count * sizeof(T));
        }
        n = count;
    }
};

// Host-to-device copy that has finished reading `src` on return (the host
// buffer may be freed or reused right after).
template <class T>
void h2d(T *dst, const T *src, size_t n, hipStream_t s) {
    if (!n) return;
    FMM_HIP(hipMemcpyAsync(dst, src, n * sizeof(T), hipMemcpyHostToDevice, s));
    FMM_HIP(hipStreamSynchronize(s));
}
template <class T>
void d2h(T *dst, const T *src, size_t n, hipStream_t s) {
    if (n) FMM_HIP(hipMemcpyAsync(dst, src, n * sizeof(T), hipMemcpyDeviceToHost, s));
    FMM_HIP(hipStreamSynchronize(s));
}
template <class T>
DBuf<T> upload(const std::vector<T> &v, hipStream_t s) {
    DBuf<T> b(v.size());
    h2d(b.p, v.data(), v.size(), s);
    return b;
}

// Copies of many small arrays in few calls. Arrays whose device buffers follow
// each other in one block (an arena hands them out in order) travel in one copy
// through a host buffer, arrays of more than 1 MB by themselves; a setup has about 100 of
// them, at some 30 us a call. flush() has finished when it returns.
class Transfers {
  public:
    // dst = a new buffer holding v, filled by flush()
    template <class T>
    void up(DBuf<T> &dst, std::vector<T> v) {
        dst.alloc(v.size());
        if (v.empty()) return;
        auto held = std::make_shared<std::vector<T>>(std::move(v));
        items_.push_back({(char *)dst.p, (char *)held->data(), dst.bytes(), block(dst), held});
    }
    // h = the contents of src, filled by flush()
    template <class T>
    void down(std::vector<T> &h, const DBuf<T> &src, size_t count) {
        h.resize(count);
        if (count) items_.push_back({(char *)src.p, (char *)h.data(), count * sizeof(T), block(src), nullptr});
    }
    void flush_up(hipStream_t s) { flush(true, s); }
    void flush_down(hipStream_t s) { flush(false, s); }

  private:
    struct Item {
        char *dev, *host;
        size_t bytes;
        const char *block;  // a copy must not span two allocations, adjacent or not
        std::shared_ptr<void> held;
    };
    template <class T>
    static const char *block(const DBuf<T> &b) {
        return b.home ? b.home->block_of(b.p) : (const char *)b.p;
    }
    void flush(bool up, hipStream_t s);
    std::vector<Item> items_;
};

// Diagnostics on stderr, on when the environment variable FMM_LOG is set to
// a value other than 0 (read once per process).
bool log_enabled();
void log_printf(const char *fmt, ...) __attribute__((format(printf, 1, 2)));
#define FMM_LOG(...)                                            \
    do {                                                        \
        if (::fmm::log_enabled()) ::fmm::log_printf(__VA_ARGS__); \
    } while (0)

inline unsigned grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    return (unsigned)(g < 1 ? 1 : g);
}

// Device-wide exclusive prefix sum (in may equal out). Returns the total when
// want_total is set (synchronises the stream), else 0.
int64_t exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, hipStream_t s, bool want_total);
int64_t exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, hipStream_t s, bool want_total);
// the same with the total left on the device (n > 0)
void exclusive_scan_i32_total(const int32_t *in, int32_t *out, int64_t n, int32_t *total, hipStream_t s);
uint32_t exclusive_scan_u32(const uint32_t *in, uint32_t *out, int64_t n, hipStream_t s, bool want_total);

// Stable LSD radix sort of (key, value) pairs by the low `bits` bits of key.
void radix_sort_pairs(uint64_t *keys, int64_t *vals, int64_t n, int bits, hipStream_t s);

}  // namespace fmm
