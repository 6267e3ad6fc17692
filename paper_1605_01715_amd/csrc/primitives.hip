// Device-wide primitives: exclusive prefix sums and a stable LSD radix sort.
//
// The Morton sort of the octree build (points mapped to a 1-D array by their
// z-value, Sec. III.B) runs on these. The radix sort is stable, so equal keys
// keep their input order, which makes the sorted order (and the tree) a pure
// function of the input.
#include "common.hpp"

#include <mutex>

namespace fmm {

namespace {

struct Kept {
    Block b;
    int age = 0;  // arenas ended since it was given back
};
constexpr size_t kPoolBytes = size_t(512) << 20;
constexpr int kPoolAge = 16;
std::mutex g_pool_mu;
// never destroyed: the HIP runtime may be gone when static objects end
std::vector<Kept> &pool() {
    static auto *v = new std::vector<Kept>();
    return *v;
}
size_t g_pool_held = 0;

// frees the kept blocks that `drop` names; the lock is held
template <class F>
void pool_drop(F &&drop) {
    auto &v = pool();
    size_t w = 0;
    for (const Kept &k : v) {
        if (drop(k)) {
            g_pool_held -= k.b.bytes;
            (void)hipFree(k.b.p);
        } else {
            v[w++] = k;
        }
    }
    v.resize(w);
}

}  // namespace

void *device_malloc(size_t bytes) {
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        block_pool_release();
        e = hipMalloc(&p, bytes);
    }
    if (e != hipSuccess) {
        (void)hipDeviceSynchronize();
        FMM_HIP(e);
    }
    return p;
}

Block block_take(size_t bytes) {
    Block b;
    FMM_HIP(hipGetDevice(&b.dev));
    {
        // the smallest kept block that fits without wasting a quarter
        std::lock_guard<std::mutex> lk(g_pool_mu);
        auto &v = pool();
        size_t best = v.size();
        for (size_t i = 0; i < v.size(); ++i) {
            const Block &k = v[i].b;
            if (k.dev == b.dev && k.bytes >= bytes && k.bytes <= bytes + bytes / 4 &&
                (best == v.size() || k.bytes < v[best].b.bytes))
                best = i;
        }
        if (best < v.size()) {
            b = v[best].b;
            g_pool_held -= b.bytes;
            v.erase(v.begin() + (ptrdiff_t)best);
            return b;
        }
    }
    b.p = device_malloc(bytes);
    b.bytes = bytes;
    return b;
}

void block_give(const Block &b) {
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        if (g_pool_held + b.bytes <= kPoolBytes) {
            try {
                pool().push_back({b, 0});
                g_pool_held += b.bytes;
                return;
            } catch (const std::bad_alloc &) {
            }
        }
    }
    (void)hipFree(b.p);
}

void block_free(const Block &b) {
    if (hipFree(b.p) != hipSuccess) (void)hipGetLastError();
}

void block_pool_tick() {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    for (Kept &k : pool()) ++k.age;
    pool_drop([](const Kept &k) { return k.age > kPoolAge; });
}

void block_pool_release() {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    pool_drop([](const Kept &) { return true; });
}

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// Inclusive scan of one value per thread across the block (Hillis-Steele in LDS).
template <class T>
__device__ T block_inclusive_scan(T v, T *sh) {
    int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        T add = (t >= off) ? sh[t - off] : T(0);
        __syncthreads();
        sh[t] += add;
        __syncthreads();
    }
    T r = sh[t];
    __syncthreads();
    return r;
}

template <class T>
__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const T *in, int64_t n, T *sums) {
    __shared__ T sh[kScanThreads];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    T acc = 0;
    for (int i = 0; i < kScanItems; ++i)
        if (base + i < n) acc += in[base + i];
    T inc = block_inclusive_scan(acc, sh);
    if (threadIdx.x == kScanThreads - 1) sums[blockIdx.x] = inc;
}

template <class T>
__global__ __launch_bounds__(kScanThreads) void k_tile_scan(const T *in, T *out, int64_t n, const T *offsets,
                                                            T *total) {
    __shared__ T sh[kScanThreads];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    T v[kScanItems];
    T acc = 0;
    for (int i = 0; i < kScanItems; ++i) {
        v[i] = (base + i < n) ? in[base + i] : T(0);
        acc += v[i];
    }
    T inc = block_inclusive_scan(acc, sh);
    T run = inc - acc + (offsets ? offsets[blockIdx.x] : T(0));
    for (int i = 0; i < kScanItems; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
        if (total && base + i == n - 1) *total = run;
    }
}

// total (may be NULL): receives the sum of all values, on the device
template <class T>
void scan_impl(const T *in, T *out, int64_t n, T *total, hipStream_t s) {
    if (n <= 0) return;
    int64_t nt = (n + kScanTile - 1) / kScanTile;
    if (nt == 1) {
        hipLaunchKernelGGL(k_tile_scan<T>, dim3(1), dim3(kScanThreads), 0, s, in, out, n, (const T *)nullptr, total);
        FMM_HIP(hipGetLastError());
        return;
    }
    DBuf<T> sums(nt, Temp{});
    hipLaunchKernelGGL(k_tile_sums<T>, dim3((unsigned)nt), dim3(kScanThreads), 0, s, in, n, sums.p);
    FMM_HIP(hipGetLastError());
    scan_impl<T>(sums.p, sums.p, nt, nullptr, s);
    hipLaunchKernelGGL(k_tile_scan<T>, dim3((unsigned)nt), dim3(kScanThreads), 0, s, in, out, n,
                       (const T *)sums.p, total);
    FMM_HIP(hipGetLastError());
    if (!sums.home) FMM_HIP(hipStreamSynchronize(s));  // `sums` is freed on return
}

template <class T>
T scan_total(const T *in, T *out, int64_t n, hipStream_t s, bool want_total) {
    if (n <= 0) return 0;
    if (!want_total) {
        scan_impl<T>(in, out, n, nullptr, s);
        return 0;
    }
    DBuf<T> total(1, Temp{});
    scan_impl<T>(in, out, n, total.p, s);
    T h = 0;
    d2h(&h, total.p, 1, s);
    return h;
}

// ---------------------------------------------------------------- radix sort
constexpr int kRsThreads = 256;
constexpr int kRsItems = 16;
constexpr int kRsTile = kRsThreads * kRsItems;

__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const uint64_t *keys, int64_t n, int shift,
                                                       uint32_t *hist, int nblk) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = (int64_t)blockIdx.x * kRsTile;
    for (int i = 0; i < kRsItems; ++i) {
        int64_t idx = base + (int64_t)i * kRsThreads + threadIdx.x;
        if (idx < n) atomicAdd(&h[(keys[idx] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter: rounds of 256 keys in input order; within a round the rank
// of a key among equal digits comes from wave ballots (lanes below it) and
// the counts of the waves before it.
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(const uint64_t *kin, const int64_t *vin,
                                                          uint64_t *kout, int64_t *vout, int64_t n,
                                                          int shift, const uint32_t *offs, int nblk) {
    __shared__ uint32_t run[256];
    __shared__ uint32_t wcnt[4][256];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    run[t] = offs[(int64_t)t * nblk + blockIdx.x];
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    int64_t base = (int64_t)blockIdx.x * kRsTile;
    for (int r = 0; r < kRsItems; ++r) {
        wcnt[0][t] = 0;
        wcnt[1][t] = 0;
        wcnt[2][t] = 0;
        wcnt[3][t] = 0;
        __syncthreads();
        int64_t idx = base + (int64_t)r * kRsThreads + t;
        bool valid = idx < n;
        uint64_t key = valid ? kin[idx] : 0ull;
        int64_t val = valid ? vin[idx] : 0;
        uint32_t d = (uint32_t)(key >> shift) & 255u;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t rank = (uint32_t)__popcll(peers & below);
        if (valid && rank == 0) wcnt[wv][d] = (uint32_t)__popcll(peers);
        __syncthreads();
        if (valid) {
            uint32_t pos = run[d] + rank;
            for (int w2 = 0; w2 < wv; ++w2) pos += wcnt[w2][d];
            kout[pos] = key;
            vout[pos] = val;
        }
        __syncthreads();
        run[t] += wcnt[0][t] + wcnt[1][t] + wcnt[2][t] + wcnt[3][t];
        __syncthreads();
    }
}

}  // namespace

void Transfers::flush(bool up, hipStream_t s) {
    constexpr size_t kLarge = size_t(1) << 20;
    const hipMemcpyKind kind = up ? hipMemcpyHostToDevice : hipMemcpyDeviceToHost;
    auto copy = [&](char *dev, char *host, size_t bytes) {
        FMM_HIP(hipMemcpyAsync(up ? dev : host, up ? host : dev, bytes, kind, s));
    };
    std::vector<std::vector<char>> held;  // host buffers in flight
    struct Part {
        size_t run;
        size_t first, last;  // items [first, last)
    };
    std::vector<Part> parts;
    try {
        for (size_t i = 0; i < items_.size();) {
            if (items_[i].bytes > kLarge) {
                copy(items_[i].dev, items_[i].host, items_[i].bytes);
                ++i;
                continue;
            }
            size_t j = i + 1;
            const char *end = items_[i].dev + items_[i].bytes;
            // the next buffer starts within the padding of the last one's end
            while (j < items_.size() && items_[j].bytes <= kLarge && items_[j].block == items_[i].block &&
                   items_[j].dev >= end && items_[j].dev - end < 256) {
                end = items_[j].dev + items_[j].bytes;
                ++j;
            }
            held.emplace_back((size_t)(end - items_[i].dev));
            char *h = held.back().data();
            if (up)
                for (size_t k = i; k < j; ++k)
                    std::memcpy(h + (items_[k].dev - items_[i].dev), items_[k].host, items_[k].bytes);
            copy(items_[i].dev, h, held.back().size());
            if (!up) parts.push_back({held.size() - 1, i, j});
            i = j;
        }
    } catch (...) {
        (void)hipStreamSynchronize(s);  // the copies queued so far still use the host buffers
        throw;
    }
    FMM_HIP(hipStreamSynchronize(s));
    for (const Part &p : parts)
        for (size_t k = p.first; k < p.last; ++k)
            std::memcpy(items_[k].host, held[p.run].data() + (items_[k].dev - items_[p.first].dev), items_[k].bytes);
    items_.clear();
}

int64_t exclusive_scan_i64(const int64_t *in, int64_t *out, int64_t n, hipStream_t s, bool want_total) {
    return scan_total<int64_t>(in, out, n, s, want_total);
}
int64_t exclusive_scan_i32(const int32_t *in, int32_t *out, int64_t n, hipStream_t s, bool want_total) {
    return scan_total<int32_t>(in, out, n, s, want_total);
}
void exclusive_scan_i32_total(const int32_t *in, int32_t *out, int64_t n, int32_t *total, hipStream_t s) {
    scan_impl<int32_t>(in, out, n, total, s);
}
uint32_t exclusive_scan_u32(const uint32_t *in, uint32_t *out, int64_t n, hipStream_t s, bool want_total) {
    return scan_total<uint32_t>(in, out, n, s, want_total);
}

void radix_sort_pairs(uint64_t *keys, int64_t *vals, int64_t n, int bits, hipStream_t s) {
    if (n <= 1) return;
    FMM_REQUIRE(n < (int64_t(1) << 31), "radix sort: more than 2^31 - 1 points");
    int nblk = (int)((n + kRsTile - 1) / kRsTile);
    DBuf<uint64_t> k2(n, Temp{});
    DBuf<int64_t> v2(n, Temp{});
    DBuf<uint32_t> hist((size_t)256 * nblk, Temp{});
    uint64_t *ka = keys, *kb = k2.p;
    int64_t *va = vals, *vb = v2.p;
    int passes = (bits + 7) / 8;
    for (int ps = 0; ps < passes; ++ps) {
        int shift = 8 * ps;
        hipLaunchKernelGGL(k_rs_hist, dim3(nblk), dim3(kRsThreads), 0, s, ka, n, shift, hist.p, nblk);
        FMM_HIP(hipGetLastError());
        scan_impl<uint32_t>(hist.p, hist.p, (int64_t)256 * nblk, nullptr, s);
        hipLaunchKernelGGL(k_rs_scatter, dim3(nblk), dim3(kRsThreads), 0, s, ka, va, kb, vb, n, shift,
                           hist.p, nblk);
        FMM_HIP(hipGetLastError());
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    if (ka != keys) {
        FMM_HIP(hipMemcpyAsync(keys, ka, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
        FMM_HIP(hipMemcpyAsync(vals, va, n * sizeof(int64_t), hipMemcpyDeviceToDevice, s));
    }
    if (!k2.home) FMM_HIP(hipStreamSynchronize(s));  // the temporaries are freed on return
}

}  // namespace fmm
