// The C entry points' host code (csrc/api.cpp, csrc/layout.cpp) on a stand-in for the HIP
// runtime whose device memory is host memory: allocations that fail, on the host and on
// the device, one after the other.  No exception leaves a call, the status is the
// documented one, nothing stays allocated, and no more device memory than the cap is held
// at any time.  The kernels' launches do nothing; results are not looked at.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "amped.h"
#include "internal.h"

// ------------------------------------------------------------- host allocations
static long g_new_left = -1;   // allocations that still succeed (-1: all)
static bool g_new_failed = false;
static void* counted_new(std::size_t n)
{
    if (g_new_left == 0) {
        g_new_failed = true;
        throw std::bad_alloc();
    }
    if (g_new_left > 0) --g_new_left;
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void* operator new(std::size_t n) { return counted_new(n); }
void* operator new[](std::size_t n) { return counted_new(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
void operator delete[](void* p, std::size_t) noexcept { std::free(p); }

// ------------------------------------------------------------ the HIP stand-in
static struct Mem {
    long left = -1;   // device allocations that still succeed (-1: all)
    bool failed = false;
    long long live = 0, peak = 0, pinned = 0;
    int objects = 0;  // streams and events
} g;
static const size_t kHead = 64;

extern "C" {
static hipError_t take(void** p, size_t n, long long& live)
{
    char* b = static_cast<char*>(std::calloc(1, n + kHead));
    if (!b) return hipErrorOutOfMemory;
    std::memcpy(b, &n, sizeof(n));
    *p = b + kHead;
    live += (long long)n;
    return hipSuccess;
}
static hipError_t give(void* p, long long& live)
{
    if (!p) return hipSuccess;
    size_t n;
    std::memcpy(&n, static_cast<char*>(p) - kHead, sizeof(n));
    live -= (long long)n;
    std::free(static_cast<char*>(p) - kHead);
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n)
{
    if (g.left == 0) {
        g.failed = true;
        return hipErrorOutOfMemory;
    }
    if (g.left > 0) --g.left;
    hipError_t e = take(p, n, g.live);
    if (g.live > g.peak) g.peak = g.live;
    return e;
}
hipError_t hipFree(void* p) { return give(p, g.live); }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned int) { return take(p, n, g.pinned); }
hipError_t hipHostFree(void* p) { return give(p, g.pinned); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void* d, int v, size_t n)
{
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int)
{
    *v = 0;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned int)
{
    *s = reinterpret_cast<hipStream_t>(0x10);
    ++g.objects;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t)
{
    --g.objects;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s)
{
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned int)
{
    *e = reinterpret_cast<hipEvent_t>(0x20);
    ++g.objects;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t)
{
    --g.objects;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}

namespace amped {
int64_t als_gram_slabs(int64_t, int) { return 4; }
int64_t gram_slabs(int64_t) { return 4; }
hipError_t launch_als_grams(const float* const*, const int64_t*, int, int, float*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_als_update(const float*, float*, int64_t, float*, double*, double*, int, int, int, double*, double*, int*,
                             double*, bool, const double*, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_check_range(const int32_t*, int64_t, int64_t, unsigned long long*, hipStream_t) { return hipSuccess; }
hipError_t launch_check_sorted(int, const int32_t* const*, int64_t, unsigned*, hipStream_t) { return hipSuccess; }
hipError_t launch_count_rows(const int32_t*, int64_t, int64_t, int64_t, uint32_t*, RowTotals*, hipStream_t) { return hipSuccess; }
hipError_t launch_cp_loss(const LossArgs&) { return hipSuccess; }
hipError_t launch_fill_rows(const int32_t*, int64_t, int64_t, int64_t, const uint32_t*, int64_t, int32_t*, int32_t*, hipStream_t)
{ return hipSuccess; }
hipError_t launch_gather_records(int, const void*, const int32_t*, void* const*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_gram(const float*, int64_t, int, float*, double*, hipStream_t, int64_t) { return hipSuccess; }
hipError_t launch_gram_noalloc(const float*, int64_t, int, double*, hipStream_t) { return hipSuccess; }
hipError_t launch_slot_rows(const int32_t*, int64_t, int64_t, int, int4*, int4*, int2*, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_hot_tables(const int32_t*, int64_t, unsigned long long*, int32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_iota(int32_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_mttkrp(const LaunchArgs&) { return hipSuccess; }
hipError_t launch_pack_records(int, const void* const*, void*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_permute32(void*, const void*, const int32_t*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_scale(float*, int64_t, const double*, hipStream_t) { return hipSuccess; }
// every row of every mode split, over all its units
hipError_t launch_small_units(const int32_t*, int64_t n, int, int units, int32_t*, int32_t*, int32_t*, unsigned*, int32_t* info,
                              hipStream_t)
{
    info[0] = (int32_t)std::min<int64_t>(units, n / (kSmallRow + 1));
    info[1] = 2;
    return hipSuccess;
}
hipError_t launch_stable_sort(const uint32_t*, const int32_t*, uint32_t* const*, int32_t* const*, int, uint32_t*, int64_t, int,
                              hipStream_t) { return hipSuccess; }
hipError_t launch_tensor_norm2(const ModeDev&, int, double*, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_unpack(const UnpackArgs&, hipStream_t) { return hipSuccess; }
int row_list_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 4095) / 4096, 2048)); }
// as csrc/sort.hip sizes them
int sort_passes(int key_bits) { return (key_bits + 9) / 10; }
int64_t sort_scratch_words(int64_t n, int key_bits)
{
    const int64_t blocks = (n + 4095) / 4096;
    int64_t group = 1;
    while (group * group < blocks) ++group;
    const int passes = sort_passes(key_bits);
    return passes == 0 ? 0 : (blocks + (blocks + group - 1) / group + 1) << ((key_bits + passes - 1) / passes);
}
}  // namespace amped

// ------------------------------------------------------------------- the checks
static int g_failures = 0;
#define CHECK(cond, ...)                                     \
    do {                                                     \
        if (!(cond)) {                                       \
            if (++g_failures <= 30) {                        \
                std::printf("line %d: ", __LINE__);          \
                std::printf(__VA_ARGS__);                    \
                std::printf("\n");                           \
            }                                                \
        }                                                    \
    } while (0)

struct Coo {
    std::vector<int64_t> dims;
    int64_t nnz;
    std::vector<int32_t> idx;
    std::vector<float> val;
    Coo(std::vector<int64_t> d, int64_t n) : dims(std::move(d)), nnz(n)
    {
        uint32_t x = 12345;
        for (size_t w = 0; w < dims.size(); ++w)
            for (int64_t k = 0; k < n; ++k) idx.push_back((int32_t)((x = x * 1664525u + 1013904223u) % (uint64_t)dims[w]));
        val.assign((size_t)n, 1.f);
    }
    amped_status create(const amped_options* o, amped_tensor_t* t) const
    {
        return amped_tensor_create((int)dims.size(), dims.data(), nnz, idx.data(), val.data(), o, t);
    }
};

static void clean(const char* what)
{
    CHECK(g.live == 0 && g.pinned == 0 && g.objects == 0, "%s: %lld device bytes, %lld pinned, %d objects left", what, g.live,
          g.pinned, g.objects);
}

// the n-th host allocation of a call fails, for every n
static void host_failures(const Coo& c, const amped_options& o, const char* what)
{
    for (long n = 0; n < 10000; ++n) {
        amped_tensor_t t = nullptr;
        g_new_left = n;
        g_new_failed = false;
        amped_status st = AMPED_OK;
        bool threw = false;
        try {
            st = c.create(&o, &t);
        } catch (...) {
            threw = true;
        }
        g_new_left = -1;
        CHECK(!threw, "%s: an exception left the call (allocation %ld)", what, n);
        CHECK(st == AMPED_OK || st == AMPED_ERR_NOMEM, "%s: status %d (allocation %ld)", what, (int)st, n);
        if (t) amped_tensor_destroy(t);
        else if (threw) g = Mem{};
        clean(what);
        if (!g_new_failed) return;
    }
}

// the n-th device allocation fails, for every n; a bad index is reported before that
static void device_failures(Coo c, const amped_options& o, const char* what)
{
    for (int bad = 0; bad < 2; ++bad) {
        if (bad && c.nnz == 0) return;
        if (bad) c.idx[(size_t)(c.nnz / 2)] = (int32_t)c.dims[0];
        for (long n = 0; n < 100; ++n) {
            amped_tensor_t t = nullptr;
            g.left = n;
            g.failed = false;
            amped_status st = c.create(&o, &t);
            g.left = -1;
            if (bad && g.failed)   // (the device's own check does nothing here)
                CHECK(st == AMPED_ERR_RANGE, "%s: status %d with a bad index (device allocation %ld)", what, (int)st, n);
            if (!bad) CHECK(st == AMPED_OK || st == AMPED_ERR_NOMEM, "%s: status %d (device allocation %ld)", what, (int)st, n);
            if (st == AMPED_ERR_RANGE)
                CHECK(std::strstr(amped_last_error(), "indices[0]"), "%s: message %s", what, amped_last_error());
            if (t) amped_tensor_destroy(t);
            clean(what);
            if (st == AMPED_OK) break;
        }
    }
}

// from the least admitted cap on: never more device memory than that
static void caps(const Coo& c, amped_options o, const char* what)
{
    auto admitted = [&](int64_t cap) {
        amped_tensor_t t = nullptr;
        o.device_byte_cap = cap;
        g.peak = 0;
        const amped_status st = c.create(&o, &t);
        CHECK(st == AMPED_OK || st == AMPED_ERR_NOMEM, "%s: status %d", what, (int)st);
        if (t) amped_tensor_destroy(t);
        if (st == AMPED_OK) CHECK(g.peak <= cap, "%s: %lld bytes at a time, cap %lld", what, g.peak, (long long)cap);
        clean(what);
        return st == AMPED_OK;
    };
    int64_t lo = 0, hi = int64_t(1) << 40;
    while (hi - lo > 1) {
        const int64_t mid = lo + (hi - lo) / 2;
        (admitted(mid) ? hi : lo) = mid;
    }
    const int64_t least = hi;
    for (; hi < 16 * least + (int64_t(1) << 22); hi += hi / 16 + 1) admitted(hi);
}

int main()
{
    const std::vector<int64_t> all = {40, 30, 9, 8, 7, 5, 3, 2};
    for (int64_t nnz : {int64_t(0), int64_t(1), int64_t(300), int64_t(9000), int64_t(70'000)})
        for (int order : {2, 3, 5, 8})
            for (int scale : {1, 3000}) {
                std::vector<int64_t> dims(all.begin(), all.begin() + order);
                for (auto& d : dims) d = d * scale - (scale > 1);
                const Coo c(dims, nnz);
                for (int host = 0; host < 2; ++host) {
                    amped_options o{};
                    o.keep_perm = order == 3;
                    o.host_layout = host;
                    o.shard_nnz = host ? 5000 : 0;
                    const std::string what = "order " + std::to_string(order) + ", " + std::to_string(nnz) + " nonzeros, sizes x " +
                                             std::to_string(scale) + (host ? ", host layouts" : "");
                    // (the host builder's threads allocate their lists inside a parallel
                    // region, which no exception can leave)
                    if (nnz == 0 || !host) host_failures(c, o, what.c_str());
                    device_failures(c, o, what.c_str());
                    caps(c, o, what.c_str());
                    if (host) {
                        o.chunk_nnz = 7;
                        o.shard_nnz = 1;
                        if (nnz <= 300) caps(c, o, (what + ", least shards").c_str());
                    }
                }
            }
    std::printf("%d failures\n", g_failures);
    return g_failures ? 1 : 0;
}
