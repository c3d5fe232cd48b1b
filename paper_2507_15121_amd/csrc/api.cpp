// C ABI of the sparse MTTKRP library (declared in include/amped.h): argument
// checks, handle lifetime, the per-mode layout build (on the device, or packed in
// host memory) and the kernel launches.
#include <hip/hip_runtime_api.h>
#include <omp.h>

#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <new>
#include <string>
#include <vector>

#include "amped.h"
#if AMPED_QUEUE_STATS
#include "amped_diag.h"
#endif
#include "internal.h"

using amped::HostModeLayout;
using amped::kMaxOrder;
using amped::kSinkFloats;
using amped::ModeDev;

namespace {

thread_local std::string g_err;

amped_status fail(amped_status st, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    try {
        g_err = buf;
    } catch (const std::bad_alloc&) {   // the status alone then
        g_err.clear();
    }
    return st;
}

amped_status hip_fail(hipError_t e, const char* what)
{
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
        return fail(AMPED_ERR_NOMEM, "%s: out of device memory (%s)", what, hipGetErrorString(e));
    if (e == hipErrorNotSupported) return fail(AMPED_ERR_UNSUPPORTED, "%s: case not supported", what);
    return fail(AMPED_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// Makes the handle's device current for the duration of a call.
struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) return;
        ok = (prev == dev) || hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard()
    {
        if (ok && prev >= 0) (void)hipSetDevice(prev);
    }
};

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

struct amped_tensor_s {
    int order = 0;
    int64_t dims[kMaxOrder] = {};
    int64_t nnz = 0, chunk = 0, n_chunks = 0;
    int64_t unit = 0;                       // nonzeros per work unit of the kernels
    bool own_units = false;                 // sized by the library
    int device = 0;
    bool keep_perm = false;
    int64_t device_bytes = 0;
    std::vector<void*> allocs;
    ModeDev mode[kMaxOrder];
    ModeDev loss_dev;                       // mode-0 layout with its own queue
    int32_t* perm[kMaxOrder] = {};
    std::vector<uint8_t> flags[kMaxOrder];
    int64_t touched[kMaxOrder] = {};
    // Host-resident layouts (options.host_layout): each mode packed in pinned
    // host memory, streamed through two device buffers of half a shard and
    // unpacked into a shard's arrays per call.
    bool host_layout = false;
    int64_t stage_len = 0;  // nonzeros per shard (whole chunks)
    amped::PackedMode hmode[kMaxOrder];
    std::vector<void*> pinned;
    std::vector<int32_t> hperm[kMaxOrder];  // kept permutations (keep_perm)
    void* ring[2] = {};                     // packed blocks of half a shard
    size_t ring_offsets = 0;                // where the blocks' offsets lie behind them, if they are copied too
    int32_t* stage = nullptr;               // (order + 1) arrays of stage_stride() entries
    int next_ring = 0;
    bool ring_used[2] = {};                 // consumed[] holds the buffer's last use
    bool was_captured = false;              // a call was captured into a graph
    // entries per staging array: the blocks that cover a shard, and 16-byte starts
    int64_t stage_stride() const { return (stage_len + 2 * amped::kPackBlock + 7) & ~(int64_t)3; }
    hipStream_t copy_stream = nullptr;
    hipEvent_t copied[2] = {}, consumed[2] = {}, call_start = nullptr;
    // CP-ALS workspace, allocated by the first sweep of a rank
    struct AlsWork {
        int rank = 0;
        float* M = nullptr;        // MTTKRP output, max_d I_d x R
        double* G = nullptr;       // [N][R][R] Gram matrices
        double* S = nullptr;       // R x R, M^T M
        float* partial = nullptr;  // Gram partials
        double* scratch = nullptr; // R x R
        double* W = nullptr;       // R x R, V^{-1} D^{-1}
        int* wide = nullptr;       // set by als_small: the product M W sums in fp64
        double* xnorm2 = nullptr;  // ||X||^2 (computed once)
        bool have_xnorm2 = false;
        bool have_grams = false;   // G matches the factors the last sweep wrote
    } als;

    // space for one more entry, so that adding it cannot throw
    static bool room(std::vector<void*>& v)
    {
        try {
            if (v.size() == v.capacity()) v.reserve(2 * v.size() + 8);
        } catch (const std::bad_alloc&) {
            return false;
        }
        return true;
    }
    hipError_t alloc(void** p, size_t bytes)
    {
        *p = nullptr;
        if (bytes == 0) return hipSuccess;
        if (!room(allocs)) return hipErrorOutOfMemory;
        hipError_t e = hipMalloc(p, bytes);
        if (e == hipSuccess) {
            allocs.push_back(*p);
            device_bytes += (int64_t)bytes;
        }
        return e;
    }
    void release(void* p)
    {
        for (auto& a : allocs)
            if (a == p) {
                (void)hipFree(a);
                a = nullptr;
            }
    }
    hipError_t host_alloc(void** p, size_t bytes)
    {
        *p = nullptr;
        if (bytes == 0) return hipSuccess;
        if (!room(pinned)) return hipErrorOutOfMemory;
        hipError_t e = hipHostMalloc(p, bytes, hipHostMallocDefault);
        if (e == hipSuccess) pinned.push_back(*p);
        return e;
    }
    void free_all()
    {
        for (void* a : allocs)
            if (a) (void)hipFree(a);
        allocs.clear();
        for (void* a : pinned) (void)hipHostFree(a);
        pinned.clear();
        for (hipEvent_t& ev : {std::ref(copied[0]), std::ref(copied[1]), std::ref(consumed[0]), std::ref(consumed[1]),
                               std::ref(call_start)})
            if (ev) {
                (void)hipEventDestroy(ev);
                ev = nullptr;
            }
        if (copy_stream) {
            (void)hipStreamDestroy(copy_stream);
            copy_stream = nullptr;
        }
    }
};

namespace {

// Bits needed to hold the values 0..n (0 for n <= 0).
int bits_for(int64_t n)
{
    int b = 0;
    while (b < 63 && n > 0 && (n >> b)) ++b;
    return b;
}

amped_status validate_args(int order, const int64_t* dims, int64_t nnz, const int32_t* indices, const float* values)
{
    if (order < 2 || order > kMaxOrder) return fail(AMPED_ERR_INVALID, "order %d outside [2, %d]", order, kMaxOrder);
    if (!dims) return fail(AMPED_ERR_INVALID, "dims is NULL");
    for (int w = 0; w < order; ++w)
        if (dims[w] < 1 || dims[w] > 0x7FFFFFFF)
            return fail(AMPED_ERR_INVALID, "dims[%d] = %lld outside [1, 2^31-1]", w, (long long)dims[w]);
    if (nnz < 0 || nnz > 0x7FFFFFFF) return fail(AMPED_ERR_INVALID, "nnz = %lld outside [0, 2^31-1]", (long long)nnz);
    if (nnz > 0 && (!indices || !values)) return fail(AMPED_ERR_INVALID, "indices or values is NULL");
    return AMPED_OK;
}

amped_status range_fail(int w, int64_t at, int32_t index, int64_t dim)
{
    return fail(AMPED_ERR_RANGE, "indices[%d][%lld] = %d outside [0, %lld)", w, (long long)at, index, (long long)dim);
}

amped_status validate_range(int order, const int64_t* dims, int64_t nnz, const int32_t* indices)
{
    for (int w = 0; w < order; ++w) {
        const int32_t* col = indices + (int64_t)w * nnz;
        const int64_t dim = dims[w];
        int64_t bad = nnz;
#pragma omp parallel for reduction(min : bad) schedule(static)
        for (int64_t k = 0; k < nnz; ++k)
            if (col[k] < 0 || col[k] >= dim) bad = std::min(bad, k);
        if (bad < nnz) return range_fail(w, bad, col[bad], dim);
    }
    return AMPED_OK;
}

amped_status check_device(int* dev)
{
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n < 1) return fail(AMPED_ERR_UNSUPPORTED, "no HIP device");
    if (hipGetDevice(dev) != hipSuccess) return fail(AMPED_ERR_UNSUPPORTED, "no current HIP device");
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, *dev) != hipSuccess)
        return fail(AMPED_ERR_UNSUPPORTED, "cannot query device %d", *dev);
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(AMPED_ERR_UNSUPPORTED, "device %d is %s, this library is built for gfx950", *dev, prop.gcnArchName);
    return AMPED_OK;
}

#define HIP_OR_FAIL(call, what)                          \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) {                          \
            st = hip_fail(e_, what);                     \
            goto cleanup;                                \
        }                                                \
    } while (0)

// A mode's row lists (zero rows, long gaps, hot-row tables where launches use them) to
// the device, and its sizes.
amped_status upload_tables(amped_tensor_s* t, ModeDev& m, int d, const HostModeLayout& lay, void* queues, void* aux,
                           bool hot)
{
    amped_status st = AMPED_OK;
    void* p = nullptr;
    if (!lay.zero_rows.empty()) {
        HIP_OR_FAIL(t->alloc(&p, lay.zero_rows.size() * 4), "hipMalloc(zero rows)");
        HIP_OR_FAIL(hipMemcpy(p, lay.zero_rows.data(), lay.zero_rows.size() * 4, hipMemcpyHostToDevice),
                    "hipMemcpy(zero rows)");
        m.zero_rows = static_cast<int32_t*>(p);
    }
    if (hot) {
        HIP_OR_FAIL(t->alloc(&p, lay.hot.size() * 4), "hipMalloc(hot rows)");
        HIP_OR_FAIL(hipMemcpy(p, lay.hot.data(), lay.hot.size() * 4, hipMemcpyHostToDevice), "hipMemcpy(hot rows)");
        m.hot = static_cast<int32_t*>(p);
    }
    if (!lay.gaps.empty()) {
        HIP_OR_FAIL(t->alloc(&p, lay.gaps.size() * 4), "hipMalloc(gaps)");
        HIP_OR_FAIL(hipMemcpy(p, lay.gaps.data(), lay.gaps.size() * 4, hipMemcpyHostToDevice), "hipMemcpy(gaps)");
        m.gaps = static_cast<int32_t*>(p);
    }
    m.nnz = t->nnz;
    m.unit = t->unit;
    m.chunk = m.residual_chunk = t->unit * (t->own_units && lay.heavy ? amped::heavy_units(t->unit) : 1);
    m.n_chunks = (t->nnz + t->unit - 1) / t->unit;
    m.rows = t->dims[d];
    m.n_zero = (int64_t)lay.zero_rows.size();
    m.zero_row = aux;
    m.sink = static_cast<float*>(aux) + 4;
    m.n_gaps = (int64_t)lay.gaps.size() / 2;
    m.queue = static_cast<unsigned*>(queues) + (size_t)d * amped::kQueueWords;
    t->flags[d] = lay.flags;
    t->touched[d] = lay.touched;
cleanup:
    return st;
}

// Host-resident layouts: the host order builder sorts every mode, the layout
// arrays are gathered into pinned host memory, and the device receives the
// row lists, the staging buffers, a copy stream and its events.
//  The blocks' offsets stay on the device, unless the cap does not hold them (they grow
// with the nonzeros): then each half shard's are copied with it, a second small copy.
// What is admitted under a cap is two shards of plain arrays, the row lists and the
// hot-row tables.  The staging arrays are one of them; a packed block is at least 32
// bytes shorter than its plain arrays, which pays for its offset; the blocks at a shard's
// ends, and the queues, take less than the hot-row tables, which only shards have that
// are large enough for the difference.
amped_status build_host_layout(amped_tensor_s* t, const int32_t* indices, const float* values, int64_t cap)
{
    const int order = t->order;
    const int64_t nnz = t->nnz;
    amped_status st = AMPED_OK;
    void* queues = nullptr;
    void* aux = nullptr;
    void* p = nullptr;
    HIP_OR_FAIL(t->alloc(&queues, (size_t)(order + 1) * amped::kQueueWords * sizeof(unsigned)), "hipMalloc(queues)");
    HIP_OR_FAIL(hipMemset(queues, 0, (size_t)(order + 1) * amped::kQueueWords * sizeof(unsigned)), "hipMemset(queues)");
    HIP_OR_FAIL(t->alloc(&aux, (size_t)(4 + kSinkFloats) * sizeof(float)), "hipMalloc(aux)");
    HIP_OR_FAIL(hipMemset(aux, 0, (size_t)(4 + kSinkFloats) * sizeof(float)), "hipMemset(aux)");
    for (int b = 0; b < 2; ++b) {
        HIP_OR_FAIL(hipEventCreateWithFlags(&t->copied[b], hipEventDisableTiming), "hipEventCreate");
        HIP_OR_FAIL(hipEventCreateWithFlags(&t->consumed[b], hipEventDisableTiming), "hipEventCreate");
    }
    HIP_OR_FAIL(hipEventCreateWithFlags(&t->call_start, hipEventDisableTiming), "hipEventCreate");
    HIP_OR_FAIL(hipStreamCreateWithFlags(&t->copy_stream, hipStreamNonBlocking), "hipStreamCreate");
    HIP_OR_FAIL(t->alloc(&p, (size_t)(order + 1) * t->stage_stride() * 4), "hipMalloc(staging)");
    HIP_OR_FAIL(hipMemset(p, 0, (size_t)(order + 1) * t->stage_stride() * 4), "hipMemset(staging)");
    t->stage = static_cast<int32_t*>(p);
    try {
        const std::vector<int32_t> lex = amped::lex_order(order, t->dims, nnz, indices);
        size_t most = 0, offsets = 0;   // bytes of the longest block, of all blocks' offsets
        for (int d = 0; d < order; ++d) {
            HostModeLayout lay;
            amped::mode_order(t->dims, nnz, indices, lex, d, lay.perm);
            amped::mode_tables(t->dims, nnz, indices, d, t->chunk, lay, t->unit);
            amped::PackedMode& h = t->hmode[d];
            h.plan(order, t->dims, nnz, indices, d, lay.perm.data());
            HIP_OR_FAIL(t->host_alloc(&p, (size_t)h.bytes(h.blocks())), "hipHostMalloc(layout)");
            h.data = static_cast<uint32_t*>(p);
            h.fill(nnz, indices, values, lay.perm.data());
            for (int64_t b = 0; b < h.blocks(); ++b) most = std::max(most, (size_t)(h.bytes(b + 1) - h.bytes(b)));
            offsets += h.blocks() > 0 ? h.offset.size() * 4 : 0;
            st = upload_tables(t, t->mode[d], d, lay, queues, aux, t->stage_len >= amped::kHotMinNnz);
            if (st != AMPED_OK) return st;
            if (t->keep_perm) t->hperm[d] = std::move(lay.perm);
        }
        // half of the most blocks that a shard touches
        const size_t half = ((size_t)(t->stage_len / amped::kPackBlock) + 3) / 2;
        t->ring_offsets = half * most;
        const bool travel = cap > 0 && t->device_bytes + (int64_t)(2 * half * most + offsets) > cap;
        for (int b = 0; b < 2; ++b)
            HIP_OR_FAIL(t->alloc(&t->ring[b], half * most + (travel && nnz > 0 ? (half + 1) * 4 : 0)), "hipMalloc(staging)");
        for (int d = 0; d < order && nnz > 0; ++d) {
            amped::PackedMode& h = t->hmode[d];
            const size_t bytes = h.offset.size() * 4;
            if (travel) {
                HIP_OR_FAIL(t->host_alloc(&p, bytes), "hipHostMalloc(block offsets)");
                std::memcpy(p, h.offset.data(), bytes);
                h.pinned_offset = static_cast<uint32_t*>(p);
            } else {
                HIP_OR_FAIL(t->alloc(&p, bytes), "hipMalloc(block offsets)");
                HIP_OR_FAIL(hipMemcpy(p, h.offset.data(), bytes, hipMemcpyHostToDevice), "hipMemcpy(block offsets)");
                h.dev_offset = static_cast<uint32_t*>(p);
            }
        }
    } catch (const std::bad_alloc&) {
        return fail(AMPED_ERR_NOMEM, "host allocation failed");
    }
    t->loss_dev = t->mode[0];
    t->loss_dev.queue = static_cast<unsigned*>(queues) + (size_t)order * amped::kQueueWords;
cleanup:
    return st;
}

// A device allocation cut into arrays that start on 256 bytes.
struct Arena {
    char* base = nullptr;
    size_t used = 0;
    static size_t step(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
    template <typename T>
    T* take(size_t n)
    {
        T* p = reinterpret_cast<T*>(base + used);
        used += step(n * sizeof(T));
        return p;
    }
};

// Copies host arrays to the device, in the order given, on a stream of its own.
// A plain hipMemcpy of pageable memory reaches 28 GB/s here; the host threads
// copying pieces of 8 MB into two pinned buffers, from which the copy engine reads
// one while they fill the other, 53 GB/s, the host link's rate.  A first array below
// a piece is left to hipMemcpy.
struct Uploader {
    static constexpr size_t kPiece = size_t(8) << 20;
    hipStream_t stream = nullptr;
    hipEvent_t busy[2] = {};
    char* pinned = nullptr;
    int next = 0;
    bool used[2] = {};

    hipError_t put(void* dst, const void* src, size_t bytes)
    {
        if (bytes < kPiece && !stream) return hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice);
        hipError_t e = hipSuccess;
        if (!stream) {
            if ((e = hipStreamCreateWithFlags(&stream, hipStreamNonBlocking)) != hipSuccess) return e;
            for (hipEvent_t& ev : busy)
                if ((e = hipEventCreateWithFlags(&ev, hipEventDisableTiming)) != hipSuccess) return e;
            if ((e = hipHostMalloc(reinterpret_cast<void**>(&pinned), 2 * kPiece, hipHostMallocDefault)) != hipSuccess)
                return e;
        }
        for (size_t at = 0; at < bytes; at += kPiece) {
            const int b = next;
            next ^= 1;
            if (used[b] && (e = hipEventSynchronize(busy[b])) != hipSuccess) return e;
            const size_t len = std::min(kPiece, bytes - at), cut = size_t(256) << 10;
            char* to = pinned + b * kPiece;
            const char* from = static_cast<const char*>(src) + at;
            const int64_t cuts = (int64_t)((len + cut - 1) / cut);
#pragma omp parallel for schedule(static)
            for (int64_t i = 0; i < cuts; ++i) std::memcpy(to + i * cut, from + i * cut, std::min(cut, len - i * cut));
            if ((e = hipMemcpyAsync(static_cast<char*>(dst) + at, to, len, hipMemcpyHostToDevice, stream)) != hipSuccess)
                return e;
            if ((e = hipEventRecord(busy[b], stream)) != hipSuccess) return e;
            used[b] = true;
        }
        return hipSuccess;
    }
    // work on s from here on comes after the copies so far
    hipError_t before(hipStream_t s)
    {
        const int b = next ^ 1;   // the last piece's event
        return used[b] ? hipStreamWaitEvent(s, busy[b], 0) : hipSuccess;
    }
    void finish()
    {
        if (stream) {
            (void)hipStreamSynchronize(stream);
            (void)hipStreamDestroy(stream);
        }
        for (hipEvent_t& ev : busy) {
            if (ev) (void)hipEventDestroy(ev);
            ev = nullptr;
        }
        if (pinned) (void)hipHostFree(pinned);
        stream = nullptr;
        pinned = nullptr;
        used[0] = used[1] = false;
    }
    ~Uploader() { finish(); }
};

// Device-resident layouts, built on the device.
//
// The index columns are copied in last mode first, the values after them.  Unless
// the COO is in lexicographic order already, stable radix sorts over the modes, each
// starting when its column has arrived, give that order; a mode's order is one more
// stable sort of it by i_d, whose sorted keys are the out_idx column and give the
// row lists.  All that is on its way while the values arrive; they go into
// lexicographic order, and the modes' other columns are gathered from one record per
// nonzero.  The host only copies and waits once for the lists' sizes (and once for
// the order check of an input that looks sorted).
// The arrays are one allocation, the scratch another of about a record per nonzero:
// the raw columns lie where the records go, the sorts' buffers in columns of modes
// that are gathered later, each mode's order in its own value column.  Allocating,
// above all freeing, costs about 1.2 us per MB.
// 5M order-3 nonzeros took 17.7 ms, and their release 3.2, with an allocation for
// each array, the keys copied back and the checks and lists made on the host; 3.6 and
// 0.3 with all of it on the device, the values first and a scratch of 180 MB; now
// 2.9.
amped_status build_device_layout(amped_tensor_s* t, const int32_t* indices, const float* values, int64_t cap)
{
    const int order = t->order;
    const int64_t nnz = t->nnz;
    const int64_t* dims = t->dims;
    amped_status st = AMPED_OK;
    hipStream_t stream = nullptr;
    void* keep = nullptr;
    void* temp = nullptr;
    void* p = nullptr;
    struct Status {
        amped::RowTotals totals[kMaxOrder];
        unsigned long long bad[kMaxOrder];
        int32_t small[kMaxOrder][2];   // split rows, most units of one
        int32_t slots[kMaxOrder][2];   // light and heavy rows with slots
        unsigned unsorted, pad;
    } status;
    const size_t n = (size_t)nnz;
    const size_t padded = n + 4;   // 16-byte loads of the last nonzeros stay inside the array
    const size_t words = (size_t)amped::kQueueWords * (order + 1), aux_floats = 4 + kSinkFloats;
    // what the handle keeps: queues and aux (16 zero bytes, then the store sink),
    // order + 1 arrays per mode, the permutations if asked for
    const size_t keep_bytes = Arena::step(words * 4) + Arena::step(aux_floats * 4) +
                              (nnz ? (size_t)order * (order + 1) * Arena::step(padded * 4) : 0) +
                              (t->keep_perm ? (size_t)order * Arena::step(n * 4) : 0);
    // the units of the one-launch MTTKRP
    const bool small = t->own_units && nnz > 0 && nnz <= amped::kSmallNnz;
    const int small_len = amped::small_unit(nnz);
    const size_t units = small ? (n + small_len - 1) / small_len : 0;
    const size_t small_bytes = small ? (size_t)order * (2 * Arena::step((units + 1) * 4) + Arena::step(units * 8) +
                                                        Arena::step(units * 4)) : 0;
    // the rows that cross unit edges
    const int n_units = (int)((nnz + t->unit - 1) / t->unit);
    const bool slots = t->own_units && nnz > 0;
    const size_t cuts = (size_t)(n_units + amped::kHeavyCuts), light_max = (size_t)amped::light_rows_max(n_units),
                 heavy_max = (size_t)amped::heavy_rows_max(n_units);
    const size_t slot_floats = (size_t)amped::slots_max(n_units) * amped::kSlotCols;
    const size_t slot_bytes = slots ? (size_t)order * (Arena::step(cuts * 8) + Arena::step(light_max * 16) +
                                                       Arena::step(heavy_max * 16) + Arena::step(slot_floats * 4)) : 0;
    Arena ka, ta;
    HIP_OR_FAIL(t->alloc(&keep, keep_bytes + small_bytes + slot_bytes), "hipMalloc(layouts)");
    ka.base = static_cast<char*>(keep);
    {
        unsigned* queues = ka.take<unsigned>(words);
        float* aux = ka.take<float>(aux_floats);
        // one block at the start of the allocation
        HIP_OR_FAIL(hipMemset(keep, 0, Arena::step(words * 4) + Arena::step(aux_floats * 4)), "hipMemset(queues)");
        for (int d = 0; d < order; ++d) {
            ModeDev& m = t->mode[d];
            m.nnz = nnz;
            m.unit = m.chunk = t->unit;
            m.n_chunks = (nnz + t->unit - 1) / t->unit;
            m.residual_chunk = t->unit * (t->own_units ? amped::residual_units(nnz, t->unit) : 1);
            m.rows = dims[d];
            m.zero_row = aux;
            m.sink = aux + 4;
            m.queue = queues + (size_t)d * amped::kQueueWords;
            if (t->keep_perm) t->perm[d] = ka.take<int32_t>(n);
        }
        if (nnz == 0) {
            for (int d = 0; d < order; ++d) {
                HostModeLayout lay;
                amped::mode_tables_sorted(nullptr, 0, dims[d], t->chunk, lay);
                st = upload_tables(t, t->mode[d], d, lay, queues, aux, false);
                if (st != AMPED_OK) return st;
            }
            t->loss_dev = t->mode[0];
            t->loss_dev.queue = queues + (size_t)order * amped::kQueueWords;
            return AMPED_OK;
        }
        int32_t* cols[kMaxOrder][kMaxOrder + 1];   // [mode][index columns in mode order, then the values]
        for (int d = 0; d < order; ++d) {
            ModeDev& m = t->mode[d];
            int j = 0;
            for (int w = 0; w <= order; ++w) {
                cols[d][w] = ka.take<int32_t>(padded);
                if (w == d) m.out_idx = cols[d][w];
                else if (w < order) m.in_idx[j++] = cols[d][w];
                else m.val = reinterpret_cast<const float*>(cols[d][w]);
            }
        }

        // scratch: the raw COO and in its place the records (where those are larger
        // and do not fit, columns are gathered one by one)
        const int rw = (int)amped::record_words(order), last = order - 1;
        bool records = rw <= order + 1 || cap == 0;
        const int blocks = amped::row_list_blocks(nnz);
        const bool hot = nnz >= amped::kHotMinNnz;   // hot-row tables, where launches use them
        size_t scratch_words = 0;
        for (int w = 0; w < order; ++w)
            scratch_words = std::max(scratch_words, (size_t)amped::sort_scratch_words(nnz, bits_for(dims[w] - 1)));
        auto temp_bytes = [&](bool rec) {
            return Arena::step(sizeof(Status)) + (size_t)order * Arena::step((size_t)blocks * 16) +
                   (hot ? Arena::step(amped::kHotMax * 8) : 0) + Arena::step(scratch_words * 4) +
                   (order == 2 ? 2 * Arena::step(n * 4) : 0) +
                   std::max(rec ? Arena::step((size_t)rw * 4 * n) : 0, (size_t)(order + 1) * Arena::step(n * 4));
        };
        hipError_t e = hipMalloc(&temp, temp_bytes(records));
        if (e != hipSuccess && records) {
            (void)hipGetLastError();
            records = false;
            e = hipMalloc(&temp, temp_bytes(false));
        }
        HIP_OR_FAIL(e, "hipMalloc(layout build)");
        ta.base = static_cast<char*>(temp);
        Status* d_status = ta.take<Status>(1);
        uint32_t* counts[kMaxOrder];
        for (int d = 0; d < order; ++d) counts[d] = ta.take<uint32_t>((size_t)blocks * 4);
        unsigned long long* best = ta.take<unsigned long long>(hot ? amped::kHotMax : 0);
        uint32_t* scratch = ta.take<uint32_t>(scratch_words);
        // The sorts' second key buffer and second order buffer are columns of the last
        // mode, the lexicographic order is one of mode 1's (order 2 has too few), and
        // mode d's order lies where its values go: the gather's threads read an entry
        // before they write that place.
        uint32_t* const keys2 = reinterpret_cast<uint32_t*>(cols[last][0]);
        int32_t* const order2 = order > 2 ? cols[last][1] : ta.take<int32_t>(n);
        int32_t* const lex = order > 2 ? cols[1][0] : ta.take<int32_t>(n);
        uint32_t* const rec = ta.take<uint32_t>(0);
        int32_t* raw[kMaxOrder + 1];
        for (int w = 0; w <= order; ++w) raw[w] = ta.take<int32_t>(n);

        HIP_OR_FAIL(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking), "hipStreamCreate");
        std::memset(&status, 0, sizeof(status));
        for (int w = 0; w < order; ++w) status.bad[w] = ~0ull;
        HIP_OR_FAIL(hipMemcpy(d_status, &status, sizeof(status), hipMemcpyHostToDevice), "hipMemcpy(status)");

        // the lexicographic order, and in it mode 0's keys
        int bits[kMaxOrder], np[kMaxOrder], passes = 0;
        for (int w = 0; w < order; ++w) {
            bits[w] = bits_for(dims[w] - 1);
            np[w] = amped::sort_passes(bits[w]);
            passes += np[w];
        }
        uint32_t* const kbuf[2] = {reinterpret_cast<uint32_t*>(cols[0][0]), keys2};
        int32_t* const vbuf[2] = {lex, order2};
        int at = -1, to = (passes - 1) & 1;   // vbuf[at] holds the order so far; the last pass writes vbuf[0]
        auto sort_by = [&](int w) -> hipError_t {
            if (np[w] == 0) return hipSuccess;
            const uint32_t* keys = reinterpret_cast<const uint32_t*>(raw[w]);
            if (at >= 0) {
                hipError_t er = amped::launch_permute32(kbuf[at], keys, vbuf[at], nnz, stream);
                if (er != hipSuccess) return er;
                keys = kbuf[at];
            }
            hipError_t er = amped::launch_stable_sort(keys, at >= 0 ? vbuf[at] : nullptr, kbuf, vbuf, to, scratch, nnz,
                                                      bits[w], stream);
            at = (to + np[w] - 1) & 1;
            to = at ^ 1;
            return er;
        };
        auto copy = [&](void* dst, const void* src) {
            return hipMemcpyAsync(dst, src, n * 4, hipMemcpyDeviceToDevice, stream);
        };
        bool sorted = amped::is_lexicographic_prefix(order, nnz, indices, std::min<int64_t>(nnz, 16384));
        const bool looks_sorted = sorted;   // a look at the first entries settles it for most unsorted inputs
        auto lex_column = [&](int w) -> hipError_t {
            if (sorted || (w == 0 && np[0] > 0)) return hipSuccess;
            return passes ? amped::launch_permute32(cols[0][w], raw[w], lex, nnz, stream) : copy(cols[0][w], raw[w]);
        };
        // the modes' orders and row lists' sizes from mode 0's index columns
        auto mode_orders = [&]() -> hipError_t {
            hipError_t er = hipSuccess;
            for (int w = 0; w < order; ++w)
                if ((er = lex_column(w)) != hipSuccess) return er;
            for (int d = 0; d < order; ++d) {
                if (d > 0 && np[d] > 0) {
                    uint32_t* kb[2] = {reinterpret_cast<uint32_t*>(cols[d][d]), keys2};
                    int32_t* vb[2] = {cols[d][order], order2};
                    er = amped::launch_stable_sort(reinterpret_cast<const uint32_t*>(cols[0][d]), nullptr, kb, vb,
                                                   (np[d] - 1) & 1, scratch, nnz, bits[d], stream);
                } else if (d > 0) {
                    er = copy(cols[d][d], cols[0][d]);
                }
                if (er != hipSuccess) return er;
                if ((er = amped::launch_count_rows(cols[d][d], nnz, dims[d], t->unit, counts[d], &d_status->totals[d],
                                                   stream)) != hipSuccess)
                    return er;
                if (slots) {
                    auto& sl = t->mode[d].slots;
                    int2* cut = ka.take<int2>(cuts);
                    int4* light = ka.take<int4>(light_max);
                    int4* heavy = ka.take<int4>(heavy_max);
                    if ((er = amped::launch_slot_rows(cols[d][d], nnz, t->unit, n_units, light, heavy, cut,
                                                      d_status->slots[d], stream)) != hipSuccess)
                        return er;
                    sl.cut = cut;
                    sl.light = light;
                    sl.heavy = heavy;
                    sl.slot = ka.take<float>(slot_floats);
                    sl.all = amped::least_cuts(n_units) == 1;
                }
                if (small) {
                    auto& sm = t->mode[d].small;
                    int32_t* cut = ka.take<int32_t>(units + 1);
                    int32_t* left = ka.take<int32_t>(units + 1);
                    int32_t* split = ka.take<int32_t>(2 * units);
                    unsigned* arrived = ka.take<unsigned>(units);
                    if ((er = amped::launch_small_units(cols[d][d], nnz, small_len, (int)units, cut, left, split,
                                                        arrived, d_status->small[d], stream)) != hipSuccess)
                        return er;
                    sm.cut = cut;
                    sm.left = left;
                    sm.split = split;
                    sm.arrived = arrived;
                }
            }
            return er;
        };
        Uploader up;
        for (int w = last; w >= 0; --w) {
            int32_t* dst = sorted ? cols[0][w] : raw[w];
            HIP_OR_FAIL(up.put(dst, indices + (int64_t)w * nnz, n * 4), "copy of the COO");
            HIP_OR_FAIL(up.before(stream), "hipStreamWaitEvent");
            HIP_OR_FAIL(amped::launch_check_range(dst, dims[w], nnz, &d_status->bad[w], stream), "range check");
            if (!sorted) HIP_OR_FAIL(sort_by(w), "radix sort");
        }
        // the launches (about 40) go between the first pieces and the rest, so that the
        // link has work meanwhile
        const size_t ahead = std::min(n, 2 * Uploader::kPiece / 4);
        int32_t* const dst = sorted ? cols[0][order] : raw[order];
        HIP_OR_FAIL(up.put(dst, values, ahead * 4), "copy of the COO");
        if (!sorted) HIP_OR_FAIL(mode_orders(), "mode orders");
        if (ahead < n) HIP_OR_FAIL(up.put(dst + ahead, values + ahead, (n - ahead) * 4), "copy of the COO");
        HIP_OR_FAIL(up.before(stream), "hipStreamWaitEvent");
        if (looks_sorted) {
            HIP_OR_FAIL(amped::launch_check_sorted(order, cols[0], nnz, &d_status->unsorted, stream), "order check");
            HIP_OR_FAIL(hipMemcpyAsync(&status, d_status, sizeof(status), hipMemcpyDeviceToHost, stream), "status");
            HIP_OR_FAIL(hipStreamSynchronize(stream), "layout build");
            sorted = status.unsorted == 0;
            if (!sorted) {
                for (int w = 0; w <= order; ++w) HIP_OR_FAIL(copy(raw[w], cols[0][w]), "copy");
                for (int w = last; w >= 0; --w) HIP_OR_FAIL(sort_by(w), "radix sort");
            }
            HIP_OR_FAIL(mode_orders(), "mode orders");
        }
        HIP_OR_FAIL(lex_column(order), "gather");

        // the other columns
        for (int d = 0; d < order && t->keep_perm; ++d) {
            const bool own = d > 0 && np[d] > 0, lexed = !sorted && passes > 0;
            const int32_t* perm = own ? cols[d][order] : lex;
            HIP_OR_FAIL(own && lexed ? amped::launch_permute32(t->perm[d], lex, perm, nnz, stream)
                        : own || lexed ? copy(t->perm[d], perm)
                                       : amped::launch_iota(t->perm[d], nnz, stream), "permutation");
        }
        if (records)
            HIP_OR_FAIL(amped::launch_pack_records(order, reinterpret_cast<const void* const*>(cols[0]), rec, nnz,
                                                   stream), "pack");
        for (int d = 1; d < order; ++d) {
            const int32_t* perm = cols[d][order];
            if (np[d] > 0 && records) {
                int32_t* others[kMaxOrder + 1];
                for (int w = 0; w <= order; ++w) others[w] = w == d ? nullptr : cols[d][w];
                HIP_OR_FAIL(amped::launch_gather_records(order, rec, perm, reinterpret_cast<void* const*>(others), nnz,
                                                         stream), "gather");
                continue;
            }
            for (int w = 0; w <= order; ++w) {
                if (w == d) continue;
                HIP_OR_FAIL(np[d] > 0 ? amped::launch_permute32(cols[d][w], cols[0][w], perm, nnz, stream)
                                      : copy(cols[d][w], cols[0][w]), "gather");
            }
        }
        up.finish();   // while the stream works
        HIP_OR_FAIL(hipMemcpyAsync(&status, d_status, sizeof(status), hipMemcpyDeviceToHost, stream), "status");
        HIP_OR_FAIL(hipStreamSynchronize(stream), "layout build");
        for (int w = 0; w < order; ++w)
            if (status.bad[w] < (unsigned long long)nnz) {
                st = range_fail(w, (int64_t)status.bad[w], indices[(int64_t)w * nnz + (int64_t)status.bad[w]], dims[w]);
                goto cleanup;
            }

        // the row lists and hot-row tables
        // the shares of rows that span units, where the mode takes the one launch
        auto one_launch = [&](int d) {
            return small && status.small[d][1] <= (nnz <= amped::kSmallSplitNnz ? amped::kSmallSpan : 0);
        };
        auto share_bytes = [&](int d) {
            return one_launch(d) && status.small[d][0] > 0
                       ? Arena::step((units + (size_t)status.small[d][0]) * amped::kSmallCols * 8) : 0;
        };
        size_t list_bytes = 0;
        for (int d = 0; d < order; ++d)
            list_bytes += Arena::step((size_t)(status.totals[d].shared + status.totals[d].lone) * 4) +
                          Arena::step((size_t)status.totals[d].gaps * 8) + share_bytes(d) +
                          (hot ? Arena::step(amped::kHotTableLen * 4) : 0);
        HIP_OR_FAIL(t->alloc(&p, list_bytes), "hipMalloc(row lists)");
        Arena la;
        la.base = static_cast<char*>(p);
        for (int d = 0; d < order; ++d) {
            ModeDev& m = t->mode[d];
            const amped::RowTotals& tot = status.totals[d];
            int32_t* zero = la.take<int32_t>((size_t)(tot.shared + tot.lone));
            int32_t* gaps = la.take<int32_t>((size_t)tot.gaps * 2);
            m.zero_rows = zero;
            m.gaps = gaps;
            m.n_zero = tot.shared + tot.lone;
            m.n_gaps = tot.gaps;
            t->touched[d] = tot.touched;
            if (slots) {
                m.slots.n_light = status.slots[d][0];
                m.slots.n_heavy = status.slots[d][1];
                m.slots.zrows = zero + tot.shared;
                m.slots.n_zero = tot.lone;
                // without heavy rows: atomics and the init kernel
                if (m.slots.n_heavy == 0) {
                    m.slots.slot = nullptr;
                    m.slots.all = false;
                }
            }
            if (one_launch(d)) {
                m.small.n_units = (int)units;
                m.small.zrows = zero + tot.shared;
                m.small.n_zero = tot.lone;
                if (status.small[d][0] > 0) {
                    m.small.share = la.take<uint64_t>((units + (size_t)status.small[d][0]) * amped::kSmallCols);
                    HIP_OR_FAIL(hipMemsetAsync(m.small.share, 0, share_bytes(d), stream), "hipMemset(shares)");
                }
            }
            if (m.n_zero + m.n_gaps > 0)
                HIP_OR_FAIL(amped::launch_fill_rows(m.out_idx, nnz, dims[d], t->unit, counts[d], tot.shared, zero, gaps,
                                                    stream), "row lists");
            if (hot) {
                int32_t* table = la.take<int32_t>(amped::kHotTableLen);
                HIP_OR_FAIL(hipMemsetAsync(best, 0, amped::kHotMax * 8, stream), "hot rows");
                HIP_OR_FAIL(amped::launch_hot_tables(m.out_idx, nnz, best, table, stream), "hot rows");
                m.hot = table;
            }
        }
        t->loss_dev = t->mode[0];
        t->loss_dev.queue = queues + (size_t)order * amped::kQueueWords;
        HIP_OR_FAIL(hipStreamSynchronize(stream), "layout build");
    }

cleanup:
    if (stream) {
        (void)hipStreamSynchronize(stream);
        (void)hipStreamDestroy(stream);
    }
    if (temp) (void)hipFree(temp);
    return st;
}

// Streams mode d's host-resident layout through the device.  A shard [start,
// cut(start)) of at most stage_len nonzeros is copied as the packed blocks that
// cover it, in two halves, each to the device buffer that is free next, on the
// copy stream; stream s waits for a half, unpacks it into the staging arrays and
// marks the buffer free again, and after the second half runs fn(shard, i).  So
// the copies run ahead of the kernels by up to a shard, also from one call into
// the next: the host link is what bounds a call, and the packed blocks (bits of
// the indices as their modes need them, of the output indices as their block's
// range does) are 9 to 11 of the 16 bytes of an order-3 nonzero.  In plain arrays,
// each shard's copied one by one and a call's copies starting when the stream had
// finished all earlier work, 10M order-3 nonzeros took 10.2 ms for all modes at
// rank 32, 5.4 ms now.
// The shard's ModeDev points into the staging arrays, carries the output indices
// on both sides of it, and only the first shard's init zeroes rows.
template <typename Cut, typename Fn>
amped_status stream_shards(amped_tensor_s* t, int d, const ModeDev& base, hipStream_t s, Cut&& cut, Fn&& fn)
{
    const int order = t->order;
    const int64_t nnz = t->nnz;
    const amped::PackedMode& h = t->hmode[d];
    if (nnz == 0) return fn(base, 0);
    hipError_t e;
    // Under capture the copies join the graph behind the stream's work so far.
    // A replay's use of the buffers is no event that a later call could wait for,
    // so from the first capture on every call starts behind its stream's work.
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if ((e = hipStreamIsCapturing(s, &cs)) != hipSuccess) return hip_fail(e, "hipStreamIsCapturing");
    if (cs != hipStreamCaptureStatusNone) t->was_captured = true;
    if (t->was_captured) {
        if ((e = hipEventRecord(t->call_start, s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
        if ((e = hipStreamWaitEvent(t->copy_stream, t->call_start, 0)) != hipSuccess)
            return hip_fail(e, "hipStreamWaitEvent");
        t->ring_used[0] = t->ring_used[1] = false;
    }
    const int64_t stride = t->stage_stride();
    amped::UnpackArgs u;
    u.order = order;
    for (int j = 0; j < order - 1; ++j) u.bits[j] = h.bits[j];
    int i = 0;
    for (int64_t start = 0; start < nnz; ++i) {
        const int64_t end = cut(start);
        if (end <= start || end - start > t->stage_len)
            return fail(AMPED_ERR_UNSUPPORTED, "a run of equal coordinates is longer than a shard (%lld nonzeros)",
                        (long long)t->stage_len);
        const int64_t b0 = start / amped::kPackBlock;
        const int64_t b1 = (end + amped::kPackBlock - 1) / amped::kPackBlock;
        const int64_t mid = b0 + (b1 - b0 + 1) / 2;
        for (int half = 0; half < 2; ++half) {
            const int64_t h0 = half ? mid : b0, h1 = half ? b1 : mid;
            if (h0 >= h1) continue;
            const int b = t->next_ring;
            t->next_ring ^= 1;
            if (t->ring_used[b] && (e = hipStreamWaitEvent(t->copy_stream, t->consumed[b], 0)) != hipSuccess)
                return hip_fail(e, "hipStreamWaitEvent");
            if ((e = hipMemcpyAsync(t->ring[b], reinterpret_cast<const char*>(h.data) + h.bytes(h0),
                                    (size_t)(h.bytes(h1) - h.bytes(h0)), hipMemcpyHostToDevice, t->copy_stream)) !=
                hipSuccess)
                return hip_fail(e, "hipMemcpyAsync(shard)");
            u.offset = h.dev_offset + h0;
            if (!h.dev_offset) {
                uint32_t* to = reinterpret_cast<uint32_t*>(static_cast<char*>(t->ring[b]) + t->ring_offsets);
                if ((e = hipMemcpyAsync(to, h.pinned_offset + h0, (size_t)(h1 - h0 + 1) * 4, hipMemcpyHostToDevice,
                                        t->copy_stream)) != hipSuccess)
                    return hip_fail(e, "hipMemcpyAsync(block offsets)");
                u.offset = to;
            }
            if ((e = hipEventRecord(t->copied[b], t->copy_stream)) != hipSuccess) return hip_fail(e, "hipEventRecord");
            if ((e = hipStreamWaitEvent(s, t->copied[b], 0)) != hipSuccess) return hip_fail(e, "hipStreamWaitEvent");
            u.packed = static_cast<const uint32_t*>(t->ring[b]);
            u.blocks = h1 - h0;
            for (int j = 0; j <= order; ++j) u.to[j] = t->stage + j * stride + (h0 - b0) * amped::kPackBlock;
            if ((e = amped::launch_unpack(u, s)) != hipSuccess) return hip_fail(e, "unpack");
            if ((e = hipEventRecord(t->consumed[b], s)) != hipSuccess) return hip_fail(e, "hipEventRecord");
            t->ring_used[b] = true;
        }
        ModeDev m = base;
        const int32_t* at = t->stage + (start - b0 * amped::kPackBlock);
        m.out_idx = at;
        for (int j = 0; j < order - 1; ++j) m.in_idx[j] = at + (1 + j) * stride;
        m.val = reinterpret_cast<const float*>(at + order * stride);
        m.nnz = end - start;
        m.n_chunks = (m.nnz + t->unit - 1) / t->unit;
        m.prev_key = start > 0 ? h.out_index(start - 1) : -1;
        m.next_key = end < nnz ? h.out_index(end) : -1;
        if (i > 0) {
            m.n_zero = 0;
            m.n_gaps = 0;
        }
        amped_status st = fn(m, i);
        if (st != AMPED_OK) return st;
        start = end;
    }
    return AMPED_OK;
}

// Shard ends for the MTTKRP-shaped kernels: whole chunks, stage_len each.
struct ChunkCut {
    int64_t nnz, len;
    int64_t operator()(int64_t start) const { return std::min(start + len, nnz); }
};

}  // namespace

extern "C" {

const char* amped_last_error(void) { return g_err.c_str(); }

const char* amped_version(void) { return "amped 0.1.0 (gfx950)"; }

amped_status amped_layout_host(int order, const int64_t* dims, int64_t nnz, const int32_t* indices, int mode,
                               int64_t chunk_nnz, int32_t* perm, uint8_t* chunk_flags)
{
    g_err.clear();
    static const float dummy = 0.f;
    amped_status st = validate_args(order, dims, nnz, indices, nnz ? &dummy : nullptr);
    if (st == AMPED_OK) st = validate_range(order, dims, nnz, indices);
    if (st != AMPED_OK) return st;
    if (mode < 0 || mode >= order) return fail(AMPED_ERR_INVALID, "mode %d outside [0, %d)", mode, order);
    if (chunk_nnz < 1) return fail(AMPED_ERR_INVALID, "chunk_nnz must be >= 1");
    try {
        std::vector<int32_t> lex = amped::lex_order(order, dims, nnz, indices);
        HostModeLayout lay;
        amped::mode_order(dims, nnz, indices, lex, mode, lay.perm);
        amped::mode_tables(dims, nnz, indices, mode, chunk_nnz, lay);
        if (perm && nnz) std::memcpy(perm, lay.perm.data(), (size_t)nnz * sizeof(int32_t));
        if (chunk_flags && !lay.flags.empty()) std::memcpy(chunk_flags, lay.flags.data(), lay.flags.size());
    } catch (const std::bad_alloc&) {
        return fail(AMPED_ERR_NOMEM, "host allocation failed");
    }
    return AMPED_OK;
}

amped_status amped_tensor_create(int order, const int64_t* dims, int64_t nnz, const int32_t* indices,
                                 const float* values, const amped_options* opts, amped_tensor_t* out)
{
    g_err.clear();
    if (!out) return fail(AMPED_ERR_INVALID, "out is NULL");
    *out = nullptr;
    amped_status st = validate_args(order, dims, nnz, indices, values);
    if (st != AMPED_OK) return st;
    // The device build checks the indices on the device; every other way out of
    // this call checks them here first, since a bad index is reported before a
    // bad option, a low cap or a missing device.
    auto unless_bad_index = [&](amped_status err) {
        std::string msg;
        msg.swap(g_err);
        const amped_status bad = validate_range(order, dims, nnz, indices);
        if (bad != AMPED_OK) return bad;
        g_err.swap(msg);
        return err;
    };
    int64_t chunk = amped::kDefaultChunk, cap = 0, shard_opt = 0;
    bool keep_perm = false, host_layout = false;
    if (opts) {
        if (opts->host_layout != 0 && opts->host_layout != 1)
            return unless_bad_index(fail(AMPED_ERR_INVALID, "host_layout must be 0 or 1"));
        host_layout = opts->host_layout == 1;
        if (opts->shard_nnz < 0) return unless_bad_index(fail(AMPED_ERR_INVALID, "shard_nnz < 0"));
        shard_opt = opts->shard_nnz;
        if (opts->chunk_nnz < 0 || opts->chunk_nnz > amped::kMaxChunk)
            return unless_bad_index(fail(AMPED_ERR_INVALID, "chunk_nnz %lld outside [0, 2^28]", (long long)opts->chunk_nnz));
        if (opts->chunk_nnz > 0) chunk = opts->chunk_nnz;
        if (opts->device_byte_cap < 0) return unless_bad_index(fail(AMPED_ERR_INVALID, "device_byte_cap < 0"));
        cap = opts->device_byte_cap;
        if (opts->keep_perm != 0 && opts->keep_perm != 1) return unless_bad_index(fail(AMPED_ERR_INVALID, "keep_perm must be 0 or 1"));
        keep_perm = opts->keep_perm == 1;
    }
    // peak device bytes: the N layouts, the kept permutations, and during the
    // build the raw COO plus one permutation; per mode at most one int per row
    // for the zero-row list and long gaps, and the hot-row tables.  (What the builds
    // take now is less; what a cap admits is unchanged, and what goes beyond the layouts
    // is left out where it does not fit: own_unit_bytes, build_host_layout.)
    const int64_t layout_bytes = (int64_t)order * (order + 1) * 4 * (nnz + 4);
    int64_t row_bytes = 0;
    for (int d = 0; d < order; ++d) row_bytes += 4 * dims[d] + 4 * amped::kHotTableLen;
    // device sort: lexicographic order, key and value ping-pong buffers, 256 counts
    // per 4096 nonzeros and their sums
    const int64_t sort_counts = (nnz + 4095) / 4096 * 256;
    const int64_t sort_bytes = 16 * nnz + 4 * (sort_counts + (sort_counts + 4095) / 4096 + 64);
    // host-resident layouts: two shard buffers of whole chunks instead (what they are
    // filled with now: build_host_layout)
    const int64_t n_chunks = (nnz + chunk - 1) / chunk;
    const int64_t shard_chunks =
        std::max<int64_t>(1, std::min(((shard_opt > 0 ? shard_opt : (int64_t)1 << 25) + chunk - 1) / chunk,
                                      std::max<int64_t>(n_chunks, 1)));
    const int64_t stage_len = shard_chunks * chunk;
    if (host_layout && stage_len > 0x7FFFFFFF - 4)
        return unless_bad_index(fail(AMPED_ERR_INVALID, "shard of %lld nonzeros too large", (long long)stage_len));
    const int64_t peak =
        host_layout ? 2 * (int64_t)(order + 1) * 4 * (stage_len + 4) + row_bytes + 4096
                    : layout_bytes + (keep_perm ? (int64_t)order * 4 * nnz : 0) + (int64_t)(order + 1) * 4 * nnz +
                          4 * nnz + (int64_t)order * ((nnz + chunk - 1) / chunk + 64) * 8 + row_bytes + sort_bytes + 4096;
    if (cap > 0 && peak > cap)
        return unless_bad_index(fail(AMPED_ERR_NOMEM, "layouts need up to %lld device bytes, cap is %lld",
                                     (long long)peak, (long long)cap));
    int dev = 0;
    st = check_device(&dev);
    if (st != AMPED_OK) return unless_bad_index(st);
    if (host_layout && (st = validate_range(order, dims, nnz, indices)) != AMPED_OK) return st;

    amped_tensor_s* t = new (std::nothrow) amped_tensor_s();
    if (!t) return fail(AMPED_ERR_NOMEM, "host allocation failed");
    t->order = order;
    for (int w = 0; w < order; ++w) t->dims[w] = dims[w];
    t->nnz = nnz;
    t->chunk = chunk;
    t->n_chunks = (nnz + chunk - 1) / chunk;
    t->unit = chunk;
    t->own_units = !opts || opts->chunk_nnz == 0;
    // under a cap that does not hold what library-sized units take beside the layouts, the
    // units are the chunks, and rows that cross them take atomics
    if (t->own_units && !host_layout && cap > 0 &&
        peak + amped::own_unit_bytes(order, nnz, amped::work_unit(nnz)) > cap)
        t->own_units = false;
    if (t->own_units)
        t->unit = host_layout ? amped::stream_work_unit(std::min(stage_len, nnz)) : amped::work_unit(nnz);
    t->device = dev;
    t->keep_perm = keep_perm;
    try {
        if (host_layout) {
            t->host_layout = true;
            t->stage_len = stage_len;
            st = build_host_layout(t, indices, values, cap);
        } else {
            st = build_device_layout(t, indices, values, cap);
        }
    } catch (const std::bad_alloc&) {
        st = fail(AMPED_ERR_NOMEM, "host allocation failed");
    }
    if (st != AMPED_OK) {
        (void)hipDeviceSynchronize();
        t->free_all();
        delete t;
        // (the build may have stopped before its own check)
        return st == AMPED_ERR_RANGE || host_layout ? st : unless_bad_index(st);
    }
    *out = t;
    return AMPED_OK;
}

amped_status amped_tensor_destroy(amped_tensor_t t)
{
    g_err.clear();
    if (!t) return AMPED_OK;
    amped_status st = AMPED_OK;
    {
        DeviceGuard guard(t->device);
        hipError_t e = hipDeviceSynchronize();
        if (e != hipSuccess) st = hip_fail(e, "hipDeviceSynchronize");
        t->free_all();
    }
    delete t;
    return st;
}

amped_status amped_tensor_info(amped_tensor_t t, int* order, int64_t* dims, int64_t* nnz, int64_t* chunk_nnz,
                               int64_t* n_chunks, int64_t* touched, int64_t* device_bytes)
{
    g_err.clear();
    if (!t) return fail(AMPED_ERR_INVALID, "tensor is NULL");
    if (order) *order = t->order;
    if (dims)
        for (int w = 0; w < t->order; ++w) dims[w] = t->dims[w];
    if (nnz) *nnz = t->nnz;
    if (chunk_nnz) *chunk_nnz = t->chunk;
    if (n_chunks) *n_chunks = t->n_chunks;
    if (touched)
        for (int w = 0; w < t->order; ++w) touched[w] = t->touched[w];
    if (device_bytes) *device_bytes = t->device_bytes;
    return AMPED_OK;
}

amped_status amped_tensor_layout(amped_tensor_t t, int mode, int32_t* perm, int32_t* out_idx, int32_t* in_idx,
                                 float* values, uint8_t* chunk_flags)
{
    g_err.clear();
    if (!t) return fail(AMPED_ERR_INVALID, "tensor is NULL");
    if (mode < 0 || mode >= t->order) return fail(AMPED_ERR_INVALID, "mode %d outside [0, %d)", mode, t->order);
    if (perm && !t->keep_perm) return fail(AMPED_ERR_INVALID, "permutation not kept (create with keep_perm=1)");
    DeviceGuard guard(t->device);
    if (!guard.ok) return fail(AMPED_ERR_HIP, "cannot select device %d", t->device);
    const ModeDev& m = t->mode[mode];
    const size_t bytes = (size_t)t->nnz * 4;
    amped_status st = AMPED_OK;
    if (t->host_layout) {
        if (bytes) {
            if (perm) std::memcpy(perm, t->hperm[mode].data(), bytes);
            t->hmode[mode].unpack(t->nnz, out_idx, in_idx, values);
        }
    } else if (bytes) {
        if (perm) HIP_OR_FAIL(hipMemcpy(perm, t->perm[mode], bytes, hipMemcpyDeviceToHost), "hipMemcpy(perm)");
        if (out_idx) HIP_OR_FAIL(hipMemcpy(out_idx, m.out_idx, bytes, hipMemcpyDeviceToHost), "hipMemcpy(out_idx)");
        if (in_idx)
            for (int j = 0; j < t->order - 1; ++j)
                HIP_OR_FAIL(hipMemcpy(in_idx + (int64_t)j * t->nnz, m.in_idx[j], bytes, hipMemcpyDeviceToHost),
                            "hipMemcpy(in_idx)");
        if (values) HIP_OR_FAIL(hipMemcpy(values, m.val, bytes, hipMemcpyDeviceToHost), "hipMemcpy(values)");
    }
    if (chunk_flags && t->host_layout) {
        if (!t->flags[mode].empty()) std::memcpy(chunk_flags, t->flags[mode].data(), t->flags[mode].size());
    } else if (chunk_flags && t->n_chunks > 0) {
        // from the output indices on both sides of every chunk edge
        try {
            std::vector<int32_t> keys((size_t)t->nnz);
            HIP_OR_FAIL(hipMemcpy(keys.data(), m.out_idx, bytes, hipMemcpyDeviceToHost), "hipMemcpy(out_idx)");
            for (int64_t k = 0; k < t->n_chunks; ++k) {
                const int64_t b = k * t->chunk, e = std::min(b + t->chunk, t->nnz);
                chunk_flags[k] = (uint8_t)((b > 0 && keys[b - 1] == keys[b] ? 1 : 0) |
                                           (e < t->nnz && keys[e - 1] == keys[e] ? 2 : 0));
            }
        } catch (const std::bad_alloc&) {
            return fail(AMPED_ERR_NOMEM, "host allocation failed");
        }
    }
    return AMPED_OK;
cleanup:
    return st;
}

namespace {

amped_status check_call(amped_tensor_t t, int mode, int rank, const void* const* factors, const void* out,
                        bool need_own, const char* out_name)
{
    if (!t) return fail(AMPED_ERR_INVALID, "tensor is NULL");
    if (mode < 0 || mode >= t->order) return fail(AMPED_ERR_INVALID, "mode %d outside [0, %d)", mode, t->order);
    if (rank < 1 || rank > 4096) return fail(AMPED_ERR_INVALID, "rank %d outside [1, 4096]", rank);
    if (!factors) return fail(AMPED_ERR_INVALID, "factors is NULL");
    for (int w = 0; w < t->order; ++w) {
        if (w == mode && !need_own) continue;
        if (!factors[w]) return fail(AMPED_ERR_INVALID, "factors[%d] is NULL", w);
        if (!aligned16(factors[w])) return fail(AMPED_ERR_INVALID, "factors[%d] is not 16-byte aligned", w);
    }
    if (!out) return fail(AMPED_ERR_INVALID, "%s is NULL", out_name);
    if (!aligned16(out)) return fail(AMPED_ERR_INVALID, "%s is not 16-byte aligned", out_name);
    return AMPED_OK;
}

amped_status run_mttkrp(amped_tensor_t t, int mode, int rank, const void* const* factors, float* out, void* stream,
                        amped::FactorType ft, amped::Kind kind, float scale, double* loss = nullptr,
                        const double* dev_scale = nullptr)
{
    const bool grad = (kind != amped::Kind::Mttkrp);
    amped_status st = check_call(t, mode, rank, factors, out, grad, grad ? "grad" : "out");
    if (st != AMPED_OK) return st;
    if (kind == amped::Kind::ResidualGradLoss && !loss) return fail(AMPED_ERR_INVALID, "loss is NULL");
    DeviceGuard guard(t->device);
    if (!guard.ok) return fail(AMPED_ERR_HIP, "cannot select device %d", t->device);
    amped::LaunchArgs a;
    a.m = &t->mode[mode];
    a.nin = t->order - 1;
    a.rank = rank;
    a.ftype = ft;
    a.kind = kind;
    int j = 0;
    for (int w = 0; w < t->order; ++w)
        if (w != mode) {
            a.in_rows[j] = t->dims[w];
            a.in_hot[j] = t->mode[w].hot;
            a.in_factors[j++] = factors[w];
        }
    a.own_factor = grad ? static_cast<const float*>(factors[mode]) : nullptr;
    a.scale = scale;
    a.dev_scale = dev_scale;
    a.out = out;
    a.loss = loss;
    a.stream = static_cast<hipStream_t>(stream);
    const char* what = kind == amped::Kind::Mttkrp ? "amped_mttkrp"
                       : kind == amped::Kind::ResidualGrad ? "amped_cp_grad" : "amped_cp_loss_grad";
    auto launch = [&](const ModeDev& m, int i) -> amped_status {
        a.m = &m;
        a.loss_accumulate = i > 0;   // later shards add to the loss of the first
        hipError_t e = amped::launch_mttkrp(a);
        return e == hipSuccess ? AMPED_OK : hip_fail(e, what);
    };
    if (t->host_layout) return stream_shards(t, mode, t->mode[mode], a.stream, ChunkCut{t->nnz, t->stage_len}, launch);
    return launch(t->mode[mode], 0);
}

}  // namespace

amped_status amped_mttkrp(amped_tensor_t t, int mode, int rank, const float* const* factors, float* out,
                          void* stream)
{
    g_err.clear();
    return run_mttkrp(t, mode, rank, reinterpret_cast<const void* const*>(factors), out, stream,
                      amped::FactorType::F32, amped::Kind::Mttkrp, 1.0f);
}

amped_status amped_mttkrp_bf16(amped_tensor_t t, int mode, int rank, const uint16_t* const* factors, float* out,
                               void* stream)
{
    g_err.clear();
    return run_mttkrp(t, mode, rank, reinterpret_cast<const void* const*>(factors), out, stream,
                      amped::FactorType::BF16, amped::Kind::Mttkrp, 1.0f);
}

amped_status amped_cp_grad(amped_tensor_t t, int mode, int rank, const float* const* factors, float scale,
                           float* grad, void* stream)
{
    g_err.clear();
    return run_mttkrp(t, mode, rank, reinterpret_cast<const void* const*>(factors), grad, stream,
                      amped::FactorType::F32, amped::Kind::ResidualGrad, scale);
}

amped_status amped_cp_grad_scaled(amped_tensor_t t, int mode, int rank, const float* const* factors, float scale,
                                  const double* dev_scale, float* grad, void* stream)
{
    g_err.clear();
    if (!dev_scale) return fail(AMPED_ERR_INVALID, "dev_scale is NULL");
    return run_mttkrp(t, mode, rank, reinterpret_cast<const void* const*>(factors), grad, stream,
                      amped::FactorType::F32, amped::Kind::ResidualGrad, scale, nullptr, dev_scale);
}

amped_status amped_scale(float* x, int64_t n, const double* dev_scale, void* stream)
{
    g_err.clear();
    if (n < 0) return fail(AMPED_ERR_INVALID, "n = %lld < 0", (long long)n);
    if (n > 0 && (!x || !dev_scale)) return fail(AMPED_ERR_INVALID, "x or dev_scale is NULL");
    if (!aligned16(x)) return fail(AMPED_ERR_INVALID, "x is not 16-byte aligned");
    int dev = 0;
    amped_status st = check_device(&dev);
    if (st != AMPED_OK) return st;
    hipError_t e = amped::launch_scale(x, n, dev_scale, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? AMPED_OK : hip_fail(e, "amped_scale");
}

amped_status amped_cp_loss_grad(amped_tensor_t t, int mode, int rank, const float* const* factors, float scale,
                                float* grad, double* loss, void* stream)
{
    g_err.clear();
    return run_mttkrp(t, mode, rank, reinterpret_cast<const void* const*>(factors), grad, stream,
                      amped::FactorType::F32, amped::Kind::ResidualGradLoss, scale, loss);
}

amped_status amped_gram(const float* A, int64_t rows, int rank, double* G, void* stream)
{
    g_err.clear();
    if (!A || !G) return fail(AMPED_ERR_INVALID, "A or G is NULL");
    if (rows < 1) return fail(AMPED_ERR_INVALID, "rows %lld < 1", (long long)rows);
    if (rank < 1 || rank > 128) return fail(AMPED_ERR_INVALID, "rank %d outside [1, 128]", rank);
    int dev = 0;
    amped_status st = check_device(&dev);
    if (st != AMPED_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t bytes = (size_t)amped::gram_slabs(rows) * rank * rank * sizeof(float);
    void* partial = nullptr;
    hipError_t e = hipMallocAsync(&partial, bytes, s);
    if (e != hipSuccess) return hip_fail(e, "hipMallocAsync(gram partials)");
    e = amped::launch_gram(A, rows, rank, static_cast<float*>(partial), G, s);
    hipError_t e2 = hipFreeAsync(partial, s);
    if (e != hipSuccess) return hip_fail(e, "amped_gram");
    if (e2 != hipSuccess) return hip_fail(e2, "hipFreeAsync(gram partials)");
    return AMPED_OK;
}

amped_status amped_gram_noalloc(const float* A, int64_t rows, int rank, double* G, void* stream)
{
    g_err.clear();
    if (!A || !G) return fail(AMPED_ERR_INVALID, "A or G is NULL");
    if (rows < 1) return fail(AMPED_ERR_INVALID, "rows %lld < 1", (long long)rows);
    if (rank < 1 || rank > 128)
        return fail(AMPED_ERR_INVALID, "rank %d outside [1, 128]: the partial sums of larger ranks do not fit the "
                    "fixed 32 MiB device scratch", rank);
    int dev = 0;
    amped_status st = check_device(&dev);
    if (st != AMPED_OK) return st;
    hipError_t e = amped::launch_gram_noalloc(A, rows, rank, G, static_cast<hipStream_t>(stream));
    if (e == hipErrorInvalidValue)
        return fail(AMPED_ERR_INVALID, "amped_gram_noalloc: %lld rows x rank %d exceed the fixed device scratch",
                    (long long)rows, rank);
    return e == hipSuccess ? AMPED_OK : hip_fail(e, "amped_gram_noalloc");
}

amped_status amped_cp_als_sweep(amped_tensor_t t, int rank, float* const* factors, double* lambda, double* fit,
                                unsigned flags, void* stream)
{
    g_err.clear();
    amped_status st = check_call(t, 0, rank, reinterpret_cast<const void* const*>(factors), lambda, true, "lambda");
    if (st != AMPED_OK) return st;
    if (rank > 128) return fail(AMPED_ERR_INVALID, "rank %d above 128 (CP-ALS)", rank);
    if (!fit) return fail(AMPED_ERR_INVALID, "fit is NULL");
    if (flags & ~AMPED_ALS_REUSE_GRAMS) return fail(AMPED_ERR_INVALID, "unknown flags 0x%x", flags);
    const bool reuse = (flags & AMPED_ALS_REUSE_GRAMS) != 0;
    if (reuse && (t->als.rank != rank || !t->als.have_grams))
        return fail(AMPED_ERR_INVALID, "no previous sweep at rank %d to reuse Gram matrices from", rank);
    DeviceGuard guard(t->device);
    if (!guard.ok) return fail(AMPED_ERR_HIP, "cannot select device %d", t->device);
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto& w = t->als;
    const int N = t->order;
    hipError_t e = hipSuccess;
    const size_t RR = (size_t)rank * rank;
    if (w.rank != rank) {
        for (void* q : {(void*)w.M, (void*)w.G, (void*)w.S, (void*)w.partial, (void*)w.scratch, (void*)w.W,
                        (void*)w.wide})
            if (q) t->release(q);
        double* keep_x = w.xnorm2;
        const bool keep_have = w.have_xnorm2;
        w = amped_tensor_s::AlsWork{};
        w.xnorm2 = keep_x;
        w.have_xnorm2 = keep_have;
        int64_t maxrows = 0, slabs = 0;
        for (int d = 0; d < N; ++d) {
            maxrows = std::max(maxrows, t->dims[d]);
            slabs += amped::als_gram_slabs(t->dims[d], rank);   // all factors' Gram matrices in one launch
        }
        void* p = nullptr;
        if ((e = t->alloc(&p, (size_t)maxrows * rank * sizeof(float))) != hipSuccess) return hip_fail(e, "als workspace");
        w.M = static_cast<float*>(p);
        if ((e = t->alloc(&p, N * RR * sizeof(double))) != hipSuccess) return hip_fail(e, "als workspace");
        w.G = static_cast<double*>(p);
        if ((e = t->alloc(&p, RR * sizeof(double))) != hipSuccess) return hip_fail(e, "als workspace");
        w.S = static_cast<double*>(p);
        if ((e = t->alloc(&p, (size_t)slabs * RR * sizeof(float))) != hipSuccess)
            return hip_fail(e, "als workspace");
        w.partial = static_cast<float*>(p);
        if ((e = t->alloc(&p, RR * sizeof(double))) != hipSuccess) return hip_fail(e, "als workspace");
        w.scratch = static_cast<double*>(p);
        if ((e = t->alloc(&p, RR * sizeof(double))) != hipSuccess) return hip_fail(e, "als workspace");
        w.W = static_cast<double*>(p);
        if ((e = t->alloc(&p, sizeof(int))) != hipSuccess) return hip_fail(e, "als workspace");
        w.wide = static_cast<int*>(p);
        if (!w.xnorm2) {
            if ((e = t->alloc(&p, sizeof(double))) != hipSuccess) return hip_fail(e, "als workspace");
            w.xnorm2 = static_cast<double*>(p);
        }
        w.rank = rank;
    }
    if (!w.have_xnorm2) {
        auto norm = [&](const ModeDev& m, int i) -> amped_status {
            hipError_t en = amped::launch_tensor_norm2(m, N - 1, w.xnorm2, i > 0, s);
            return en == hipSuccess ? AMPED_OK : hip_fail(en, "tensor norm");
        };
        if (t->host_layout) {
            // shards end between runs of equal coordinates (each run is summed
            // before squaring)
            const auto& h = t->hmode[0];
            auto same = [&](int64_t p, int64_t q) {
                if (h.out_index(p) != h.out_index(q)) return false;
                for (int j = 0; j < N - 1; ++j)
                    if (h.in_index(j, p) != h.in_index(j, q)) return false;
                return true;
            };
            auto cut = [&](int64_t start) {
                int64_t end = std::min(start + t->stage_len, t->nnz);
                if (end < t->nnz)
                    while (end > start && same(end - 1, end)) --end;
                return end;
            };
            st = stream_shards(t, 0, t->mode[0], s, cut, norm);
        } else {
            st = norm(t->mode[0], 0);
        }
        if (st != AMPED_OK) return st;
        w.have_xnorm2 = true;
    }
    w.have_grams = false;   // stays false if the sweep stops part-way
    if (!reuse) {
        if ((e = amped::launch_als_grams(factors, t->dims, N, rank, w.partial, w.G, s)) != hipSuccess)
            return hip_fail(e, "gram");
    }
    for (int d = 0; d < N; ++d) {
        st = run_mttkrp(t, d, rank, reinterpret_cast<const void* const*>(factors), w.M, stream,
                        amped::FactorType::F32, amped::Kind::Mttkrp, 1.0f);
        if (st != AMPED_OK) return st;
        if ((e = amped::launch_als_update(w.M, factors[d], t->dims[d], w.partial, w.G, w.S, N, d, rank, w.scratch, w.W,
                                          w.wide, lambda, d == N - 1, w.xnorm2, fit, s)) != hipSuccess)
            return hip_fail(e, "als update");
    }
    w.have_grams = true;   // G now holds the Gram matrices of the factors just written
    return AMPED_OK;
}

#if AMPED_QUEUE_STATS
amped_status amped_queue_stats(uint64_t* records, int64_t max_records, int64_t* n_records, int32_t* waves_per_block,
                               double* clock_hz)
{
    g_err.clear();
    if (!n_records || !waves_per_block || !clock_hz) return fail(AMPED_ERR_INVALID, "NULL output");
    if (records && max_records < 0) return fail(AMPED_ERR_INVALID, "max_records < 0");
    int dev = 0, khz = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess) return hip_fail(e, "wall clock rate");
    *clock_hz = 1e3 * khz;
    int wpb = 0;
    e = amped::queue_stats_copy(reinterpret_cast<unsigned long long*>(records), max_records, n_records, &wpb);
    *waves_per_block = wpb;
    return e == hipSuccess ? AMPED_OK : hip_fail(e, "amped_queue_stats");
}
#endif

amped_status amped_cp_loss(amped_tensor_t t, int rank, const float* const* factors, double* loss, void* stream)
{
    g_err.clear();
    amped_status st = check_call(t, 0, rank, reinterpret_cast<const void* const*>(factors), loss, true, "loss");
    if (st != AMPED_OK) return st;
    DeviceGuard guard(t->device);
    if (!guard.ok) return fail(AMPED_ERR_HIP, "cannot select device %d", t->device);
    amped::LossArgs a;
    a.m = &t->loss_dev;
    a.order = t->order;
    a.rank = rank;
    a.own_factor = factors[0];
    for (int w = 1; w < t->order; ++w) {
        a.in_factors[w - 1] = factors[w];
        a.in_rows[w - 1] = t->dims[w];
    }
    a.loss = loss;
    a.stream = static_cast<hipStream_t>(stream);
    auto launch = [&](const ModeDev& m, int i) -> amped_status {
        a.m = &m;
        a.accumulate = i > 0;
        hipError_t e = amped::launch_cp_loss(a);
        return e == hipSuccess ? AMPED_OK : hip_fail(e, "amped_cp_loss");
    };
    if (t->host_layout) return stream_shards(t, 0, t->loss_dev, a.stream, ChunkCut{t->nnz, t->stage_len}, launch);
    return launch(t->loss_dev, 0);
}

}  // extern "C"
