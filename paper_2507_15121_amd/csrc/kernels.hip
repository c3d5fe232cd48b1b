// The launches of the sparse MTTKRP, its bfloat16-factor form, the fused residual + MTTKRP
// gradient and the sparse CP loss: which instance, grid and addressing a call takes, and
// the small kernels before and after it (init, close, scale) and of the layout build
// (permute).  The work decomposition and the kernel itself are in kernel_impl.h, the
// one-launch form of small tensors in k_small.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <unordered_map>
#include <utility>

#include "kernel_impl.h"

#ifndef AMPED_BUFFER_LOADS
#define AMPED_BUFFER_LOADS 1
#endif

namespace amped {
namespace dev {

// ----------------------------------------------------------------- init kernel
// Resets the work-queue counters (and the loss) and zeroes the output rows
// the MTTKRP kernel does not store: rows that several units add into,
// untouched rows of short runs (both in the zero-row list) and long runs of
// untouched rows.  vec4: ld, col0 and ncols are multiples of 4 (16-byte stores).
__global__ void __launch_bounds__(kBlock) init_kernel(float* out, int64_t ld, int col0, int ncols, bool vec4,
                                                      const int32_t* zrows, int64_t n_zero,
                                                      const int32_t* gaps, int64_t n_gaps, unsigned* queue,
                                                      double* loss)
{
    if (blockIdx.x == 0) {
        if (queue && threadIdx.x < kQueueSlots) queue[threadIdx.x * kQueueStride] = 0u;
        if (loss && threadIdx.x == 0) *loss = 0.0;
    }
    if (out) zero_rows(out, ld, col0, ncols, vec4, zrows, n_zero, gaps, n_gaps, blockIdx.x, gridDim.x);
}

// A factor of `rows` rows is read through a 32-bit buffer offset when one
// more row still fits: padding entries use row -1, whose offset (2^32 - one
// row + column bytes) then lies past the end and reads zeros.
bool fits_buffer(int64_t rows, int rank, int elem_bytes)
{
    return (uint64_t)(rows + 1) * (uint64_t)rank * (uint64_t)elem_bytes <= (1ull << 32);
}

// Launch shape of an MTTKRP-kernel instance on the current device: the
// hot-row cache slots K (largest power of two whose LDS, with the kernel's
// static LDS, fits one block; capped by AMPED_HOT_MAX if set, 0 = no cache),
// the dynamic LDS bytes and the persistent grid (every CU filled to the
// occupancy that LDS allows).
struct Shape {
    int hot_k = 0;
    size_t dyn = 16;
    int grid = 0;
};

// Work-queue stripes per launch (1..kQueueSlots): AMPED_QUEUE_STRIPES, read
// once per process, else the default.
#ifndef AMPED_DEFAULT_STRIPES
#define AMPED_DEFAULT_STRIPES 8
#endif
int queue_stripes()
{
    static const int n = [] {
        const char* e = std::getenv("AMPED_QUEUE_STRIPES");
        const int v = (e && *e) ? std::atoi(e) : AMPED_DEFAULT_STRIPES;
        return std::max(1, std::min(v, kQueueSlots));
    }();
    return n;
}

#if AMPED_QUEUE_STATS
// Diagnostic build: the per-wave records of the last MTTKRP-shaped launch.
struct QueueStats {
    unsigned long long* dev = nullptr;
    int64_t cap = 0, n = 0;
    int waves_per_block = 0;
} g_qstats;
std::mutex g_qstats_mu;

hipError_t qstats_attach(KParams& k, int grid, int block, hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_qstats_mu);
    const int64_t n = (int64_t)grid * (block / 64);
    if (n > g_qstats.cap) {
        if (g_qstats.dev) (void)hipFree(g_qstats.dev);
        g_qstats.dev = nullptr;
        g_qstats.cap = 0;
        hipError_t e = hipMalloc(&g_qstats.dev, (size_t)n * 4 * sizeof(unsigned long long));
        if (e != hipSuccess) return e;
        g_qstats.cap = n;
    }
    g_qstats.n = n;
    g_qstats.waves_per_block = block / 64;
    k.qstats = g_qstats.dev;
    return hipMemsetAsync(g_qstats.dev, 0, (size_t)n * 4 * sizeof(unsigned long long), st);
}
#endif

int hot_cap()
{
    static const int cap = [] {
        const char* e = std::getenv("AMPED_HOT_MAX");
        if (!e || !*e) return kHotMax;
        const int v = std::atoi(e);
        return v < 0 ? 0 : std::min(v, kHotMax);
    }();
    return cap;
}

Shape launch_shape(KernelFn fn, int block, int nin, int row_bytes, bool cache)
{
    static std::mutex mu;
    static std::map<std::tuple<int, const void*, int, int, bool>, Shape> memo;
    int dev = 0;
    Shape sh;
    if (hipGetDevice(&dev) != hipSuccess) return sh;
    const void* f = reinterpret_cast<const void*>(fn);
    std::lock_guard<std::mutex> lk(mu);
    const auto key = std::make_tuple(dev, f, nin, row_bytes, cache);
    auto it = memo.find(key);
    if (it != memo.end()) return it->second;
    int cus = 0, max_lds = 0;
    hipFuncAttributes attr{};
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess ||
        hipFuncGetAttributes(&attr, f) != hipSuccess)
        return sh;
    if (cache) {
        for (int k = hot_cap(); k >= 16; k >>= 1)
            if (attr.sharedSizeBytes + hot_lds_bytes(nin, k, row_bytes) <= (size_t)max_lds) {
                sh.hot_k = k;
                break;
            }
    }
    // hot_cap() may not be a power of two: round down
    while (sh.hot_k & (sh.hot_k - 1)) sh.hot_k &= sh.hot_k - 1;
    sh.dyn = hot_lds_bytes(nin, sh.hot_k, row_bytes);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, block, sh.dyn) != hipSuccess || nb < 1) nb = 1;
    sh.grid = nb * cus;
    memo.emplace(key, sh);
    return sh;
}

// Blocks of a launch: the persistent grid, or a block per chunk when there are
// fewer chunks (one wave of each block then has work: the chunks spread over
// the CUs).
int launch_grid(const Shape& sh, const KParams& k) { return (int)std::min<int64_t>(sh.grid, k.n_chunks); }

// Whether a launch's part of every output row is whole 16-byte pieces.
bool whole_vectors(const float* out, int64_t ld, int col0, int ncols)
{
    return ld % 4 == 0 && col0 % 4 == 0 && ncols % 4 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
}

hipError_t launch_init(const ModeDev& m, float* out, int64_t ld, int col0, int ncols, double* loss,
                       hipStream_t st)
{
    const bool vec4 = whole_vectors(out, ld, col0, ncols);
    const int64_t work = std::max<int64_t>(m.n_zero * (vec4 ? ncols / 4 : ncols), m.n_gaps * kBlock);
    int grid = (int)std::min<int64_t>(std::max<int64_t>(1, (work + kBlock - 1) / kBlock), 4096);
    hipLaunchKernelGGL(init_kernel, dim3(grid), dim3(kBlock), 0, st, out, ld, col0, ncols, vec4, m.zero_rows,
                       out ? m.n_zero : 0, m.gaps, out ? m.n_gaps : 0, m.queue, loss);
    return hipGetLastError();
}

// Point the kernel at the K-slot hot tables of its inputs (K = 0: no cache;
// also when a table is missing).
void set_hot(KParams& k, int hot_k, const int32_t* const* in_hot, int nin)
{
    for (int w = 0; w < nin; ++w)
        if (!in_hot[w]) hot_k = 0;
    k.hot_k = hot_k;
    for (int w = 0; w < nin; ++w) k.hot[w] = hot_k ? in_hot[w] + (hot_k - 1) : nullptr;
}

// Rows that cross the edge of a chunk of several units cross a unit's edge, so
// they are in the zero-row list.
KParams base_params(const ModeDev& m, int64_t chunk)
{
    KParams k{};
    k.out_idx = m.out_idx;
    for (int w = 0; w < kMaxIn; ++w) k.in_idx[w] = m.in_idx[w];
    k.val = m.val;
    k.queue = m.queue;
    k.n_stripes = queue_stripes();
    k.chunk = chunk;
    k.n_chunks = (m.nnz + chunk - 1) / chunk;
    k.stripe_len = (int)((k.n_chunks + k.n_stripes - 1) / k.n_stripes);
    k.nnz = m.nnz;
    k.rows = m.rows;
    k.zero_row = m.zero_row;
    k.sink = m.sink;
    k.prev_key = m.prev_key;
    k.next_key = m.next_key;
    k.per_chunk = 1;
    if (m.slots.slot) {
        k.cut = m.slots.cut;
        k.slot = m.slots.slot;
        k.per_chunk = (int)(chunk / m.unit);
    }
    return k;
}

// A gradient that was computed before its factor was known.  That factor is 1 when
// the loss itself is differentiated, and the pass over the matrix then left out
// (54 us of a step's 984 for a 1M x 32 factor).
__global__ void __launch_bounds__(kBlock) scale_kernel(float* x, int64_t n, const double* s)
{
    const double d = *s;
    if (d == 1.0) return;
    const float f = (float)d;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, n4 = n / 4;
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float4* x4 = reinterpret_cast<float4*>(x);
    for (int64_t i = i0; i < n4; i += stride) {
        float4 v = x4[i];
        v.x *= f; v.y *= f; v.z *= f; v.w *= f;
        x4[i] = v;
    }
    for (int64_t i = 4 * n4 + i0; i < n; i += stride) x[i] *= f;
}

// The output rows whose pieces have slots, each piece a chunk's (per_chunk units) sum, in
// fp64 and in one order whatever the waves' was; and the untouched rows, where the init
// kernel is left out.  Blocks: one per heavy row and 32 columns, then those of the light
// rows (a wave each), then those that zero.  cw lanes of 4 columns hold a piece, a wave's or
// block's pieces lie side by side, a heavy row's 8 deep; sums by shuffles, then through
// LDS.  What bounds it is latency: the row, then one round of loads (a heavy row's 8 BLOCK
// / cw pieces) of slots that other XCDs have just written.  4.8 us for 23 heavy rows of up
// to 185 pieces at rank 32 (a mode of 5M nonzeros, whose kernel takes 76), 12 for 195 rows
// of up to 1500 at rank 64 (20M, 315), 84 for one of 18,900 (1B, 16,200); blocks of 1024
// threads where a row may have thousands.  With 16, 8 and 4 columns per block the second
// took 13, 23 and 45 us.
constexpr int kCloseCols = 32;
struct CloseParams {
    const int4* heavy;
    const int4* light;
    int n_heavy, n_light, heavy_blocks, light_blocks;
    const float* slot;
    float* out;
    int64_t ld;
    int stride, col0, ncols, cw, per_chunk;
    bool vec4;
    const int32_t* zrows;
    const int32_t* gaps;
    int64_t n_zero, n_gaps;
};
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK) close_kernel(const CloseParams p)
{
    constexpr int kWaves = BLOCK / 64;
    __shared__ double s[kWaves][kCloseCols];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, block = blockIdx.x;
    if (block >= p.heavy_blocks + p.light_blocks) {
        const int first = p.heavy_blocks + p.light_blocks;
        zero_rows(p.out, p.ld, p.col0, p.ncols, p.vec4, p.zrows, p.n_zero, p.gaps, p.n_gaps, block - first,
                  gridDim.x - first);
        return;
    }
    const bool is_heavy = block < p.heavy_blocks;
    const int index = is_heavy ? block % p.n_heavy : (block - p.heavy_blocks) * kWaves + wave;
    if (!is_heavy && index >= p.n_light) return;
    const int4 r = is_heavy ? p.heavy[index] : p.light[index];
    // piece 0 is the first unit's, the others those of the chunks that start after it
    const int chunk0 = r.y / p.per_chunk, pieces = r.z / p.per_chunk - chunk0 + 1;
    const int c4 = lane & (p.cw - 1);
    const float* src = p.slot + (int64_t)r.w * p.stride + 4 * c4;
    auto at = [&](int k) { return (int64_t)(k == 0 ? 0 : (chunk0 + k) * p.per_chunk - r.y) * p.stride; };
    float* const row = p.out + (int64_t)r.x * p.ld + p.col0;
    double acc[4];
    // pieces first, first + step, ... of the columns from col on, D of them in flight
    auto sum = [&](int col, int first, int step, auto depth) {
        constexpr int D = decltype(depth)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = 0.0;
        for (int k0 = first; k0 < pieces; k0 += D * step) {
            float4 v[D];
#pragma unroll
            for (int u = 0; u < D; ++u)
                v[u] = col + 4 * c4 < p.stride && k0 + u * step < pieces
                           ? *reinterpret_cast<const float4*>(src + col + at(k0 + u * step))
                           : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < D; ++u) {
                acc[0] += (double)v[u].x;
                acc[1] += (double)v[u].y;
                acc[2] += (double)v[u].z;
                acc[3] += (double)v[u].w;
            }
        }
        for (int m = p.cw; m < 64; m <<= 1)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += __shfl_xor(acc[i], m, 64);
    };
    if (is_heavy) {
        const int col = block / p.n_heavy * kCloseCols;
        sum(col, tid / p.cw, BLOCK / p.cw, std::integral_constant<int, 8>{});
        if (lane < p.cw)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[wave][4 * lane + i] = acc[i];
        __syncthreads();
        if (tid < 4 * p.cw && col + tid < p.ncols) {
            double x = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) x += s[w][tid];
            row[col + tid] = (float)x;
        }
        return;
    }
    for (int col = 0; col < p.ncols; col += kCloseCols) {
        sum(col, lane / p.cw, 64 / p.cw, std::integral_constant<int, 1>{});
        if (lane < p.cw)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (col + 4 * lane + i < p.ncols) row[col + 4 * lane + i] = (float)acc[i];
    }
}

hipError_t launch_close(const ModeDev& m, const KParams& k, hipStream_t st)
{
    CloseParams c{};
    c.heavy = m.slots.heavy;
    c.light = m.slots.light;
    c.n_heavy = m.slots.n_heavy;
    c.n_light = m.slots.n_light;
    c.heavy_blocks = c.n_heavy * ((k.ncols + kCloseCols - 1) / kCloseCols);
    const int block = m.slots.all ? 256 : 1024;
    c.light_blocks = (c.n_light + block / 64 - 1) / (block / 64);
    c.slot = m.slots.slot;
    c.out = k.out;
    c.ld = k.ld;
    c.stride = slot_stride(k.ncols);
    c.col0 = k.col0;
    c.ncols = k.ncols;
    c.cw = 1;
    while (4 * c.cw < std::min(k.ncols, kCloseCols)) c.cw *= 2;
    c.per_chunk = k.per_chunk;
    int64_t zero_blocks = 0;
    if (m.slots.all) {
        c.vec4 = whole_vectors(k.out, k.ld, k.col0, k.ncols);
        c.zrows = m.slots.zrows;
        c.gaps = m.gaps;
        c.n_zero = m.slots.n_zero;
        c.n_gaps = m.n_gaps;
        const int64_t stores = (c.n_zero * (c.vec4 ? k.ncols / 4 : k.ncols) + block - 1) / block;
        zero_blocks = std::min<int64_t>(std::max(stores, c.n_gaps), 4096);
    }
    const int64_t grid = c.heavy_blocks + c.light_blocks + zero_blocks;
    if (grid == 0) return hipSuccess;
    if (block == 256) hipLaunchKernelGGL(close_kernel<256>, dim3((unsigned)grid), dim3(256), 0, st, c);
    else hipLaunchKernelGGL(close_kernel<1024>, dim3((unsigned)grid), dim3(1024), 0, st, c);
    return hipGetLastError();
}

// dst[p] = src[perm[p]] for 32-bit words (layout build).
__global__ void __launch_bounds__(kBlock) permute_kernel(uint32_t* dst, const uint32_t* src, const int32_t* perm,
                                                         int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) dst[p] = src[perm[p]];
}

KernelFn pick_mttkrp(int nin, FactorType ft, Kind kind, Lanes v, bool buf)
{
    if (kind == Kind::ResidualGrad) return ft == FactorType::F32 ? pick_grad(nin, v, buf) : nullptr;
    if (kind == Kind::ResidualGradLoss) return ft == FactorType::F32 ? pick_grad_loss(nin, v, buf) : nullptr;
    return ft == FactorType::F32 ? pick_mttkrp_f32(nin, v, buf) : pick_mttkrp_bf16(nin, v, buf);
}

}  // namespace dev

using namespace dev;

hipError_t launch_permute32(void* dst, const void* src, const int32_t* perm, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((n + kBlock - 1) / kBlock, 8192);
    hipLaunchKernelGGL(permute_kernel, dim3(grid), dim3(kBlock), 0, st, static_cast<uint32_t*>(dst),
                       static_cast<const uint32_t*>(src), perm, n);
    return hipGetLastError();
}

hipError_t launch_scale(float* x, int64_t n, const double* s, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((n / 4 + kBlock - 1) / kBlock, 2048));
    hipLaunchKernelGGL(scale_kernel, dim3(grid), dim3(kBlock), 0, st, x, n, s);
    return hipGetLastError();
}

// MTTKRP of a small tensor in one launch per column tile.
static hipError_t launch_small(const LaunchArgs& a, SmallFn fn, int tile, int eb)
{
    const ModeDev& m = *a.m;
    SmallParams k{};
    k.out_idx = m.out_idx;
    for (int w = 0; w < a.nin; ++w) {
        k.in_idx[w] = m.in_idx[w];
        k.fac[w] = a.in_factors[w];
        k.fbytes[w] = (uint32_t)((uint64_t)a.in_rows[w] * a.rank * eb);
    }
    k.val = m.val;
    k.out = a.out;
    k.ld = a.rank;
    k.nnz = (int)m.nnz;
    k.n_units = m.small.n_units;
    k.cut = m.small.cut;
    k.left = m.small.left;
    k.split = m.small.split;
    k.arrived = m.small.arrived;
    k.share = m.small.share;
    k.zrows = m.small.zrows;
    k.n_zero = m.small.n_zero;
    k.gaps = m.gaps;
    k.n_gaps = m.n_gaps;
    for (int col0 = 0; col0 < a.rank; col0 += tile) {
        k.col0 = col0;
        k.ncols = std::min(tile, a.rank - col0);
        k.vec4 = a.rank % 4 == 0 && col0 % 4 == 0 && k.ncols % 4 == 0;
        // blocks beside the units' for the untouched rows: 8 stores per lane, or a range
        const int64_t stores = (k.n_zero * (k.vec4 ? k.ncols / 4 : k.ncols) + 511) / 512;
        const int64_t grid = std::max<int64_t>(k.n_units, std::min<int64_t>(4096, std::max(stores, k.n_gaps)));
        void* args[] = {&k};
        hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)grid), dim3(64), args, 0, a.stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_mttkrp(const LaunchArgs& a)
{
    const ModeDev& m = *a.m;
    const int eb = (a.ftype == FactorType::F32) ? 4 : 2;
    // buffer addressing when every factor the kernel reads fits in 32-bit
    // offsets with one row to spare
    bool buf = AMPED_BUFFER_LOADS != 0;
    for (int w = 0; w < a.nin; ++w)
        if (!fits_buffer(a.in_rows[w], a.rank, eb)) buf = false;
    const bool grad = a.kind != Kind::Mttkrp;   // the residual forms read the output mode's factor
    if (grad && !fits_buffer(m.rows, a.rank, 4)) buf = false;
    auto [tile, v] = split_columns(a.rank, a.ftype, a.nin);
    // (the load-balance build records the queue's kernel at every size)
    if (!AMPED_QUEUE_STATS && !grad && buf && v.lpr && m.small.n_units > 0)
        if (SmallFn small = pick_small(a.nin, a.ftype, v)) return launch_small(a, small, tile, eb);
    // An exact rank's instance with the hot-row cache is used where the cache
    // is; the residual forms (no cache) always take the exact one.
    if (!grad && buf && m.nnz < kHotMinNnz) v.exact = false;
    KernelFn fn = v.lpr ? pick_mttkrp(a.nin, a.ftype, a.kind, v, buf) : nullptr;
    const bool scalar = (fn == nullptr);
    // the fused residual form needs the whole row in one launch (rank <= 64
    // on the scalar path)
    if (scalar && grad && a.rank > 64) return hipErrorNotSupported;
    if (scalar) {
        v = Lanes{};
        tile = std::min(64, a.rank);
        fn = pick_mttkrp(a.nin, a.ftype, a.kind, v, false);
    }
    if (!fn) return hipErrorNotSupported;
    KParams k = base_params(m, grad ? m.residual_chunk : m.chunk);
    for (int w = 0; w < a.nin; ++w) {
        k.fac[w] = a.in_factors[w];
        k.fbytes[w] = buf ? (uint32_t)((uint64_t)a.in_rows[w] * a.rank * eb) : 0u;
    }
    k.own = a.own_factor;
    k.own_bytes = (buf && grad) ? (uint32_t)((uint64_t)m.rows * a.rank * 4) : 0u;
    k.out = a.out;
    k.loss = a.kind == Kind::ResidualGradLoss ? a.loss : nullptr;
    k.ld = a.rank;
    k.scale = a.scale;
    k.dev_scale = a.dev_scale;
    const bool cache = !grad && v.exact;
    const int block = mttkrp_block(cache);
    const Shape sh = launch_shape(fn, block, a.nin, v.lpr * v.rpl * eb, cache && !scalar && m.nnz >= kHotMinNnz);
    if (sh.grid <= 0) return hipErrorInvalidDevice;
    set_hot(k, sh.hot_k, a.in_hot, a.nin);
    // more units than waves: the queue's counters are used, so they are reset first
    const bool queued = k.n_chunks > (int64_t)launch_grid(sh, k) * (block / 64);
    for (int col0 = 0; col0 < a.rank; col0 += tile) {
        const int ncols = std::min(tile, a.rank - col0);
        // the loss (one launch: the residual forms never tile columns) is reset
        // by the init kernel unless this launch adds to it
        double* const loss = a.loss_accumulate ? nullptr : k.loss;
        hipError_t e = hipSuccess;
        if (!m.slots.all) e = launch_init(m, a.out, a.rank, col0, ncols, loss, a.stream);
        else if (loss || queued) e = launch_init(m, nullptr, 0, 0, 0, loss, a.stream);
        if (e != hipSuccess) return e;
        if (m.n_chunks == 0) continue;
        k.col0 = col0;
        k.ncols = ncols;
#if AMPED_QUEUE_STATS
        if ((e = qstats_attach(k, launch_grid(sh, k), block, a.stream)) != hipSuccess) return e;
#endif
        void* args[] = {&k};
        e = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3(launch_grid(sh, k)), dim3(block), args, sh.dyn,
                            a.stream);
        if (e != hipSuccess) return e;
        if (k.cut && (e = launch_close(m, k, a.stream)) != hipSuccess) return e;
    }
    return hipSuccess;
}

#if AMPED_QUEUE_STATS
hipError_t queue_stats_copy(unsigned long long* host, int64_t max_records, int64_t* n_records, int* waves_per_block)
{
    std::lock_guard<std::mutex> lk(g_qstats_mu);
    *n_records = g_qstats.n;
    *waves_per_block = g_qstats.waves_per_block;
    if (!host || g_qstats.n == 0) return hipSuccess;
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    const int64_t n = std::min(max_records, g_qstats.n);
    return hipMemcpy(host, g_qstats.dev, (size_t)n * 4 * sizeof(unsigned long long), hipMemcpyDeviceToHost);
}
#endif

hipError_t launch_cp_loss(const LossArgs& a)
{
    const ModeDev& m = *a.m;
    bool buf = AMPED_BUFFER_LOADS != 0 && fits_buffer(m.rows, a.rank, 4);
    for (int w = 0; w < a.order - 1; ++w)
        if (!fits_buffer(a.in_rows[w], a.rank, 4)) buf = false;
    const Lanes v = choose_lanes(a.rank, FactorType::F32, a.order - 1);
    KernelFn fn = v.lpr ? pick_loss(a.order - 1, v, buf) : nullptr;
    const bool scalar = (fn == nullptr);
    if (scalar && a.rank > 64) return hipErrorNotSupported;
    if (scalar) fn = pick_loss(a.order - 1, Lanes{}, false);
    if (!fn) return hipErrorNotSupported;
    KParams k = base_params(m, m.residual_chunk);
    for (int w = 0; w < a.order - 1; ++w) {
        k.fac[w] = a.in_factors[w];
        k.fbytes[w] = buf ? (uint32_t)((uint64_t)a.in_rows[w] * a.rank * 4) : 0u;
    }
    k.own = a.own_factor;
    k.own_bytes = buf ? (uint32_t)((uint64_t)m.rows * a.rank * 4) : 0u;
    k.loss = a.loss;
    k.ld = a.rank;
    k.col0 = 0;
    k.ncols = a.rank;
    hipError_t e = launch_init(m, nullptr, 0, 0, 0, a.accumulate ? nullptr : a.loss, a.stream);
    if (e != hipSuccess) return e;
    if (m.n_chunks == 0) return hipSuccess;
    const int block = mttkrp_block(false);
    const Shape sh = launch_shape(fn, block, a.order - 1, a.rank * 4, false);
    if (sh.grid <= 0) return hipErrorInvalidDevice;
#if AMPED_QUEUE_STATS
    if ((e = qstats_attach(k, launch_grid(sh, k), block, a.stream)) != hipSuccess) return e;
#endif
    void* args[] = {&k};
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3(launch_grid(sh, k)), dim3(block), args, sh.dyn,
                           a.stream);
}

}  // namespace amped
