#pragma once
// Device code shared by the gfx950 kernel translation units: sparse MTTKRP (Eq. 1, Sec. 2.1), its bfloat16-factor
// form, the sparse CP loss and the fused residual + MTTKRP gradient.
//
// Work decomposition (one GPU's share of the paper's scheme, Sec. 3-4):
//  * A mode's nonzeros are sorted by output index (Sec. 3.1: all nonzeros of
//    one output index together) and cut into units of equal nonzero counts,
//    the inter-shard partitions of Sec. 3.1/3.2.  (The layout contract's chunks
//    are those units where a caller names their length; the kernels' `chunk`
//    is always the unit.)
//  * A persistent grid of wave64s replaces the hardware block scheduler of
//    Sec. 4.2: each wave starts with a unit of its own and takes further ones
//    from device atomic counters until none is left, so skewed slices spread
//    over all CUs.
//  * Inside a unit the wave is G groups of LPR lanes.  Each lane holds RPL
//    consecutive columns of a factor row (16 bytes; 8 for bf16 rows of 32
//    bytes, and of 64 bytes when at most two factors are gathered), so a group
//    loads a whole row with one coalesced access.  Group g walks its own contiguous run of
//    the unit's nonzeros in order and keeps the running sum of the current
//    output row in registers (the elementwise computation, EC of Sec. 3,
//    reduced over consecutive equal output indices instead of one atomic per
//    nonzero as in Alg. 2).
//  * A row that starts and ends inside one group's run is written once with a
//    plain store.  Pieces of rows that cross group boundaries are parked in
//    LDS and summed at the end of the unit; only rows that cross a unit's
//    boundary are added to memory with fp32 atomics (Sec. 3.2 uses atomics
//    between SMs), after the init kernel has zeroed them.  Where the library
//    sizes the units the pieces of rows that span many of them, or of all that
//    cross an edge, go to slots instead, which close_kernel adds in fp64.
//  * Untouched output rows are zeroed once, by the init kernel or close_kernel.
//  * From 32M nonzeros on, MTTKRP keeps the most-used rows of each input factor
//    in LDS (hot-row cache); their gathers issue no memory request.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "lanes.h"

namespace amped {
namespace dev {

constexpr int kBlock = 256;  // init and permute kernels
// MTTKRP kernel blocks: the waves of a block share only the hot-row cache,
// so the MTTKRP instances that have it run 512-thread blocks, one per CU beside
// a large cache, and the others (the residual and loss forms, whose extra
// own-row registers leave them short of waves otherwise, and MTTKRP without the
// cache) 256-thread blocks.
#ifndef AMPED_BLOCK
#define AMPED_BLOCK 512
#endif
#ifndef AMPED_BLOCK_OWN
#define AMPED_BLOCK_OWN 256
#endif
__host__ __device__ constexpr int mttkrp_block(bool cache) { return cache ? AMPED_BLOCK : AMPED_BLOCK_OWN; }
// Instances with the hot-row cache: MTTKRP of the exact ranks.
__host__ __device__ constexpr bool has_hot_cache(int kind, bool exact) { return kind == 0 && exact; }
// Compile-time knobs, off by default (both measured slower): non-temporal
// output-row stores, and the cache-policy bits of factor-row gathers.
#ifndef AMPED_OUT_NT
#define AMPED_OUT_NT 0
#endif
#ifndef AMPED_GATHER_AUX
#define AMPED_GATHER_AUX 0
#endif
// Diagnostic build: every wave of the MTTKRP-shaped kernels records how many
// chunks and nonzeros it took from the work queue and when it took its first
// chunk and exited (constant-rate wall clock), for the load-balance report.
#ifndef AMPED_QUEUE_STATS
#define AMPED_QUEUE_STATS 0
#endif
constexpr int kMaxIn = kMaxOrder - 1;

// Tuning knobs (compile-time): nonzeros per group whose gathers are issued
// together (MTTKRP, then the residual gradient, with up to 2 input modes; the
// loss and higher orders use the third value), and the waves per SIMD the
// register allocation must allow (0 = compiler's choice).
#ifndef AMPED_UMAX
#define AMPED_UMAX 4
#endif
#ifndef AMPED_UMAX_GRAD
#define AMPED_UMAX_GRAD 4
#endif
#ifndef AMPED_UMAX_OWN
#define AMPED_UMAX_OWN 2
#endif
#ifndef AMPED_UMAX_NIN
#define AMPED_UMAX_NIN 2   // most input modes that still get AMPED_UMAX
#endif
#ifndef AMPED_MIN_WAVES
#define AMPED_MIN_WAVES 2   // an instance that takes more than 256 registers runs one wave per SIMD
#endif
// Spread each tile's metadata loads over its batch pairs (see the tile loop).
#ifndef AMPED_META_SPREAD
#define AMPED_META_SPREAD 1
#endif
#if AMPED_MIN_WAVES > 0
#define AMPED_OCCUPANCY __attribute__((amdgpu_waves_per_eu(AMPED_MIN_WAVES)))
#else
#define AMPED_OCCUPANCY
#endif

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

struct KParams {
    const int32_t* out_idx;
    const int32_t* in_idx[kMaxIn];
    const float* val;
    const void* fac[kMaxIn];
    const float* own;
    float* out;
    double* loss;
    unsigned* queue;  // n_stripes counters, kQueueStride words apart
    int n_stripes;    // contiguous chunk stripes, one counter each (1..kQueueSlots)
    int stripe_len;   // chunks per stripe
    int64_t nnz, chunk, n_chunks, rows;
    int64_t ld;     // row stride of factors and output, in elements
    int col0;       // first column handled by this launch
    int ncols;      // columns handled by this launch
    float scale;
    const double* dev_scale;  // multiplies scale (NULL: 1)
    uint32_t fbytes[kMaxIn];  // input factor sizes in bytes (buffer addressing)
    uint32_t own_bytes;
    const void* zero_row;     // 16 zero bytes: what padding entries read on the 64-bit path
    float* sink;              // 64 * 8 floats that absorb stores which must not land
    const int2* cut;          // where units start inside rows with slots (NULL: none; launch_slot_rows)
    float* slot;              // the slots, of slot_stride(ncols) floats each
    int per_chunk;            // units per chunk
    int prev_key;             // output index just before position 0 of these arrays (-1: none)
    int next_key;             // output index just after position nnz - 1 (-1: none)
    const int32_t* hot[kMaxIn];  // per input: direct-mapped table of hot_k rows kept in LDS
    int hot_k;                // LDS row-cache slots per input (power of two; 0 = none)
#if AMPED_QUEUE_STATS
    unsigned long long* qstats;  // per wave: chunks, nonzeros, first-pop and exit times
#endif
};

// Dynamic LDS of the MTTKRP kernel: 16 zero bytes, then (vector path, K > 0)
// the tags [NIN][K] and rows [NIN][K][row bytes] of the hot-row cache.
__host__ __device__ constexpr size_t hot_tag_offset() { return 16; }
__host__ __device__ constexpr size_t hot_row_offset(int nin, int k) { return (16 + (size_t)nin * k * 4 + 15) & ~(size_t)15; }
__host__ __device__ constexpr size_t hot_lds_bytes(int nin, int k, int row_bytes)
{
    return k > 0 ? hot_row_offset(nin, k) + (size_t)nin * k * row_bytes : 16;
}

// A row piece's slot: whole 16 bytes.
__host__ __device__ constexpr int slot_stride(int ncols) { return (ncols + 3) & ~3; }

// Raw buffer resource over [base, base + bytes): word 3 is the gfx9-family
// default for untyped dword access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// ------------------------------------------------------------ compile-time loops
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// One product or sum rounded by itself (never contracted into an fma).
__device__ __forceinline__ float mul_rounded(float a, float b)
{
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float add_rounded(float a, float b)
{
#pragma clang fp contract(off)
    return a + b;
}

template <int LPR>
__device__ __forceinline__ float group_sum(float x)
{
#pragma unroll
    for (int m = 1; m < LPR; m <<= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// ------------------------------------------------------------------ row access
// Row<T, RPL>: RPL consecutive columns of a factor row as fp32, read from a
// 64-bit address (load_ptr) or a buffer resource and 32-bit byte offset
// (load_buf, vector forms only).
template <typename T, int RPL> struct Row;


template <> struct Row<float, 4> {
    using Raw = float4;
    // bitwise OR with the same lane's 16 bytes of an LDS row (one side is 0)
    static __device__ __forceinline__ Raw merge_lds(const Raw& a, const char* lds)
    {
        const u32x4 b = *reinterpret_cast<const u32x4*>(lds);
        return make_float4(__uint_as_float(__float_as_uint(a.x) | b.x), __uint_as_float(__float_as_uint(a.y) | b.y),
                           __uint_as_float(__float_as_uint(a.z) | b.z), __uint_as_float(__float_as_uint(a.w) | b.w));
    }
    static __device__ __forceinline__ Raw load_buf(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, AMPED_GATHER_AUX);
        return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    }
    static __device__ __forceinline__ Raw load_ptr(const char* a) { return *reinterpret_cast<const float4*>(a); }
    static __device__ __forceinline__ void unpack(const Raw& r, float (&v)[4])
    {
        v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w;
    }
};

template <> struct Row<uint16_t, 8> {  // bfloat16 bit patterns, widened exactly
    using Raw = uint4;
    static __device__ __forceinline__ Raw merge_lds(const Raw& a, const char* lds)
    {
        const u32x4 b = *reinterpret_cast<const u32x4*>(lds);
        return make_uint4(a.x | b.x, a.y | b.y, a.z | b.z, a.w | b.w);
    }
    static __device__ __forceinline__ Raw load_buf(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, AMPED_GATHER_AUX);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    static __device__ __forceinline__ Raw load_ptr(const char* a) { return *reinterpret_cast<const uint4*>(a); }
    static __device__ __forceinline__ void unpack(const Raw& r, float (&v)[8])
    {
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
};

template <> struct Row<uint16_t, 4> {  // 4 bfloat16 per lane (rows of up to 64 bytes)
    using Raw = uint2;
    static __device__ __forceinline__ Raw merge_lds(const Raw& a, const char* lds)
    {
        const u32x2 b = *reinterpret_cast<const u32x2*>(lds);
        return make_uint2(a.x | b.x, a.y | b.y);
    }
    static __device__ __forceinline__ Raw load_buf(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, AMPED_GATHER_AUX);
        return make_uint2(v.x, v.y);
    }
    static __device__ __forceinline__ Raw load_ptr(const char* a) { return *reinterpret_cast<const uint2*>(a); }
    static __device__ __forceinline__ void unpack(const Raw& r, float (&v)[4])
    {
        v[0] = __uint_as_float(r.x << 16);
        v[1] = __uint_as_float(r.x & 0xFFFF0000u);
        v[2] = __uint_as_float(r.y << 16);
        v[3] = __uint_as_float(r.y & 0xFFFF0000u);
    }
};

template <> struct Row<float, 1> {
    using Raw = float;
    static __device__ __forceinline__ Raw load_buf(__amdgpu_buffer_rsrc_t, uint32_t) { return 0.f; }
    static __device__ __forceinline__ Raw load_ptr(const char* a) { return *reinterpret_cast<const float*>(a); }
    static __device__ __forceinline__ void unpack(const Raw& r, float (&v)[1]) { v[0] = r; }
};

template <> struct Row<uint16_t, 1> {
    using Raw = uint32_t;
    static __device__ __forceinline__ Raw load_buf(__amdgpu_buffer_rsrc_t, uint32_t) { return 0u; }
    static __device__ __forceinline__ Raw load_ptr(const char* a) { return *reinterpret_cast<const uint16_t*>(a); }
    static __device__ __forceinline__ void unpack(const Raw& r, float (&v)[1]) { v[0] = __uint_as_float(r << 16); }
};

// Output row pieces: RPL fp32 columns of row `row`, starting at column c.
template <int RPL>
__device__ __forceinline__ void store_vec(float* p, const float (&v)[RPL]);
template <int RPL>
__device__ __forceinline__ void store_cols(float* out, int64_t row, int64_t ld, int c, const float (&v)[RPL])
{
    store_vec<RPL>(out + row * ld + c, v);
}

// RPL fp32 values of an output row to a lane's own address.
template <int RPL>
__device__ __forceinline__ void store_vec(float* p, const float (&v)[RPL])
{
    if constexpr (RPL % 4 == 0) {
#pragma unroll
        for (int i = 0; i < RPL; i += 4) {
            // rows of ranks that are no multiple of 4 are only 4-byte aligned,
            // which 16-byte global accesses of gfx950 take
            const f32x4_a4 x = {v[i], v[i + 1], v[i + 2], v[i + 3]};
            if constexpr (AMPED_OUT_NT != 0) __builtin_nontemporal_store(x, reinterpret_cast<f32x4_a4*>(p + i));
            else *reinterpret_cast<f32x4_a4*>(p + i) = x;
        }
    } else {
#pragma unroll
        for (int i = 0; i < RPL; ++i) p[i] = v[i];
    }
}
template <int RPL>
__device__ __forceinline__ void lds_store(float* p, const float (&v)[RPL])
{
    if constexpr (RPL % 4 == 0) {
#pragma unroll
        for (int i = 0; i < RPL; i += 4)
            *reinterpret_cast<float4*>(p + i) = make_float4(v[i], v[i + 1], v[i + 2], v[i + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < RPL; ++i) p[i] = v[i];
    }
}

// U consecutive ints of an LDS ring row (16-byte aligned when U % 4 == 0,
// 8-byte aligned when U == 2) with the widest reads that fit.
template <int U>
__device__ __forceinline__ void lds_vec(const int* p, int (&v)[U])
{
    if constexpr (U % 4 == 0) {
#pragma unroll
        for (int i = 0; i < U; i += 4) {
            const i32x4 x = *reinterpret_cast<const i32x4*>(p + i);
            v[i] = x.x; v[i + 1] = x.y; v[i + 2] = x.z; v[i + 3] = x.w;
        }
    } else if constexpr (U == 2) {
        const int2 x = *reinterpret_cast<const int2*>(p);
        v[0] = x.x; v[1] = x.y;
    } else {
#pragma unroll
        for (int i = 0; i < U; ++i) v[i] = p[i];
    }
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Work distribution.  The chunks are split into S contiguous stripes, each with
// its own counter.  A wave's first chunk is fixed by its place in the grid; the
// next ones come from the counter of its home stripe (with one stripe per XCD
// the consecutive chunks of a stripe, neighbouring output rows or, for a heavy
// row, neighbouring input indices, are taken by one XCD's CUs while any chunk
// is left on it), and when that runs dry from the stripe with most chunks left,
// so no CU idles while any chunk is left anywhere.
//
// What bounds it: an atomic on one cache line takes 12 ns, one after the other,
// whatever the wave.  So every counter has a line of its own, the first chunks
// and a grid with a wave for every chunk need no atomic, and a wave looks at all
// counters with one load (lane x reads stripe x) before it takes from another
// stripe.  Counters side by side in one line, with every wave ending by a
// failing atomic on each of the 8, took 2048 * 8 * 12 ns = 195 us at the end of
// every launch, whatever its work: 228 us instead of 48 us for 25 chunks
// (100k nonzeros, rank 16), 273 instead of 102 us for 5M nonzeros at rank 32,
// 2.95 instead of 2.86 ms for 200M.  The next chunk is asked for before the
// current one is worked on, so the atomic's latency is hidden.
//
// A counter grows only by its stripe's chunks and by at most one failing add per
// wave of the grid (a stripe once seen empty is not asked again), so it stays
// below 2^32 (chunks < 2^31).
struct ChunkQueue {
    unsigned* q;
    unsigned n, len;      // chunks; chunks per stripe: stripe x holds [x * len, min((x + 1) * len, n))
    unsigned S, home;     // stripes, this wave's stripe
    unsigned per, rest;   // waves of the grid per stripe, and stripes with one block of waves more
    unsigned waves;       // per block
    bool more;            // the home stripe may have more chunks
    unsigned asked;       // lane 0: the home counter's value

    __device__ __forceinline__ unsigned size(unsigned x) const { return min(n, (x + 1) * len) - min(n, x * len); }
    // chunks of stripe x that are first chunks of its waves, outside the counter
    __device__ __forceinline__ unsigned fixed(unsigned x) const { return per + (x < rest ? waves : 0u); }

    // the wave's first chunk, or -1
    __device__ __forceinline__ int start(const KParams& p, unsigned block, unsigned wave, unsigned waves_per_block)
    {
        const unsigned blocks = gridDim.x;
        q = p.queue;
        n = (unsigned)p.n_chunks;
        S = (unsigned)p.n_stripes;
        len = (unsigned)p.stripe_len;
        waves = waves_per_block;
        home = block % S;
        per = blocks / S * waves;
        rest = blocks % S;
        asked = 0;
        more = n > blocks * waves;
        if (!more) {   // a wave for every chunk: no counter (S = 0: none to look at)
            S = 0;
            const unsigned c = wave * blocks + block;   // spread over the CUs first
            return c < n ? (int)c : -1;
        }
        const unsigned i = block / S * waves + wave;
        return i < size(home) ? (int)(home * len + i) : take(0u);
    }
    // asks for the home stripe's next chunk; next() gets the answer
    __device__ __forceinline__ void ask(int lane)
    {
        if (more && lane == 0) asked = atomicAdd(q + home * kQueueStride, 1u);
    }
    __device__ __forceinline__ int next()
    {
        if (more) {
            const unsigned i = (unsigned)__builtin_amdgcn_readfirstlane((int)asked) + fixed(home);
            if (i < size(home)) return (int)(home * len + i);
        }
        return S == 0 ? -1 : take(1u << home);
    }
    // a chunk of the stripe with most left, or -1 when none is left anywhere
    // (dry: bits of stripes seen empty)
    __device__ __forceinline__ int take(unsigned dry)
    {
        more = false;
        const unsigned lane = threadIdx.x & 63;
        for (;;) {
            unsigned best = lane & 7;
            if (lane < S && !((dry >> lane) & 1u)) {
                const unsigned c = __hip_atomic_load(q + lane * kQueueStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                                   fixed(lane);
                const unsigned sz = size(lane);
                best |= c < sz ? min(sz - c, 0x0FFFFFFFu) << 3 : 0u;
            }
#pragma unroll
            for (int m = 1; m < 8; m <<= 1) best = max(best, (unsigned)__shfl_xor((int)best, m, 64));
            best = (unsigned)__builtin_amdgcn_readfirstlane((int)best);
            if (best < 8) return -1;
            const unsigned x = best & 7;
            unsigned c = 0;
            if (lane == 0) c = atomicAdd(q + x * kQueueStride, 1u);
            c = (unsigned)__builtin_amdgcn_readfirstlane((int)c) + fixed(x);
            if (c < size(x)) return (int)(x * len + c);
            dry |= 1u << x;
        }
    }
};

// --------------------------------------------------------------- MTTKRP kernel
// KIND 0: MTTKRP.  KIND 1: scale * MTTKRP of the residuals val - CP model,
// recomputed per nonzero from all factor rows.  KIND 2: the sparse CP loss,
// sum over nonzeros of (val - CP model)^2 (per-entry work in fp32, each
// squared residual added in fp64, one fp64 atomic per wave; no output
// matrix).  KIND 3: KIND 1 and KIND 2 in one pass (every mode's layout holds
// every nonzero, so the residuals the gradient computes give the loss too).
//
// Memory accesses are software-pipelined:
//  * the nonzero metadata of tile tau+2 is loaded (VGPRs) while tile tau is
//    processed and parked in a 2-slot LDS ring at the start of tile tau+1, so
//    its latency is hidden behind at least two batches of work;
//  * the factor-row gathers of batch q+1 are issued before batch q is
//    consumed (two register buffers), so a wave always has a batch in flight.
// A tile is TS >= 2U nonzeros per group, a batch U nonzeros per group.
//
// The inner loop has no per-nonzero bounds test: ring entries past the end of
// a group's run are padding that carries the run's last output index, a zero
// value and the row index -1, whose gather returns zeros (past the end of the
// buffer resource, or redirected to a zero row on the 64-bit path).  Padding
// therefore adds exact zeros to the open row and never starts a new one.
//
// EXACT: the launch's columns are LPR * RPL (or, on the column-tile path, RPL is
// 1).  Otherwise they are any number up to that, from RPL on: lane s reads RPL
// columns from min(s * RPL, columns - RPL), so the lanes of a group still cover
// the row with one load each, the last ones overlapping; all loads stay inside
// the row, a column held twice gets the same value twice, and sums over the
// columns leave the second one out.
template <int NIN, int LPR, int RPL, typename T, int KIND, bool BUF, bool EXACT>
__global__ void __launch_bounds__(mttkrp_block(has_hot_cache(KIND, EXACT))) AMPED_OCCUPANCY
mttkrp_kernel(const KParams p)
{
    constexpr bool HOT = has_hot_cache(KIND, EXACT) && RPL > 1;
    constexpr int kMttkrpBlock = mttkrp_block(has_hot_cache(KIND, EXACT));
    constexpr int kWaves = kMttkrpBlock / 64;
    constexpr int G = 64 / LPR;
    constexpr int RT = LPR * RPL;
    // nonzeros per group per batch: the loss and high orders keep fewer rows
    // in flight per batch
    constexpr int U = (KIND != 2 && NIN <= AMPED_UMAX_NIN) ? (KIND == 0 ? AMPED_UMAX : AMPED_UMAX_GRAD)
                                                          : AMPED_UMAX_OWN;
    constexpr bool GRAD = KIND == 1 || KIND == 3;                // residual gradient: output scaled by p.scale
    constexpr bool LOSS = KIND == 2 || KIND == 3;                // squared residuals summed into p.loss
    constexpr int TS = (4 * LPR > 2 * U) ? 4 * LPR : 2 * U;      // nonzeros per group per tile
    constexpr int Q4 = TS / (4 * LPR);                           // 16-byte metadata loads per lane and field
    constexpr int NB = TS / U;                                   // batches per tile (even)
    constexpr int NF = NIN + 2;                                  // key, input indices, value
    constexpr int FS = G * TS;                                   // ring entries per field
    constexpr bool VEC = RPL > 1;
    using RowT = Row<T, RPL>;
    constexpr bool OWN = KIND >= 1;                              // the output mode's row is read too
    constexpr bool OUT = KIND != 2;                              // an output matrix is written
    using OwnRow = Row<float, OWN ? RPL : 1>;
    constexpr int kMetaNT = 2;                                   // non-temporal cache policy
    static_assert(KIND == 0 || std::is_same<T, float>::value, "residual and loss forms are fp32 only");
    static_assert(NB % 2 == 0, "batches per tile must be even");
    static_assert(TS % 4 == 0 && (U == 1 || U == 2 || U % 4 == 0), "ring rows must be vector aligned");
    static_assert(!BUF || VEC, "buffer addressing is for the vector path");
    static_assert(EXACT || (VEC && BUF), "other ranks take the vector path with buffer addressing");

    __shared__ int s_key[kWaves][2 * G];
    __shared__ int s_ext[kWaves][2 * G];
    __shared__ __align__(16) float s_acc[kWaves][2 * G][RT];    // slot 2g+1 is also the in-loop park sink
    __shared__ __align__(16) int s_meta[kWaves][2][NF][FS];     // [slot][field][group*TS + j]

    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int g = lane / LPR;
    const int s = lane % LPR;
    const bool lane_on = VEC || (s * RPL < p.ncols);
    const int c = p.col0 + (EXACT ? (lane_on ? s * RPL : 0) : min(s * RPL, p.ncols - RPL));
    const int64_t ld = VEC && EXACT ? (int64_t)RT : p.ld;
    const int over = EXACT ? 0 : p.col0 + s * RPL - c;   // leading columns that an earlier lane holds
    const uint64_t rb = (uint64_t)ld * sizeof(T);
    const uint64_t rb_own = (uint64_t)ld * sizeof(float);
    const float oscale = !GRAD ? 1.0f : p.dev_scale ? (float)((double)p.scale * *p.dev_scale) : p.scale;
    const char* lbase[NIN];
#pragma unroll
    for (int w = 0; w < NIN; ++w) lbase[w] = static_cast<const char*>(p.fac[w]) + (int64_t)c * sizeof(T);
    const char* obase = OWN ? reinterpret_cast<const char*>(p.own + c) : nullptr;
    const char* zrow = static_cast<const char*>(p.zero_row);
    float* const gsink = p.sink + s * RPL;
    double lsum = 0.0;  // LOSS: sum of squared residuals (each group's value in all its LPR lanes)
    // BUF: every factor is below 4 GiB, so rows are read with buffer loads
    // addressed by a 32-bit byte offset (row * row_bytes + column bytes)
    __amdgpu_buffer_rsrc_t rsrc[NIN];
    __amdgpu_buffer_rsrc_t rsrc_own;
    const uint32_t cb = (uint32_t)c * (uint32_t)sizeof(T);
    const uint32_t cb_own = (uint32_t)c * (uint32_t)sizeof(float);
    if constexpr (BUF) {
#pragma unroll
        for (int w = 0; w < NIN; ++w) rsrc[w] = make_rsrc(p.fac[w], p.fbytes[w]);
        if constexpr (OWN) rsrc_own = make_rsrc(p.own, p.own_bytes);
    }
    // Hot-row cache (vector path): the K rows of each input factor named by
    // the direct-mapped table p.hot[w] are copied to LDS once per block; ring
    // entries that name a cached row are rewritten to -2 - slot when parked.
    extern __shared__ __align__(16) char s_dyn[];
    constexpr int RB = RT * (int)sizeof(T);  // row bytes on the vector path
    const int K = HOT ? p.hot_k : 0;
    const int* const htag = reinterpret_cast<const int*>(s_dyn + hot_tag_offset());
    const uint32_t hrow = (uint32_t)hot_row_offset(NIN, K);  // byte offset of the cached rows
    if constexpr (HOT) {
        if (threadIdx.x < 4) reinterpret_cast<int*>(s_dyn)[threadIdx.x] = 0;
        {
            if (K > 0) {
                int* tag = reinterpret_cast<int*>(s_dyn + hot_tag_offset());
#pragma unroll
                for (int w = 0; w < NIN; ++w) {
                    for (int i = threadIdx.x; i < K; i += kMttkrpBlock) tag[w * K + i] = p.hot[w][i];
                    // 4 pieces per thread at a time, their loads in flight together
                    constexpr int PR = RB / 16;   // 16-byte pieces per row
                    for (int i0 = threadIdx.x; i0 < K * PR; i0 += 4 * kMttkrpBlock) {
                        int row[4];
                        u32x4 v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int i = i0 + u * kMttkrpBlock;
                            row[u] = i < K * PR ? p.hot[w][i / PR] : kHotEmpty;
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int piece = (i0 + u * kMttkrpBlock) % PR;
                            v[u] = u32x4{0u, 0u, 0u, 0u};
                            if (row[u] >= 0)
                                v[u] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(p.fac[w]) +
                                                                        (uint64_t)row[u] * RB + piece * 16);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int i = i0 + u * kMttkrpBlock;
                            if (i < K * PR)
                                *reinterpret_cast<u32x4*>(s_dyn + hrow + ((size_t)w * K + i / PR) * RB + (i % PR) * 16) = v[u];
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    // one factor-row gather: row >= 0 from memory, -1 (padding) zeros, <= -2
    // cache slot -2 - row from LDS (its memory read then returns zeros: past
    // the buffer's end, or the zero row on the 64-bit path).  Without EXACT the
    // ring holds byte offsets (row * row bytes, multiplied once when parked).
    const int pad = EXACT ? -1 : -(int)rb;
    auto gather = [&](int w, int ix) -> typename RowT::Raw {
        typename RowT::Raw r;
        if constexpr (!EXACT) r = RowT::load_buf(rsrc[w], (uint32_t)ix + cb);
        else if constexpr (BUF) r = RowT::load_buf(rsrc[w], (uint32_t)max(ix, -1) * (uint32_t)rb + cb);
        else r = RowT::load_ptr(ix < 0 ? zrow : lbase[w] + (uint64_t)(uint32_t)ix * rb);
        if constexpr (HOT) {
            constexpr uint32_t LB = RPL * sizeof(T);   // bytes per lane
            const uint32_t la = ix <= -2 ? hrow + (uint32_t)(w * K + (-2 - ix)) * RB + (uint32_t)s * LB : 0u;
            r = RowT::merge_lds(r, s_dyn + la);
        }
        return r;
    };
    auto gather_own = [&](int k) -> typename OwnRow::Raw {
        if constexpr (BUF) return OwnRow::load_buf(rsrc_own, (uint32_t)k * (uint32_t)rb_own + cb_own);
        else return OwnRow::load_ptr(k < 0 ? zrow : obase + (uint64_t)(uint32_t)k * rb_own);
    };
    const bool vec_meta = (p.chunk & 3) == 0;

#if AMPED_QUEUE_STATS
    unsigned long long st_chunks = 0, st_nnz = 0, st_first = 0;
#endif
    ChunkQueue cq;
    for (int chunk = cq.start(p, blockIdx.x, wv, kWaves); chunk >= 0; chunk = cq.next()) {
        cq.ask(lane);
        const int64_t cs = (int64_t)chunk * p.chunk;
        const int clen = (int)(min(cs + p.chunk, p.nnz) - cs);
#if AMPED_QUEUE_STATS
        if (st_chunks == 0) st_first = (unsigned long long)wall_clock64();
        ++st_chunks;
        st_nnz += (unsigned long long)clen;
#endif
        const int Lg = ((clen + FS - 1) / FS) * TS;            // run length per group, whole tiles
        const int goff = g * Lg;                                // group's first position in the chunk
        const int len = max(0, min(Lg, clen - goff));           // nonzeros in the group's run
        const bool gon = len > 0;
        const int ntiles = Lg / TS;
        const int nbatch = ntiles * NB;
        const int64_t gs = cs + goff;
        const int64_t ge = gs + len;
        // metadata of this chunk as buffers over [cs, cs + clen rounded up to
        // 4); reads past that return zeros, so no load needs a bounds branch
        const uint32_t mbytes = (uint32_t)((clen + 3) & ~3) * 4u;
        __amdgpu_buffer_rsrc_t mr[NF];
        mr[0] = make_rsrc(p.out_idx + cs, mbytes);
#pragma unroll
        for (int w = 0; w < NIN; ++w) mr[1 + w] = make_rsrc(p.in_idx[w] + cs, mbytes);
        mr[NF - 1] = make_rsrc(p.val + cs, mbytes);

        int open_key = -1, last_key = -1;
        int first_open = 1;  // the open row is the run's first
        int lsh = 0;         // the run's first row continues from the previous position
        float acc[RPL];
        float cur_own[RPL];  // own row of the entry consumed last (forms that read it)
        int own_key = -1;
#pragma unroll
        for (int i = 0; i < RPL; ++i) acc[i] = cur_own[i] = 0.f;
        // the output indices at and beside the ends of the group's run: loaded
        // here, looked at once the first tile's loads are on their way too (a
        // unit's start and end are chains of memory latencies: this and the
        // combine below take 1M nonzeros at rank 32 from 32 to 24 us per mode)
        int k_first = 0, k_prev = 0, k_last = 0, k_next = 0;
        if constexpr (OUT) {
            const int64_t top = p.nnz - 1;
            k_first = p.out_idx[min(gs, top)];
            k_prev = p.out_idx[max(min(gs, p.nnz) - 1, (int64_t)0)];
            k_last = p.out_idx[max(min(ge, p.nnz) - 1, (int64_t)0)];
            k_next = p.out_idx[min(ge, top)];
        }
        // the slots of the rows that the unit starts and ends in
        int h_left = kNoSlot, h_right = kNoSlot;
        if constexpr (OUT) {
            if (p.cut) {
                h_left = p.cut[(int64_t)chunk * p.per_chunk].y;
                h_right = p.cut[((int64_t)chunk + 1) * p.per_chunk].x;
            }
        }
        auto open_run = [&]() {
            if constexpr (OUT) {
                if (gon) {
                    last_key = k_last;
                    lsh = ((gs > 0 ? k_prev : p.prev_key) == k_first) ? 1 : 0;
                    open_key = k_first;
                }
                // slot 2g: the run's first row when it continues from the left
                // (bit 0: from the previous chunk); slot 2g+1: the run's last row
                if (s == 0) {
                    s_key[wv][2 * g] = lsh ? open_key : -1;
                    s_ext[wv][2 * g] = (g == 0) ? 1 : 0;
                    s_key[wv][2 * g + 1] = -1;
                }
            }
        };

        // ---- metadata: VGPR staging -> LDS ring.  Lane s of group g holds
        // nonzeros gs + t*TS + k*4*LPR + 4s .. +3 of each field, read with one
        // 16-byte load when chunk starts are 4-aligned.
        i32x4 vm[Q4][NF];
        auto load_meta = [&](int t) {
            if (t < ntiles) {
#pragma unroll
                for (int kq = 0; kq < Q4; ++kq) {
                    const uint32_t off = (uint32_t)(goff + t * TS + kq * 4 * LPR + 4 * s) * 4u;
                    if (vec_meta) {
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(mr[f], (int)off, 0, kMetaNT);
                            vm[kq][f] = i32x4{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                        }
                    } else {
#pragma unroll
                        for (int f = 0; f < NF; ++f)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                vm[kq][f][e] = (int)__builtin_amdgcn_raw_buffer_load_b32(mr[f], (int)(off + 4 * e), 0,
                                                                                         kMetaNT);
                    }
                }
            } else {
#pragma unroll
                for (int kq = 0; kq < Q4; ++kq)
#pragma unroll
                    for (int f = 0; f < NF; ++f) vm[kq][f] = i32x4{0, 0, 0, 0};
            }
        };
        // Items [L0, L1) of tile t's metadata (item l = 16-byte load kq = l / NF
        // of field l % NF), issued whatever t is: past the last tile the offset
        // is pushed out of the buffer (2^30 >= any chunk's metadata bytes), so
        // the loads return zeros and cost no memory traffic.
        auto load_meta_part = [&](int t, auto l0, auto l1) {
            constexpr int L0 = decltype(l0)::value, L1 = decltype(l1)::value;
            const uint32_t bias = t < ntiles ? 0u : (1u << 30);
            static_for<L1 - L0>([&](auto li) {
                constexpr int l = L0 + decltype(li)::value;
                constexpr int kq = l / NF, f = l % NF;
                const uint32_t off = (uint32_t)(goff + t * TS + kq * 4 * LPR + 4 * s) * 4u + bias;
                if (vec_meta) {
                    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(mr[f], (int)off, 0, kMetaNT);
                    vm[kq][f] = i32x4{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        vm[kq][f][e] = (int)__builtin_amdgcn_raw_buffer_load_b32(mr[f], (int)(off + 4 * e), 0, kMetaNT);
                }
            });
        };
        // tile t to ring slot t & 1, entries past the end of the run padded
        // here (a tile after its loads were issued, so they have landed)
        auto park_meta = [&](int t) {
#pragma unroll
            for (int kq = 0; kq < Q4; ++kq) {
                const int rel = t * TS + kq * 4 * LPR + 4 * s;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool past = rel + e >= len;
                    vm[kq][0][e] = past ? last_key : vm[kq][0][e];
#pragma unroll
                    for (int w = 0; w < NIN; ++w) {
                        int ix = vm[kq][1 + w][e];
                        if constexpr (!EXACT) ix = (int)((uint32_t)ix * (uint32_t)rb);
                        vm[kq][1 + w][e] = past ? pad : ix;
                    }
                    vm[kq][NF - 1][e] = past ? 0 : vm[kq][NF - 1][e];
                }
                if constexpr (HOT) {
                    if (K > 0) {
                        // rows held in the LDS cache become -2 - slot (tags
                        // are rows or -2, so padding -1 never matches)
#pragma unroll
                        for (int w = 0; w < NIN; ++w)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int ix = vm[kq][1 + w][e];
                                const int slot = ix & (K - 1);
                                vm[kq][1 + w][e] = (htag[w * K + slot] == ix) ? -2 - slot : ix;
                            }
                    }
                }
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    *reinterpret_cast<i32x4*>(&s_meta[wv][t & 1][f][g * TS + kq * 4 * LPR + 4 * s]) = vm[kq][f];
            }
            wave_lds_sync();
        };

        typename RowT::Raw rawA[U][NIN], rawB[U][NIN];
        typename OwnRow::Raw ownA[U], ownB[U];

        // issue the gathers of batch q
        auto issue = [&](int q, typename RowT::Raw (&raw)[U][NIN], typename OwnRow::Raw (&own)[U]) {
            const int t = q / NB;
            const int j0 = (q % NB) * U;
            const int* mrow = &s_meta[wv][t & 1][0][g * TS + j0];
            int ix[NIN][U];
#pragma unroll
            for (int w = 0; w < NIN; ++w) lds_vec<U>(mrow + (1 + w) * FS, ix[w]);
            int kk[U];
            int kprev = 0;   // key of the entry before the batch (same tile)
            if constexpr (OWN) {
                lds_vec<U>(mrow, kk);
                kprev = mrow[j0 > 0 ? -1 : 0];
            }
#pragma unroll
            for (int ju = 0; ju < U; ++ju) {
#pragma unroll
                for (int w = 0; w < NIN; ++w) raw[ju][w] = gather(w, ix[w][ju]);
                if constexpr (OWN) {
                    // the own row is read where the key changes (and at a
                    // tile's first entry); elsewhere consume reuses the row
                    // it holds.  Lanes that need none load at -1 (zeros), and
                    // when no group of the wave needs one the load instruction
                    // is skipped altogether (a wave-uniform branch, so the
                    // address unit does no work for it)
                    const bool same = j0 + ju > 0 && kk[ju] == (ju == 0 ? kprev : kk[ju > 0 ? ju - 1 : 0]);
                    const bool need = !(ix[0][ju] == pad || same);
                    if (__builtin_amdgcn_ballot_w64(need) != 0) own[ju] = gather_own(need ? kk[ju] : -1);
                    else own[ju] = typename OwnRow::Raw{};
                }
            }
        };

        // a finished row: stored, or parked in LDS when it is the run's first
        // row and continues from the left (the store then goes to a sink).
        // Unneeded parks go to slot 2g+1, which is only filled at the run's end.
        auto flush = [&]() {
            const bool pk = (first_open & lsh) != 0;
            float* lp = &s_acc[wv][2 * g + (pk ? 0 : 1)][s * RPL];
            lds_store<RPL>(lp, acc);
            float v[RPL];
#pragma unroll
            for (int i = 0; i < RPL; ++i) v[i] = acc[i] * oscale;
            float* gp = (pk || !lane_on) ? gsink : p.out + (int64_t)open_key * ld + c;
            store_vec<RPL>(gp, v);
        };

        // consume batch q from its buffers: Hadamard, scale, running row sum
        auto consume = [&](int q, typename RowT::Raw (&raw)[U][NIN], typename OwnRow::Raw (&own)[U]) {
            const int t = q / NB;
            const int j0 = (q % NB) * U;
            const int* mrow = &s_meta[wv][t & 1][0][g * TS + j0];
            int key[U], vbits[U];
            if constexpr (OUT || OWN) lds_vec<U>(mrow, key);
            lds_vec<U>(mrow + (NF - 1) * FS, vbits);
#pragma unroll
            for (int ju = 0; ju < U; ++ju) {
                const float val = __int_as_float(vbits[ju]);
                float prod[RPL];
                RowT::unpack(raw[ju][0], prod);
#pragma unroll
                for (int w = 1; w < NIN; ++w) {
                    float rw[RPL];
                    RowT::unpack(raw[ju][w], rw);
#pragma unroll
                    for (int i = 0; i < RPL; ++i) prod[i] *= rw[i];
                }
                float coef = val;
                if constexpr (OWN) {
                    // same rule as in issue: a fresh row where the key changes
                    // or the tile starts, else the row of the previous entry
                    const bool fresh = j0 + ju == 0 || key[ju] != own_key;
                    float ow[RPL];
                    OwnRow::unpack(own[ju], ow);
#pragma unroll
                    for (int i = 0; i < RPL; ++i) cur_own[i] = fresh ? ow[i] : cur_own[i];
                    own_key = key[ju];
                    float part = 0.f;
                    if constexpr (EXACT) {
#pragma unroll
                        for (int i = 0; i < RPL; ++i) part = fmaf(prod[i], cur_own[i], part);
                    } else {
                        // the columns' tree of the column-tile path: rounded
                        // products, neighbours added first
                        float term[RPL];
#pragma unroll
                        for (int i = 0; i < RPL; ++i) term[i] = i < over ? 0.f : mul_rounded(prod[i], cur_own[i]);
#pragma unroll
                        for (int m = 1; m < RPL; m <<= 1)
#pragma unroll
                            for (int i = 0; i < RPL; i += 2 * m) term[i] = add_rounded(term[i], term[i + m]);
                        part = term[0];
                    }
                    if constexpr (!VEC) part = lane_on ? part : 0.f;
                    coef = val - group_sum<LPR>(part);
                }
                if constexpr (LOSS) lsum = fma((double)coef, (double)coef, lsum);
                if constexpr (OUT) {
                    if (key[ju] != open_key) {
                        flush();
#pragma unroll
                        for (int i = 0; i < RPL; ++i) acc[i] = 0.f;
                        open_key = key[ju];
                        first_open = 0;
                    }
#pragma unroll
                    for (int i = 0; i < RPL; ++i) acc[i] = fmaf(coef, prod[i], acc[i]);
                }
            }
        };

        // With at most 8 batch pairs per tile, the tile is unrolled and the
        // loads of tile t+2's metadata are spread over its batch pairs at
        // fixed places, so every pass of the tile loop issues the same loads
        // and the compiler's load-counter waits are exact; otherwise tile
        // t+2 is loaded at once at the start of tile t.
        constexpr int IT = NB / 2;
        constexpr bool SPREAD = AMPED_META_SPREAD != 0 && IT <= 8;
        if (SPREAD && nbatch > 0) {
            constexpr int NL = Q4 * NF;
            load_meta(0);
            open_run();
            park_meta(0);
            load_meta(1);
            issue(0, rawA, ownA);
#pragma unroll 1
            for (int t = 0; t < ntiles; ++t) {
                park_meta(t + 1);
                static_for<IT>([&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    const int q = t * NB + 2 * K;
                    issue(q + 1, rawB, ownB);
                    load_meta_part(t + 2, std::integral_constant<int, K * NL / IT>{},
                                   std::integral_constant<int, (K + 1) * NL / IT>{});
                    consume(q, rawA, ownA);
                    issue(q + 2, rawA, ownA);   // past the last batch: padding only
                    consume(q + 1, rawB, ownB);
                });
            }
        } else if (nbatch > 0) {
            load_meta(0);
            open_run();
            park_meta(0);
            load_meta(1);
            issue(0, rawA, ownA);
#pragma unroll 1
            for (int q = 0; q < nbatch; q += 2) {
                // start of tile t: tile t+1 goes to the ring, tile t+2 is
                // loaded after the next batch's gathers (loads complete in
                // order, so consuming batch q then does not wait for it)
                const bool tile_start = (q % NB) == 0;
                if (tile_start) park_meta(q / NB + 1);
                issue(q + 1, rawB, ownB);
                if (tile_start) load_meta(q / NB + 2);
                consume(q, rawA, ownA);
                // unconditional, so the wait before the next consume counts
                // the same loads on every pass; past the last batch the ring
                // slot holds padding only (its gathers read nothing)
                issue(q + 2, rawA, ownA);
                consume(q + 1, rawB, ownB);
            }
        }

        if constexpr (!OUT) continue;

        // end of the run: the open row
        bool parked = false;
        if (gon) {
            const int nextk = ge < p.nnz ? k_next : p.next_key;
            const bool right_shared = (nextk == open_key);
            const bool left_open = first_open && lsh;  // the run is one row, continued from the left
            if (left_open && s == 0) s_key[wv][2 * g] = -1;
            if (left_open || right_shared) {
                float* dst = &s_acc[wv][2 * g + 1][s * RPL];
#pragma unroll
                for (int i = 0; i < RPL; ++i) dst[i] = acc[i];
                if (s == 0) {
                    s_key[wv][2 * g + 1] = open_key;
                    s_ext[wv][2 * g + 1] = ((left_open && g == 0) ? 1 : 0) | ((right_shared && ge == cs + clen) ? 2 : 0);
                }
            } else if (lane_on) {
                float v[RPL];
#pragma unroll
                for (int i = 0; i < RPL; ++i) v[i] = acc[i] * oscale;
                store_cols<RPL>(p.out, open_key, ld, c, v);
            }
            parked = lsh || right_shared;
        }

        if (__builtin_amdgcn_ballot_w64(parked) != 0) {
            wave_lds_sync();
            // the pieces in slot order, a lane per column (CL columns with more
            // than 64), so a row takes one store or atomic instruction; the
            // slots' keys sit in lane registers
            constexpr int CL = (RT + 63) / 64;
            constexpr bool FULL = RT >= 64;
            static_assert(EXACT || VEC, "");
            const int kq = lane < 2 * G ? s_key[wv][lane] : -1;
            const int eq = lane < 2 * G ? s_ext[wv][lane] : 0;
            // where column `lane + 64 i` sits in a slot (the last lanes' columns
            // overlap), and whether the launch has it
            bool col_on[CL];
            int at[CL];
#pragma unroll
            for (int i = 0; i < CL; ++i) {
                const int cc = lane + 64 * i;
                if constexpr (EXACT) {
                    col_on[i] = (FULL || cc < RT) && (VEC || cc < p.ncols);
                    at[i] = FULL || cc < RT ? cc : 0;
                } else {
                    const int full = (p.ncols / RPL) * RPL;   // columns that only their own lane holds
                    col_on[i] = cc < p.ncols;
                    at[i] = !col_on[i] ? 0 : cc < full ? cc : cc + full + RPL - p.ncols;
                }
            }
            int cur = -1, cur_ext = 0;
            float cacc[CL];
#pragma unroll
            for (int i = 0; i < CL; ++i) cacc[i] = 0.f;
            auto emit = [&]() {
                if (cur < 0) return;
                float* o = p.out + (int64_t)cur * ld + p.col0 + lane;
                bool add = cur_ext != 0;
                if (add) {
                    // a piece with a slot is stored there: the row's first one if it
                    // starts here, else that of the unit's first position
                    const int h = cur_ext & 1 ? h_left : h_right;
                    if (h != kNoSlot) {
                        const int slot = cur_ext & 1 ? h + chunk * p.per_chunk : h;
                        o = p.slot + (int64_t)slot * slot_stride(p.ncols) + lane;
                        add = false;
                    }
                }
#pragma unroll
                for (int i = 0; i < CL; ++i) {
                    if (!col_on[i]) continue;
                    const float v = cacc[i] * oscale;
                    if (add) atomicAdd(o + 64 * i, v);
                    else o[64 * i] = v;
                }
            };
            for (uint64_t left = __builtin_amdgcn_ballot_w64(kq >= 0); left != 0; left &= left - 1) {
                const int qq = __builtin_ctzll(left);
                const int k = __builtin_amdgcn_readlane(kq, qq), e = __builtin_amdgcn_readlane(eq, qq);
                const float* src = s_acc[wv][qq];
                if (k != cur) {
                    emit();
                    cur = k;
                    cur_ext = e;
#pragma unroll
                    for (int i = 0; i < CL; ++i) cacc[i] = src[at[i]];
                } else {
                    cur_ext |= e;
#pragma unroll
                    for (int i = 0; i < CL; ++i) cacc[i] += src[at[i]];
                }
            }
            emit();
        }
        wave_lds_sync();
    }
#if AMPED_QUEUE_STATS
    if (lane == 0 && p.qstats) {
        unsigned long long* r = p.qstats + ((size_t)blockIdx.x * kWaves + wv) * 4;
        r[0] = st_chunks;
        r[1] = st_nnz;
        r[2] = st_first;
        r[3] = (unsigned long long)wall_clock64();
    }
#endif
    if constexpr (LOSS) {
        // wave sum in fp64.  The first log2(LPR) steps add equal values (every
        // lane of a group holds the group's sum), so they are exact doublings
        // undone by the final 1/LPR.  One atomic per block: atomics on one
        // address take 12 ns each, one after the other.
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) lsum += __shfl_xor(lsum, m, 64);
        lsum *= 1.0 / LPR;
        __shared__ double s_loss[kWaves];
        if (lane == 0) s_loss[wv] = lsum;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int w = 0; w < kWaves; ++w) sum += s_loss[w];
            if (sum != 0.0) atomicAdd(p.loss, sum);
        }
    }
}

using KernelFn = void (*)(const KParams);

// Zeroes listed rows and (start, length) ranges of rows, nblocks blocks together (a
// range, at most about kGapPiece rows, is one block's work), of which this is `block`.  vec4:
// ld, col0 and ncols are multiples of 4 (16-byte stores).
__device__ __forceinline__ void zero_rows(float* out, int64_t ld, int col0, int ncols, bool vec4, const int32_t* zrows,
                                          int64_t n_zero, const int32_t* gaps, int64_t n_gaps, int64_t block,
                                          int64_t nblocks)
{
    const int64_t nthreads = nblocks * blockDim.x;
    const int nv = vec4 ? ncols / 4 : ncols;  // stores per row
    const int64_t total = n_zero * nv;
    for (int64_t i = block * blockDim.x + threadIdx.x; i < total; i += nthreads) {
        const int64_t r = zrows[i / nv];
        const int j = (int)(i % nv);
        if (vec4) *reinterpret_cast<float4*>(out + r * ld + col0 + 4 * j) = make_float4(0.f, 0.f, 0.f, 0.f);
        else out[r * ld + col0 + j] = 0.f;
    }
    for (int64_t gi = block; gi < n_gaps; gi += nblocks) {
        const int64_t start = gaps[2 * gi], len = gaps[2 * gi + 1];
        const int64_t n = len * nv;
        for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
            const int64_t r = start + i / nv;
            const int j = (int)(i % nv);
            if (vec4) *reinterpret_cast<float4*>(out + r * ld + col0 + 4 * j) = make_float4(0.f, 0.f, 0.f, 0.f);
            else out[r * ld + col0 + j] = 0.f;
        }
    }
}

// MTTKRP in one launch (small_kernel).
struct SmallParams {
    const int32_t* out_idx;
    const int32_t* in_idx[kMaxIn];
    const float* val;
    const void* fac[kMaxIn];
    uint32_t fbytes[kMaxIn];
    float* out;
    int64_t ld;
    int nnz, col0, ncols;
    int n_units;
    const int32_t* cut;      // [n_units + 1] positions
    const int32_t* left;     // [n_units + 1] the split row that cut k lies in, or -1
    const int32_t* split;    // per split row: its first unit, its number of units
    unsigned* arrived;       // per split row, 0 between launches
    uint64_t* share;         // [n_units + split rows][kSmallCols]: unit u's of split row h is u + h; 0 between launches
    bool vec4;
    const int32_t* zrows;
    const int32_t* gaps;
    int64_t n_zero, n_gaps;
};
using SmallFn = void (*)(const SmallParams);

// Vector instances exist for up to 4 input modes; every other case takes the
// column-tile path.
constexpr int kMaxVecNin = 4;

// Kernel pickers, one translation unit each (compiled in parallel).
KernelFn pick_mttkrp_f32(int nin, Lanes v, bool buf);
KernelFn pick_mttkrp_bf16(int nin, Lanes v, bool buf);
KernelFn pick_grad(int nin, Lanes v, bool buf);
KernelFn pick_loss(int nin, Lanes v, bool buf);
KernelFn pick_grad_loss(int nin, Lanes v, bool buf);
SmallFn pick_small(int nin, FactorType ft, Lanes v);

template <int NIN, int LPR, int RPL, typename T, int KIND>
KernelFn pick_buf(bool exact, bool buf)
{
    // 2 lanes and 64 lanes, and bfloat16 with 32, have no exact instance: their
    // ranks take the other one, which the residual forms have up to rank 64
    constexpr bool kExact = LPR >= 4 && LPR <= (sizeof(T) == 4 ? 32 : 16);
    constexpr bool kAny = KIND == 0 || LPR <= 16;
    if constexpr (kExact) {
        if (exact) return buf ? mttkrp_kernel<NIN, LPR, RPL, T, KIND, true, true>
                              : mttkrp_kernel<NIN, LPR, RPL, T, KIND, false, true>;
    }
    if constexpr (kAny) {
        if (buf) return mttkrp_kernel<NIN, LPR, RPL, T, KIND, true, false>;
    }
    return nullptr;
}

template <int NIN, typename T, int KIND>
KernelFn pick_vec(Lanes v, bool buf)
{
    if constexpr (NIN > kMaxVecNin) {
        return nullptr;
    } else {
        if (v.rpl == 4) {
            switch (v.lpr) {
            case 2: return pick_buf<NIN, 2, 4, T, KIND>(v.exact, buf);
            case 4: return pick_buf<NIN, 4, 4, T, KIND>(v.exact, buf);
            case 8:
                if constexpr (std::is_same<T, float>::value || NIN <= 2)
                    return pick_buf<NIN, 8, 4, T, KIND>(v.exact, buf);
                break;
            case 16:
                if constexpr (std::is_same<T, float>::value) return pick_buf<NIN, 16, 4, T, KIND>(v.exact, buf);
                break;
            case 32:
                if constexpr (std::is_same<T, float>::value) return pick_buf<NIN, 32, 4, T, KIND>(v.exact, buf);
                break;
            case 64:
                if constexpr (std::is_same<T, float>::value) return pick_buf<NIN, 64, 4, T, KIND>(v.exact, buf);
                break;
            default: break;
            }
        } else if constexpr (std::is_same<T, uint16_t>::value) {
            switch (v.lpr) {
            case 4:
                if constexpr (NIN > 2) return pick_buf<NIN, 4, 8, T, KIND>(v.exact, buf);
                break;
            case 8: return pick_buf<NIN, 8, 8, T, KIND>(v.exact, buf);
            case 16: return pick_buf<NIN, 16, 8, T, KIND>(v.exact, buf);
            case 32: return pick_buf<NIN, 32, 8, T, KIND>(v.exact, buf);
            default: break;
            }
        }
        return nullptr;
    }
}

template <int NIN, typename T, int KIND>
KernelFn pick_nin(Lanes v, bool buf)
{
    if (v.lpr == 0) return mttkrp_kernel<NIN, 64, 1, T, KIND, false, true>;
    return pick_vec<NIN, T, KIND>(v, buf);
}

template <typename T, int KIND>
KernelFn pick_any(int nin, Lanes v, bool buf)
{
    switch (nin) {
    case 1: return pick_nin<1, T, KIND>(v, buf);
    case 2: return pick_nin<2, T, KIND>(v, buf);
    case 3: return pick_nin<3, T, KIND>(v, buf);
    case 4: return pick_nin<4, T, KIND>(v, buf);
    case 5: return pick_nin<5, T, KIND>(v, buf);
    case 6: return pick_nin<6, T, KIND>(v, buf);
    case 7: return pick_nin<7, T, KIND>(v, buf);
    default: return nullptr;
    }
}

}  // namespace dev
}  // namespace amped
