// Device side of the per-mode layout builder (preprocessing, Sec. 5.7; not
// part of the timed MTTKRP): a stable least-significant-digit radix sort of
// (key, value) pairs, up to 10 bits per pass.
//
// One pass over n pairs, with tiles of kTile consecutive pairs per block, each
// wave owning a quarter of the tile:
//   1. histogram: each block counts the digits of its tile and writes its counts,
//      hist[block * digits + digit];
//   2. scan, down the columns of that array: groups of blocks, then the groups'
//      sums and the digits' starts;
//   3. scatter: each wave walks its quarter in order, 64 pairs per round.  A pair's
//      rank among equal digits of the quarter is the count from earlier rounds +
//      from earlier lanes (lanes with the same digit are found by matching the
//      digit's bits with ballots; the first of them adds their number to the wave's
//      counter), so equal digits keep their input order and every pass, hence the
//      whole sort, is stable.  The tile is put in digit order in LDS and leaves as
//      one run per digit.
// All accesses but the runs' ends are whole lines, and no pass has a step that a
// crowded digit makes serial.  With 8 bits per pass, counts digit-major, one LDS
// atomic per key in the histogram and rounds of 256 pairs written straight to
// their places, a pass over 5M pairs took 60 to 95 us (20 histogram, 12 scan, 25
// to 68 scatter); now 45 to 60 (6 to 10, 10, 25 to 40), and 17 to 20 bits need two
// passes instead of three.
//
// Beside the sort: the check of the coordinates (range, lexicographic order),
// the gather of a mode's arrays through its order (a nonzero as one record of
// 16 bytes or a multiple, so that a random place costs one line, not one per
// column: 15 gathers of 4-byte columns took 1.07 ms for 5M order-3 nonzeros),
// and the row lists and hot-row tables from a mode's sorted keys.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <vector>

#include "internal.h"

namespace amped {
namespace {

constexpr int kSortBlock = 256;
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kRounds = 16;
constexpr int64_t kTile = (int64_t)kSortBlock * kRounds;  // pairs per block
constexpr int kMaxDigitBits = 10;

// The lanes of `among` whose digit equals this lane's.
template <int B>
__device__ __forceinline__ uint64_t match_digit(uint32_t dg, uint64_t among)
{
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const bool bit = (dg >> b) & 1u;
        const uint64_t ones = __ballot(bit);
        among &= bit ? ones : ~ones;
    }
    return among;
}

// B: the most bits a digit may have; bits: those it has.  The lanes count in several
// copies, on different banks: one copy takes a wave's equal digits one at a time, and
// matching the digits with ballots first (as the scatter does) costs the same 10 us
// of a pass over 5M keys.
template <int B>
__global__ void __launch_bounds__(kSortBlock) radix_histogram(const uint32_t* keys, int64_t n, int shift, int bits,
                                                              uint32_t* hist)
{
    constexpr int kCopies = B <= 8 ? 16 : 8, LD = (1 << B) + 2;
    __shared__ uint32_t h[kCopies * LD];
    const int tid = threadIdx.x, nd = 1 << bits;
    for (int d = tid; d < kCopies * LD; d += kSortBlock) h[d] = 0;
    __syncthreads();
    uint32_t* const mine = h + (tid & (kCopies - 1)) * LD;
    const int64_t t0 = (int64_t)blockIdx.x * kTile + tid;
    uint32_t key[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) key[r] = t0 + r * kSortBlock < n ? keys[t0 + r * kSortBlock] : 0u;
#pragma unroll
    for (int r = 0; r < kRounds; ++r)
        if (t0 + r * kSortBlock < n) atomicAdd(&mine[(key[r] >> shift) & (nd - 1)], 1u);
    __syncthreads();
    for (int d = tid; d < nd; d += kSortBlock) {
        uint32_t x = 0;
#pragma unroll
        for (int c = 0; c < kCopies; ++c) x += h[c * LD + d];
        hist[(int64_t)blockIdx.x * nd + d] = x;
    }
}

// Exclusive sums, per digit, over a group's blocks, in place; the group's total
// goes to sums[group * digits + digit].
__global__ void __launch_bounds__(kSortBlock) scan_groups(uint32_t* hist, int64_t nblocks, int64_t group, int nd,
                                                          uint32_t* sums)
{
    const int d = blockIdx.y * kSortBlock + threadIdx.x;
    if (d >= nd) return;
    const int64_t b0 = (int64_t)blockIdx.x * group, b1 = min(b0 + group, nblocks);
    uint32_t run = 0;
    for (int64_t b = b0; b < b1; b += 8) {
        uint32_t x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = b + k < b1 ? hist[(b + k) * nd + d] : 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (b + k < b1) hist[(b + k) * nd + d] = run;
            run += x[k];
        }
    }
    sums[(int64_t)blockIdx.x * nd + d] = run;
}

// The same over the groups, by one block with a thread per digit; starts[digit] is
// where the digit's pairs start.
__global__ void __launch_bounds__(1 << kMaxDigitBits) scan_digits(uint32_t* sums, int64_t groups, int nd,
                                                                  uint32_t* starts)
{
    __shared__ uint32_t s_wave[(1 << kMaxDigitBits) / 64];
    const int d = threadIdx.x, lane = d & 63, wave = d >> 6;
    uint32_t run = 0;
    if (d < nd) {
        for (int64_t g = 0; g < groups; g += 8) {
            uint32_t x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = g + k < groups ? sums[(g + k) * nd + d] : 0u;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (g + k < groups) sums[(g + k) * nd + d] = run;
                run += x[k];
            }
        }
    }
    uint32_t incl = run;
    for (int m = 1; m < 64; m <<= 1) {
        const uint32_t y = __shfl_up(incl, m, 64);
        incl += lane >= m ? y : 0u;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += s_wave[w];
    if (d < nd) starts[d] = incl - run;
}

// vals_in NULL: the values are the positions.
template <int B>
__global__ void __launch_bounds__(kSortBlock) radix_scatter(const uint32_t* keys_in, const int32_t* vals_in,
                                                            uint32_t* keys_out, int32_t* vals_out, int64_t n,
                                                            int shift, int bits, const uint32_t* hist,
                                                            const uint32_t* sums, const uint32_t* starts,
                                                            int64_t group)
{
    constexpr int D = 1 << B, PER = (D + kSortBlock - 1) / kSortBlock;
    constexpr int kWords = kSortWaves * D > 2 * (int)kTile ? kSortWaves * D : 2 * (int)kTile;
    __shared__ uint32_t s_mem[kWords];     // digit counts per wave, then the tile in digit order
    __shared__ uint32_t s_delta[D];        // a digit's place in the output minus its place in the tile
    __shared__ uint32_t s_wave[kSortWaves];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, nd = 1 << bits;
    const int64_t first = (int64_t)blockIdx.x * kTile;
    const int count = (int)min((int64_t)kTile, n - first);
    const int p0 = wave * (64 * kRounds) + lane;
    uint32_t keys[kRounds], rank[kRounds];
    int32_t vals[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = p0 + r * 64;
        keys[r] = p < count ? keys_in[first + p] : 0u;
        vals[r] = p < count ? (vals_in ? vals_in[first + p] : (int32_t)(first + p)) : 0;
    }
    uint32_t out[PER];   // where the digits tid * PER ... of this tile start
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = tid * PER + k;
        out[k] = d < nd ? hist[(int64_t)blockIdx.x * nd + d] + sums[((int64_t)blockIdx.x / group) * nd + d] + starts[d]
                        : 0u;
    }
    for (int d = tid; d < kSortWaves * D; d += kSortBlock) s_mem[d] = 0;
    __syncthreads();
    uint32_t* const cnt = s_mem + wave * D;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool valid = p0 + r * 64 < count;
        const uint32_t dg = (keys[r] >> shift) & (nd - 1);
        const uint64_t same = match_digit<B>(dg, __ballot(valid));
        const uint64_t below = same & ((1ull << lane) - 1);
        uint32_t before = 0;
        if (valid && below == 0) before = atomicAdd(&cnt[dg], (uint32_t)__popcll(same));
        const int leader = valid ? __ffsll((unsigned long long)same) - 1 : lane;
        rank[r] = __shfl(before, leader, 64) + (uint32_t)__popcll(below);
    }
    __syncthreads();
    // places in the tile: digits in order, within a digit the waves in order
    uint32_t total = 0, tot[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = tid * PER + k;
        tot[k] = 0;
        if (d < D) {
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) tot[k] += s_mem[w * D + d];
        }
        total += tot[k];
    }
    uint32_t at = total;
    for (int m = 1; m < 64; m <<= 1) {
        const uint32_t y = __shfl_up(at, m, 64);
        at += lane >= m ? y : 0u;
    }
    if (lane == 63) s_wave[wave] = at;
    __syncthreads();
    for (int w = 0; w < wave; ++w) at += s_wave[w];
    at -= total;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = tid * PER + k;
        if (d < D) {
            s_delta[d] = out[k] - at;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const uint32_t x = s_mem[w * D + d];
                s_mem[w * D + d] = at;
                at += x;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) rank[r] += cnt[(keys[r] >> shift) & (nd - 1)];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        if (p0 + r * 64 >= count) continue;
        s_mem[rank[r]] = keys[r];
        s_mem[kTile + rank[r]] = (uint32_t)vals[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int p = r * kSortBlock + tid;
        if (p >= count) continue;
        const uint32_t key = s_mem[p];
        const uint32_t to = s_delta[(key >> shift) & (nd - 1)] + (uint32_t)p;
        keys_out[to] = key;
        vals_out[to] = (int32_t)s_mem[kTile + p];
    }
}

__global__ void __launch_bounds__(kSortBlock) iota_kernel(int32_t* a, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = (int32_t)i;
}

int grid_for(int64_t items, int64_t per_block)
{
    return (int)std::max<int64_t>(1, (items + per_block - 1) / per_block);
}

}  // namespace

// Blocks per group of the column scans: about as many groups as blocks in one.
static int64_t scan_group(int64_t nblocks)
{
    int64_t g = 1;
    while (g * g < nblocks) ++g;
    return g;
}

int64_t sort_scratch_words(int64_t n, int key_bits)
{
    const int64_t nblocks = (n + kTile - 1) / kTile, group = scan_group(nblocks);
    const int passes = sort_passes(key_bits);
    if (passes == 0) return 0;
    return (nblocks + (nblocks + group - 1) / group + 1) << ((key_bits + passes - 1) / passes);
}

hipError_t launch_iota(int32_t* a, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(iota_kernel, dim3(std::min(grid_for(n, kSortBlock), 8192)), dim3(kSortBlock), 0, st, a, n);
    return hipGetLastError();
}

int sort_passes(int key_bits) { return (key_bits + kMaxDigitBits - 1) / kMaxDigitBits; }

hipError_t launch_stable_sort(const uint32_t* keys, const int32_t* vals, uint32_t* const* kbuf, int32_t* const* vbuf,
                              int first, uint32_t* scratch, int64_t n, int key_bits, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t nblocks = (n + kTile - 1) / kTile, group = scan_group(nblocks);
    const int64_t groups = (nblocks + group - 1) / group;
    const int passes = sort_passes(key_bits);
    int to = first;
    for (int p = 0; p < passes; ++p) {
        // the key's bits in equal parts
        const int shift = key_bits * p / passes, bits = key_bits * (p + 1) / passes - shift, nd = 1 << bits;
        uint32_t* hist = scratch;
        uint32_t* sums = hist + nblocks * nd;
        uint32_t* starts = sums + groups * nd;
        auto pass = [&](auto histogram, auto scatter) {
            hipLaunchKernelGGL(histogram, dim3((unsigned)nblocks), dim3(kSortBlock), 0, st, keys, n, shift, bits, hist);
            hipLaunchKernelGGL(scan_groups, dim3((unsigned)groups, (nd + kSortBlock - 1) / kSortBlock),
                               dim3(kSortBlock), 0, st, hist, nblocks, group, nd, sums);
            hipLaunchKernelGGL(scan_digits, dim3(1), dim3(1 << kMaxDigitBits), 0, st, sums, groups, nd, starts);
            hipLaunchKernelGGL(scatter, dim3((unsigned)nblocks), dim3(kSortBlock), 0, st, keys, vals, kbuf[to],
                               vbuf[to], n, shift, bits, hist, sums, starts, group);
        };
        if (bits <= 8) pass(radix_histogram<8>, radix_scatter<8>);
        else pass(radix_histogram<kMaxDigitBits>, radix_scatter<kMaxDigitBits>);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        keys = kbuf[to];
        vals = vbuf[to];
        to ^= 1;
    }
    return hipSuccess;
}

// ------------------------------------------------------------ coordinate check
namespace {

struct Columns {
    const int32_t* col[kMaxOrder];
};

__global__ void __launch_bounds__(kSortBlock) check_range(const int32_t* col, int64_t dim, int64_t n,
                                                          unsigned long long* bad)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int32_t x = col[i];
        if (x < 0 || x >= dim) atomicMin(bad, (unsigned long long)i);
    }
}

__global__ void __launch_bounds__(kSortBlock) check_sorted(Columns c, int order, int64_t n, unsigned* unsorted)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x + 1; i < n; i += stride) {
        int cmp = 0;
        for (int w = 0; w < order && cmp == 0; ++w) {
            const int32_t a = c.col[w][i - 1], b = c.col[w][i];
            cmp = (a < b) ? -1 : (a > b) ? 1 : 0;
        }
        bad |= cmp > 0;
    }
    if (bad) *unsorted = 1u;
}

// ------------------------------------------------------------- record gathers
// A nonzero's record: its order indices, then its value, padded to V times 16 bytes.
template <int V>
struct alignas(16) Record {
    uint4 v[V];
};

struct Split {
    uint32_t* to[kMaxOrder + 1];   // where word j of the records goes (NULL: nowhere)
    const uint32_t* from[kMaxOrder + 1];
    int words;
};

template <int V>
__global__ void __launch_bounds__(kSortBlock) pack_records(Split s, Record<V>* rec, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint32_t w[4 * V];
#pragma unroll
        for (int j = 0; j < 4 * V; ++j) w[j] = j < s.words ? s.from[j][i] : 0u;
        Record<V> r;
#pragma unroll
        for (int q = 0; q < V; ++q) r.v[q] = make_uint4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
        rec[i] = r;
    }
}

// Record perm[p] to place p of the columns.
template <int V>
__global__ void __launch_bounds__(kSortBlock) gather_records(const Record<V>* rec, const int32_t* perm, Split s,
                                                             int64_t n)
{
    constexpr int U = 4;   // records in flight per thread
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n; i0 += U * stride) {
        int32_t at[U];
        Record<V> r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) at[u] = i0 + u * stride < n ? perm[i0 + u * stride] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = rec[at[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * stride;
            if (i >= n) continue;
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const uint32_t w[4] = {r[u].v[q].x, r[u].v[q].y, r[u].v[q].z, r[u].v[q].w};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * q + j < s.words && s.to[4 * q + j]) s.to[4 * q + j][i] = w[j];
            }
        }
    }
}

// ------------------------------------------------------------------ row lists
// What position p of the sorted keys adds to the lists: the gap of untouched
// rows before its row (the last position: also the one after it) and whether its
// row is shared by two work units and p is the first unit start inside it.
struct RowStep {
    int64_t gap0 = 0, gap1 = 0;    // untouched rows [start0, start0 + gap0), [start1, ...)
    int64_t start0 = 0, start1 = 0;
    int32_t shared = -1;           // the shared row
    bool first = false;            // p is the first of its row
};
__device__ __forceinline__ RowStep row_step(const int32_t* keys, int64_t p, int64_t n, int64_t rows, int64_t unit,
                                            int64_t cur, int64_t prev)   // keys[p], keys[p - 1] (p = 0: -1)
{
    RowStep s;
    s.first = cur != prev;
    if (s.first) {
        s.start0 = prev + 1;
        s.gap0 = max((int64_t)0, cur - prev - 1);
    } else if (p % unit == 0 && (p == unit || keys[p - unit - 1] != cur)) {
        s.shared = (int32_t)cur;
    }
    if (p == n - 1) {
        s.start1 = cur + 1;
        s.gap1 = max((int64_t)0, rows - cur - 1);
    }
    return s;
}
__device__ __forceinline__ uint32_t gap_pieces(int64_t gap)
{
    return gap >= kLongGap ? (uint32_t)((gap + kGapPiece - 1) / kGapPiece) : 0u;
}
__device__ __forceinline__ uint32_t lone_rows(int64_t gap) { return gap < kLongGap ? (uint32_t)gap : 0u; }

// Per block (a contiguous range of positions): entries of each list.
// counts[block]: shared rows, lone rows, gap pieces, touched rows.
__global__ void __launch_bounds__(kSortBlock) count_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit,
                                                         int64_t len, uint4* counts)
{
    __shared__ uint32_t s_sum[4][kSortWaves];
    const int64_t p1 = min((int64_t)(blockIdx.x + 1) * len, n);
    uint32_t c[4] = {0, 0, 0, 0};
    for (int64_t p = (int64_t)blockIdx.x * len + threadIdx.x; p < p1; p += kSortBlock) {
        const RowStep s = row_step(keys, p, n, rows, unit, keys[p], p > 0 ? keys[p - 1] : -1);
        c[0] += s.shared >= 0;
        c[1] += lone_rows(s.gap0) + lone_rows(s.gap1);
        c[2] += gap_pieces(s.gap0) + gap_pieces(s.gap1);
        c[3] += s.first;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        for (int m = 1; m < 64; m <<= 1) c[k] += __shfl_xor(c[k], m, 64);
        if ((threadIdx.x & 63) == 0) s_sum[k][threadIdx.x >> 6] = c[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t[4] = {0, 0, 0, 0};
        for (int k = 0; k < 4; ++k)
            for (int w = 0; w < kSortWaves; ++w) t[k] += s_sum[k][w];
        counts[blockIdx.x] = make_uint4(t[0], t[1], t[2], t[3]);
    }
}

// Exclusive sums of the blocks' counts in place, and their totals.
__global__ void __launch_bounds__(kSortBlock) scan_counts(uint4* counts, int nblocks, RowTotals* totals)
{
    __shared__ int64_t s[4][kSortBlock];
    const int per = (nblocks + kSortBlock - 1) / kSortBlock;
    const int b0 = min(nblocks, (int)threadIdx.x * per), b1 = min(nblocks, b0 + per);
    int64_t c[4] = {0, 0, 0, 0};
    for (int b = b0; b < b1; ++b) {
        const uint4 v = counts[b];
        c[0] += v.x; c[1] += v.y; c[2] += v.z; c[3] += v.w;
    }
    for (int k = 0; k < 4; ++k) s[k][threadIdx.x] = c[k];
    __syncthreads();
    int64_t e[4] = {0, 0, 0, 0};
    for (int k = 0; k < 4; ++k)
        for (int i = 0; i < (int)threadIdx.x; ++i) e[k] += s[k][i];
    if (threadIdx.x == kSortBlock - 1) {
        totals->shared = e[0] + c[0];
        totals->lone = e[1] + c[1];
        totals->gaps = e[2] + c[2];
        totals->touched = e[3] + c[3];
    }
    for (int b = b0; b < b1; ++b) {
        const uint4 v = counts[b];
        counts[b] = make_uint4((uint32_t)e[0], (uint32_t)e[1], (uint32_t)e[2], (uint32_t)e[3]);
        e[0] += v.x; e[1] += v.y; e[2] += v.z; e[3] += v.w;
    }
}

// The lists in position order: zero = shared rows, then lone rows (from
// n_shared on); gaps = (start, length) pairs of at most about kGapPiece rows,
// as push_gap of the host builder cuts them.
__global__ void __launch_bounds__(kSortBlock) fill_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit,
                                                        int64_t len, const uint4* offsets, int64_t n_shared,
                                                        int32_t* zero, int32_t* gaps)
{
    __shared__ uint32_t s_sum[3][kSortWaves];
    __shared__ uint32_t s_base[3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) {
        const uint4 o = offsets[blockIdx.x];
        s_base[0] = o.x;
        s_base[1] = o.y;
        s_base[2] = o.z;
    }
    __syncthreads();
    const int64_t pa = (int64_t)blockIdx.x * len, p1 = min(pa + len, n);
    // the next round's keys are loaded while a round is computed: 36 us for 5M keys
    // without, 24 with
    int32_t cur = 0, prev = -1;
    auto load = [&](int64_t p) {
        if (p >= p1) return;
        cur = keys[p];
        prev = p > 0 ? keys[p - 1] : -1;
    };
    load(pa + threadIdx.x);
    for (int64_t q = pa; q < p1; q += kSortBlock) {
        const int64_t p = q + threadIdx.x;
        RowStep s;
        const int32_t cur0 = cur, prev0 = prev;
        load(p + kSortBlock);
        if (p < p1) s = row_step(keys, p, n, rows, unit, cur0, prev0);
        uint32_t c[3] = {s.shared >= 0 ? 1u : 0u, lone_rows(s.gap0) + lone_rows(s.gap1),
                         gap_pieces(s.gap0) + gap_pieces(s.gap1)};
        uint32_t at[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            uint32_t x = c[k];   // inclusive sum over the wave
            if (__ballot(x != 0)) {
                for (int m = 1; m < 64; m <<= 1) {
                    const uint32_t y = __shfl_up(x, m, 64);
                    x += lane >= m ? y : 0u;
                }
            }
            at[k] = x - c[k];
            if (lane == 63) s_sum[k][wave] = x;
        }
        __syncthreads();
        uint32_t tot[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            at[k] += s_base[k];
            tot[k] = 0;
            for (int w = 0; w < kSortWaves; ++w) {
                at[k] += w < wave ? s_sum[k][w] : 0u;
                tot[k] += s_sum[k][w];
            }
        }
        if (s.shared >= 0) zero[at[0]] = s.shared;
        int64_t z = n_shared + at[1];
        for (uint32_t j = 0; j < lone_rows(s.gap0); ++j) zero[z++] = (int32_t)(s.start0 + j);
        for (uint32_t j = 0; j < lone_rows(s.gap1); ++j) zero[z++] = (int32_t)(s.start1 + j);
        // a wave writes its lanes' gaps together: one may have a million pieces
        for (int side = 0; side < 2; ++side) {
            const int64_t gap = side ? s.gap1 : s.gap0, start = side ? s.start1 : s.start0;
            const uint32_t np = gap_pieces(gap);
            const uint32_t g0 = at[2] + (side ? gap_pieces(s.gap0) : 0u);
            for (uint64_t left = __ballot(np > 0); left != 0; left &= left - 1) {
                const int l = __ffsll((unsigned long long)left) - 1;
                const int64_t ggap = __shfl(gap, l, 64), gstart = __shfl(start, l, 64);
                const uint32_t gn = __shfl(np, l, 64), gat = __shfl(g0, l, 64);
                for (uint32_t i = lane; i < gn; i += 64) {
                    const int64_t a = gstart + ggap * i / gn, b = gstart + ggap * (i + 1) / gn;
                    gaps[2 * ((int64_t)gat + i)] = (int32_t)a;
                    gaps[2 * ((int64_t)gat + i) + 1] = (int32_t)(b - a);
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            s_base[0] += tot[0];
            s_base[1] += tot[1];
            s_base[2] += tot[2];
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------- hot-row tables
// best[s] = max over rows r = s (mod kHotMax) of (uses << 32 | ~r): the row that
// the most nonzeros use, ties to the smaller row.  A row's uses are its run's
// length, found from the run's start by doubling steps and bisection.
__global__ void __launch_bounds__(kSortBlock) hot_runs(const int32_t* keys, int64_t n, unsigned long long* best)
{
    __shared__ unsigned long long s_best[kHotMax];
    for (int i = threadIdx.x; i < kHotMax; i += kSortBlock) s_best[i] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int32_t row = keys[p];
        if (p > 0 && keys[p - 1] == row) continue;
        int64_t lo = p, step = 1;   // keys[lo] == row
        while (lo + step < n && keys[lo + step] == row) {
            lo += step;
            step *= 2;
        }
        int64_t hi = min(lo + step, n);   // past the run
        while (hi - lo > 1) {
            const int64_t mid = lo + (hi - lo) / 2;
            if (keys[mid] == row) lo = mid;
            else hi = mid;
        }
        const unsigned long long e = (unsigned long long)(hi - p) << 32 | (uint32_t)~(uint32_t)row;
        const int s = row & (kHotMax - 1);
        if (e > s_best[s]) atomicMax(&s_best[s], e);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHotMax; i += kSortBlock)
        if (s_best[i] > best[i]) atomicMax(&best[i], s_best[i]);
}

// The tables of every K from the largest one's: slot s of K takes the better of
// slots s and s + K of 2K.
__global__ void __launch_bounds__(kHotMax) hot_tables(const unsigned long long* best, int32_t* hot)
{
    __shared__ unsigned long long s[kHotMax];
    const int i = threadIdx.x;
    s[i] = best[i];
    __syncthreads();
    for (int K = kHotMax;; K >>= 1) {
        if (i < K) hot[K - 1 + i] = s[i] ? (int32_t)~(uint32_t)s[i] : kHotEmpty;
        if (K == 1) break;
        if (i < K / 2) s[i] = max(s[i], s[i + K / 2]);
        __syncthreads();
    }
}

// ------------------------------------------------------------------ small units
// One block.  Cut k is the start of the row at position k * unit, or that position
// itself inside a row longer than kSmallRow (a split row).  Such a row's units
// are the one before its first cut to the one after its last.
__global__ void __launch_bounds__(1024) small_units(const int32_t* keys, int n, int unit, int units, int32_t* cut,
                                                    int32_t* left, int32_t* split, unsigned* arrived, int32_t* info)
{
    __shared__ int s_sum[1024];
    __shared__ int s_most;
    const int tid = threadIdx.x;
    if (tid == 0) s_most = 0;
    const int per = (units + 1 + 1023) / 1024;
    const int k0 = min(units + 1, tid * per), k1 = min(units + 1, k0 + per);
    // left[k] for now: the start of the split row that cut k lies in, or -1
    for (int k = k0; k < k1; ++k) {
        const int x = (int)min((int64_t)k * unit, (int64_t)n);
        int c = x, in = -1;
        if (x < n) {
            const int32_t row = keys[x];
            int lo = -1, hi = x;                     // first position of the row
            while (hi - lo > 1) {
                const int mid = lo + (hi - lo) / 2;
                if (keys[mid] < row) lo = mid;
                else hi = mid;
            }
            // longer than kSmallRow: its entry kSmallRow past the first is still the row
            if (hi + kSmallRow < n && keys[hi + kSmallRow] == row) in = x > hi ? hi : -1;
            else c = hi;
        }
        cut[k] = c;
        left[k] = in;
    }
    __syncthreads();
    // split rows in order: cut k is the first of its row
    auto first = [&](int k) { return left[k] >= 0 && left[k - 1] != left[k]; };   // left[0] = -1
    int c = 0;
    for (int k = max(k0, 1); k < k1; ++k) c += first(k);
    s_sum[tid] = c;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const int y = tid >= off ? s_sum[tid - off] : 0;
        __syncthreads();
        s_sum[tid] += y;
        __syncthreads();
    }
    int id = s_sum[tid] - c;
    // (the rows' starts stay in left[] until every thread has read them)
    for (int k = max(k0, 1); k < k1; ++k)
        if (first(k)) {
            int e = k + 1;
            while (e <= units && left[e] == left[k]) ++e;
            split[2 * id] = k - 1;
            split[2 * id + 1] = e - k + 1;
            arrived[id] = 0u;
            atomicMax(&s_most, e - k + 1);
            ++id;
        }
    __syncthreads();
    // left[k] = the row's id: those of earlier threads' rows come first
    id = s_sum[tid] - c - 1;
    int32_t own[8];   // per <= 5 (units <= 4096)
    for (int k = k0; k < k1; ++k) {
        if (k >= 1 && first(k)) ++id;
        own[k - k0] = left[k] >= 0 ? id : -1;
    }
    __syncthreads();
    for (int k = k0; k < k1; ++k) left[k] = own[k - k0];
    if (tid == 0) {
        info[0] = s_sum[1023];
        info[1] = s_most;
    }
}

// ------------------------------------------------------------- rows with slots
// One block.  The cuts inside a row are consecutive; its last one is found by doubling
// steps and bisection.  (Indices out of range may leave the keys unsorted; the call then
// fails, after this kernel, which stays inside its arrays whatever the keys are.)
__global__ void __launch_bounds__(1024) slot_rows(const int32_t* keys, int64_t n, int64_t unit, int units, int4* light,
                                                  int4* heavy, int2* cut, int32_t* counts)
{
    __shared__ int s_sum[3][1024];   // light rows, heavy rows, slots
    const int tid = threadIdx.x, least = least_cuts(units), most_heavy = (int)heavy_rows_max(units);
    for (int k = tid; k < units + kHeavyCuts; k += 1024) cut[k] = make_int2(kNoSlot, kNoSlot);
    const int per = (units + 1023) / 1024;
    const int k0 = min(units, tid * per), k1 = min(units, k0 + per);
    // whether cut k is the first one inside a row with slots
    auto first = [&](int k) {
        if (k < 1 || k + least - 1 >= units) return false;
        const int64_t p = (int64_t)k * unit;
        const int32_t row = keys[p];
        return keys[p - 1] == row && (k == 1 || keys[p - unit - 1] != row) && keys[p + (least - 1) * unit] == row;
    };
    auto last = [&](int k) {
        const int32_t row = keys[(int64_t)k * unit];
        int lo = k + least - 1, step = 1;
        while (lo + step < units && keys[(int64_t)(lo + step) * unit] == row) {
            lo += step;
            step *= 2;
        }
        int hi = min(lo + step, units);
        while (hi - lo > 1) {
            const int mid = lo + (hi - lo) / 2;
            if (keys[(int64_t)mid * unit] == row) lo = mid;
            else hi = mid;
        }
        return lo;
    };
    int c[3] = {0, 0, 0};
    for (int k = k0; k < k1; ++k)
        if (first(k)) {
            const int cuts = last(k) - k + 1;
            ++c[cuts < kHeavyCuts ? 0 : 1];
            c[2] += cuts + 1;
        }
#pragma unroll
    for (int i = 0; i < 3; ++i) s_sum[i][tid] = c[i];
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        int x[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) x[i] = tid >= off ? s_sum[i][tid - off] : 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 3; ++i) s_sum[i][tid] += x[i];
        __syncthreads();
    }
    int nl = s_sum[0][tid] - c[0], nh = s_sum[1][tid] - c[1], slot = s_sum[2][tid] - c[2];
    for (int k = k0; k < k1; ++k)
        if (first(k)) {
            const int e = last(k);
            const int4 v = make_int4(keys[(int64_t)k * unit], k - 1, e, slot);
            if (e - k + 1 < kHeavyCuts) {
                light[nl++] = v;
                for (int j = k; j <= e; ++j) cut[j] = make_int2(v.w, v.w - v.y);
            } else {
                if (nh < most_heavy) heavy[nh] = v;
                ++nh;
            }
            slot += e - k + 2;
        }
    __syncthreads();
    const int total = min(s_sum[1][1023], most_heavy);
    for (int r = tid >> 6; r < total; r += 16) {
        const int4 v = heavy[r];
        for (int k = v.y + 1 + (tid & 63); k <= v.z; k += 64) cut[k] = make_int2(v.w, v.w - v.y);
    }
    if (tid == 0) {
        counts[0] = s_sum[0][1023];
        counts[1] = total;
    }
}

int stream_grid(int64_t n, int per_thread)
{
    const int64_t per_block = (int64_t)kSortBlock * per_thread;
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + per_block - 1) / per_block, 8192));
}

template <int V>
hipError_t gather_v(const Split& s, bool pack, void* rec, const int32_t* perm, int64_t n, hipStream_t st)
{
    Record<V>* r = static_cast<Record<V>*>(rec);
    if (pack) hipLaunchKernelGGL(pack_records<V>, dim3(stream_grid(n, 1)), dim3(kSortBlock), 0, st, s, r, n);
    else
        hipLaunchKernelGGL(gather_records<V>, dim3(stream_grid(n, 4)), dim3(kSortBlock), 0, st, r, perm, s, n);
    return hipGetLastError();
}
hipError_t gather_any(const Split& s, bool pack, void* rec, const int32_t* perm, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    switch (record_words(s.words - 1) / 4) {
    case 1: return gather_v<1>(s, pack, rec, perm, n, st);
    case 2: return gather_v<2>(s, pack, rec, perm, n, st);
    default: return gather_v<3>(s, pack, rec, perm, n, st);
    }
}

}  // namespace

// ------------------------------------------------------------ packed layouts
namespace {

// A wave per block of 256 nonzeros; lane l unpacks its entries 4 l .. 4 l + 3 of
// every column, from a 64-bit window each (the word after a column's last one is
// the next column's or a value's), and stores them with one 16-byte store.
__global__ void __launch_bounds__(256) unpack_kernel(UnpackArgs u)
{
    const int lane = threadIdx.x & 63;
    const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (k >= u.blocks) return;
    const uint32_t* w = u.packed + (int64_t)(u.offset[k] - u.offset[0]) * 8;
    const uint32_t base = w[0], kb = w[1];
    w += 8;
    auto column = [&](uint32_t b, uint32_t add, int32_t* to) {
        int v[4];
        const uint32_t mask = b ? 0xFFFFFFFFu >> (32 - b) : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t bit = (4 * lane + j) * b;
            const uint64_t x = (uint64_t)w[(bit >> 5) + 1] << 32 | w[bit >> 5];
            v[j] = (int)(((uint32_t)(x >> (bit & 31)) & mask) + add);
        }
        *reinterpret_cast<int4*>(to + k * kPackBlock + 4 * lane) = make_int4(v[0], v[1], v[2], v[3]);
        w += 8 * b;
    };
    column(kb, base, u.to[0]);
    for (int j = 0; j < u.order - 1; ++j) column((uint32_t)u.bits[j], 0u, u.to[1 + j]);
    *reinterpret_cast<int4*>(u.to[u.order] + k * kPackBlock + 4 * lane) = *reinterpret_cast<const int4*>(w + 4 * lane);
}

}  // namespace

hipError_t launch_unpack(const UnpackArgs& u, hipStream_t st)
{
    if (u.blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)((u.blocks + 3) / 4)), dim3(256), 0, st, u);
    return hipGetLastError();
}

hipError_t launch_check_range(const int32_t* col, int64_t dim, int64_t n, unsigned long long* bad, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(check_range, dim3(stream_grid(n, 4)), dim3(kSortBlock), 0, st, col, dim, n, bad);
    return hipGetLastError();
}

hipError_t launch_check_sorted(int order, const int32_t* const* cols, int64_t n, unsigned* unsorted, hipStream_t st)
{
    if (n <= 1) return hipSuccess;
    Columns c{};
    for (int w = 0; w < order; ++w) c.col[w] = cols[w];
    hipLaunchKernelGGL(check_sorted, dim3(stream_grid(n, 4)), dim3(kSortBlock), 0, st, c, order, n, unsorted);
    return hipGetLastError();
}

hipError_t launch_pack_records(int order, const void* const* cols, void* rec, int64_t n, hipStream_t st)
{
    Split s{};
    s.words = order + 1;
    for (int j = 0; j <= order; ++j) s.from[j] = static_cast<const uint32_t*>(cols[j]);
    return gather_any(s, true, rec, nullptr, n, st);
}

hipError_t launch_gather_records(int order, const void* rec, const int32_t* perm, void* const* cols, int64_t n,
                                 hipStream_t st)
{
    Split s{};
    s.words = order + 1;
    for (int j = 0; j <= order; ++j) s.to[j] = static_cast<uint32_t*>(cols[j]);
    return gather_any(s, false, const_cast<void*>(rec), perm, n, st);
}

hipError_t launch_small_units(const int32_t* keys, int64_t n, int unit, int units, int32_t* cut, int32_t* left,
                              int32_t* split, unsigned* arrived, int32_t* info, hipStream_t st)
{
    if (n < 1 || n > kSmallNnz || units < 1 || units > 4096) return hipErrorInvalidValue;
    hipLaunchKernelGGL(small_units, dim3(1), dim3(1024), 0, st, keys, (int)n, unit, units, cut, left, split, arrived, info);
    return hipGetLastError();
}

hipError_t launch_slot_rows(const int32_t* keys, int64_t n, int64_t unit, int n_units, int4* light, int4* heavy, int2* cut,
                            int32_t* counts, hipStream_t st)
{
    if (n_units < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(slot_rows, dim3(1), dim3(1024), 0, st, keys, n, unit, n_units, light, heavy, cut, counts);
    return hipGetLastError();
}

int row_list_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 4095) / 4096, 2048)); }

hipError_t launch_count_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit, uint32_t* counts,
                             RowTotals* totals, hipStream_t st)
{
    const int nb = row_list_blocks(n);
    const int64_t len = (n + nb - 1) / nb;
    uint4* c = reinterpret_cast<uint4*>(counts);
    hipLaunchKernelGGL(count_rows, dim3(nb), dim3(kSortBlock), 0, st, keys, n, rows, unit, len, c);
    hipLaunchKernelGGL(scan_counts, dim3(1), dim3(kSortBlock), 0, st, c, nb, totals);
    return hipGetLastError();
}

hipError_t launch_fill_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit, const uint32_t* counts,
                            int64_t n_shared, int32_t* zero, int32_t* gaps, hipStream_t st)
{
    const int nb = row_list_blocks(n);
    const int64_t len = (n + nb - 1) / nb;
    hipLaunchKernelGGL(fill_rows, dim3(nb), dim3(kSortBlock), 0, st, keys, n, rows, unit, len,
                       reinterpret_cast<const uint4*>(counts), n_shared, zero, gaps);
    return hipGetLastError();
}

hipError_t launch_hot_tables(const int32_t* keys, int64_t n, unsigned long long* best, int32_t* hot, hipStream_t st)
{
    hipLaunchKernelGGL(hot_runs, dim3((unsigned)std::min<int64_t>((n + kSortBlock - 1) / kSortBlock, 1024)),
                       dim3(kSortBlock), 0, st, keys, n, best);
    hipLaunchKernelGGL(hot_tables, dim3(1), dim3(kHotMax), 0, st, best, hot);
    return hipGetLastError();
}

}  // namespace amped
