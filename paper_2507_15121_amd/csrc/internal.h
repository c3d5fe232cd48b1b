// Internal interfaces shared by the C-ABI layer, the host layout builder and
// the HIP kernel launchers.  Not installed; not part of the ABI.
#pragma once

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>

namespace amped {

constexpr int kMaxOrder = 8;
constexpr int64_t kDefaultChunk = 4096;
// Largest chunk: a chunk's metadata arrays stay below 2^30 bytes, so 32-bit
// buffer offsets into them (with an out-of-range bias) never wrap.
constexpr int64_t kMaxChunk = int64_t(1) << 28;
// Nonzeros per work unit (what one wave takes from the queue) of a layout of nnz
// nonzeros, when the caller leaves the chunk size to the library.  A unit costs
// a wave about 3 us beside 6 us for each 256 nonzeros (rank 32).  Up to 5.2M
// nonzeros each of the 2048 waves of the grid gets one unit of whole tiles: fewer
// or more of them leave waves idle at the end.  Above that waves that meet fewer
// cache hits take longer, and small units off the queue even that out; from 32M
// on more of a heavy row's neighbours share a unit of 2048.  All modes at rank 32,
// units of 4096, one unit per wave, 1024 and 2048: 1M nonzeros 95, 63, 73 us and
// more; 2M 103 us (one per wave), 128 us (512); 5M 309, 233, 248 us; 10M 600, 446,
// 428, 450 us (order 4: 740, 703, 740 us with the last three); 20M 868 us (5120),
// 809, 830; rank 64 with bfloat16 factors 1002, 934, 955; 50M 2090, -, 2071, 2045;
// 200M 8694, -, 8756, 8626 (units of 2048).  From 64M on the unit is 4096 all the same:
// with one fp32 atomic per unit into a heavy row their rounding decided the result's error
// (40M nonzeros, units of 2048 and 4096: 4.0e-7 and 4.1e-7 of the outputs' norm; 100M
// 4.7e-7 and 4.4e-7; 200M 5.6e-7 and 4.9e-7; 8192, whose sums in registers are longer,
// 5.2e-7 to 5.6e-7).  Shorter units have not been measured since heavy rows have slots.
constexpr int64_t kGridWaves = 2048;
constexpr int64_t kTileNnz = 256;      // a unit is whole tiles of the kernel
constexpr int64_t kMaxRoundUnit = 2560;
inline int64_t work_unit(int64_t nnz)
{
    if (nnz > kGridWaves * kMaxRoundUnit)
        return nnz < (int64_t(32) << 20) ? 1024 : nnz < (int64_t(64) << 20) ? 2048 : 4096;
    const int64_t tiles = (nnz + kGridWaves * kTileNnz - 1) / (kGridWaves * kTileNnz);
    return kTileNnz * (tiles > 0 ? tiles : 1);
}
// Units that a wave of the residual and loss forms takes at a time: a unit costs
// them more (their own rows start anew).  All gradients at rank 32 with 1, 2 and
// this many units of 1024: 10M nonzeros 509, 502, 485 us (one chunk per wave), 20M
// 965, 950, 950 us.
inline int64_t residual_units(int64_t nnz, int64_t unit)
{
    if (nnz <= kGridWaves * kMaxRoundUnit || nnz >= (int64_t(32) << 20)) return 1;
    if (nnz <= kGridWaves * 5120) return (nnz + kGridWaves * unit - 1) / (kGridWaves * unit);
    return 2;
}
// The same for layouts that are streamed in shards of whole chunks of 4096: a
// power of two, so that shards end at unit ends too.
inline int64_t stream_work_unit(int64_t shard)
{
    int64_t u = kTileNnz;
    while (u < kDefaultChunk && u * kGridWaves < shard) u *= 2;
    return u;
}
// Heavy rows: those with kHeavyCuts or more edges of units that the library sizes
// inside.  One fp32 atomic per unit would make their error grow with the number of
// units (factors in (0, 1), a row of 199k nonzeros, rank 32: units of 512, 1024, 2048,
// 4096 2.9e-7, 2.5e-7, 1.4e-7, 1.1e-7 of the row), so in a mode that has such rows the
// pieces of rows with least_cuts or more edges inside go to slots, which close_kernel adds
// in fp64 (3.6e-8 at any unit).
//  With a wave for every unit that is every row that crosses an edge: the launch after the
// kernel then zeroes the untouched rows, too, and the one before it, which zeroes what
// atomics add to, is left out.  With more units than that the launch before is needed for
// the queue, and rows with few edges stay atomics.  All modes of 300k, 1M and 3M nonzeros
// with Zipf rows at rank 32: atomics only 37, 64 and 139 us; so 43, 72 and 150; with both
// launches 48, 74 and 152 (a closing launch takes 4 to 6 us, 1.5 more than one that has
// nothing to add).  10M, ALS sweep: 699 and 720 us; 20M rank 64 bfloat16: 945 and 981;
// 200M, units of 4096: 8437 and 8504, its error 5.3e-7 and 3.7e-7 of the outputs' norm
// (factors in (-1, 1)).
//  Streamed layouts have no slots: there a mode with a heavy row takes heavy_units units at
// a time, whole chunks or a little more.
constexpr int kHeavyCuts = 8;          // residual_units() is at most this
constexpr int kSlotCols = 256;         // columns of a launch at most
inline int64_t heavy_units(int64_t unit) { return (kDefaultChunk + unit - 1) / unit; }
constexpr int least_cuts(int64_t n_units) { return n_units <= kGridWaves ? 1 : kHeavyCuts; }
// Least nonzeros of a launch that keeps the most-used factor rows in LDS.  Every
// block copies them first, about 10 us, and the instances with the copy hold 70
// more registers; all modes at rank 32 without and with it: 5M nonzeros 235 and
// 258 us, 10M 456 and 469, 20M 875 and 893, 50M 2175 and 2118, 200M 9146 and 8650
// (order 4, 10M: 764 and 827; rank 64 with bfloat16 factors, 20M: 1027 and 1088).
#ifndef AMPED_HOT_MIN_NNZ
#define AMPED_HOT_MIN_NNZ (int64_t(32) << 20)
#endif
constexpr int64_t kHotMinNnz = AMPED_HOT_MIN_NNZ;

// Tensors whose MTTKRP is one launch of one wave per unit (small_kernel).  The
// unit's nominal length leaves at most 2048 units; a row of up to kSmallRow
// nonzeros lies in one unit, longer ones span units, and their shares' round trip
// takes 2 us or more: up to 2^17 nonzeros a mode takes the one launch unless a row
// spans more than kSmallSpan units, up to 2^18 only if no row spans any.  Kernels
// of a mode without and with the one launch: 2000 nonzeros at rank 16 9.3 and 6.0
// us, 100k 9.1 and 6.6 us (uniform), 20k with heavy rows 9.3 and 8.1 us (and 2.5
// us less in the call); 250k with every row split 10.2 and 9.0 us at rank 16, but
// 19 and 22 us at 128; 500k 15.5 and 15.5 us at rank 32, 10.6 and 14.6 us split.
#ifndef AMPED_SMALL_NNZ
#define AMPED_SMALL_NNZ (int64_t(1) << 18)
#endif
constexpr int64_t kSmallNnz = AMPED_SMALL_NNZ;
constexpr int64_t kSmallSplitNnz = int64_t(1) << 17;
constexpr int kSmallRow = 192;
constexpr int kSmallSpan = 64;
constexpr int kSmallCols = 256;        // columns of a launch
inline int small_unit(int64_t nnz) { return nnz <= (1 << 17) ? 64 : 128; }

// Hot-row tables: for every power of two K <= kHotMax, a direct-mapped table
// of K slots; slot s names the row r with r % K == s that the most nonzeros
// use in this mode (kHotEmpty if no row maps to s).  The tables of all K are
// stored back to back, the one for K at offset K - 1.
constexpr int kHotMax = 1024;
constexpr int kHotTableLen = 2 * kHotMax - 1;
constexpr int32_t kHotEmpty = -2;
// Scratch floats each tensor keeps for stores that must not land (64 lanes x 8).
constexpr int kSinkFloats = 512;
// The init kernel zeroes untouched output rows: runs at least this long as
// (start, length) ranges, shorter runs row by row from the zero-row list.
// A range is one workgroup's work, so longer runs are cut into ranges of
// about kGapPiece rows (each at least kLongGap): an untouched run of millions
// of rows (say, the unused tail of an index space) is then spread over the
// whole grid instead of one workgroup.
constexpr int kLongGap = 16;
constexpr int kGapPiece = 2048;
// Work-queue counters per layout: the chunks are split into at most this many
// contiguous stripes, each with its own counter (one stripe per XCD).
constexpr int kQueueSlots = 8;
// Words between two counters: a cache line each, so that atomics on different
// counters do not wait for each other.
constexpr int kQueueStride = 32;
constexpr int kQueueWords = kQueueSlots * kQueueStride;

// ----------------------------------------------------------------- host layout
struct HostModeLayout {
    std::vector<int32_t> perm;        // position -> input nonzero
    std::vector<uint8_t> flags;       // per chunk: bit0 head continues, bit1 tail continues
    std::vector<int32_t> zero_rows;   // rows shared by two or more work units, then untouched rows of short runs
    std::vector<int32_t> gaps;        // (start, length) pairs of long untouched-row runs
    std::vector<int32_t> hot;         // hot-row tables of this mode's rows [kHotTableLen]
    bool heavy = false;               // some row is a heavy row
    int64_t touched = 0;              // distinct output indices
};

// Position order of the input sorted lexicographically by (i_0, ..., i_{N-1}),
// stable; an empty vector means the input already is in that order.
std::vector<int32_t> lex_order(int order, const int64_t* dims, int64_t nnz, const int32_t* idx);

// Stable order by i_mode of `base` (identity when base is empty).
void mode_order(const int64_t* dims, int64_t nnz, const int32_t* idx, const std::vector<int32_t>& base,
                int mode, std::vector<int32_t>& perm);

// Chunk flags, zero-row list (of units of `unit` nonzeros; 0: of the chunks),
// long gaps, hot-row tables and touched count of a mode order.
void mode_tables(const int64_t* dims, int64_t nnz, const int32_t* idx, int mode, int64_t chunk,
                 HostModeLayout& lay, int64_t unit = 0);

// The same tables from the mode's sorted output-index column keys[nnz].
void mode_tables_sorted(const int32_t* keys, int64_t nnz, int64_t rows, int64_t chunk, HostModeLayout& lay,
                        int64_t unit = 0);

// True when the COO is already in lexicographic order of (i_0, ..., i_{N-1}).
bool is_lexicographic(int order, int64_t nnz, const int32_t* idx);
// The same of its first len entries only, one after the other.
bool is_lexicographic_prefix(int order, int64_t nnz, const int32_t* idx, int64_t len);

// Device layout build: a stable LSD radix sort of n (key, value) pairs by the
// low key_bits bits of the keys, in sort_passes(key_bits) passes (at least one must
// be needed).  The first pass reads (keys, vals) and writes
// (kbuf[first], vbuf[first]), the next ones alternate between the two buffer
// pairs; vals NULL: the positions.  keys or vals may be a buffer of the pair that
// is not written first.  scratch holds sort_scratch_words(n, key_bits) 32-bit words.
int64_t sort_scratch_words(int64_t n, int key_bits);
int sort_passes(int key_bits);
hipError_t launch_stable_sort(const uint32_t* keys, const int32_t* vals, uint32_t* const* kbuf, int32_t* const* vbuf,
                              int first, uint32_t* scratch, int64_t n, int key_bits, hipStream_t st);
// *bad = min(*bad, least position whose index is outside [0, dim)).
hipError_t launch_check_range(const int32_t* col, int64_t dim, int64_t n, unsigned long long* bad, hipStream_t st);
// *unsorted = 1 when the coordinates are not in lexicographic order.
hipError_t launch_check_sorted(int order, const int32_t* const* cols, int64_t n, unsigned* unsorted, hipStream_t st);
// A nonzero's record: order indices and the value, record_words(order) words of
// whole 16 bytes.  pack: columns (order index columns, then the values) to
// records; gather: record perm[p] to place p of the columns (NULL: not wanted).
inline int64_t record_words(int order) { return (order + 4) / 4 * 4; }
hipError_t launch_pack_records(int order, const void* const* cols, void* rec, int64_t n, hipStream_t st);
hipError_t launch_gather_records(int order, const void* rec, const int32_t* perm, void* const* cols, int64_t n,
                                 hipStream_t st);
// Row lists of a mode from its sorted keys, in two steps: the entries' totals
// (counts: 4 * row_list_blocks(n) words, 16-byte aligned, kept for the second
// step), then the lists themselves (zero: shared + lone rows; gaps: pairs).
struct RowTotals {
    int64_t shared, lone, gaps, touched;
};
int row_list_blocks(int64_t n);
hipError_t launch_count_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit, uint32_t* counts,
                             RowTotals* totals, hipStream_t st);
hipError_t launch_fill_rows(const int32_t* keys, int64_t n, int64_t rows, int64_t unit, const uint32_t* counts,
                            int64_t n_shared, int32_t* zero, int32_t* gaps, hipStream_t st);
// The units of small_kernel from sorted keys: cut and left [units + 1], split and
// arrived (zeroed) for at most `units` split rows; info[0] = split rows, info[1] =
// most units of one.
hipError_t launch_small_units(const int32_t* keys, int64_t n, int unit, int units, int32_t* cut, int32_t* left,
                              int32_t* split, unsigned* arrived, int32_t* info, hipStream_t st);
// The rows of a mode with n_units units that have slots, from sorted keys, those with fewer
// than kHeavyCuts unit edges inside (light, none when least_cuts is kHeavyCuts) and the
// others: (row, its first and last unit, the slot of its first unit's piece); unit k's
// piece has that slot plus k minus the first.  For k < n_units + kHeavyCuts cut[k] = (that
// slot, the same less the first unit) where unit k starts inside such a row, else kNoSlot
// twice.  counts = light rows, heavy rows.
constexpr int kNoSlot = -0x7FFFFFFF;
constexpr int64_t light_rows_max(int64_t n_units) { return least_cuts(n_units) == 1 ? n_units : 0; }
constexpr int64_t heavy_rows_max(int64_t n_units) { return n_units / kHeavyCuts + 1; }
constexpr int64_t slots_max(int64_t n_units) { return n_units + light_rows_max(n_units) + heavy_rows_max(n_units); }
hipError_t launch_slot_rows(const int32_t* keys, int64_t n, int64_t unit, int n_units, int4* light, int4* heavy, int2* cut,
                            int32_t* counts, hipStream_t st);
// The most device bytes that units sized by the library take beside the layouts: the
// tables and slots of rows that cross units, the tables and shares of the one-launch MTTKRP.
inline int64_t own_unit_bytes(int order, int64_t nnz, int64_t unit)
{
    const int64_t n = (nnz + unit - 1) / unit;
    int64_t mode = 8 * (n + kHeavyCuts) + 16 * (light_rows_max(n) + heavy_rows_max(n)) + slots_max(n) * kSlotCols * 4 + 4 * 256;
    if (nnz > 0 && nnz <= kSmallNnz) {
        const int64_t u = (nnz + small_unit(nnz) - 1) / small_unit(nnz), split = std::min(u, nnz / (kSmallRow + 1));
        mode += 8 * (u + 1) + 12 * u + (u + split) * kSmallCols * 8 + 5 * 256;
    }
    return order * mode;
}
// Hot-row tables (kHotTableLen entries) from sorted keys; best: kHotMax zeros.
hipError_t launch_hot_tables(const int32_t* keys, int64_t n, unsigned long long* best, int32_t* hot, hipStream_t st);
// a[i] = i for i < n.
hipError_t launch_iota(int32_t* a, int64_t n, hipStream_t st);

// Gather src[perm[p]] for p in [p0, p1) into dst (the host check's reference of a
// layout column; the packed layouts gather as they pack).
void gather_i32(const int32_t* src, const int32_t* perm, int64_t p0, int64_t p1, int32_t* dst);

// A mode's layout packed for the host link: blocks of kPackBlock nonzeros, each
//   8 words   the block's first output index, the bits b of the others above it
//   8 b       words: output indices minus the first, b bits each
//   8 bits[j] words: input indices j, bits[j] each (as its mode needs)
//   256       words: the values
// every column's entries one after the other, lowest bits first.  A block is never
// longer than its plain arrays.  offset[k] is where block k starts, in 8 words.
constexpr int kPackBlock = 256;
struct PackedMode {
    int nin = 0;
    int bits[kMaxOrder - 1] = {};
    int mode = 0, in_mode[kMaxOrder - 1] = {};
    std::vector<uint32_t> offset;          // [blocks + 1]
    uint32_t* data = nullptr;
    uint32_t* dev_offset = nullptr;        // offset on the device, or (dev_offset NULL)
    uint32_t* pinned_offset = nullptr;     // in pinned memory, copied with the blocks

    int64_t blocks() const { return offset.empty() ? 0 : (int64_t)offset.size() - 1; }
    int64_t bytes(int64_t block) const { return offset.empty() ? 0 : (int64_t)offset[block] * 32; }
    void plan(int order, const int64_t* dims, int64_t nnz, const int32_t* idx, int mode, const int32_t* perm);
    void fill(int64_t nnz, const int32_t* idx, const float* val, const int32_t* perm);
    int32_t out_index(int64_t p) const;
    int32_t in_index(int j, int64_t p) const;
    // out_idx [nnz], in_idx [nin][nnz], val [nnz], each nullable
    void unpack(int64_t nnz, int32_t* out_idx, int32_t* in_idx, float* val) const;
};

// -------------------------------------------------------------- device layout
// The blocks at `packed` (block k starts 8 (offset[k] - offset[0]) words in) to plain
// arrays: to[0] output indices, then the input indices, then the values.
struct UnpackArgs {
    int order = 0;
    int bits[kMaxOrder - 1] = {};
    const uint32_t* packed = nullptr;
    const uint32_t* offset = nullptr;
    int64_t blocks = 0;
    int32_t* to[kMaxOrder + 1] = {};
};
hipError_t launch_unpack(const UnpackArgs& u, hipStream_t st);

struct ModeDev {
    const int32_t* out_idx = nullptr;              // [nnz]
    const int32_t* in_idx[kMaxOrder - 1] = {};     // other modes ascending, each [nnz]
    const float* val = nullptr;                    // [nnz]
    const int32_t* zero_rows = nullptr;            // [n_zero]
    const int32_t* gaps = nullptr;                 // [2 * n_gaps]
    int64_t nnz = 0, rows = 0, n_zero = 0, n_gaps = 0;
    int64_t chunk = 0, n_chunks = 0;               // nonzeros per work unit, work units
    int64_t residual_chunk = 0;                    // the same for the residual and loss forms (whole units)
    unsigned* queue = nullptr;                     // kQueueSlots device work-queue counters, kQueueStride words apart
    const int32_t* hot = nullptr;                  // hot-row tables of this mode [kHotTableLen]
    const void* zero_row = nullptr;                // 16 zero bytes
    float* sink = nullptr;                         // kSinkFloats floats of write-only scratch
    // Rows whose pieces have slots (slot NULL: none do)
    struct Slots {
        int n_light = 0, n_heavy = 0;
        const int4* light = nullptr;
        const int4* heavy = nullptr;
        const int2* cut = nullptr;
        float* slot = nullptr;             // slots of at most kSlotCols floats
        bool all = false;                  // every row that crosses a unit edge has them
        const int32_t* zrows = nullptr;    // all: the untouched rows of the zero-row list
        int64_t n_zero = 0;
    } slots;
    int64_t unit = 0;                              // nonzeros per unit (chunk: per unit of a launch)
    // MTTKRP in one launch (n_units = 0: not for this mode)
    struct Small {
        int n_units = 0;
        const int32_t* cut = nullptr;      // [n_units + 1] positions
        const int32_t* left = nullptr;     // [n_units + 1] the split row that a cut lies in, or -1
        const int32_t* split = nullptr;    // pairs: a split row's first unit, its number of units
        unsigned* arrived = nullptr;       // per split row, 0 between launches
        uint64_t* share = nullptr;         // [n_units + split rows][kSmallCols], 0 between launches, when any row is split
        const int32_t* zrows = nullptr;    // the untouched rows of the zero-row list
        int64_t n_zero = 0;
    } small;
    // A shard of a longer layout (whole chunks of it): the output indices just
    // before and after the shard, -1 at the layout's ends.  Rows that cross a
    // shard edge cross a chunk edge, so they are in the zero-row list and every
    // shard adds into them.
    int prev_key = -1, next_key = -1;
};

enum class FactorType { F32 = 0, BF16 = 1 };
// ResidualGradLoss: the residual gradient that also sums the squared
// residuals into `loss` (the sparse CP loss) in the same pass.
enum class Kind { Mttkrp = 0, ResidualGrad = 1, ResidualGradLoss = 3 };

struct LaunchArgs {
    const ModeDev* m = nullptr;
    int nin = 0;                                   // number of input modes (order - 1)
    int rank = 0;
    FactorType ftype = FactorType::F32;
    Kind kind = Kind::Mttkrp;
    const void* in_factors[kMaxOrder - 1] = {};    // input-mode factors, modes ascending
    int64_t in_rows[kMaxOrder - 1] = {};           // their row counts
    const int32_t* in_hot[kMaxOrder - 1] = {};     // their hot-row tables
    const float* own_factor = nullptr;             // factor of the output mode (ResidualGrad)
    float scale = 1.0f;                            // ResidualGrad output scale
    const double* dev_scale = nullptr;             // a device-resident factor of it (nullable)
    float* out = nullptr;
    double* loss = nullptr;                        // ResidualGradLoss: fp64 loss
    bool loss_accumulate = false;                  // add to *loss instead of resetting it
    hipStream_t stream = nullptr;
};

// Enqueue init + MTTKRP (or fused residual gradient).  Returns hipSuccess or the
// launch error.
hipError_t launch_mttkrp(const LaunchArgs& a);

// x[i] *= (float)*s for i < n; nothing is read or written when *s is 1.
hipError_t launch_scale(float* x, int64_t n, const double* s, hipStream_t st);

// Enqueue the CP loss over the given layout (any mode's layout holds every
// nonzero once).  all_factors are in mode order with the layout's output mode
// first resolved by the caller: own_factor = factor of the layout's mode.
struct LossArgs {
    const ModeDev* m = nullptr;
    int order = 0;
    int rank = 0;
    const float* own_factor = nullptr;
    const float* in_factors[kMaxOrder - 1] = {};
    int64_t in_rows[kMaxOrder - 1] = {};
    double* loss = nullptr;
    bool accumulate = false;                       // add to *loss instead of resetting it
    hipStream_t stream = nullptr;
};
hipError_t launch_cp_loss(const LossArgs& a);

#if AMPED_QUEUE_STATS
// Diagnostic build: copy the per-wave work-queue records of the last
// MTTKRP-shaped launch (4 words each: chunks, nonzeros, first-pop time, exit
// time) after synchronising the device.
hipError_t queue_stats_copy(unsigned long long* host, int64_t max_records, int64_t* n_records, int* waves_per_block);
#endif

// CP-ALS building blocks (csrc/als.hip).  G = A^T A (fp64) of a rows x R fp32
// matrix, R <= 128, via gram_slabs(rows) x R x R fp32 partials.
int64_t gram_slabs(int64_t rows);
hipError_t launch_gram(const float* A, int64_t rows, int R, float* partial, double* G, hipStream_t st,
                       int64_t nslab = 0);
// The sweep's Gram matrices: G[m] = A[m]^T A[m] for n matrices in one launch, via
// (sum of als_gram_slabs(rows[m], R)) x R x R fp32 partials.
int64_t als_gram_slabs(int64_t rows, int R);
hipError_t launch_als_grams(const float* const* A, const int64_t* rows, int n, int R, float* partial, double* G,
                            hipStream_t st);
// launch_gram with the partial sums in the library's fixed device array (no
// allocation): at most gram_noalloc_slabs(rows, R) <= gram_slabs(rows) slabs,
// so that they fit its 32 MiB.
int64_t gram_noalloc_slabs(int64_t rows, int R);
hipError_t launch_gram_noalloc(const float* A, int64_t rows, int R, double* G, hipStream_t st);
// The mode-d update from M (rows x R): S = M^T M, the R x R algebra (scratch: R x R
// doubles) and A = M W, the sums in fp64 when it sets *wide (V ill-conditioned),
// else in fp32.  G is [N][R][R] and G[d] is replaced by the Gram matrix of the new
// factor; partial as for launch_als_grams.
hipError_t launch_als_update(const float* M, float* A, int64_t rows, float* partial, double* G, double* S, int N, int d,
                             int R, double* scratch, double* W, int* wide, double* lambda, bool last,
                             const double* xnorm2, double* fit, hipStream_t st);
// ||X||^2 over a layout whose exact duplicates are adjacent (accumulate: add
// to *result; no run of duplicates may cross the layout's ends then).
hipError_t launch_tensor_norm2(const ModeDev& m, int nin, double* result, bool accumulate, hipStream_t st);

// dst[p] = src[perm[p]] for p < n, 32-bit words, on the device.
hipError_t launch_permute32(void* dst, const void* src, const int32_t* perm, int64_t n, hipStream_t st);

}  // namespace amped
