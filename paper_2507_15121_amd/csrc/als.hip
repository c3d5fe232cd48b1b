// gfx950 kernels for one CP-ALS sweep around the sparse MTTKRP (CPD by
// alternating least squares, Sec. 2.1; the mode loop of Alg. 1).  After the
// MTTKRP of mode d (M = X_(d) times the Khatri-Rao product of the others):
//
//   V   = Hadamard over w != d of G_w,  G_w = A_w^T A_w          (R x R)
//   A_d = M V^{-1}, then unit-norm columns with the norms in lambda
//
// Nothing per row is read twice more than needed: with S = M^T M,
// P = V^{-1} S V^{-1} is the Gram matrix of the unnormalised update, so
// lambda_r = sqrt(P_rr), the new G_d = D^{-1} P D^{-1} (D = diag(lambda)) and
// A_d = M W with W = V^{-1} D^{-1} come from R x R algebra; the big matrices
// pass through memory once each for S and once for A_d = M W.
//
// Kernels:
//  * gram_partial: A^T A of a rows x R fp32 matrix on the matrix cores.  Each
//    wave takes a slab of rows and one group of up to four 32 x 32 output tiles;
//    v_mfma_f32_32x32x2f32 consumes two rows per instruction, with lane l
//    supplying A[row0 + l/32][tile*32 + l%32] as both operands (the K index of
//    the product is the row).  Per-slab fp32 partials are summed in fp64 by
//    gram_reduce, in slab order (deterministic).
//  * als_small: one block, fp64 in registers: V, V^{-1} (Gauss-Jordan), P, lambda,
//    the new G_d, W and, after the last mode, the fit; in small modes also the
//    partials' sum and, in as many blocks as the rows need, A_d.
//  * als_solve: A_d = M W, a persistent grid over tiles of rows (256 at
//    R <= 32) staged through LDS beside W; the next tile's rows are loaded
//    into registers while the current one is computed.
//  * tensor_norm2: ||X||^2 over the mode-0 layout, exact duplicates (adjacent
//    there) summed before squaring.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace amped {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kGramMaxPairs = 4;   // 32x32 output tiles per wave (4 x 16 accumulators)

// f(j) for j = 0 .. N - 1 as compile-time constants
template <typename F, int... Is>
__device__ __forceinline__ void for_pairs_impl(F&& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void for_pairs(F&& f)
{
    for_pairs_impl(f, std::make_integer_sequence<int, N>{});
}

// Upper-triangle tile pair p of T x T tiles (G is symmetric): row-major over
// tm <= tn.
__host__ __device__ constexpr int tri_tm(int T, int p)
{
    int tm = 0;
    while (p >= T - tm) {
        p -= T - tm;
        ++tm;
    }
    return tm;
}
__host__ __device__ constexpr int tri_tn(int T, int p)
{
    int tm = 0;
    while (p >= T - tm) {
        p -= T - tm;
        ++tm;
    }
    return tm + p;
}

// The Gram matrices of one launch: matrix m's slabs are blocks [begin, next
// matrix's begin) of gram_partial, its partials are stored there too.
constexpr int kGramMany = kMaxOrder;
struct GramSet {
    const float* A[kGramMany];
    int64_t rows[kGramMany], slab_rows[kGramMany];
    int64_t begin[kGramMany + 1];
    double* G[kGramMany];
    int n;
};

// T = number of 32-column tiles (R <= 32 T).  Grid (slabs, tile groups);
// four waves per block each take a quarter of the slab's rows and keep up to
// kGramMaxPairs 32x32 tiles in MFMA accumulators, with kGramBatch row pairs of
// loads in flight before their MFMAs.  The four waves' tiles are then summed
// through LDS in wave order (deterministic) into the slab's partial.
constexpr int kGramBatch = 8;
template <int T, int GROUP>
__device__ __forceinline__ void gram_slab(const GramSet& set, int R, float* partial,
                                          float (&s_t)[4][T * (T + 1) / 2 < kGramMaxPairs ? T * (T + 1) / 2 : kGramMaxPairs][32 * 32])
{
    int mat = 0;
    while (mat + 1 < set.n && (int64_t)blockIdx.x >= set.begin[mat + 1]) ++mat;
    const float* const A = set.A[mat];
    const int64_t rows = set.rows[mat], slab_rows = set.slab_rows[mat];
    constexpr int NP = T * (T + 1) / 2;                               // upper-triangle tiles
    constexpr int P0 = GROUP * kGramMaxPairs;                         // this group's tiles: P0 .. P0 + NPB
    constexpr int NPB = NP - P0 < kGramMaxPairs ? NP - P0 : kGramMaxPairs;
    constexpr int T0 = tri_tm(T, P0);                                 // first column tile that they need
    constexpr int B = T <= 2 ? kGramBatch : kGramBatch / 2;          // row pairs per load batch
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t b0 = ((int64_t)blockIdx.x - set.begin[mat]) * slab_rows;
    const int64_t b1 = std::max(b0, std::min<int64_t>(b0 + slab_rows, rows));
    const int64_t q = ((slab_rows + 3) / 4 + 1) & ~(int64_t)1;   // even rows per wave, 4 q >= slab_rows
    const int64_t r0 = std::min<int64_t>(b0 + wave * q, b1);
    const int64_t r1 = std::min<int64_t>(r0 + q, b1);
    f32x16 acc[NPB];
#pragma unroll
    for (int j = 0; j < NPB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
    const int col = lane & 31;
    const int kk = lane >> 5;
    // batches of B row pairs, double-buffered: batch k+1 is loaded while
    // batch k feeds the MFMAs
    auto load = [&](float (&x)[B][T], int64_t i) {
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int64_t row = i + 2 * u + kk;
            const bool rv = row < r1;
#pragma unroll
            for (int t = T0; t < T; ++t) {
                const int c = t * 32 + col;
                x[u][t] = (rv && c < R) ? A[row * R + c] : 0.f;
            }
        }
    };
    auto fma_batch = [&](const float (&x)[B][T]) {
#pragma unroll
        for (int u = 0; u < B; ++u)
            for_pairs<NPB>([&](auto j) {
                constexpr int p = P0 + decltype(j)::value;
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[u][tri_tm(T, p)], x[u][tri_tn(T, p)], acc[j], 0, 0, 0);
            });
    };
    float xa[B][T], xb[B][T];
    if (r0 < r1) load(xa, r0);
    for (int64_t i = r0; i < r1; i += 4 * B) {
        load(xb, i + 2 * B);      // rows past r1 read as zeros
        fma_batch(xa);
        if (i + 4 * B < r1) load(xa, i + 4 * B);
        fma_batch(xb);
    }
    // lane l holds output column l%32; value v sits in row 8(v/4) + 4(l/32) + v%4
#pragma unroll
    for (int j = 0; j < NPB; ++j) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s_t[wave][j][(8 * (v >> 2) + 4 * kk + (v & 3)) * 32 + col] = acc[j][v];
    }
    __syncthreads();
    float* out = partial + (int64_t)blockIdx.x * R * R;
    for_pairs<NPB>([&](auto jj) {
        constexpr int j = decltype(jj)::value, p = P0 + j;
        for (int e = threadIdx.x; e < 1024; e += 256) {
            const int m = e >> 5, n = e & 31;
            const float sum = ((s_t[0][j][e] + s_t[1][j][e]) + s_t[2][j][e]) + s_t[3][j][e];
            const int r = tri_tm(T, p) * 32 + m, c = tri_tn(T, p) * 32 + n;
            if (r < R && c < R) {
                out[r * R + c] = sum;
                out[c * R + r] = sum;   // the mirrored tile (the same entry on the diagonal tiles)
            }
        }
    });
}

// The tile groups of a slab differ in blockIdx.y: each has code of its own, so
// that the tiles of a matrix instruction are fixed registers (chosen at run time,
// 50,000 rows of rank 100 took 1570 us in amped_gram's slabs, now 316 us).
template <int T>
__global__ void __launch_bounds__(256) gram_partial(GramSet set, int R, float* partial)
{
    constexpr int NP = T * (T + 1) / 2;
    __shared__ float s_t[4][NP < kGramMaxPairs ? NP : kGramMaxPairs][32 * 32];
    if (blockIdx.y == 0) gram_slab<T, 0>(set, R, partial, s_t);
    if constexpr (NP > kGramMaxPairs) {
        if (blockIdx.y == 1) gram_slab<T, 1>(set, R, partial, s_t);
    }
    if constexpr (NP > 2 * kGramMaxPairs) {
        if (blockIdx.y == 2) gram_slab<T, 2>(set, R, partial, s_t);
    }
}

// G[m][e] = sum over matrix m's slabs of partial[slab][e] in fp64.  A block takes
// 32 consecutive entries of one matrix; its 32 slab lanes add every 32nd slab,
// then the 32 sums are added in lane order (deterministic).
__global__ void __launch_bounds__(1024) gram_reduce(GramSet set, int R, const float* partial)
{
    __shared__ double s[32][33];
    const int e32 = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const int e = blockIdx.x * 32 + e32;
    const int RR = R * R;
    const int m = blockIdx.y;
    const int64_t nslab = set.begin[m + 1] - set.begin[m];
    const float* src = partial + set.begin[m] * RR;
    double acc = 0.0;
    if (e < RR) {
        // 8 loads in flight, added in slab order
        int64_t k = sl;
        for (; k + 224 < nslab; k += 256) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = src[(k + 32 * u) * RR + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += (double)v[u];
        }
        for (; k < nslab; k += 32) acc += (double)src[k * RR + e];
    }
    s[sl][e32] = acc;
    __syncthreads();
    if (sl == 0 && e < RR) {
        double t = 0.0;
        for (int j = 0; j < 32; ++j) t += s[j][e32];
        set.G[m][e] = t;
    }
}

// Largest 1-norm condition number of V for which the update's product M W
// keeps fp32 sums (als_solve).  The sum over k of M[i, k] W[k, r] cancels by
// up to about sqrt(kappa) when V is ill-conditioned (nearly collinear factor
// columns); fp32 sums then lose that many ulps, so above this bound the sums
// are taken in fp64.  At kappa = 1e4 the fp32 rounding of M W stays below the
// fp32 error of M itself (about 1e-6 relative).
constexpr double kSolveFp32MaxCond = 1e4;

// R x R fp64 algebra of one mode update, one block: V, V^{-1}, P = V^{-1} S
// V^{-1}, lambda, the new G[d], W and after the last mode the fit.
// G: [N][R][R] (G[d] is replaced); T: R x R doubles of scratch.
//
// Thread (ti, tj) of a TI x TI grid holds the entries (ti + TI a, tj + TI b),
// a, b < RA, of the RP x RP matrix (RP = TI RA >= R, padded by the identity) in
// registers, through the elimination and both products; LDS carries what other
// threads need.  What bounds it is the chain of R pivots, so a pivot is one LDS
// round trip and one barrier (row k, column k in two buffers), on as many threads
// as leave each one to four entries (16 above rank 96).  With the matrices in
// LDS, or above rank 64 in global memory, and three barriers per pivot it took 62
// us at rank 32 and about 5 ms at rank 100; now 19 us and 171 us (57 us at 64).
//
// Two launches of a small mode are left out.  With `nslab` partials given S is their
// sum (in slab order, as gram_reduce adds up to 32 slabs).  With M given, every block
// of the grid does the same algebra and then computes its own `per` rows of A = M W,
// with als_solve's sums in its order; block 0 alone writes the R x R results (no block
// reads G_d).  A sweep of 100k nonzeros at rank 16 takes 92.5 instead of 109.5 us.
struct SmallMode {
    const float* partial;    // [nslab][R][R], or NULL
    int nslab;
    const float* M;          // rows x R, or NULL
    float* A;
    int rows;
    int per;                 // rows per block: at most kSolvePerThread entries per thread
};
constexpr int kFoldSlabs = 8;
constexpr int kSolvePerThread = 4;
constexpr int kSolveBlocks = 256;   // at most: one per CU

template <int RA, int TI>
__global__ void __launch_bounds__(TI * TI) als_small(double* G, const double* S, int N, int d, int R, double* T,
                                                     double* W, int* wide, double* lambda, int last,
                                                     const double* xnorm2, double* fit, SmallMode mode)
{
    constexpr int RP = RA * TI, NT = TI * TI, LD = RP + 1;
    constexpr bool ST = RP <= 64;                           // S, then T, in LDS too
    extern __shared__ __align__(16) double s_inv[];        // V^{-1}, row stride LD; then (ST) S and T
    double* const s_st = s_inv + RP * LD;
    __shared__ double s_row[2][RP], s_col[2][RP];
    __shared__ double s_lam[RP], s_tr[RP], s_red[NT / 64];
    double(*const s_part)[RP] = reinterpret_cast<double(*)[RP]>(s_inv);   // TI x RP, until s_inv is filled
    const int tid = threadIdx.x, ti = tid / TI, tj = tid % TI;
    const int RR = R * R;
    float* const s_m = reinterpret_cast<float*>(s_st + RP * LD);   // this block's rows of M
    int rows_here = 0;
    if constexpr (ST) {
        if (mode.M) {
            const int r0 = (int)blockIdx.x * mode.per;
            rows_here = min(mode.per, mode.rows - r0);
            const float* src = mode.M + (int64_t)r0 * R;
#pragma unroll
            for (int k = 0; k < kSolvePerThread; ++k) {
                const int e = tid + k * NT;
                if (e < rows_here * R) s_m[e] = src[e];
            }
        }
        for (int e = tid; e < RR; e += NT) {
            double x = 0.0;
            if (mode.partial) {
                float v[kFoldSlabs];
#pragma unroll
                for (int k = 0; k < kFoldSlabs; ++k) v[k] = k < mode.nslab ? mode.partial[k * RR + e] : 0.f;
#pragma unroll
                for (int k = 0; k < kFoldSlabs; ++k) x += (double)v[k];
            } else {
                x = S[e];
            }
            s_st[e / R * LD + e % R] = x;
        }
    }
    auto row_of = [&](int x) { return ti + TI * x; };
    auto col_of = [&](int x) { return tj + TI * x; };

    // largest value over the block's threads
    auto block_max = [&](double x) {
        for (int m = 1; m < 64; m <<= 1) x = fmax(x, __shfl_xor(x, m, 64));
        if ((tid & 63) == 0) s_red[tid >> 6] = x;
        __syncthreads();
        x = s_red[0];
        for (int w = 1; w < NT / 64; ++w) x = fmax(x, s_red[w]);
        __syncthreads();
        return x;
    };
    // largest column sum of |x| over the R x R part
    auto norm1 = [&](const double (&x)[RA][RA]) {
#pragma unroll
        for (int j = 0; j < RA; ++j) {
            double sum = 0.0;
#pragma unroll
            for (int i = 0; i < RA; ++i) sum += row_of(i) < R ? fabs(x[i][j]) : 0.0;
            s_part[ti][col_of(j)] = sum;
        }
        __syncthreads();
        double most = 0.0;
        for (int c = tid; c < R; c += NT) {
            double sum = 0.0;
            for (int i = 0; i < TI; ++i) sum += s_part[i][c];
            most = sum > most || !(sum == sum) ? sum : most;   // a NaN stays
        }
        __syncthreads();
        const bool bad = __syncthreads_or(most == most ? 0 : 1) != 0;
        most = block_max(bad ? 0.0 : most);
        return bad ? __longlong_as_double(0x7ff8000000000000LL) : most;
    };

    double v[RA][RA], diag = 0.0;
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < RA; ++j) {
            const int r = row_of(i), c = col_of(j);
            double x = r == c ? 1.0 : 0.0;
            if (r < R && c < R) {
                x = 1.0;
                for (int w = 0; w < N; ++w)
                    if (w != d) x *= G[(int64_t)w * RR + r * R + c];
                if (r == c) diag = fmax(diag, fabs(x));
            }
            v[i][j] = x;
        }
    const double vmax = block_max(diag);
    const double vnorm = norm1(v);

    // V^{-1} in place by Gauss-Jordan elimination without pivoting (V is
    // symmetric positive semi-definite).  A pivot that is not positive (V
    // singular, e.g. a zero factor column) is replaced by a tiny one, so that row
    // and column of V^{-1} stay apart from the rest.
    const double tiny = (vmax > 0.0 ? vmax : 1.0) * 1e-30;
#pragma unroll
    for (int ka = 0; ka < RA; ++ka) {
        for (int kt = 0; kt < TI; ++kt) {
            const int k = ka * TI + kt;
            if (k >= R) break;
            double* row = s_row[k & 1];
            double* col = s_col[k & 1];
            if (ti == kt) {
#pragma unroll
                for (int j = 0; j < RA; ++j) row[col_of(j)] = v[ka][j];
            }
            if (tj == kt) {
#pragma unroll
                for (int i = 0; i < RA; ++i) col[row_of(i)] = v[i][ka];
            }
            __syncthreads();
            const double pv = row[k];
            const double inv = 1.0 / (pv > tiny ? pv : tiny);
            double rk[RA], ck[RA];
#pragma unroll
            for (int j = 0; j < RA; ++j) rk[j] = (j == ka && tj == kt ? 1.0 : row[col_of(j)]) * inv;
#pragma unroll
            for (int i = 0; i < RA; ++i) ck[i] = col[row_of(i)];
#pragma unroll
            for (int i = 0; i < RA; ++i)
#pragma unroll
                for (int j = 0; j < RA; ++j) {
                    const double base = j == ka && tj == kt ? 0.0 : v[i][j];
                    v[i][j] = i == ka && ti == kt ? rk[j] : base - ck[i] * rk[j];
                }
        }
    }
    // The 1-norm condition number kappa = ||V||_1 ||V^{-1}||_1 picks the
    // precision of the update's product M W (als_solve): fp32 sums while kappa
    // <= kSolveFp32MaxCond, fp64 sums above (or when kappa is not finite).
    const double kappa = vnorm * norm1(v);
    const bool is_wide = !(kappa <= kSolveFp32MaxCond);   // NaN: fp64
    const bool first = blockIdx.x == 0;
    if (first && tid == 0) *wide = is_wide ? 1 : 0;
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < RA; ++j) s_inv[row_of(i) * LD + col_of(j)] = v[i][j];
    __syncthreads();
    // T = S V^{-1} (S is symmetric: column r of it is read as row r), then
    // P = V^{-1} T (V^{-1} is symmetric)
    double p[RA][RA];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int j = 0; j < RA; ++j) p[i][j] = 0.0;
    };
    clear();
#pragma unroll 4
    for (int k = 0; k < R; ++k) {
        double x[RA], y[RA];
#pragma unroll
        for (int i = 0; i < RA; ++i) x[i] = ST ? s_st[k * LD + row_of(i)] : S[k * R + min(row_of(i), R - 1)];
#pragma unroll
        for (int j = 0; j < RA; ++j) y[j] = s_inv[k * LD + col_of(j)];
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int j = 0; j < RA; ++j) p[i][j] = fma(x[i], y[j], p[i][j]);
    }
    if constexpr (ST) __syncthreads();   // S read by all
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < RA; ++j) {
            const int r = row_of(i), c = col_of(j);
            if constexpr (ST) s_st[r * LD + c] = p[i][j];
            else if (r < R && c < R) T[r * R + c] = p[i][j];
            if (r == c) s_tr[r] = p[i][j];
        }
    __syncthreads();
    clear();
#pragma unroll 4
    for (int k = 0; k < R; ++k) {
        double x[RA], y[RA];
#pragma unroll
        for (int i = 0; i < RA; ++i) x[i] = s_inv[k * LD + row_of(i)];
#pragma unroll
        for (int j = 0; j < RA; ++j) y[j] = ST ? s_st[k * LD + col_of(j)] : T[k * R + min(col_of(j), R - 1)];
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
            for (int j = 0; j < RA; ++j) p[i][j] = fma(x[i], y[j], p[i][j]);
    }
    // lambda = sqrt(diag P)
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < RA; ++j)
            if (row_of(i) == col_of(j)) s_lam[row_of(i)] = p[i][j] > 0.0 ? sqrt(p[i][j]) : 0.0;
    __syncthreads();
    if (first)
        for (int r = tid; r < R; r += NT) lambda[r] = s_lam[r];
    double xh = 0.0;
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < RA; ++j) {
            const int r = row_of(i), c = col_of(j);
            if (r >= R || c >= R) continue;
            const double lr = s_lam[r], lc = s_lam[c];
            const double g = (lr > 0.0 && lc > 0.0) ? p[i][j] / (lr * lc) : 0.0;
            const double x = lc > 0.0 ? v[i][j] / lc : 0.0;
            if constexpr (ST) s_inv[r * LD + c] = x;   // V^{-1} is no longer read
            if (!first) continue;
            G[(int64_t)d * RR + r * R + c] = g;
            W[r * R + c] = x;
            if (last) {
                double h = g;
                for (int w = 0; w < N; ++w)
                    if (w != d) h *= G[(int64_t)w * RR + r * R + c];
                xh += lr * lc * h;
            }
        }
    if (last && first) {
        // <X, Xhat> = sum_r lambda_r (S W)_rr = trace(S V^{-1}) over columns
        // with lambda_r > 0; ||Xhat||^2 = lambda^T (Hadamard of all G) lambda,
        // its per-thread sums added in a fixed order.
        for (int m = 1; m < 64; m <<= 1) xh += __shfl_xor(xh, m, 64);
        if ((tid & 63) == 0) s_red[tid >> 6] = xh;
        __syncthreads();
        if (tid == 0) {
            double model = 0.0, inner = 0.0;
            for (int w = 0; w < NT / 64; ++w) model += s_red[w];
            for (int r = 0; r < R; ++r)
                if (s_lam[r] > 0.0) inner += s_tr[r];
            const double x2 = *xnorm2;
            const double res = x2 - 2.0 * inner + model;
            *fit = x2 > 0.0 ? 1.0 - sqrt(res > 0.0 ? res : 0.0) / sqrt(x2) : 0.0;
        }
    }
    if constexpr (ST) {
        if (mode.M) {
            __syncthreads();
            float* dst = mode.A + (int64_t)blockIdx.x * mode.per * R;
            for (int e = tid; e < rows_here * R; e += NT) {
                const int c = e % R;
                const float* m = s_m + (e - c);
                if (is_wide) {
                    double x = 0.0;
#pragma unroll 4
                    for (int k = 0; k < R; ++k) x = fma((double)m[k], s_inv[k * LD + c], x);
                    dst[e] = (float)x;
                } else {
                    float x = 0.f;
#pragma unroll 8
                    for (int k = 0; k < R; ++k) x = fmaf(m[k], (float)s_inv[k * LD + c], x);
                    dst[e] = x;
                }
            }
        }
    }
}

// A = M W for a rows x R fp32 matrix M and an R x R fp64 matrix W.  W =
// V^{-1} D^{-1} has large entries of opposite sign when V is ill-conditioned
// (nearly collinear factor columns), and the sum over k then cancels: when
// als_small flagged V (*wide != 0) the products and sums are fp64 and A is
// rounded to fp32 once, otherwise W is rounded to fp32 and the sums are fp32.
// A block of 256 threads stages RB rows of M (row stride R + 1 in LDS, so the
// rows a wave reads fall in different banks) and W; thread (g, c8) computes
// RPT rows and 8 columns from registers.
template <int RPT, typename Acc>
__device__ __forceinline__ void solve_tile(const Acc* sW, int RW, const float* sM, int R, int i0, int nr, int c8,
                                           float* A, int64_t r0)
{
    Acc acc[RPT][8];
#pragma unroll
    for (int j = 0; j < RPT; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[j][c] = Acc(0);
    for (int k = 0; k < R; ++k) {
        Acc w[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) w[c] = sW[k * RW + 8 * c8 + c];
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const Acc m = (i0 + j < nr) ? (Acc)sM[(i0 + j) * (R + 1) + k] : Acc(0);
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[j][c] = fma(m, w[c], acc[j][c]);
        }
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        if (i0 + j >= nr) continue;
        float* out = A + (r0 + i0 + j) * R + 8 * c8;
        if ((R & 7) == 0) {   // 32-byte aligned run of 8 columns
            *reinterpret_cast<float4*>(out) = make_float4((float)acc[j][0], (float)acc[j][1], (float)acc[j][2],
                                                          (float)acc[j][3]);
            *reinterpret_cast<float4*>(out + 4) = make_float4((float)acc[j][4], (float)acc[j][5], (float)acc[j][6],
                                                              (float)acc[j][7]);
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (8 * c8 + c < R) out[c] = (float)acc[j][c];
        }
    }
}

// Persistent: block b takes tiles b, b + grid, ... of RB rows.  W goes to LDS
// once per block.  With R % 4 == 0 each thread holds its part of the next
// tile's rows of M (up to 8 float4) in registers, loaded before the current
// tile is computed, so the loads overlap the arithmetic and the stores.
template <int RPT>
__global__ void __launch_bounds__(256) als_solve(const float* M, const double* W, const int* wide_flag, float* A,
                                                 int64_t rows, int R, int RB, int64_t ntiles)
{
    extern __shared__ __align__(16) double s_solve[];
    const int C8 = (R + 7) / 8;                 // column groups of 8
    const int RW = 8 * C8;                      // padded row length of W
    const bool wide = *wide_flag != 0;          // the same for every thread
    double* sW = s_solve;                       // [R][RW] fp64, or fp32 in the first half
    float* sWf = reinterpret_cast<float*>(s_solve);
    float* sM = reinterpret_cast<float*>(s_solve + R * RW);   // [RB][R + 1]
    const int tid = threadIdx.x;
    for (int e = tid; e < R * RW; e += 256) {
        const int k = e / RW, c = e % RW;
        const double w = c < R ? W[k * R + c] : 0.0;
        if (wide) sW[e] = w;
        else sWf[e] = (float)w;
    }
    const bool vec = (R & 3) == 0;
    const float4* M4 = reinterpret_cast<const float4*>(M);
    float4 v[8];   // RB * R / 4 <= 8 * 256 (launch_als_solve)
    auto fetch = [&](int64_t t) {
        const int64_t r0 = t * RB;
        const int n4 = t < ntiles ? (int)(std::min<int64_t>(RB, rows - r0) * R / 4) : 0;
        const float4* src = M4 + (t < ntiles ? r0 * (R / 4) : 0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = u * 256 + tid;
            v[u] = e < n4 ? src[e] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    if (vec) fetch(blockIdx.x);
    const int g = tid / C8, c8 = tid % C8;
    const int i0 = RPT * g;
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        const int64_t r0 = t * RB;
        const int nr = (int)std::min<int64_t>(RB, rows - r0);
        __syncthreads();   // W staged; the previous tile's reads of sM done
        if (vec) {
            const int n4 = nr * R / 4;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = u * 256 + tid;
                if (e < n4) {
                    const int i = (4 * e) / R, k = (4 * e) % R;
                    float* d = &sM[i * (R + 1) + k];
                    d[0] = v[u].x; d[1] = v[u].y; d[2] = v[u].z; d[3] = v[u].w;
                }
            }
        } else {
            for (int e = tid; e < nr * R; e += 256) sM[(e / R) * (R + 1) + e % R] = M[r0 * R + e];
        }
        __syncthreads();
        if (vec) fetch(t + gridDim.x);
        if (i0 < nr) {
            if (wide) solve_tile<RPT, double>(sW, RW, sM, R, i0, nr, c8, A, r0);
            else solve_tile<RPT, float>(sWf, RW, sM, R, i0, nr, c8, A, r0);
        }
    }
}

// ||X||^2 over a layout whose exact duplicates are adjacent (mode 0's).
struct InIdx {
    const int32_t* p[kMaxOrder - 1];
};

__global__ void __launch_bounds__(256) tensor_norm2(const int32_t* out_idx, InIdx in_idx, int nin,
                                                    const float* val, int64_t nnz, double* result)
{
    __shared__ double part[4];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    double s = 0.0;
    auto same = [&](int64_t a, int64_t b) {
        if (out_idx[a] != out_idx[b]) return false;
        for (int w = 0; w < nin; ++w)
            if (in_idx.p[w][a] != in_idx.p[w][b]) return false;
        return true;
    };
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += stride) {
        if (p > 0 && same(p - 1, p)) continue;
        double v = val[p];
        for (int64_t q = p + 1; q < nnz && same(p, q); ++q) v += val[q];
        s += v * v;
    }
    for (int m = 1; m < 64; m <<= 1) s += __shfl_xor(s, m, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(result, part[0] + part[1] + part[2] + part[3]);
}

}  // namespace

int64_t gram_slabs(int64_t rows)
{
    // about 8192 rows per slab; above 256 slabs a multiple of 256, so every
    // CU of the 256 gets the same number of slabs
    int64_t n = (rows + 8191) / 8192;
    if (n > 256) n = (n + 255) / 256 * 256;
    return std::max<int64_t>(1, std::min<int64_t>(n, 2048));
}

int64_t als_gram_slabs(int64_t rows, int R)
{
    // The sweep's Gram matrices need not have amped_gram's bits, and slabs of 8192
    // rows leave most CUs idle: 80 us for 100k rows of rank 32 on 13 blocks, 86 us
    // for 500k on 62 (8 and 19 us here).  So from 256 rows on (64 per wave), up to a few blocks per
    // CU; wide ranks have several tile groups per slab and larger partials.
    int64_t n = std::min<int64_t>((rows + 255) / 256, R <= 64 ? 1024 : 512);
    if (n > 256) n = (n + 255) / 256 * 256;
    return std::max<int64_t>(gram_slabs(rows), n);
}

static hipError_t launch_gram_set(GramSet& set, const int64_t* nslab, int R, float* partial, hipStream_t st,
                                  bool reduce = true)
{
    if (R < 1 || R > 128 || set.n < 1 || set.n > kGramMany) return hipErrorInvalidValue;
    set.begin[0] = 0;
    for (int m = 0; m < set.n; ++m) {
        set.begin[m + 1] = set.begin[m] + nslab[m];
        set.slab_rows[m] = (set.rows[m] + nslab[m] - 1) / nslab[m];
        set.slab_rows[m] += set.slab_rows[m] & 1;
    }
    const int T = (R + 31) / 32;
    const int groups = (T * (T + 1) / 2 + kGramMaxPairs - 1) / kGramMaxPairs;
    dim3 grid((unsigned)set.begin[set.n], (unsigned)groups);
    switch (T) {
    case 1: hipLaunchKernelGGL(gram_partial<1>, grid, dim3(256), 0, st, set, R, partial); break;
    case 2: hipLaunchKernelGGL(gram_partial<2>, grid, dim3(256), 0, st, set, R, partial); break;
    case 3: hipLaunchKernelGGL(gram_partial<3>, grid, dim3(256), 0, st, set, R, partial); break;
    default: hipLaunchKernelGGL(gram_partial<4>, grid, dim3(256), 0, st, set, R, partial); break;
    }
    if (reduce) hipLaunchKernelGGL(gram_reduce, dim3((R * R + 31) / 32, set.n), dim3(1024), 0, st, set, R, partial);
    return hipGetLastError();
}

hipError_t launch_gram(const float* A, int64_t rows, int R, float* partial, double* G, hipStream_t st,
                       int64_t nslab)
{
    GramSet set{};
    set.n = 1;
    set.A[0] = A;
    set.rows[0] = rows;
    set.G[0] = G;
    if (nslab <= 0) nslab = gram_slabs(rows);
    return launch_gram_set(set, &nslab, R, partial, st);
}

hipError_t launch_als_grams(const float* const* A, const int64_t* rows, int n, int R, float* partial, double* G,
                            hipStream_t st)
{
    GramSet set{};
    int64_t nslab[kGramMany] = {};
    if (n > kGramMany) return hipErrorInvalidValue;
    set.n = n;
    for (int m = 0; m < n; ++m) {
        set.A[m] = A[m];
        set.rows[m] = rows[m];
        set.G[m] = G + (int64_t)m * R * R;
        nslab[m] = als_gram_slabs(rows[m], R);
    }
    return launch_gram_set(set, nslab, R, partial, st);
}

// ------------------------------------------------ Gram without allocation
// The partial sums of amped_gram_noalloc live in this fixed device array
// instead of memory allocated per call: kGramScratchFloats floats (32 MiB) on
// every device the library runs on, held until the process ends.  Every call
// on a device shares its array; gram_partial overwrites every entry the
// reduction reads, so nothing has to be cleared between calls, and calls that
// overlap on one device race on it.
constexpr int64_t kGramScratchFloats = int64_t(8) << 20;
static __device__ __align__(256) float scratch[kGramScratchFloats];

namespace {
// Device address of `scratch` per device, looked up once per device with that
// device current (the host-side name is not a device address).
constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;
}  // namespace

int64_t gram_noalloc_slabs(int64_t rows, int R)
{
    const int64_t fit = kGramScratchFloats / ((int64_t)R * R);
    return std::min(gram_slabs(rows), fit);
}

hipError_t launch_gram_noalloc(const float* A, int64_t rows, int R, double* G, hipStream_t st)
{
    if (R < 1 || R > 128 || rows < 1) return hipErrorInvalidValue;
    const int64_t nslab = gram_noalloc_slabs(rows, R);
    if (nslab < 1 || nslab * (int64_t)R * R > kGramScratchFloats) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    float* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            g_scratch_ptr[dev] = static_cast<float*>(p);
        }
        ptr = g_scratch_ptr[dev];
    }
    return launch_gram(A, rows, R, ptr, G, st, nslab);
}

static hipError_t launch_als_solve(const float* M, const double* W, const int* wide, float* A, int64_t rows, int R,
                                   hipStream_t st);

hipError_t launch_als_update(const float* M, float* A, int64_t rows, float* partial, double* G, double* S, int N, int d,
                             int R, double* scratch, double* W, int* wide, double* lambda, bool last,
                             const double* xnorm2, double* fit, hipStream_t st)
{
    const int64_t nslab = als_gram_slabs(rows, R);
    SmallMode mode{};
    GramSet set{};
    set.n = 1;
    set.A[0] = M;
    set.rows[0] = rows;
    set.G[0] = S;
    const bool fold = R <= 64 && nslab <= kFoldSlabs;
    hipError_t e = launch_gram_set(set, &nslab, R, partial, st, !fold);
    if (e != hipSuccess) return e;
    if (fold) {
        mode.partial = partial;
        mode.nslab = (int)nslab;
    }
    // rank 64's block has 1024 threads, so 4096 entries of M; up to rank 32 it has 256
    const int block = R <= 32 ? 256 : 1024;
    const int64_t per = std::max(1, kSolvePerThread * block / R);
    const int64_t nblock = (rows + per - 1) / per;
    const bool solve = R <= 64 && nblock <= kSolveBlocks;
    if (solve) {
        mode.M = M;
        mode.A = A;
        mode.rows = (int)rows;
        mode.per = (int)per;
    }
    auto launch = [&](auto kernel, int rp, int threads) {
        const size_t lds = (size_t)rp * (rp + 1) * sizeof(double) * (rp <= 64 ? 2 : 1) +
                           (rp <= 64 ? (size_t)kSolvePerThread * threads * sizeof(float) : 0);
        hipLaunchKernelGGL(kernel, dim3(solve ? (unsigned)nblock : 1), dim3(threads), lds, st, G, S, N, d, R, scratch,
                           W, wide, lambda, last ? 1 : 0, xnorm2, fit, mode);
    };
    // one to four entries per thread while the block has them: fewer waves have
    // cheaper barriers but more arithmetic per pivot (rank 32: one wave of 16
    // entries per thread 46 us, four waves of 4 entries 19 us); 16 above rank 96
    if (R <= 16) launch(als_small<1, 16>, 16, 256);
    else if (R <= 32) launch(als_small<2, 16>, 32, 256);
    else if (R <= 64) launch(als_small<2, 32>, 64, 1024);
    else if (R <= 96) launch(als_small<3, 32>, 96, 1024);
    else launch(als_small<4, 32>, 128, 1024);
    if ((e = hipGetLastError()) != hipSuccess || solve) return e;
    return launch_als_solve(M, W, wide, A, rows, R, st);
}

static hipError_t launch_als_solve(const float* M, const double* W, const int* wide, float* A, int64_t rows, int R,
                            hipStream_t st)
{
    if (rows <= 0) return hipSuccess;
    const int C8 = (R + 7) / 8;
    // rows per thread: 4, or 2 above R = 64 so that the fp64 W (R x 8 C8
    // doubles) and the staged rows of M fit one block's LDS
    const int rpt = R > 64 ? 2 : 4;
    const int RB = rpt * (256 / C8);    // rows per block
    const size_t lds = (size_t)R * 8 * C8 * sizeof(double) + (size_t)RB * (R + 1) * sizeof(float);
    if ((int64_t)RB * R > 8 * 256 * 4) return hipErrorInvalidValue;   // the kernel holds 8 float4 per thread
    const int64_t ntiles = (rows + RB - 1) / RB;
    // persistent grid: as many blocks as fit on the GPU at once
    int dev = 0, cus = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = rpt == 4 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, als_solve<4>, 256, lds)
                     : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, als_solve<2>, 256, lds);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(ntiles, (int64_t)std::max(per_cu, 1) * cus)));
    if (rpt == 4) hipLaunchKernelGGL(als_solve<4>, grid, dim3(256), lds, st, M, W, wide, A, rows, R, RB, ntiles);
    else hipLaunchKernelGGL(als_solve<2>, grid, dim3(256), lds, st, M, W, wide, A, rows, R, RB, ntiles);
    return hipGetLastError();
}

hipError_t launch_tensor_norm2(const ModeDev& m, int nin, double* result, bool accumulate, hipStream_t st)
{
    hipError_t e = accumulate ? hipSuccess : hipMemsetAsync(result, 0, sizeof(double), st);
    if (e != hipSuccess || m.nnz == 0) return e;
    InIdx ii{};
    for (int w = 0; w < nin; ++w) ii.p[w] = m.in_idx[w];
    const int grid = (int)std::min<int64_t>((m.nnz + 255) / 256, 4096);
    hipLaunchKernelGGL(tensor_norm2, dim3(grid), dim3(256), 0, st, m.out_idx, ii, nin, m.val, m.nnz, result);
    return hipGetLastError();
}

}  // namespace amped
