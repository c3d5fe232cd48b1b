// MTTKRP of tensors of up to kSmallNnz nonzeros, in one launch.
//
// What bounds such a call is latency: the launches, and in them one chain of
// memory accesses.  So:
//  * one wave per unit, one unit per block, no queue: 1500 waves for 100k
//    nonzeros, each with a few batches to go;
//  * units are cut at row starts (built with the layout), so an output row has
//    one writer and nothing has to be zeroed before it is added to; the untouched
//    rows are zeroed here, by the waves that are done;
//  * a row longer than kSmallRow spans units: each writes its sum to a slot of its
//    own and counts itself in, and the last one adds the slots in unit order and
//    stores the row (so the sums do not depend on the waves' order);
//  * a lane group reads its nonzeros' metadata straight into registers, and the
//    code is a rolled loop of 4 nonzeros per group, a quarter of the large
//    kernel's, which a cold instruction cache takes in sooner.
// With the init kernel and the queue's kernel, a mode of 100k nonzeros at rank 16
// took 2.3 + 7.4 us of kernels and 9.5 us of host time in the call; 6.3 us and 6.6.
#include "kernel_impl.h"

namespace amped {
namespace dev {

constexpr uint64_t kShareMark = uint64_t(1) << 32;
constexpr int kShareTries = 1 << 14;

// Lane s of a group reads RPL columns from min(s RPL, ncols - RPL) on, as the
// large kernel's instances for any rank do.
template <int NIN, int LPR, int RPL, typename T>
__global__ void __launch_bounds__(64) small_kernel(const SmallParams p)
{
    constexpr int G = 64 / LPR, RT = LPR * RPL, U = 4;
    using RowT = Row<T, RPL>;
    __shared__ int s_key[2 * G];
    __shared__ __align__(16) float s_acc[2 * G][RT];

    const int lane = threadIdx.x & 63;
    const int g = lane / LPR, s = lane % LPR;
    const int c = p.col0 + min(s * RPL, p.ncols - RPL);
    const int64_t ld = p.ld;
    const uint32_t rb = (uint32_t)ld * (uint32_t)sizeof(T), cb = (uint32_t)c * (uint32_t)sizeof(T);
    const int unit = blockIdx.x;
    const int cs = unit < p.n_units ? p.cut[unit] : 0;
    const int clen = unit < p.n_units ? p.cut[unit + 1] - cs : 0;
    if (clen > 0) {
        const int Lg = (clen + U * G - 1) / (U * G) * U;    // a group's run, whole batches
        const int goff = g * Lg;
        const int len = max(0, min(Lg, clen - goff));
        const bool gon = len > 0;
        const uint32_t mbytes = (uint32_t)((clen + 3) & ~3) * 4u;   // the arrays carry 4 entries of padding
        __amdgpu_buffer_rsrc_t rk = make_rsrc(p.out_idx + cs, mbytes), rv = make_rsrc(p.val + cs, mbytes);
        __amdgpu_buffer_rsrc_t ri[NIN], rf[NIN];
#pragma unroll
        for (int w = 0; w < NIN; ++w) {
            ri[w] = make_rsrc(p.in_idx[w] + cs, mbytes);
            rf[w] = make_rsrc(p.fac[w], p.fbytes[w]);
        }
        struct Meta {
            int key[U], val[U], ix[NIN][U];
        };
        // nonzeros j .. j + 3 of the group's run; past its end a value of 0, the
        // last key and a row whose offset is past the factor's end (reads zeros)
        auto load = [&](Meta& m, int j) {
            const int off = j < Lg ? (goff + j) * 4 : 0x40000000;
            const u32x4 k = __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0);
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0);
#pragma unroll
            for (int e = 0; e < U; ++e) {
                m.key[e] = (int)k[e];
                m.val[e] = (int)v[e];
            }
#pragma unroll
            for (int w = 0; w < NIN; ++w) {
                const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(ri[w], off, 0, 0);
#pragma unroll
                for (int e = 0; e < U; ++e) m.ix[w][e] = (int)x[e];
            }
        };
        auto issue = [&](typename RowT::Raw (&raw)[U][NIN], const Meta& m, int j) {
#pragma unroll
            for (int e = 0; e < U; ++e)
#pragma unroll
                for (int w = 0; w < NIN; ++w) {
                    const uint32_t row = j + e < len ? (uint32_t)m.ix[w][e] : ~0u;
                    raw[e][w] = RowT::load_buf(rf[w], row * rb + cb);
                }
        };

        Meta m0, m1, m2;
        typename RowT::Raw ra[U][NIN], rbuf[U][NIN];
        load(m0, 0);
        // the keys at the ends of the run and beside them, and the unit's edges
        const int top = p.nnz - 1;
        const int gs = cs + goff, ge = gs + len;
        const int k_first = p.out_idx[min(gs, top)], k_prev = p.out_idx[max(min(gs, p.nnz) - 1, 0)];
        const int k_last = p.out_idx[max(min(ge, p.nnz) - 1, 0)], k_next = p.out_idx[min(ge, top)];
        const int left = p.left[unit], right = p.left[unit + 1];   // split rows at the unit's ends, or -1
        load(m1, U);
        issue(ra, m0, 0);

        // the row that is open, and whether it began before the run (in an earlier
        // group or unit)
        int open_key = k_first, first_open = 1;
        const int lsh = gon && gs > 0 && k_prev == k_first ? 1 : 0;
        float acc[RPL];
#pragma unroll
        for (int i = 0; i < RPL; ++i) acc[i] = 0.f;
        if (s == 0) s_key[2 * g] = s_key[2 * g + 1] = -1;
        wave_lds_sync();
        auto consume = [&](typename RowT::Raw (&raw)[U][NIN], const Meta& m, int j) {
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const bool in = j + e < len;
                const float val = in ? __int_as_float(m.val[e]) : 0.f;
                const int key = in ? m.key[e] : k_last;
                float prod[RPL];
                RowT::unpack(raw[e][0], prod);
#pragma unroll
                for (int w = 1; w < NIN; ++w) {
                    float rw[RPL];
                    RowT::unpack(raw[e][w], rw);
#pragma unroll
                    for (int i = 0; i < RPL; ++i) prod[i] *= rw[i];
                }
                if (gon && key != open_key) {
                    if (first_open & lsh) {
                        lds_store<RPL>(&s_acc[2 * g][s * RPL], acc);
                        if (s == 0) s_key[2 * g] = open_key;
                    } else {
                        store_vec<RPL>(p.out + (int64_t)open_key * ld + c, acc);
                    }
#pragma unroll
                    for (int i = 0; i < RPL; ++i) acc[i] = 0.f;
                    open_key = key;
                    first_open = 0;
                }
#pragma unroll
                for (int i = 0; i < RPL; ++i) acc[i] = fmaf(val, prod[i], acc[i]);
            }
        };
        // the metadata of batch q + 2 goes out before the gathers of q + 1, so the
        // wait for it leaves those in flight
#pragma unroll 1
        for (int j = 0; j < Lg; j += 2 * U) {
            load(m2, j + 2 * U);
            issue(rbuf, m1, j + U);
            consume(ra, m0, j);
            m0 = m1;
            m1 = m2;
            if (j + U >= Lg) break;
            load(m2, j + 3 * U);
            issue(ra, m1, j + 2 * U);
            consume(rbuf, m0, j + U);
            m0 = m1;
            m1 = m2;
        }

        // end of the run: the open row is stored, or parked when it goes on
        if (gon) {
            const bool more = ge < p.nnz && k_next == open_key;
            if (more || (first_open & lsh)) {
                lds_store<RPL>(&s_acc[2 * g + 1][s * RPL], acc);
                if (s == 0) s_key[2 * g + 1] = open_key;
            } else {
                store_vec<RPL>(p.out + (int64_t)open_key * ld + c, acc);
            }
        }
        wave_lds_sync();
        // the parked pieces in slot order, a lane per column; the row that came in
        // from the left unit or goes on into the right one is a split row
        const int kq = lane < 2 * G ? s_key[lane] : -1;
        uint64_t slots = __builtin_amdgcn_ballot_w64(kq >= 0);
        if (slots != 0) {
            constexpr int CL = (RT + 63) / 64;
            const int full = p.ncols / RPL * RPL;   // columns that only their own lane holds
            int at[CL];
            float sum[CL];
#pragma unroll
            for (int i = 0; i < CL; ++i) {
                const int cc = lane + 64 * i;
                at[i] = cc >= p.ncols ? 0 : cc < full ? cc : cc + full + RPL - p.ncols;
                sum[i] = 0.f;
            }
            int cur = -1;
            const int left_key = left >= 0 ? p.out_idx[cs] : -1, right_key = right >= 0 ? p.out_idx[cs + clen] : -1;
            auto put = [&](int row, const float (&x)[CL]) {
#pragma unroll
                for (int i = 0; i < CL; ++i)
                    if (lane + 64 * i < p.ncols) p.out[(int64_t)row * ld + p.col0 + lane + 64 * i] = x[i];
            };
            auto emit = [&]() {
                if (cur < 0) return;
                const bool from_left = cur == left_key;
                if (!from_left && cur != right_key) {
                    put(cur, sum);
                    return;
                }
                // This unit's share of split row h, then the unit is counted in; the last
                // one to arrive adds all shares.  The counter says who adds, not that the
                // others' shares are visible yet: relaxed atomics on different locations
                // have no order between blocks.  So a share is one 64-bit atomic of its
                // value and a mark, and the adder reads a share until the mark is there,
                // which is the order of a single location; the share's wave has counted
                // itself in and waits for nobody, so it comes.  (No fences: an agent-scope
                // release writes an L2 back, which took split modes of 250k nonzeros from 9
                // to 18 us.)  The adder clears the marks for the next launch.
                const int h = from_left ? left : right;
                uint64_t* mine = p.share + (int64_t)(unit + h) * kSmallCols + lane;
#pragma unroll
                for (int i = 0; i < CL; ++i)
                    __hip_atomic_store(mine + 64 * i, kShareMark | __float_as_uint(sum[i]), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                const int f = p.split[2 * h], n = p.split[2 * h + 1];   // its first unit and how many
                unsigned before = 0;
                if (lane == 0)
                    before = __hip_atomic_fetch_add(p.arrived + h, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                before = (unsigned)__builtin_amdgcn_readfirstlane((int)before);
                if (before + 1 != (unsigned)n) return;
                double total[CL];   // fp64: the error does not grow with the units
#pragma unroll
                for (int i = 0; i < CL; ++i) total[i] = 0.0;
                uint64_t* const all = p.share + (int64_t)(f + h) * kSmallCols + lane;
                for (int k0 = 0; k0 < n; k0 += 8) {
                    uint64_t x[8][CL];
                    bool here = false;
                    // (bounded all the same: calls of one mode at once, which the API
                    // forbids, could leave a mark out for good)
                    for (int tries = 0; !here && tries < kShareTries; ++tries) {
                        here = true;
#pragma unroll
                        for (int k = 0; k < 8; ++k)
#pragma unroll
                            for (int i = 0; i < CL; ++i) {
                                x[k][i] = k0 + k < n ? __hip_atomic_load(all + (int64_t)(k0 + k) * kSmallCols + 64 * i,
                                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                     : kShareMark;
                            }
#pragma unroll
                        for (int k = 0; k < 8; ++k)
#pragma unroll
                            for (int i = 0; i < CL; ++i) here = here && (x[k][i] & kShareMark) != 0;
                        here = __builtin_amdgcn_ballot_w64(!here) == 0;
                    }
#pragma unroll
                    for (int k = 0; k < 8; ++k)
#pragma unroll
                        for (int i = 0; i < CL; ++i) {
                            total[i] += (double)__uint_as_float((uint32_t)x[k][i]);
                            if (k0 + k < n)
                                __hip_atomic_store(all + (int64_t)(k0 + k) * kSmallCols + 64 * i, uint64_t(0),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                }
#pragma unroll
                for (int i = 0; i < CL; ++i) sum[i] = (float)total[i];
                put(cur, sum);
                if (lane == 0)   // for the next launch
                    __hip_atomic_store(p.arrived + h, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            for (;;) {
                const int q = slots != 0 ? __builtin_ctzll(slots) : 0;
                const int k = slots != 0 ? __builtin_amdgcn_readlane(kq, q) : -2;
                if (k != cur) {
                    emit();
                    if (slots == 0) break;
                    cur = k;
#pragma unroll
                    for (int i = 0; i < CL; ++i) sum[i] = 0.f;
                }
#pragma unroll
                for (int i = 0; i < CL; ++i) sum[i] += s_acc[q][at[i]];
                slots &= slots - 1;
            }
        }
    }
    zero_rows(p.out, ld, p.col0, p.ncols, p.vec4, p.zrows, p.n_zero, p.gaps, p.n_gaps, blockIdx.x, gridDim.x);
}

template <int NIN, typename T>
SmallFn pick_small_vec(Lanes v)
{
    if (v.rpl == 4) {
        switch (v.lpr) {
        case 2: return small_kernel<NIN, 2, 4, T>;
        case 4: return small_kernel<NIN, 4, 4, T>;
        case 8: return small_kernel<NIN, 8, 4, T>;
        case 16:
            if constexpr (sizeof(T) == 4) return small_kernel<NIN, 16, 4, T>;
            break;
        case 32:
            if constexpr (sizeof(T) == 4) return small_kernel<NIN, 32, 4, T>;
            break;
        case 64:
            if constexpr (sizeof(T) == 4) return small_kernel<NIN, 64, 4, T>;
            break;
        default: break;
        }
    } else if constexpr (sizeof(T) == 2) {
        switch (v.lpr) {
        case 4: return small_kernel<NIN, 4, 8, T>;
        case 8: return small_kernel<NIN, 8, 8, T>;
        case 16: return small_kernel<NIN, 16, 8, T>;
        case 32: return small_kernel<NIN, 32, 8, T>;
        default: break;
        }
    }
    return nullptr;
}

template <typename T>
SmallFn pick_small_nin(int nin, Lanes v)
{
    switch (nin) {
    case 1: return pick_small_vec<1, T>(v);
    case 2: return pick_small_vec<2, T>(v);
    case 3: return pick_small_vec<3, T>(v);
    case 4: return pick_small_vec<4, T>(v);
    default: return nullptr;
    }
}

SmallFn pick_small(int nin, FactorType ft, Lanes v)
{
    return ft == FactorType::F32 ? pick_small_nin<float>(nin, v) : pick_small_nin<uint16_t>(nin, v);
}

}  // namespace dev
}  // namespace amped
