// The column-list kernel (see spd_match.h).  Included by the spd_match_*.hip translation units.
#pragma once
#include "spd_match.h"
#include "spd_scan_impl.h"

namespace spd {

__device__ __forceinline__ int64_t clamp_i64(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// (LDS by address: an offset from a __shared__ array costs another addition)
template <typename T> __device__ __forceinline__ __attribute__((address_space(3))) T *lds_at(uint32_t address) {
    return (__attribute__((address_space(3))) T *)(uintptr_t)address;
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
// A strip holds a pair's sums in planes, one for each number of Op<OP>::Acc (its doubles, then its count), so that the
// rows of neighbouring lanes lie in different banks.  `at`: LDS address of the strip, `plane`: bytes of a plane of doubles.
// Fixed: one sum in fixed point in the place of the double.
struct Fixed { long long v; };
struct Ranked { uint32_t m, met_a, met_b; };         // Chebyshev: the maximum (a float's bits), which of the rows' largest entries were met
template <int OP> struct Sums {
    static constexpr bool FIX = match_fixed(OP);
    using Acc = std::conditional_t<FIX, Fixed, std::conditional_t<OP == OP_CHEB, Ranked, typename Op<OP>::Acc>>;
    static_assert(!FIX || (match_doubles(OP) == 1 && match_counts(OP) == 0), "one sum");
    static __device__ __forceinline__ void init(Acc &x) {
        if constexpr (FIX) x.v = 0; else if constexpr (OP == OP_CHEB) x = Ranked{0u, 0u, 0u}; else Op<OP>::init(x);
    }
    static __device__ __forceinline__ void combine(Acc &x, const Acc &y) {
        if constexpr (FIX) x.v += y.v; else if constexpr (OP != OP_CHEB) Op<OP>::combine(x, y);
    }
    static constexpr int kDoubles = match_doubles(OP), kCounts = match_counts(OP);
    static constexpr bool kOne = kDoubles + kCounts == 1;
    static constexpr bool kAnyOrder = FIX || kDoubles == 0;       // integers: their sums come out the same in any order
    static constexpr uint32_t kUnit = kDoubles ? 8u : 4u;          // bytes from a row's first number to the next row's
    static __device__ __forceinline__ Acc get(uint32_t at, uint32_t plane, uint32_t row) {
        Acc x;
        init(x);
        if constexpr (OP == OP_CHEB) {
            return Ranked{*lds_at<uint32_t>(at + row * 4u), *lds_at<uint32_t>(at + plane / 2u + row * 4u), *lds_at<uint32_t>(at + plane + row * 4u)};
        }
#pragma unroll
        for (int p = 0; p < kDoubles; ++p) {
            const double v = *lds_at<double>(at + (uint32_t)p * plane + row * 8u);
            __builtin_memcpy(reinterpret_cast<unsigned char *>(&x) + 8 * p, &v, 8);
        }
        if constexpr (kCounts == 1) {
            const int v = *lds_at<int>(at + (uint32_t)kDoubles * plane + row * 4u);
            __builtin_memcpy(reinterpret_cast<unsigned char *>(&x) + 8 * kDoubles, &v, 4);
        }
        return x;
    }
    static __device__ __forceinline__ void put(uint32_t at, uint32_t plane, uint32_t row, const Acc &x) {
        if constexpr (OP == OP_CHEB) {
            *lds_at<uint32_t>(at + row * 4u) = x.m;
            *lds_at<uint32_t>(at + plane / 2u + row * 4u) = x.met_a;
            *lds_at<uint32_t>(at + plane + row * 4u) = x.met_b;
            return;
        }
#pragma unroll
        for (int p = 0; p < kDoubles; ++p) {
            double v;
            __builtin_memcpy(&v, reinterpret_cast<const unsigned char *>(&x) + 8 * p, 8);
            *lds_at<double>(at + (uint32_t)p * plane + row * 8u) = v;
        }
        if constexpr (kCounts == 1) {
            int v;
            __builtin_memcpy(&v, reinterpret_cast<const unsigned char *>(&x) + 8 * kDoubles, 4);
            *lds_at<int>(at + (uint32_t)kDoubles * plane + row * 4u) = v;
        }
    }
    // Adds to the sums of the row whose first number lies `offset` bytes into the strip.
    static __device__ __forceinline__ void add(uint32_t at, uint32_t plane, uint32_t offset, const Acc &x) {
        if constexpr (OP == OP_CHEB) {
            (void)__hip_atomic_fetch_max(lds_at<uint32_t>(at + offset), x.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            (void)__hip_atomic_fetch_or(lds_at<uint32_t>(at + plane / 2u + offset), x.met_a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            (void)__hip_atomic_fetch_or(lds_at<uint32_t>(at + plane + offset), x.met_b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return;
        }
        if constexpr (FIX) {
            __hip_atomic_fetch_add(lds_at<unsigned long long>(at + offset), (unsigned long long)x.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return;
        }
#pragma unroll
        for (int p = 0; p < kDoubles; ++p) {
            double v;
            __builtin_memcpy(&v, reinterpret_cast<const unsigned char *>(&x) + 8 * p, 8);
            __hip_atomic_fetch_add(lds_at<double>(at + (uint32_t)p * plane + offset), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if constexpr (kCounts == 1) {
            int v;
            __builtin_memcpy(&v, reinterpret_cast<const unsigned char *>(&x) + 8 * kDoubles, 4);
            __hip_atomic_fetch_add(lds_at<int>(at + (uint32_t)kDoubles * plane + (kDoubles ? offset >> 1 : offset)), v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    // A strip of one number: the row's, which becomes zero bits (what init() makes).
    static __device__ __forceinline__ Acc take(uint32_t at) {
        Acc x;
        if constexpr (kDoubles) {
            const unsigned long long v = __hip_atomic_exchange(lds_at<unsigned long long>(at), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_memcpy(&x, &v, 8);
        } else {
            const uint32_t v = __hip_atomic_exchange(lds_at<uint32_t>(at), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            __builtin_memcpy(&x, &v, 4);
        }
        return x;
    }
    static __device__ __forceinline__ bool is_zero(const Acc &x) {
        if constexpr (kDoubles) {
            unsigned long long v;
            __builtin_memcpy(&v, &x, 8);
            return v == 0ull;
        } else {
            uint32_t v;
            __builtin_memcpy(&v, &x, 4);
            return v == 0u;
        }
    }
};

// One column both rows store: the products of Op<OP>, without the tests for absent entries that the
// staged scan needs (neither lists nor rows hold zeros, nor for Jensen-Shannon and KL what is not positive).  match_walks: whether any column of an entry of A can count.
template <int OP> __device__ __forceinline__ bool match_walks(float a) { return OP == OP_JS || OP == OP_KL ? a > 0.0f : a != 0.0f; }
template <int OP> __device__ __forceinline__ void match_visit(typename Op<OP>::Acc &x, float a, float b, const OpParams &q) {
    if constexpr (OP == OP_CNT) {
        x.c = 1;
    } else if constexpr (OP == OP_HAMM) {
        x.c = (a != b) ? -1 : -2;
    } else if constexpr (OP == OP_JS) {
        x.v = (double)Op<OP>::term(a, b) - ((double)a + (double)b);
    } else if constexpr (OP == OP_KL) {
        x.v = (double)(a * fast_log2(divide(a, divisor_of(b))));
        x.hits = 1;
    } else if constexpr (OP == OP_MINK) {
        Op<OP>::init(x);
        for_degree(q.p, [&](auto tag) { Op<OP>::template visit_as<decltype(tag)::value>(x, a, Op<OP>::prep(b, q), q); });
    } else {
        Op<OP>::init(x);
        Op<OP>::visit(x, a, Op<OP>::prep(b, q), q);
    }
}

// A row of A as the sums in fixed point take it (match_fixed): a term x of the row stands as `offset` + `factor` * x, in [2, 4)
// and thus in units of 2^-51; `unit` is what one of them is worth.  `wild`: Canberra, see match_wild.
struct Scale { double factor, offset, unit; bool wild; };
__device__ __forceinline__ double power_of_two(int e) { return __hiloint2double((1023 + e) << 20, 0); }
template <int OP> __device__ __forceinline__ Scale scale_of(int e, int len) {
    Scale s{1.0, 2.0, 1.0, OP == OP_CANB && e != 0};
    if constexpr (match_fixed(OP)) {
        const int k = OP == OP_CANB ? match_canberra_scale(len) : e;
        s.factor = power_of_two(-k);
        s.unit = power_of_two(k - 51);
        if constexpr (OP == OP_CANB) { s.offset += 2.0 * s.factor; s.factor = -s.factor; }
    }
    return s;
}
// The words of a double in [2, 4) are 2^62 and its mantissa, which counts units of 2^-51: a sum of such words modulo 2^62 is
// the sum of the units.
template <int OP> __device__ __forceinline__ Fixed fixed_visit(float a, float b, const Scale &s) {
    double t;
    if constexpr (OP == OP_L1) {
        t = fma((double)fabsf(median_with_zero(a, b)), s.factor, 2.0);
    } else {
        t = fma((double)fast_div(fabsf(a - b), fabsf(a) + fabsf(b)), s.factor, s.offset);
    }
    long long w;
    __builtin_memcpy(&w, &t, 8);
    return Fixed{w};
}
// The same for a column of a row that is wild: |a - b| / (|a| + |b|) of numbers that are brought to where neither the sum nor its reciprocal
// leaves single precision (one that is 2^53 below the other adds nothing to the ratio of 1).
__device__ __forceinline__ Fixed wild_visit(float a, float b, const Scale &s) {
    const float by = fabsf(a) < 1.0f && fabsf(b) < 1.0f ? 0x1p96f : 0x1p-96f;
    return fixed_visit<OP_CANB>(a * by, b * by, s);
}
// A sum of Op<OP>, formed in fp64, in units.
template <int OP> __device__ __forceinline__ Fixed fixed_sum(const typename Op<OP>::Acc &x, const Scale &s) {
    return Fixed{(long long)__builtin_rint(x.v * (s.factor * 0x1p51))};
}
// The units of a sum.
__device__ __forceinline__ double units_of(const Fixed &x) { return (double)(unsigned long long)(x.v & ((1ll << 62) - 1)); }
// What a distance reads of a row of B: nothing, the first norm, the second one (cosine: it is 0 where the first is), or both.
// They lie in planes, so that a row of the tile costs 8 bytes where the two together were 16.
enum NormsRead { READ_NONE = 0, READ_FIRST, READ_SECOND, READ_BOTH };
SPD_HD constexpr int norms_read(int metric) {
    switch (metric) {
    case MT_INNER: case MT_KL: case MT_KL_STRICT: case MT_RUSSELL_RAO: case MT_CHEBYSHEV: return READ_NONE;
    case MT_COSINE: return READ_SECOND;
    case MT_CORRELATION: case MT_MINKOWSKI: case MT_L2_UNEXPANDED: return READ_BOTH;
    default: return READ_FIRST;
    }
}
// ... `x` the first of what is read, `y` the second norm.
struct RowNorms { double x, y; };
// The distance of a pair from its sums and the rows' norms.
template <int OP, int MT>
__device__ __forceinline__ float distance_of(const OpParams &q, const typename Sums<OP>::Acc &c, double unit, double na0, double na1, const RowNorms &b) {
    constexpr int R = norms_read(MT);
    const double a0 = R == READ_SECOND ? na1 : na0, b1 = R == READ_SECOND ? b.x : b.y;
    if constexpr (match_fixed(OP)) {
        return finish_as<MT>(q, units_of(c) * unit, 0.0, 0.0, a0, na1, b.x, b1);
    } else if constexpr (OP == OP_CHEB) {
        return 0.0f;                                               // (not formed from these: finish_ranked)
    } else {
        using O = Op<OP>;
        return finish_as<MT>(q, O::v0(c), O::v1(c), O::v2(c), a0, na1, b.x, b1);
    }
}

// Lane l receives lane 63 - l's value.
__device__ __forceinline__ uint64_t wave_reverse(uint64_t v) {
    const int from = (63 - (int)__lane_id()) << 2;
    return ((uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)v);
}
constexpr int kMatchLocks = 32;          // k-NN: locks of a workgroup, by row

// One column of A against a row that may not store it (b = 0, which adds nothing).
template <int OP> __device__ __forceinline__ void dense_visit(typename Op<OP>::Acc &x, float a, float b, const OpParams &q) {
    if constexpr (OP == OP_MINK) {
        for_degree(q.p, [&](auto tag) { Op<OP>::template visit_as<decltype(tag)::value>(x, a, Op<OP>::prep(b, q), q); });
    } else {
        Op<OP>::visit(x, a, Op<OP>::prep(b, q), q);
    }
}

// Keeps what is computed into t and cell where the source has it (else it sinks into the branch that uses it).
template <typename Acc> __device__ __forceinline__ void pin(Acc &t, uint32_t &cell) {
    constexpr int N = (int)(sizeof(Acc) / 4);
    uint32_t w[N];
    __builtin_memcpy(w, &t, sizeof(Acc));
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(w[i]));
    asm volatile("" : "+v"(cell));
    __builtin_memcpy(&t, w, sizeof(Acc));
}

// Inclusive sum and maximum over the wavefront's lanes (the maximum of values that are not negative).
template <int CTRL, int ROWS> __device__ __forceinline__ int dpp_or_zero(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_scan_add(int v) {
    v += dpp_or_zero<0x111, 0xf>(v);                   // row_shr:1, 2, 4, 8
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);                   // row_bcast:15 into rows 1 and 3, row_bcast:31 into 2 and 3
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ int wave_scan_max(int v) {
    v = max(v, dpp_or_zero<0x111, 0xf>(v));
    v = max(v, dpp_or_zero<0x112, 0xf>(v));
    v = max(v, dpp_or_zero<0x114, 0xf>(v));
    v = max(v, dpp_or_zero<0x118, 0xf>(v));
    v = max(v, dpp_or_zero<0x142, 0xa>(v));
    v = max(v, dpp_or_zero<0x143, 0xc>(v));
    return v;
}
// h + w in one instruction, whatever the upper half of h's register holds.  (A half is a register's lower half to the compiler; a
// 16-bit integer it would clear the upper half of first.)
__device__ __forceinline__ uint32_t plus_half(_Float16 h, uint32_t w) {
    uint32_t r;
    asm("v_mad_u32_u16 %0, %1, 1, %2" : "=v"(r) : "v"(h), "s"(w));
    return r;
}
// Lane I of every row of 16 lanes, in all lanes of the row (row_newbcast).
template <int I> __device__ __forceinline__ uint32_t row_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + I, 0xf, 0xf, true);
}
template <int I> __device__ __forceinline__ float row_lane(float v) { return __uint_as_float(row_lane<I>(__float_as_uint(v))); }

constexpr int kMatchUnroll = 4;          // list steps whose loads are in flight together

// BOTH: k-NN whose distances read both norms (Minkowski's and correlation).
template <int OP, bool KNN, bool BOTH>
__global__ void __launch_bounds__(match_waves(match_cell_bytes(OP)) * kWave) spd_match_kernel(const MatchArgs args) {
    using O = Op<OP>;
    using S = Sums<OP>;
    constexpr bool FIX = S::FIX;
    using Acc = typename S::Acc;
    static_assert(S::kAnyOrder || !match_any_order(OP), "rows are shared from half the length on where the wavefronts add to one strip");
    // D: 64-row pieces of a dense column that are summed in registers together; the largest tiles hold 19 for one
    // fp64 sum (one round of 19 against two of 10: 2,048 queries of 300,000 rows of 230, 10.5 -> 10.2 ms; 13 and 6
    // leave half a round idle: 11.3) and 39 for a count; a sum and a count have 13 and Minkowski's three numbers 10, in two rounds of 7
    // (Jensen-Shannon needs its registers for the logarithms)
    constexpr int U = kMatchUnroll, D = S::kOne ? (OP == OP_JS ? 10 : (S::kDoubles ? 19 : 13)) : 7, nw = match_waves(match_cell_bytes(OP));
    extern __shared__ __align__(16) unsigned char dyn[];
    __shared__ int s_next;
    __shared__ int s_lock[KNN ? kMatchLocks : 1];
    __shared__ uint16_t s_owner[nw][kWave];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6);
    const int T = args.b.shape.tile_rows;
    const uint32_t strip_bytes = match_strip_bytes(match_cell_bytes(OP), T), plane = (uint32_t)(T + 1) * 8u;
    const uint32_t strips_at = lds_address(dyn), strip_at = (uint32_t)wave_uniform((int)(strips_at + (uint32_t)wave * strip_bytes));
    // Workgroups go round the eight XCDs in turn: with `by_xcd` the slices of one group of tiles, which
    // read the same lists at about the same time, share an XCD and its L2.
    int group, slice;
    if (args.by_xcd) {
        const int xcd = (int)blockIdx.x & 7, within = (int)blockIdx.x >> 3;
        slice = within % args.slices;
        group = within / args.slices * 8 + xcd;
    } else {
        slice = (int)blockIdx.x % args.slices;
        group = (int)blockIdx.x / args.slices;
    }
    if (group >= args.b.shape.n_tiles) return;
    const int my_tiles = (args.b.shape.n_tiles - group + args.groups - 1) / args.groups;      // group, group + groups, ...
    Acc zero;
    S::init(zero);
    for (int i = lane; i <= T; i += kWave) S::put(strip_at, plane, (uint32_t)i, zero);
    if (tid == 0) s_next = 0;
    if (KNN && tid < kMatchLocks) s_lock[tid] = 0;
    __syncthreads();

    // 64 entries of a row of A, one per lane, on their way to the strip: first the entries, then the lists of
    // their columns, then the lists' entries.  Each stage is loaded while the stage before it is at work on
    // something else, so that the three round trips to memory are not waited for in turn.
    // (`met`: Chebyshev, the bit of the entry's rank)
    struct Entries { uint32_t c; float v; uint32_t met; };
    struct Lists { uint32_t first, last; float a; uint32_t met; };
    auto load_entries = [&](int64_t start, int len, int e0) {
        Entries x{0xFFFFFFFFu, 0.0f, 0u};
        if (e0 + lane < len) {
            x.c = (uint32_t)args.a_indices[start + e0 + lane];
            x.v = args.a_values[start + e0 + lane];
            if constexpr (OP == OP_CHEB) {
                const uint32_t rank = args.ranks_a[start + e0 + lane];
                x.met = rank < (uint32_t)kRanks ? 1u << rank : 0u;
            }
        }
        return x;
    };
    auto load_lists = [&](int tile, const Entries &x) {
        const uint32_t *__restrict__ ptr = args.b.ptr + (size_t)tile * (size_t)args.b.shape.ptr_stride;
        Lists y{0u, 0u, 0.0f, 0u};
        if (x.c < args.k) {
            const uint32_t at = x.c + (x.c >> args.b.shape.block_shift);
            // (both in one load: 64 lanes at as many lines take the L1 as long for four bytes as for eight)
            struct __attribute__((packed, aligned(4))) Two { uint32_t first, last; };
            const Two two = *reinterpret_cast<const Two *>(ptr + at);
            y.first = two.first;
            y.last = two.last;
        }
        y.a = x.v;
        y.met = x.met;
        return y;
    };
    // The batch's dense columns: one value per row of the tile, lane by lane, summed in registers; then the strip.
    auto walk_dense = [&](const unsigned char *__restrict__ values, uint32_t first4, float a, uint64_t mask, const Scale &scale, uint32_t to) {
        const uint32_t lane4 = (uint32_t)lane * 4u;
        for (int i0 = 0; i0 < T; i0 += D * kWave) {
            typename O::Acc sum[D];
            float cur[D];
#pragma unroll
            for (int d = 0; d < D; ++d) O::init(sum[d]);
            // (past the tile's end what lies behind the column is read, or the spare entries at the end of the lists, and not added)
            auto fetch = [&](float (&into)[D], int e) {
                const unsigned char *col = values + ((uint32_t)__builtin_amdgcn_readlane((int)first4, e) + (uint32_t)i0 * 4u);
#pragma unroll
                for (int d = 0; d < D; ++d) into[d] = *reinterpret_cast<const float *>(col + lane4 + d * (kWave * 4));
            };
            auto visit = [&](const float (&from)[D], int e) {
                const float ae = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), e));
#pragma unroll
                for (int d = 0; d < D; ++d) dense_visit<OP>(sum[d], ae, from[d], args.q);
            };
            uint64_t left = mask;
            if constexpr (KNN && D == 19) {                       // (no registers for a second column in flight)
                for (; left; left &= left - 1) {
                    const int e = (int)__builtin_ctzll(left);
                    fetch(cur, e);
                    visit(cur, e);
                }
            } else {
                float nxt[D];
                int e = (int)__builtin_ctzll(left);
                fetch(cur, e);
                for (;;) {
                    left &= left - 1;
                    const int e1 = left ? (int)__builtin_ctzll(left) : e;
                    fetch(nxt, e1);
                    __builtin_amdgcn_sched_barrier(0);
                    visit(cur, e);
                    if (!left) break;
                    left &= left - 1;
                    e = left ? (int)__builtin_ctzll(left) : e1;
                    fetch(cur, e);
                    __builtin_amdgcn_sched_barrier(0);
                    visit(nxt, e1);
                    if (!left) break;
                }
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (i0 + d * kWave < T) {
                    const uint32_t i = (uint32_t)(i0 + lane + d * kWave);
                    if constexpr (FIX) {
                        S::add(to, plane, i * S::kUnit, fixed_sum<OP>(sum[d], scale));
                    } else if constexpr (S::kAnyOrder) {
                        if constexpr (OP != OP_CHEB) S::add(to, plane, i * S::kUnit, sum[d]);          // (which has no dense columns)
                    } else {
                        Acc acc = S::get(to, plane, i);
                        S::combine(acc, sum[d]);
                        S::put(to, plane, i, acc);
                    }
                }
        }
    };
    // The lists are cut into chunks of 16 entries, and a step is four chunks, one to a quarter of the
    // wavefront, whichever lists they belong to (a step of one list alone is filled to 62 % by 300,000 rows of 230 and to 28 %
    // by ratings; its 13 vector instructions are 8 here: 10,000 x 10,000 rows of 38, L1, 421 -> 340 us a call, 1,024 x 300,000
    // rows of 230, cosine, 6.6 -> 5.6 ms, 1,531 x 28,301 ratings, Canberra, 1.13 -> 0.75 ms).  Entries of six bytes
    // in two arrays and sums in fixed point: L1 of 10,000 x 10,000 rows of 38 355 -> 327 us, of 4,096 x 65,536 rows of 1,820 29.3 -> 25.2
    // ms.  What bounds a step now: nine to ten vector instructions and the chunks' share of those that describe them, 9 to 11 cache
    // lines looked up by the L1, 13 clocks of an LDS add, all of them clocks of a compute unit.
    // 64 chunks are described at a time, a chunk to a lane: lane 16 g + i
    // holds chunk 4 i + g, so that step i finds its four descriptions in lane i of each quarter (a DPP broadcast).  Chunks
    // follow one another over the steps and over the lanes of a step in the order of A's columns, and LDS serves the
    // lanes that meet in one sum in ascending order: a sum is formed in the order of A's columns here too.
    // What a walk of no more than four steps leaves behind for the k-NN's finish: the chunks it took, and the lanes' entries.
    struct Few { int total; uint32_t cell[U], left[U]; };
    auto walk_chunks = [&](const unsigned char *__restrict__ values, const unsigned char *__restrict__ rows, uint32_t first, uint32_t last, float a,
                           uint32_t met, const Scale &scale, uint32_t to, Few &few) {
        const int chunks = (int)((last - first + 15u) >> 4);
        const int incl = wave_scan_add(chunks), excl = incl - chunks;
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (KNN) few.total += total;
        if (total == 0) return;
        const uint32_t base4 = first * 4u - 64u * (uint32_t)excl;                // chunk q reads values from byte base4 + 64 q on
        const uint32_t last4 = last * 4u;
        const int turned = ((lane & 15) << 2) | (lane >> 4);
        const uint32_t lane4 = (uint32_t)(lane & 15) * 4u;
        struct Chunk { uint32_t at, left; float a; uint32_t met; };                            // left: bytes of its list's values from `at` on
        struct Entry { _Float16 cell; float v; };
        // (16 bits: 64 lists of a tile are 64 * 156 chunks at most, the last group's tag is below 2^14)
        uint16_t *owner = s_owner[wave];
        owner[lane] = 0;
        int tag = 64, carry = 0;
        // Which list a chunk belongs to: every list marks its first chunk with its lane, and a running maximum carries the
        // marks on (a mark of an earlier group is below the tag).
        auto describe = [&](int q0) {
            const uint32_t start = (uint32_t)(excl - q0);
            if (chunks > 0 && start < 64u) owner[start] = (uint16_t)(tag + lane);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            int e = owner[lane];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            e = wave_scan_max(max(e, tag + carry));
            carry = __builtin_amdgcn_readlane(e, 63) & 63;
            tag += 64;
            const int from = (__builtin_amdgcn_ds_bpermute(turned << 2, e) & 63) << 2;
            const int q = q0 + turned;
            Chunk c;
            c.at = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)base4) + 64u * (uint32_t)q;
            c.left = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)last4) - c.at;
            c.a = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(a)));
            c.met = 0u;
            if constexpr (OP == OP_CHEB) c.met = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)met);
            if (q >= total) { c.at = 0u; c.left = 0u; }
            return c;
        };
        auto fetch_one = [&](uint32_t chunk_at) {
            const uint32_t at = chunk_at + lane4;
            Entry x{*reinterpret_cast<const _Float16 *>(rows + (at >> 1)), 0.0f};
            if constexpr (OP != OP_CNT) x.v = *reinterpret_cast<const float *>(values + at);
            return x;
        };
        auto fetch = [&](Entry (&into)[U], const Chunk &c, auto block) {
            constexpr int I = decltype(block)::value * U;
            into[0] = fetch_one(row_lane<I>(c.at));
            into[1] = fetch_one(row_lane<I + 1>(c.at));
            into[2] = fetch_one(row_lane<I + 2>(c.at));
            into[3] = fetch_one(row_lane<I + 3>(c.at));
        };
        auto add_one = [&](const Entry &from, uint32_t left, float av, uint32_t met) {
            // (everything but the LDS add itself is done for all lanes: a branch around it costs more)
            Acc t;
            uint32_t at;
            if constexpr (OP == OP_CHEB) {
                const uint32_t cell = __builtin_bit_cast(uint16_t, from.cell), rank = cell >> kRankShift;
                const float d = fabsf(av - from.v);
                t = Ranked{__float_as_uint(d), met, rank < (uint32_t)kRanks ? 1u << (rank & 31u) : 0u};
                at = (cell & ((1u << kRankShift) - 1u)) * 4u;
                const bool counts = d == d;                       // (as a maximum passes over what is not a number)
                pin(t, at);
                if (lane4 < left && counts) S::add(to, plane, at, t);
                return;
            }
            if constexpr (FIX) t = fixed_visit<OP>(av, from.v, scale);
            else if constexpr (OP != OP_CHEB) match_visit<OP>(t, av, from.v, args.q);
            if constexpr (S::kOne) at = plus_half(from.cell, to); else at = __builtin_bit_cast(uint16_t, from.cell);
            pin(t, at);
            if (lane4 < left) {
                if constexpr (S::kOne) S::add(0u, plane, at, t); else S::add(to, plane, at, t);
            }
        };
        auto add = [&](const Entry (&from)[U], const Chunk &c, auto block) {
            constexpr int I = decltype(block)::value * U;
            add_one(from[0], row_lane<I>(c.left), row_lane<I>(c.a), OP == OP_CHEB ? row_lane<I>(c.met) : 0u);
            add_one(from[1], row_lane<I + 1>(c.left), row_lane<I + 1>(c.a), OP == OP_CHEB ? row_lane<I + 1>(c.met) : 0u);
            add_one(from[2], row_lane<I + 2>(c.left), row_lane<I + 2>(c.a), OP == OP_CHEB ? row_lane<I + 2>(c.met) : 0u);
            add_one(from[3], row_lane<I + 3>(c.left), row_lane<I + 3>(c.a), OP == OP_CHEB ? row_lane<I + 3>(c.met) : 0u);
        };
        constexpr std::integral_constant<int, 0> b0{};
        constexpr std::integral_constant<int, 1> b1{};
        constexpr std::integral_constant<int, 2> b2{};
        constexpr std::integral_constant<int, 3> b3{};
        Entry x[U], y[U];
        Chunk c = describe(0);
        fetch(x, c, b0);
        if (total <= 4 * U) {                                   // a few entries: no more steps than they take
            if constexpr (KNN) {
#pragma unroll
                for (int u = 0; u < U; ++u) few.cell[u] = __builtin_bit_cast(uint16_t, x[u].cell);
                few.left[0] = row_lane<0>(c.left);
                few.left[1] = row_lane<1>(c.left);
                few.left[2] = row_lane<2>(c.left);
                few.left[3] = row_lane<3>(c.left);
            }
            add_one(x[0], row_lane<0>(c.left), row_lane<0>(c.a), OP == OP_CHEB ? row_lane<0>(c.met) : 0u);
            if (total <= 4) return;
            add_one(x[1], row_lane<1>(c.left), row_lane<1>(c.a), OP == OP_CHEB ? row_lane<1>(c.met) : 0u);
            if (total <= 8) return;
            add_one(x[2], row_lane<2>(c.left), row_lane<2>(c.a), OP == OP_CHEB ? row_lane<2>(c.met) : 0u);
            if (total <= 12) return;
            add_one(x[3], row_lane<3>(c.left), row_lane<3>(c.a), OP == OP_CHEB ? row_lane<3>(c.met) : 0u);
            return;
        }
        fetch(y, c, b1);
        for (int left = total;;) {                              // chunks from this group on
            Chunk next = c;
            if (left > 64) next = describe(total - left + 64);
            __builtin_amdgcn_sched_barrier(0);                  // (keep the loads ahead of the arithmetic)
            add(x, c, b0);
            if (left <= 16) break;
            fetch(x, c, b2);
            __builtin_amdgcn_sched_barrier(0);
            add(y, c, b1);
            if (left <= 32) break;
            fetch(y, c, b3);
            __builtin_amdgcn_sched_barrier(0);
            add(x, c, b2);
            if (left <= 48) break;
            fetch(x, next, b0);
            __builtin_amdgcn_sched_barrier(0);
            add(y, c, b3);
            left -= 64;
            if (left <= 0) break;
            fetch(y, next, b1);
            c = next;
        }
    };
    // The batch's lists and dense columns of a row that is wild, one after the other.
    auto walk_wild = [&](const unsigned char *__restrict__ values, const unsigned char *__restrict__ rows, uint32_t first, uint32_t last, bool dense,
                         float a, const Scale &scale, uint32_t to) {
        if constexpr (OP == OP_CANB) {
            const uint32_t end = dense ? first + (uint32_t)T : last;
            const uint64_t dense_mask = __ballot(dense);
#pragma unroll 1
            for (uint64_t left = __ballot(first < end); left; left &= left - 1) {
                const int e = (int)__builtin_ctzll(left);
                const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)first, e), to_end = (uint32_t)__builtin_amdgcn_readlane((int)end, e);
                const float ae = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), e));
#pragma unroll 1
                for (uint32_t i = from + (uint32_t)lane; i < to_end; i += kWave) {
                    const float b = reinterpret_cast<const float *>(values)[i];
                    if (b == 0.0f) continue;
                    const uint32_t cell = (dense_mask >> e) & 1u ? (i - from) * S::kUnit : (uint32_t)reinterpret_cast<const uint16_t *>(rows)[i];
                    S::add(to, plane, cell, wild_visit(ae, b, scale));
                }
            }
        }
    };
    // (`to`: the strip)
    auto walk_lists = [&](int tile, const Lists &y, const Scale &scale, uint32_t to, Few &few) {
        const int64_t tile_first = args.b.shape.room_of(clamp_i64(args.b_indptr[(int64_t)tile * T], 0, args.b_nnz)) + tile * args.b.shape.tile_extra;
        const unsigned char *__restrict__ values = reinterpret_cast<const unsigned char *>(args.b.values + tile_first);
        const unsigned char *__restrict__ rows = reinterpret_cast<const unsigned char *>(args.b.rows + tile_first);
        const uint32_t list_n = (uint32_t)(args.b.shape.list_entries(args.b_nnz) - kMatchSpare - tile_first);     // (no access leaves the lists)
        const float a = transform_value(args.transform, y.a);
        const uint32_t position = args.b.shape.position_bits(), gap = args.b.shape.gap_bits();
        const uint32_t first = min(y.first & position, list_n);
        const uint32_t end = (y.last & position) - ((y.last >> kMatchGapShift) & gap);
        const bool dense = (y.first & kMatchDense) != 0u && match_walks<OP>(a) && first + (uint32_t)T <= list_n;
        const uint64_t dense_mask = __ballot(dense);
        if (OP == OP_CANB && scale.wild) {
            const uint32_t last = match_walks<OP>(a) && (y.first & kMatchDense) == 0u ? max(first, min(end, list_n)) : first;
            walk_wild(values, rows, first, last, dense, a, scale, to);
            if (KNN) few.total += 4 * U + 1;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            return;
        }
        if constexpr (OP != OP_CHEB) {
            if (dense_mask != 0) {
                if (KNN) few.total += 4 * U + 1;
                walk_dense(values, first * 4u, a, dense_mask, scale, to);
            }
        }
        const uint32_t last = match_walks<OP>(a) && (y.first & kMatchDense) == 0u ? max(first, min(end, list_n)) : first;
        walk_chunks(values, rows, first, last, a, y.met, scale, to, few);
        // (a lane reads later what other lanes of its wavefront wrote: LDS serves a wavefront in order, the
        // fence keeps the compiler to that order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    // What finish() reads of a row of A, loaded while the row's last lists are walked.
    struct RowOf { double na0, na1; uint64_t bound; };
    auto load_scale = [&](int row) { return FIX ? (int)args.scales_a[row] : 0; };
    auto load_row = [&](int row) {
        RowOf r{args.norms_a[row], args.norms_a[(size_t)args.m + (size_t)row], kKnnUnused};
        if constexpr (KNN) r.bound = (uint64_t)__atomic_load_n(&args.knn_tau[row], __ATOMIC_RELAXED);
        return r;
    };
    // k-NN: what the tiles of a row's run have found so far.
    uint64_t bound = kKnnUnused;          // no key above it can be among the k best
    uint64_t best = kKnnUnused;           // the k best, ascending over the lanes ...
    uint64_t queue = kKnnUnused;          // ... and `queued` keys that are not merged yet
    int queued = 0;
    bool any = false;
    // Chebyshev: the distances of the 64 rows from `from` on, and of those `step` further ..., from the strip at `at`, whose places are
    // cleared.  All of them are formed before the first is stored.
    auto finish_ranked = [&](int tile, int row, int64_t a_begin, int a_len, uint32_t at, int from, int step) {
      if constexpr (OP == OP_CHEB) {
        constexpr int G = kRankedRows / kWave;
        const int64_t j0 = (int64_t)tile * T;
        const int tile_n = (int)min((int64_t)T, args.n - j0);
        const float top_a = lane < kRanks ? args.tops_a[(size_t)row * kRanks + (size_t)lane] : 0.0f;
        float d[G];
        uint32_t doubt = 0u;                                     // (a bit a round) all of a row's largest entries were met, and smaller ones may exceed d
#pragma unroll
        for (int g = 0; g < G; ++g) {
            d[g] = 0.0f;
            const int i = from + g * step + lane;
            if (from + g * step >= T) continue;
            const Acc c = S::get(at, plane, (uint32_t)i);
            S::put(at, plane, (uint32_t)i, zero);
            const uint32_t first_a = ~c.met_a ? (uint32_t)__builtin_ctz(~c.met_a) : (uint32_t)kRanks, first_b = ~c.met_b ? (uint32_t)__builtin_ctz(~c.met_b) : (uint32_t)kRanks;
            const float next_a = __shfl(top_a, (int)min(first_a, (uint32_t)kRanks - 1u));
            const float next_b = args.b.tops[(size_t)min(first_b, (uint32_t)kRanks - 1u) * (size_t)args.n + (size_t)(j0 + min(i, tile_n - 1))];
            float most = __uint_as_float(c.m);
            most = first_a < (uint32_t)kRanks ? fmaxf(most, next_a) : most;
            most = first_b < (uint32_t)kRanks ? fmaxf(most, next_b) : most;
            d[g] = most;
            if ((first_a == (uint32_t)kRanks && next_a > most) || (first_b == (uint32_t)kRanks && next_b > most)) doubt |= 1u << g;
        }
        if (__ballot(doubt != 0u) != 0) {
            // The largest entry of one row, beyond what the pair has, in a column that the other does not store: by the whole wavefront.
            // Rows that are all met are mostly alike: an entry is looked for at its own place in the other row first, then next
            // to it, then outwards, and the other way round only where the columns are not the same ones.  (1,000 x 1,000 rows of 100
            // ones over one support: 2,513 us with both ways always and a reduction through LDS, 1,320 by the staged scan, 560 now, of which
            // the grid gives half; over supports that differ by a column 1,936, 884 and 610.  Both rows in one pass: 677 and 523, but ratings,
            // whose pairs' first pass mostly settles the second, 347 -> 406.)
            auto stored = [](const int32_t *yi, const float *yv, int y1, int guess, int32_t at_guess, int32_t col) {
                const bool up = at_guess < col;
                int lo = 0, hi = y1, step = 1;
                const int next = up ? guess + 1 : guess - 1;
                if (next < 0 || next >= y1) return false;
                const int32_t c = yi[next];
                const float w = yv[next];
                if (c == col) return w != 0.0f;
                if (up) {
                    if (c > col) return false;
                    lo = next + 1;
                    while (hi - lo > step && yi[lo + step] < col) { lo += step + 1; step *= 2; }
                    hi = min(hi, lo + step + 1);
                } else {
                    if (c < col) return false;
                    hi = next;
                    while (hi - lo > step && yi[hi - step] >= col) { hi -= step; step *= 2; }
                    lo = max(lo, hi - step);
                }
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (yi[mid] < col) lo = mid + 1; else hi = mid;
                }
                return lo < y1 && yi[lo] == col && yv[lo] != 0.0f;
            };
            // (`alike`: whether the entries of both rows are the same columns', and no stored zero hides one of the other's)
            auto beyond = [&](const int32_t *xi, const float *xv, int lx, const int32_t *yi, const float *yv, int ly, float most, bool &alike) {
                alike = lx == ly;
                for (int e = lane; e < lx; e += 2 * kWave) {
                    float v[2], w[2];
                    int32_t col[2], at_guess[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int x = e + u * kWave, guess = max(min(x, ly - 1), 0);
                        v[u] = x < lx ? fabsf(xv[x]) : 0.0f;
                        col[u] = x < lx ? xi[x] : 0;
                        at_guess[u] = ly > 0 ? yi[guess] : -1;
                        w[u] = ly > 0 ? yv[guess] : 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int x = e + u * kWave;
                        const bool here = at_guess[u] == col[u];
                        alike &= x >= lx || (here && v[u] != 0.0f);
                        if (v[u] > most && !(here ? w[u] != 0.0f : stored(yi, yv, ly, min(x, ly - 1), at_guess[u], col[u]))) most = v[u];
                    }
                }
                alike = __ballot(!alike) == 0;
                return __int_as_float(__builtin_amdgcn_readlane(wave_scan_max(__float_as_int(most)), 63));          // (none is negative)
            };
#pragma unroll 1
            for (int g = 0; g < G; ++g) {
                uint64_t left = __ballot((doubt >> g) & 1u);
                if (left == 0) continue;
                const int64_t j = j0 + min(from + g * step + lane, tile_n - 1);
                const int64_t first = clamp_i64(args.b_indptr[j], 0, args.b_nnz), last = clamp_i64(args.b_indptr[j + 1], first, args.b_nnz);
                for (; left; left &= left - 1) {
                    const int l = (int)__builtin_ctzll(left), i = from + g * step + l;
                    if (i >= tile_n) continue;
                    const int64_t b0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(first >> 32), l) << 32) |
                                                 (uint32_t)__builtin_amdgcn_readlane((int)first, l));
                    const int lb = __builtin_amdgcn_readlane((int)(last - first), l);
                    float mine = 0.0f;
#pragma unroll
                    for (int u = 0; u < G; ++u) mine = u == g ? d[u] : mine;
                    float most = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mine), l));
                    bool alike;
                    most = beyond(args.a_indices + a_begin, args.a_values + a_begin, a_len, args.b_indices + b0, args.b_values + b0, lb, most, alike);
                    if (!alike) most = beyond(args.b_indices + b0, args.b_values + b0, lb, args.a_indices + a_begin, args.a_values + a_begin, a_len, most, alike);
#pragma unroll
                    for (int u = 0; u < G; ++u) d[u] = u == g && lane == l ? most : d[u];
                }
            }
        }
        float *__restrict__ out = args.out + (size_t)row * (size_t)args.n + (size_t)j0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = from + g * step + lane;
            if (i < tile_n) __builtin_nontemporal_store(d[g], out + i);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    };
    // The tile's distances from the wavefront's strip, in row order: one coalesced store per 64 rows; the
    // strip is clear again afterwards.  `flush`: the row's run of tiles ends here; `lock`: k-NN, of a row that other workgroups
    // take in other tiles, else null.
    auto finish = [&](int tile, int row, const RowOf &of, const Scale &scale, const Few &few, bool flush, int *lock) {
        // (hidden from the compiler: it would keep the addresses of every loop below in registers through the whole kernel, 50 more than
        // there are.  k-NN by fp64 sums has them: 4,096 x 663,000 n-grams, cosine, 2,083 -> 2,032 us)
        int lane = (int)threadIdx.x & 63;
        if constexpr (!KNN || FIX) asm volatile("" : "+v"(lane));
        const int64_t j0 = (int64_t)tile * T;
        const int tile_n = (int)min((int64_t)T, args.n - j0);
        const double na0 = of.na0, na1 = of.na1, unit = (OP == OP_L1 ? -2.0 : -1.0) * scale.unit;            // (the sum enters the distance with that factor)
        constexpr int F = 4;                                      // rows of a lane that are in flight together
        // F rows of a lane from row i0 of the tile on: their sums and norms, by constant offsets from one address each (the
        // rows beyond the tile's last repeat it), and their places cleared again.  (With an address and a bound for every row,
        // 25 vector instructions per 64 rows, a call on 10,000 x 10,000 rows of 38 spent more on this than on the lists.)
        const uint32_t lane4 = (uint32_t)lane * 4u;
        auto load_norms = [&](const double *first, bool both, int i0, RowNorms (&nb)[F]) {
            const unsigned char *const first_at = reinterpret_cast<const unsigned char *>(first + j0);
            const unsigned char *const second_at = reinterpret_cast<const unsigned char *>(args.b.norms + args.n + j0);
            auto load = [&](auto at) {
#pragma unroll
                for (int u = 0; u < F; ++u) nb[u].x = *reinterpret_cast<const double *>(first_at + at(u, 8u));
                if (both) {
#pragma unroll
                    for (int u = 0; u < F; ++u) nb[u].y = *reinterpret_cast<const double *>(second_at + at(u, 8u));
                }
            };
            if (i0 + F * kWave <= tile_n) {
                load([&](int u, uint32_t size) { return (uint32_t)(i0 + lane) * size + (uint32_t)(u * kWave) * size; });
            } else {
                load([&](int u, uint32_t size) { return (uint32_t)min(i0 + u * kWave + lane, tile_n - 1) * size; });
            }
        };
        auto load_sums = [&](int i0, Acc (&c)[F]) {
            if (i0 + F * kWave <= tile_n) {
#pragma unroll
                for (int u = 0; u < F; ++u) c[u] = S::get(strip_at, plane, (uint32_t)(i0 + lane + u * kWave));
            } else {
#pragma unroll
                for (int u = 0; u < F; ++u) c[u] = S::get(strip_at, plane, (uint32_t)min(i0 + u * kWave + lane, tile_n - 1));
            }
        };
        auto clear_round = [&](int i0) {
#pragma unroll
            for (int u = 0; u < F; ++u)
                if (i0 + u * kWave < T) S::put(strip_at, plane, (uint32_t)(i0 + lane + u * kWave), zero);          // (a tile is whole wavefronts of rows)
        };
        // Dense columns add behind the last tile's end too: 0, unless the entry of A is not finite.  Nothing reads these sums
        // here, but the wavefront's next tile may be an earlier one, which has rows there.
        auto clear_behind = [&]() {
            for (int i0 = (tile_n + F * kWave - 1) / (F * kWave) * (F * kWave); i0 < T; i0 += F * kWave) clear_round(i0);
        };
        if constexpr (!KNN) {
            for_metric_of<OP>(args.q.metric, [&](auto metric_tag) {
                constexpr int MT = decltype(metric_tag)::value;
                constexpr int R = norms_read(MT);
                float *__restrict__ out = args.out + (size_t)row * (size_t)args.n + (size_t)j0;
                // A round's norms are loaded before the round ahead stores its distances: what is loaded after a store is at hand only when the
                // store has reached memory (10,000 x 10,000 rows of 38, L1, 327 us a call with that wait in every round, 316
                // without).  The first of the whole rounds stands before the loop, so that every turn of the loop has the same loads
                // and stores in flight.
                const int whole = tile_n / (F * kWave) * (F * kWave);
                RowNorms nb[F], ahead[F];
                auto load = [&](int i0, RowNorms (&into)[F]) {
                    if constexpr (R != READ_NONE) load_norms(args.b.norms + (R == READ_SECOND ? args.n : 0), R == READ_BOTH, i0, into);
                };
                auto round = [&](int i0, int next) {
                    Acc c[F];
                    load_sums(i0, c);
                    load(next, ahead);
                    __builtin_amdgcn_sched_barrier(0);
                    unsigned char *to = reinterpret_cast<unsigned char *>(out + i0);
#pragma unroll
                    for (int u = 0; u < F; ++u)
                        __builtin_nontemporal_store(distance_of<OP, MT>(args.q, c[u], unit, na0, na1, nb[u]),
                                                    reinterpret_cast<float *>(to + lane4 + u * (kWave * 4)));
                    clear_round(i0);
#pragma unroll
                    for (int u = 0; u < F; ++u) nb[u] = ahead[u];
                };
                load(0, nb);
                if (whole > 0) {
                    round(0, F * kWave < tile_n ? F * kWave : 0);
#pragma unroll 1
                    for (int i0 = F * kWave; i0 < whole; i0 += F * kWave) round(i0, i0 + F * kWave < tile_n ? i0 + F * kWave : i0);
                }
                if (whole < tile_n) {
                    Acc c[F];
                    load_sums(whole, c);
                    unsigned char *to = reinterpret_cast<unsigned char *>(out + whole);
#pragma unroll
                    for (int u = 0; u < F; ++u)
                        if (whole + u * kWave + lane < tile_n)
                            __builtin_nontemporal_store(distance_of<OP, MT>(args.q, c[u], unit, na0, na1, nb[u]),
                                                        reinterpret_cast<float *>(to + lane4 + u * (kWave * 4)));
                    clear_round(whole);
                }
            });
            clear_behind();
        } else {
            // (the metric is settled where distances are formed: an instance of all this for each of the dot product's is
            // too much to be inlined, and what it then keeps in memory cost 4,096 x 663,000 n-grams 8.5 ms for 2.0)
            const int k = args.knn_k;
            auto kth_of = [&](uint64_t sorted, int at) {
                return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(sorted >> 32), at) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sorted, at);
            };
            bound = of.bound < bound ? of.bound : bound;          // (the tightest k-th key of any list of this row so far)
            auto merge = [&]() {
                const uint64_t c = wave_sort_desc(lane < queued ? queue : kKnnUnused, lane);
                best = wave_merge_asc(c < best ? c : best, lane);
                if (lane >= k) best = kKnnUnused;
                const uint64_t now = kth_of(best, k - 1);
                bound = now < bound ? now : bound;
                queued = 0;
            };
            auto distances = [&](auto &d, const auto &c, const auto &nb) {
                for_metric_of<OP>(args.q.metric, [&](auto metric_tag) {
                    constexpr int MT = decltype(metric_tag)::value;
                    if constexpr (BOTH != (norms_read(MT) == READ_BOTH)) return;
#pragma unroll
                    for (int u = 0; u < (int)(sizeof(d) / sizeof(d[0])); ++u) {
                        d[u] = distance_of<OP, MT>(args.q, c[u], unit, na0, na1, nb[u]);
                        if constexpr (MT == MT_INNER) d[u] = 0.0f - d[u];
                    }
                });
            };
            // Whether a row that shares no column could pass: the distances of one sum grow with the row's first norm, so none is
            // nearer than the tile's row of the least.  (Correlation's do not: few_only stands for one norm a row.)
            bool few_only = false;
            if constexpr (S::kOne) {
                if (!BOTH && few.total <= 4 * F) {
                    float d[1] = {0.0f};
                    const Acc c[1] = {zero};
                    const RowNorms nb[1] = {{args.b.least[(size_t)tile * 2 + (args.norms_b != args.b.norms ? 1 : 0)], args.b.least[(size_t)tile * 2 + 1]}};
                    distances(d, c, nb);
                    few_only = d[0] == d[0] && knn_key(d[0], (int)j0) > bound;
                }
            }
            // The row's first tile goes twice through the strip: first the distances replace the sums and every lane keeps the
            // smallest of its rows' (the first of equal ones); the k-th smallest of the lanes' smallest keys bounds the
            // tile's k-th (k rows of this tile lie at or below it; at k = 32 of 1,216 rows some 44 do).
            bool first = !few_only && bound == kKnnUnused, stored = false;
            float least_d = __builtin_huge_valf();
            int least_i = -1;
            const int last0 = few_only ? 0 : (tile_n - 1) / (F * kWave) * (F * kWave);
            for (int i0 = few_only && few.total == 0 ? -1 : last0; i0 >= 0;) {
                float d[F];
                int i[F];
                if (stored) {
#pragma unroll
                    for (int u = 0; u < F; ++u) {
                        i[u] = i0 + u * kWave + lane;
                        d[u] = *lds_at<float>(strip_at + (uint32_t)min(i[u], tile_n - 1) * S::kUnit);
                        d[u] = i[u] < tile_n ? d[u] : __builtin_nanf("");
                    }
                } else if (S::kOne && few_only && few.total <= 4) {
                    // One step of entries met the row, as mostly where they are few: one lane of those that met a sum takes it and leaves its
                    // place clear.
                    if constexpr (S::kOne) {
                        Acc met[1] = {zero};
                        if ((uint32_t)(lane & 15) * 4u < few.left[0]) met[0] = S::take(strip_at + few.cell[0]);
                        i[0] = S::is_zero(met[0]) ? tile_n : (int)(few.cell[0] / S::kUnit);
                        const int64_t j = j0 + min(i[0], tile_n - 1);
                        const RowNorms nb[1] = {{args.norms_b[j], 0.0}};
                        float formed[1] = {0.0f};
                        distances(formed, met, nb);
                        d[0] = i[0] < tile_n ? formed[0] : __builtin_nanf("");
#pragma unroll
                        for (int u = 1; u < F; ++u) { d[u] = __builtin_nanf(""); i[u] = tile_n; }
                    }
                } else {
                    Acc c[F];
                    RowNorms nb[F];
                    if (S::kOne && few_only) {
                        // A few entries met the row: one lane of those that met a sum takes it and leaves its place clear
                        if constexpr (S::kOne) {
                            static_assert(F == U, "a step's entries to a place of the round");
#pragma unroll
                            for (int u = 0; u < F; ++u) {
                                c[u] = zero;
                                if (few.total > 4 * u && (uint32_t)(lane & 15) * 4u < few.left[u]) c[u] = S::take(strip_at + few.cell[u]);
                            }
#pragma unroll
                            for (int u = 0; u < F; ++u) {
                                i[u] = S::is_zero(c[u]) ? tile_n : (int)(few.cell[u] / S::kUnit);
                                nb[u] = RowNorms{0.0, 0.0};
                                if (few.total > 4 * u) nb[u].x = args.norms_b[j0 + min(i[u], tile_n - 1)];
                            }
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < F; ++u) i[u] = i0 + u * kWave + lane;
                        load_sums(i0, c);
                        load_norms(args.norms_b, BOTH, i0, nb);
                    }
                    distances(d, c, nb);
#pragma unroll
                    for (int u = 0; u < F; ++u) d[u] = i[u] < tile_n ? d[u] : __builtin_nanf("");
                }
                if (first && !stored) {
#pragma unroll
                    for (int u = F - 1; u >= 0; --u) {
                        if (i[u] < tile_n) *lds_at<float>(strip_at + (uint32_t)i[u] * S::kUnit) = d[u];
                        const bool closer = d[u] <= least_d;
                        least_d = closer ? d[u] : least_d;
                        least_i = closer ? i[u] : least_i;
                    }
                } else {
                    if (!few_only) clear_round(i0);
                    const float nearest = fminf(fminf(d[0], d[1]), fminf(d[2], d[3]));        // (ignores what is not a number)
                    if (__ballot(nearest <= float_from_order_key((uint32_t)(bound >> 32))) != 0) {
#pragma unroll 1
                        for (int u = 0; u < F; ++u) {
                            const float du = u < 2 ? (u == 0 ? d[0] : d[1]) : (u == 2 ? d[2] : d[3]);
                            const int iu = u < 2 ? (u == 0 ? i[0] : i[1]) : (u == 2 ? i[2] : i[3]);
                            if (__ballot(du <= float_from_order_key((uint32_t)(bound >> 32))) == 0) continue;
                            const uint64_t key = knn_key(du, (int)(j0 + iu));
                            bool pass = du == du && key <= bound;
                            uint64_t mask = __ballot(pass);
                            if (mask == 0) continue;
                            any = true;
                            if (queued + (int)__popcll(mask) > kWave) {
                                merge();
                                pass = pass && key <= bound;
                                mask = __ballot(pass);
                                if (mask == 0) continue;
                            }
                            // the passing lanes' keys go to the queue's next places (a permutation of the lanes)
                            const int n_pass = (int)__popcll(mask);
                            const int to = pass ? queued + (int)lane_rank_in(mask) : queued + n_pass + (int)lane_rank_in(~mask);
                            const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_permute((to & 63) << 2, (int)(uint32_t)key);
                            const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_permute((to & 63) << 2, (int)(uint32_t)(key >> 32));
                            if (lane >= queued && lane < queued + n_pass) queue = ((uint64_t)hi << 32) | lo;
                            queued += n_pass;
                        }
                    }
                }
                i0 -= F * kWave;
                if (i0 < 0) {
                    if (!first || stored) break;
                    stored = true;
                    const uint64_t least = least_i >= 0 ? knn_key(least_d, (int)(j0 + least_i)) : kKnnUnused;
                    const uint64_t kth = kth_of(wave_sort_desc(least, lane), kWave - k);
                    bound = kth < bound ? kth : bound;
                    i0 = last0;
                }
            }
            if (!few_only) clear_behind();                        // (few entries: no dense column)
            if (flush && any) {
                merge();                                          // (what is queued joins the run's list, if it has one)
                // into the row's list of this group, under a lock (two wavefronts of the workgroup may be at one row, in
                // different tiles, or of several workgroups, where the lock lies in memory); the holder waits for nothing
                const bool in_memory = lock != nullptr;
                int *const row_lock = &s_lock[row & (kMatchLocks - 1)];
                int first_lane = lane;
                asm volatile("" : "+v"(first_lane));              // (see the claim below)
                if (first_lane == 0) {
                    int spins = 0;
                    if (in_memory) {
                        while (atomicCAS(lock, 0, 1) != 0 && ++spins < kKnnLockSpins) __builtin_amdgcn_s_sleep(1);
                    } else {
                        while (atomicCAS(row_lock, 0, 1) != 0 && ++spins < kKnnLockSpins) __builtin_amdgcn_s_sleep(1);
                    }
                }
                if (in_memory) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); else __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                KnnEntry *part = args.knn_part + ((size_t)row * (size_t)args.groups + (size_t)group) * (size_t)k;
                const uint64_t theirs = lane < k ? knn_key(part[lane].d, part[lane].j) : kKnnUnused;
                const uint64_t turned = wave_reverse(theirs);
                best = wave_merge_asc(turned < best ? turned : best, lane);
                if (lane >= k) best = kKnnUnused;
                if (lane < k) part[lane] = KnnEntry{float_from_order_key((uint32_t)(best >> 32)), (int)(uint32_t)best};
                if (in_memory) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent"); else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                const uint64_t now = kth_of(best, k - 1);
                if (first_lane == 0) {
                    if (in_memory) __hip_atomic_store(lock, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else __atomic_store_n(row_lock, 0, __ATOMIC_RELAXED);
                    if (now < kKnnUnused) atomicMin(&args.knn_tau[row], (unsigned long long)now);
                }
            }
            if (flush) {
                bound = best = queue = kKnnUnused;
                queued = 0;
                any = false;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };

    // ---- the longest rows: an even share of the row to each wavefront ---------------------------------
    // (a wavefront alone would hold its workgroup up long after the others are done)
    int owner = 0;
    // A workgroup takes a (tile, row) of its group after another, the longest rows of a tile first: the slice that has
    // the longest row of all would be the last by far, and the workgroups of an XCD would drift apart in their tiles.  (1,531 x 28,301
    // ratings, Canberra, 488 -> 404 us; 4,096 x 500,000 sets, Jaccard, k-NN 8.46 -> 7.65 ms.  Sums in fp64, which are formed in the same order
    // whichever workgroup takes the row: the same ratings, cosine, 460 -> 384, KL 708 -> 510, k-NN 752 -> 584; 979 x 88,197 rows of 230,
    // cosine, 1,926 -> 1,647; 10,000 x 10,000 rows of 38 313 -> 317.)  Not with k-NN over few tiles: a row's first
    // tiles would be gone through at once, without a bound (10,000 x 10,000 rows of 38, cosine by sums in fixed point 510 -> 579 us).
    const bool taken = !KNN || args.by_xcd != 0;
    __shared__ int s_item[2];
    int item = 0, turn = 0;
    if (taken && args.m_shared > 0) {
        if (tid == 0) s_item[0] = (int)atomicAdd(&args.next[group], 1u);
        __syncthreads();
        item = s_item[0];
    }
    for (int ti = taken ? item / max(args.m_shared, 1) : 0; ti < my_tiles;) {
        const int tile = group + ti * args.groups;
        for (int at = taken ? item - ti * args.m_shared : slice; at < args.m_shared; at += args.slices) {
            int next = 0;
            if (taken && tid == 0) next = (int)atomicAdd(&args.next[group], 1u);
            const MatchRow rw = args.rows[at];
            const int row = wave_uniform(rw.row), len = wave_uniform(rw.len);
            const int begin = (int)((int64_t)len * wave / nw), end = (int)((int64_t)len * (wave + 1) / nw);
            Entries x = load_entries(rw.start + begin, end - begin, 0);
            const Scale scale = scale_of<OP>(wave_uniform(load_scale(row)), len);
            // Sums that come out the same in any order go to one strip, the next row's to the next one: one wait a row.  Others are
            // formed strip by strip and the strips summed in a fixed order.
            const uint32_t owners_at = (uint32_t)wave_uniform((int)(strips_at + (uint32_t)owner * strip_bytes));
            Few few{};
            for (int e0 = 0; e0 < end - begin; e0 += kWave) {
                const Lists y = load_lists(tile, x);
                x = load_entries(rw.start + begin, end - begin, e0 + kWave);
                walk_lists(tile, y, scale, S::kAnyOrder ? owners_at : strip_at, few);
            }
            few.total = 4 * U + 1;
            if (taken && tid == 0) s_item[turn ^ 1] = next;
            __syncthreads();
            if constexpr (!S::kAnyOrder) {
                for (int i = tid; i < T; i += nw * kWave) {
                    Acc sum = S::get(strips_at, plane, (uint32_t)i);
                    S::put(strips_at, plane, (uint32_t)i, zero);
#pragma unroll
                    for (int w = 1; w < nw; ++w) {
                        S::combine(sum, S::get(strips_at + (uint32_t)w * strip_bytes, plane, (uint32_t)i));
                        S::put(strips_at + (uint32_t)w * strip_bytes, plane, (uint32_t)i, zero);
                    }
                    S::put(owners_at, plane, (uint32_t)i, sum);
                }
                __syncthreads();
            }
            if constexpr (OP == OP_CHEB) {
                finish_ranked(tile, row, rw.start, len, owners_at, wave * kWave, nw * kWave);
            } else if constexpr (S::kAnyOrder && !KNN) {
                // (the distances by all wavefronts: by one they held the next row up; 10,000 x 10,000 rows of 38, L1, with the one strip 313 -> 298 us a call)
                const RowOf of = load_row(row);
                const int64_t j0 = (int64_t)tile * T;
                const int tile_n = (int)min((int64_t)T, args.n - j0);
                const double unit = (OP == OP_L1 ? -2.0 : -1.0) * scale.unit;
                for_metric_of<OP>(args.q.metric, [&](auto metric_tag) {
                    constexpr int MT = decltype(metric_tag)::value, R = norms_read(MT);
                    float *__restrict__ out = args.out + (size_t)row * (size_t)args.n + (size_t)j0;
                    for (int i = tid; i < T; i += nw * kWave) {
                        if (i < tile_n) {
                            RowNorms nb{0.0, 0.0};
                            if (R != READ_NONE) nb.x = args.b.norms[(R == READ_SECOND ? args.n : 0) + j0 + i];
                            if (R == READ_BOTH) nb.y = args.b.norms[args.n + j0 + i];
                            __builtin_nontemporal_store(distance_of<OP, MT>(args.q, S::get(owners_at, plane, (uint32_t)i), unit, of.na0, of.na1, nb), out + i);
                        }
                        S::put(owners_at, plane, (uint32_t)i, zero);
                    }
                });
            } else if (wave == owner) {
                if constexpr (OP != OP_CHEB) finish(tile, row, load_row(row), scale, few, true, taken ? reinterpret_cast<int *>(args.next) + args.groups + group * kMatchRowLocks + (row & (kMatchRowLocks - 1)) : nullptr);
            }
            owner = owner + 1 < nw ? owner + 1 : 0;
            if (taken) {
                turn ^= 1;
                item = s_item[turn];
                break;
            }
        }
        ti = taken ? (args.m_shared > 0 ? item / args.m_shared : my_tiles) : ti + 1;
    }
    if (taken && !KNN && args.m_shared > 0) __syncthreads();          // (a strip may be another wavefront's to clear)

    // ---- the other rows: one wavefront each, no waiting for one another ------------------------------
    const int rows_here = args.m - args.m_shared > slice ? (args.m - args.m_shared - slice + args.slices - 1) / args.slices : 0;
    if (rows_here == 0) return;
    // A wavefront takes a row and a run of tiles after another and goes through their batches of 64 entries as one
    // stream: while the lists of one batch are walked, the list bounds of the next one and the entries of
    // the one after that are on their way.
    struct Place { int tile, row, len, e0, tiles; int64_t start; int scale; };       // e0: of the batch; tiles: left of the run; row < 0: there is none
    auto claim = [&]() {
        // (the lane number is hidden from the compiler here: were `lane == 0` also to close the loop's body,
        // it would thread the two tests together and let the other lanes round the loop ahead of lane 0)
        int at = 0, claimer = lane;
        asm volatile("" : "+v"(claimer));
        if (claimer == 0) at = atomicAdd(&s_next, 1);
        at = wave_uniform(at);
        const int run = at / rows_here, ti = run * args.run;
        Place p{0, -1, 0, 0, 0, 0, 0};
        if (ti < my_tiles) {
            const MatchRow rw = args.rows[args.m_shared + slice + (at - run * rows_here) * args.slices];
            p.tile = group + ti * args.groups;
            p.tiles = min(args.run, my_tiles - ti);
            p.row = wave_uniform(rw.row);
            p.len = wave_uniform(rw.len);
            p.start = rw.start;
            p.scale = load_scale(p.row);
        }
        return p;
    };
    Place ahead = claim();                       // where the stream goes on once the run below is through
    auto advance = [&](const Place &p) {         // the batch after p
        Place q = p;
        q.e0 += kWave;
        if (q.row >= 0 && q.e0 >= q.len) {
            if (q.tiles > 1) {
                q.e0 = 0;
                --q.tiles;
                q.tile += args.groups;
            } else {
                q = ahead;
                ahead = claim();
            }
        }
        return q;
    };
    Place p0 = ahead;
    ahead = claim();
    Entries x = load_entries(p0.start, p0.len, 0);
    Place p1 = advance(p0);
    Lists y = load_lists(p0.tile, x);
    x = load_entries(p1.start, p1.len, p1.e0);
    Few few{};
    while (p0.row >= 0) {
        const Place p2 = advance(p1);
        const Lists y1 = load_lists(p1.tile, x);
        x = load_entries(p2.start, p2.len, p2.e0);
        const RowOf of = load_row(p0.row);
        const Scale scale = scale_of<OP>(wave_uniform(p0.scale), p0.len);
        walk_lists(p0.tile, y, scale, strip_at, few);
        if (p0.e0 + kWave >= p0.len) {
            if constexpr (OP == OP_CHEB) finish_ranked(p0.tile, p0.row, p0.start, p0.len, strip_at, 0, kWave);
            else finish(p0.tile, p0.row, of, scale, few, p0.tiles <= 1, nullptr);
            few.total = 0;
        } else if (KNN) {
            few.total += 4 * U + 1;                             // (the entries of several batches are not at hand together)
        }
        p0 = p1;
        p1 = p2;
        y = y1;
    }
}

// Raises a kernel's LDS limit, once per device (`allowed`: the instance's own).
constexpr int kMatchDevices = 64;
template <typename Kernel> static hipError_t allow_lds(Kernel kern, std::atomic<uint32_t> (&allowed)[kMatchDevices], uint32_t bytes,
                                                            uint32_t static_bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool known = dev >= 0 && dev < kMatchDevices;
    if (known && allowed[dev].load(std::memory_order_acquire) >= bytes) return hipSuccess;
    // to the most any launch may ask for, so that no two launches set it against each other
    const uint32_t want = std::max<uint32_t>(bytes, 160u * 1024u - static_bytes);
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)want);
    if (e == hipSuccess) {
        if (known) allowed[dev].store(want, std::memory_order_release);
        return e;
    }
    // a device with less LDS: ask for what this launch needs
    (void)hipGetLastError();
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int OP, bool KNN, bool BOTH> static hipError_t launch_match_op(hipStream_t st, const MatchArgs &args, uint32_t lds_bytes) {
    auto kern = spd_match_kernel<OP, KNN, BOTH>;
    static std::atomic<uint32_t> allowed[kMatchDevices];
    hipError_t e = allow_lds(kern, allowed, lds_bytes, (uint32_t)match_static_lds(match_cell_bytes(OP)));
    if (e != hipSuccess) return e;
    const int64_t groups = args.by_xcd ? (args.groups + 7) / 8 * 8 : args.groups;
    hipLaunchKernelGGL(kern, dim3((unsigned)(groups * args.slices)), dim3((unsigned)(match_waves(match_cell_bytes(OP)) * kWave)), lds_bytes, st, args);
    return hipGetLastError();
}
template <int OP> static hipError_t launch_match_either(hipStream_t st, const MatchArgs &args, uint32_t lds_bytes) {
    if (args.knn_k <= 0) return launch_match_op<OP, false, false>(st, args, lds_bytes);
    if constexpr (OP == OP_DOT) {
        if (args.q.metric == MT_CORRELATION) return launch_match_op<OP, true, true>(st, args, lds_bytes);
    }
    return launch_match_op<OP, true, OP == OP_MINK || OP == OP_MINK_ANY>(st, args, lds_bytes);
}

}  // namespace spd
