// The column lists of B (a transpose per tile of rows), row norms, and the dispatch of the column-list
// kernel to its products.
#include <cmath>

#include "spd_match_impl.h"

namespace spd {

// ------------------------------------------------------------------------------------
// row pointers that the host has not seen yet
// ------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) spd_match_look_at_rows_kernel(const int64_t *__restrict__ a, int64_t m, int64_t a_nnz,
                                                                     const int64_t *__restrict__ b, int64_t n, int64_t b_nnz, uint32_t *word,
                                                                     uint32_t malformed) {
    const int64_t all = m + 1 + (b ? n + 1 : 0), step = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < all; i += step) {
        const bool of_a = i <= m;
        const int64_t *p = of_a ? a : b;
        const int64_t r = of_a ? i : i - (m + 1), rows = of_a ? m : n, nnz = of_a ? a_nnz : b_nnz;
        const int64_t at = p[r], before = r > 0 ? p[r - 1] : 0;
        if ((r == 0 && at != 0) || at < before || (r == rows && at != nnz)) __atomic_store_n(word, malformed, __ATOMIC_RELAXED);
    }
}
hipError_t launch_match_look_at_rows(hipStream_t st, const int64_t *a, int64_t m, int64_t a_nnz, const int64_t *b, int64_t n, int64_t b_nnz,
                                     uint32_t *word, uint32_t malformed) {
    const int64_t all = m + 1 + (b ? n + 1 : 0);
    hipLaunchKernelGGL(spd_match_look_at_rows_kernel, dim3((unsigned)std::min<int64_t>(4096, (all + 255) / 256)), dim3(256), 0, st, a, m, a_nnz, b, n,
                       b_nnz, word, malformed);
    return hipGetLastError();
}
__device__ __forceinline__ bool rows_malformed(const RowsVerdict &seen) { return seen.word && *seen.word == seen.malformed; }

// ------------------------------------------------------------------------------------
// row norms.  The sums of a row: entries from `from` on, `stride` apart, U of a lane in flight.
// ------------------------------------------------------------------------------------
struct NormSums { double s0, s1; float most, least; };
struct NormArgs {
    const int64_t *indptr;
    const float *values;
    int64_t n_rows, nnz;
    int metric, transform, norm;
    float p;
    double k;
    RowsVerdict seen;
    double *norms;
    int16_t *scales;
};
template <bool SCALES> __device__ __forceinline__ void norm_add(const NormArgs &a, float v, NormSums &x) {          // (v = 0 adds nothing)
    const float t = transform_value(a.transform, v);
    norm_accumulate(a.norm, t, a.p, x.s0, x.s1);
    if constexpr (SCALES) {
        x.most = fmaxf(x.most, fabsf(t));
        x.least = t != 0.0f ? fminf(x.least, fabsf(t)) : x.least;
    }
}
template <bool SCALES, int U> __device__ __forceinline__ void norm_sums(const NormArgs &a, int64_t from, int64_t end, int stride, NormSums &x) {
    for (int64_t e = from; e < end; e += U * stride) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = e + u * stride < end ? a.values[e + u * stride] : 0.0f;
#pragma unroll
        for (int u = 0; u < U; ++u) norm_add<SCALES>(a, v[u], x);
    }
}
// Over the lanes of a wavefront, to its last one.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_add(double v) {
    return v + __hiloint2double(dpp_or_zero<CTRL, ROWS>(__double2hiint(v)), dpp_or_zero<CTRL, ROWS>(__double2loint(v)));
}
__device__ __forceinline__ double wave_sum_last(double v) {
    v = dpp_add<0x111, 0xf>(v);                             // row_shr:1, 2, 4, 8; row_bcast:15, row_bcast:31
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    return dpp_add<0x143, 0xc>(v);
}
template <bool SCALES> __device__ __forceinline__ void norm_reduce_last(int norm, NormSums &x) {
    x.s0 = wave_sum_last(x.s0);
    if (norm == NORM_SUM_SUMSQ || norm == NORM_SUM_POW || norm >= NORM_SEMI) x.s1 = wave_sum_last(x.s1);
    if constexpr (SCALES) {                                  // (magnitudes: their bits are in their order)
        x.most = __int_as_float(wave_scan_max(__float_as_int(x.most)));
        x.least = __int_as_float(INT32_MAX - wave_scan_max(INT32_MAX - __float_as_int(x.least)));
    }
}
template <bool SCALES> __device__ __forceinline__ void norm_write(const NormArgs &a, int64_t r, const NormSums &x) {
    double d0, d1;
    norm_derive(a.metric, a.k, x.s0, x.s1, d0, d1);
    if constexpr (SCALES) a.scales[r] = (int16_t)(a.metric == MT_CANBERRA ? match_wild(x.least, x.most) : match_scale(x.most, x.s0));
    a.norms[r] = d0;
    a.norms[a.n_rows + r] = d1;
}
// A row by all 256 lanes of a workgroup: its wavefronts' sums in a fixed order.  (All of them come here, and wait for one another.)
template <bool SCALES> __device__ __forceinline__ void norm_by_all(const NormArgs &a, int64_t r, NormSums (&s_part)[256 / kWave]) {
    const int tid = (int)threadIdx.x;
    const int64_t begin = clamp_i64(a.indptr[r], 0, a.nnz), end = clamp_i64(a.indptr[r + 1], begin, a.nnz);
    NormSums x{0.0, 0.0, 0.0f, 1.0f};
    norm_sums<SCALES, 8>(a, begin + tid, end, 256, x);
    norm_reduce_last<SCALES>(a.norm, x);
    if (tid % kWave == kWave - 1) s_part[tid / kWave] = x;
    __syncthreads();
    if (tid == 0) {
        NormSums all{0.0, 0.0, 0.0f, 1.0f};
#pragma unroll
        for (int w = 0; w < 256 / kWave; ++w) {
            all.s0 += s_part[w].s0;
            all.s1 += s_part[w].s1;
            all.most = fmaxf(all.most, s_part[w].most);
            all.least = fminf(all.least, s_part[w].least);
        }
        norm_write<SCALES>(a, r, all);
    }
    __syncthreads();
}
// A workgroup to the row.
template <bool SCALES> __global__ void __launch_bounds__(256) spd_match_norms_kernel(const NormArgs a) {
    if (rows_malformed(a.seen)) return;
    __shared__ NormSums s_part[256 / kWave];
    norm_by_all<SCALES>(a, blockIdx.x, s_part);
}
// A wavefront to `per_wave` rows that follow one another: the next one's entries are on their way while one is summed, and the numbers
// that distances read are derived for all of them together, a row to a lane (a wavefront each, with sums through LDS and square roots for one lane of
// it, 300,000 rows of 230 entries: 157 us, 109 now).  Rows of more than 4,096 entries wait for the whole workgroup, one after
// the other (500,000 rows of 1 to 50,000 entries: 332 us while a wavefront went through the longest alone, 250, 219 now).
constexpr int kNormRows = 8;
template <bool SCALES> __global__ void __launch_bounds__(256) spd_match_norms_rows_kernel(const NormArgs a, int per_wave) {
    if (rows_malformed(a.seen)) return;
    constexpr int kLong = 64 * kWave;
    __shared__ NormSums s_part[256 / kWave];
    __shared__ int s_long[256 / kWave * kNormRows], s_longs;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6);
    const int64_t block_first = (int64_t)blockIdx.x * (256 / kWave) * per_wave, first = block_first + (int64_t)wave * per_wave;
    const int rows = (int)max((int64_t)0, min((int64_t)per_wave, a.n_rows - first));
    if (tid == 0) s_longs = 0;
    __syncthreads();
    // lane i: where row i begins; the last one's end with the lane behind
    const int64_t begins = lane <= rows && first <= a.n_rows ? clamp_i64(a.indptr[first + min(lane, rows)], 0, a.nnz) : 0;
    auto bound = [&](int i) {
        return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(begins >> 32), i) << 32) | (uint32_t)__builtin_amdgcn_readlane((int)begins, i));
    };
    auto fetch = [&](int i, int64_t &begin, int64_t &end, float (&v)[4]) {
        begin = bound(i);
        end = max(begin, bound(i + 1));
        if (end - begin > kLong) {
            if (lane == 0) s_long[atomicAdd(&s_longs, 1)] = wave * per_wave + i;
            end = begin;
        }
        const int64_t e = begin + lane;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = e + u * kWave < end ? a.values[e + u * kWave] : 0.0f;
    };
    NormSums mine{0.0, 0.0, 0.0f, 1.0f};
    float cur[4], ahead[4];
    int64_t begin = 0, end = 0;
    if (rows > 0) fetch(0, begin, end, cur);
    for (int i = 0; i < rows; ++i) {
        int64_t begin1 = 0, end1 = 0;
        if (i + 1 < rows) fetch(i + 1, begin1, end1, ahead);
        NormSums x{0.0, 0.0, 0.0f, 1.0f};
#pragma unroll
        for (int u = 0; u < 4; ++u) norm_add<SCALES>(a, cur[u], x);
        norm_sums<SCALES, 4>(a, begin + 4 * kWave + lane, end, kWave, x);
        norm_reduce_last<SCALES>(a.norm, x);
        auto last = [&](double v) { return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63), __builtin_amdgcn_readlane(__double2loint(v), 63)); };
        auto last_of = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)); };
        // (the last lane's sums are read by all lanes: within the branch they would not be formed there)
        const NormSums row{last(x.s0), last(x.s1), last_of(x.most), last_of(x.least)};
        if (lane == i) mine = row;
        begin = begin1;
        end = end1;
#pragma unroll
        for (int u = 0; u < 4; ++u) cur[u] = ahead[u];
    }
    const int64_t behind = clamp_i64(__shfl_down((long long)begins, 1), begins, INT64_MAX);
    if (lane < rows && behind - begins <= kLong) norm_write<SCALES>(a, first + lane, mine);
    __syncthreads();
    const int longs = s_longs;
    for (int at = 0; at < longs; ++at) norm_by_all<SCALES>(a, block_first + s_long[at], s_part);
}
// Four lanes to a row of few entries; rows of more than 256 wait for the whole workgroup.
template <bool SCALES> __global__ void __launch_bounds__(256) spd_match_norms_short_kernel(const NormArgs a) {
    if (rows_malformed(a.seen)) return;
    constexpr int G = 4, kRows = 256 / G, kLong = 64 * G;
    __shared__ NormSums s_part[256 / kWave];
    __shared__ int s_long[kRows], s_longs;
    const int tid = (int)threadIdx.x, sub = tid % G;
    const int64_t row0 = (int64_t)blockIdx.x * kRows, row = row0 + tid / G;
    int64_t begin = 0, end = 0;
    if (row < a.n_rows) {
        begin = clamp_i64(a.indptr[row], 0, a.nnz);
        end = clamp_i64(a.indptr[row + 1], begin, a.nnz);
    }
    if (tid == 0) s_longs = 0;
    __syncthreads();
    const bool is_long = end - begin > kLong;
    if (is_long && sub == 0) s_long[atomicAdd(&s_longs, 1)] = tid / G;
    NormSums x{0.0, 0.0, 0.0f, 1.0f};
    norm_sums<SCALES, 4>(a, begin + sub, is_long ? begin : end, G, x);
#pragma unroll
    for (int d = G / 2; d >= 1; d >>= 1) {
        x.s0 += __shfl_xor(x.s0, d);
        x.s1 += __shfl_xor(x.s1, d);
        if constexpr (SCALES) {
            x.most = fmaxf(x.most, __shfl_xor(x.most, d));
            x.least = fminf(x.least, __shfl_xor(x.least, d));
        }
    }
    if (row < a.n_rows && !is_long && sub == 0) norm_write<SCALES>(a, row, x);
    __syncthreads();
    const int longs = s_longs;
    for (int at = 0; at < longs; ++at) norm_by_all<SCALES>(a, row0 + s_long[at], s_part);
}

// ------------------------------------------------------------------------------------
// Chebyshev: every entry's rank by magnitude in its row, and the row's largest magnitudes.  A wavefront to the row.  The 32nd largest
// of what the lanes' largest entries are bounds the row's 32nd; what reaches it is queued and merged with the 64 largest so far when 64
// are waiting, so that a long row is sorted two or three times and not for every 64 entries (7,777 rows of 37, the longest
// 2,000, and 3,333 of them, a launch each, sorted for every 64 entries: 28 us each; 17 for both now).
// ------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) spd_match_ranks_kernel(const RankedRows first, const RankedRows second, const RowsVerdict seen) {
    if (rows_malformed(seen)) return;
    const int lane = (int)threadIdx.x & 63;
    const int64_t at = (int64_t)blockIdx.x * 4 + wave_uniform((int)threadIdx.x >> 6);
    const bool is_first = at < first.n_rows;
    const RankedRows &o = is_first ? first : second;
    const int64_t row = is_first ? at : at - first.n_rows;
    if (row >= o.n_rows) return;
    const int64_t begin = clamp_i64(o.indptr[row], 0, o.nnz), end = clamp_i64(o.indptr[row + 1], begin, o.nnz);
    constexpr uint64_t kNone = ~0ull;                              // (keys ascend with falling magnitudes; then by place)
    auto key_of = [&](int64_t e, float v) { return e < end && v != 0.0f ? ((uint64_t)~__float_as_uint(fabsf(v)) << 32) | (uint32_t)(e - begin) : kNone; };
    auto kth = [&](uint64_t sorted) {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(sorted >> 32), kRanks - 1) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sorted, kRanks - 1);
    };
    uint64_t best = kNone, bar = kNone, queue = kNone;
    int queued = 0;
    auto merge = [&]() {
        const uint64_t c = wave_sort_desc(lane < queued ? queue : kNone, lane);
        best = wave_merge_asc(c < best ? c : best, lane);
        const uint64_t now = kth(best);
        bar = now < bar ? now : bar;
        queued = 0;
    };
    if (end - begin > 2 * kWave) {
        uint64_t mine = kNone;
        for (int64_t e0 = begin + lane; e0 < end; e0 += 4 * kWave) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = e0 + u * kWave < end ? o.values[e0 + u * kWave] : 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t key = key_of(e0 + u * kWave, v[u]);
                mine = key < mine ? key : mine;
            }
        }
        bar = kth(wave_merge_asc(wave_sort_desc(mine, lane), lane));
    }
    for (int64_t e0 = begin; e0 < end; e0 += 4 * kWave) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = e0 + u * kWave + lane < end ? o.values[e0 + u * kWave + lane] : 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t e = e0 + u * kWave + lane;
            if (e < end) o.ranks[e] = 255;
            const uint64_t key = key_of(e, v[u]);
            bool pass = key != kNone && key <= bar;
            uint64_t mask = __ballot(pass);
            if (mask == 0) continue;
            if (queued + (int)__popcll(mask) > kWave) {
                merge();
                pass = pass && key <= bar;
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
    merge();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");          // (an entry's rank replaces what another lane wrote there)
    if (lane < kRanks) {
        if (best != kNone) o.ranks[begin + (int64_t)(uint32_t)best] = (uint8_t)lane;
        o.tops[o.by_row ? row * kRanks + lane : (int64_t)lane * o.n_rows + row] = best != kNone ? __uint_as_float(~(uint32_t)(best >> 32)) : 0.0f;
    }
}
static int64_t match_ranks_grid(int64_t rows) { return (rows + 3) / 4; }
hipError_t launch_match_ranks(hipStream_t st, const RankedRows &first, const RankedRows &second, const RowsVerdict &seen) {
    const int64_t rows = first.n_rows + second.n_rows;
    if (rows <= 0) return hipSuccess;
    hipLaunchKernelGGL(spd_match_ranks_kernel, dim3((unsigned)match_ranks_grid(rows)), dim3(256), 0, st, first, second, seen);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------
// B: a tile's entries by column.  A workgroup takes a run of column blocks of one tile.  The rows ascend in
// their columns, so a row's entries of a block are a stretch of it, whose end a lane to the row searches from where the block before ended.  The
// stretches are lined up one behind the other, and the lanes take their entries as they stand in this line, every entry once: it is counted, the
// count before it is its place in its column's list, and it waits in registers for the lists' starts.  Counters and the block's
// piece of the lists lie in LDS and the piece is written out whole.  (Counters in memory that eight XCDs share
// run at 2.6e10 atomics a second: 300,000 rows of 230 entries took 7.1 ms; one workgroup per tile with
// scattered 8-byte stores 1.74 ms; a few lanes to every row, which went through its stretch twice, 1.06, with 240 vector instructions an entry.)
// The order inside a list is whatever the wavefronts make it: no sum depends on it, because a row of B appears in a list at most once.
// ------------------------------------------------------------------------------------
// Two workgroups to a compute unit, as far as LDS and registers go: what a block takes is mostly waiting, for one load after the other and at barriers.  (With one
// of 1,024 lanes / two of 512, when they were compared, us: 10,000 rows of 38 46 / 23, 7,777 of them 41 / 20, 28,301 ratings 95 / 72, 663,000 n-grams 96 / 44, 300,000
// rows of 230 936 / 850, 65,536 of 1,820 917 / 805, 500,000 sets 895 / 860; a few lanes to every row 49, 36, 131, 81, 1,096, 972, 1,582.)
constexpr int kBuildThreads = 512;
constexpr int build_rows(int tile_rows) { return tile_rows <= kBuildThreads ? 1 : (tile_rows <= 3 * kBuildThreads ? 3 : 5); }          // of a lane
// Entries that a lane holds: fewer of a lane with more rows, whose ends take registers too, but where half as many again make blocks of twice the columns.  (All instances
// take the 128 registers that four wavefronts to a SIMD leave: with 16 entries and three rows 6 are spilled, with 24 52.)
constexpr int kBuildHeld = 16, kBuildHeldMore = 24;
constexpr int build_held(int rows) { return rows == 1 ? kBuildHeldMore : kBuildHeld; }
constexpr int kBuildProbe = 8;                                              // entries that a lane looks at together
// A block of more entries than the lanes hold is gone through twice, so many at a time.
constexpr uint32_t kBuildWindow = 8192;
constexpr int kAgain = 4;                                                   // ... and of a lane's so many in flight together

// (a norm that is not a number is the least: the distances turn a sum that is not a number into 0)
__device__ __forceinline__ bool less_norm(double a, double than) { return !(a >= than) && than == than; }
// The norms of a tile's row of the least first norm, by a whole workgroup.
__device__ __forceinline__ void tile_least(const double *__restrict__ norms, const double *__restrict__ second, int rows, double *__restrict__ least, double (*s_least)[2]) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double d0 = __builtin_huge_val(), d1 = 0.0;
    for (int r = tid; r < rows; r += kBuildThreads) {
        const double nb = norms[r];
        if (less_norm(nb, d0)) { d0 = nb; d1 = second[r]; }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const double o0 = __shfl_xor(d0, d), o1 = __shfl_xor(d1, d);
        if (less_norm(o0, d0)) { d0 = o0; d1 = o1; }
    }
    if (lane == 0) { s_least[wave][0] = d0; s_least[wave][1] = d1; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kBuildThreads / kWave; ++w)
            if (less_norm(s_least[w][0], d0)) { d0 = s_least[w][0]; d1 = s_least[w][1]; }
        least[0] = d0;
        least[1] = d1;
    }
}

// Lists that follow one another: entries before the first that begins at a line (kMatchLine), and from there on (-1: none does).
struct Stretch { uint32_t before; int32_t after; };
__device__ __forceinline__ uint32_t to_line(uint32_t at) { return (at + kMatchLine - 1u) & ~(kMatchLine - 1u); }
__device__ __forceinline__ uint32_t end_of(uint32_t at, const Stretch &x) { return x.after < 0 ? at + x.before : to_line(at + x.before) + (uint32_t)x.after; }
__device__ __forceinline__ Stretch then(const Stretch &x, const Stretch &y) {
    if (x.after < 0) return Stretch{x.before + y.before, y.after};
    return Stretch{x.before, (int32_t)end_of((uint32_t)x.after, y)};
}

// Sixteen bytes at once.
struct __align__(16) Eight { uint16_t v[8]; };
struct __align__(16) Four { float v[4]; };

template <int R, int K>
__global__ void __launch_bounds__(kBuildThreads, 4) spd_match_build_kernel(const int64_t *__restrict__ indptr, const int32_t *__restrict__ indices,
                                                                        const float *__restrict__ values, int64_t n_rows, int64_t nnz,
                                                                        uint32_t most_cols, MatchB b, uint32_t blocks_per_wg, uint32_t wgs, int unit,
                                                                        int transform, bool with_values, bool positive, const RowsVerdict seen) {
    if (rows_malformed(seen)) return;
    constexpr int nw = kBuildThreads / kWave;
    extern __shared__ __align__(16) unsigned char s_raw[];
    __shared__ uint32_t s_wave[nw], s_second[nw], s_lens[R][nw], s_first[nw], s_dense[kBuildDense];
    __shared__ double s_least[nw][2];
    const MatchShape &shape = b.shape;
    const uint8_t *const ranks = b.ranks;
    const uint32_t cols = b.cols ? min(*b.cols, most_cols) : most_cols;
    const uint32_t block_cols = 1u << shape.block_shift, blocks = min((uint32_t)shape.blocks, (cols + block_cols - 1u) >> shape.block_shift);
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6);
    const int T = shape.tile_rows;
    // Workgroups go round the eight XCDs in turn: an XCD takes an eighth of the (tile, part)s that follow one another, so that the
    // lines which two blocks of a row share come from its L2 (300,000 rows of 230 entries: misses 40 -> 21 million).  Not where they are hardly more
    // than the 256 compute units: in the order of the grid the few that take a second
    // turn are of the last tile, which is short (KL, 260 workgroups for 10,000 rows, 41 -> 32 us; L1, 360 of them, 46 in either order, and
    // the walk after it 2 us longer).
    const uint32_t of_xcd = (gridDim.x + 7u) >> 3, at_wg = gridDim.x > 288u ? (blockIdx.x & 7u) * of_xcd + (blockIdx.x >> 3) : blockIdx.x;
    const int tile = (int)(at_wg / wgs), part = (int)(at_wg % wgs);
    if (tile >= shape.n_tiles) return;
    const int64_t j0 = (int64_t)tile * T;
    const int rows = (int)min((int64_t)T, n_rows - j0);
    const int64_t row_first = clamp_i64(indptr[j0], 0, nnz);             // of the rows' entries
    const int64_t first = shape.room_of(row_first) + tile * shape.tile_extra;            // of the tile's lists
    const int64_t list_end = shape.list_entries(nnz) - kMatchSpare;
    float *s_value = reinterpret_cast<float *>(s_raw);                              // stage entries, a multiple of 8
    uint16_t *s_row = reinterpret_cast<uint16_t *>(s_value + shape.stage);
    uint32_t *s_count = reinterpret_cast<uint32_t *>(s_row + shape.stage);    // block_cols counters, a multiple of 4
    uint32_t *s_delta = s_count + block_cols;                                 // from a place in the line of stretches to the row's entry there
    uint32_t *ptr = b.ptr + (size_t)tile * (size_t)shape.ptr_stride;
    // (positions are below 2^29: the tile's entries by byte offsets of 32 bits)
    const unsigned char *const tile_columns = reinterpret_cast<const unsigned char *>(indices + row_first);
    const unsigned char *const tile_values = reinterpret_cast<const unsigned char *>(values + row_first);
    const uint8_t *const tile_ranks = ranks + row_first;
    if (part == 0 && b.least) tile_least(b.norms + j0, b.norms + n_rows + j0, rows, b.least + (size_t)tile * 2, s_least);
    const uint32_t block_first = (uint32_t)part * blocks_per_wg;
    const uint32_t block_last = min(block_first + blocks_per_wg, blocks);
    if (block_first >= block_last) return;
    // Rows tid, tid + kBuildThreads, ...: where the block's entries begin, and where the row ends.
    uint32_t cur[R], row_end[R];
    // The first entry from `at` on, where column `from_col` begins, whose column is not below `target`, of all the lane's rows at once: by the entries round where it should lie, then where these
    // say it should, then by halves.
    auto find = [&](uint32_t (&at)[R], uint32_t target, uint32_t from_col) {
        constexpr int N = kBuildProbe;
        struct __attribute__((packed, aligned(4))) Probe { uint32_t c[N]; };
        if (nnz < N) {
#pragma unroll
            for (int j = 0; j < R; ++j)
                while (at[j] < row_end[j] && (uint32_t)indices[row_first + at[j]] < target) ++at[j];
            return;
        }
        const int last = (int)min(nnz - N - row_first, (int64_t)INT32_MAX);          // (may lie before the tile)
        uint32_t hi[R];
        int guess[R];
        float per_col[R];                          // entries to a column
        const float share = 1.0f / (float)(cols - from_col), ahead = (float)(target - from_col);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            hi[j] = row_end[j];
            per_col[j] = (float)(hi[j] - at[j]) * share;
            guess[j] = (int)at[j] + (int)(per_col[j] * ahead);
        }
        for (int round = 0;; ++round) {
            bool open = false;
            Probe x[R];
            int from[R];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (at[j] >= hi[j]) continue;
                from[j] = min(max((int)at[j], min(guess[j] - N / 2, (int)hi[j] - N)), last);
                x[j] = *reinterpret_cast<const Probe *>(tile_columns + (int64_t)from[j] * 4);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (at[j] >= hi[j]) continue;
                int less = 0;
#pragma unroll
                for (int u = 0; u < N; ++u) less += from[j] + u < (int)at[j] || (from[j] + u < (int)hi[j] && x[j].c[u] < target) ? 1 : 0;
                if (less == 0) {
                    hi[j] = (uint32_t)from[j];
                    guess[j] = from[j] - 1 - (int)((float)(x[j].c[0] - target) * per_col[j]);
                } else if (less == N) {
                    at[j] = min((uint32_t)(from[j] + N), hi[j]);
                    guess[j] = from[j] + N + (int)((float)(target - x[j].c[N - 1]) * per_col[j]);
                } else {
                    at[j] = hi[j] = (uint32_t)(from[j] + less);
                }
                if (round >= 2) guess[j] = (int)((at[j] + hi[j]) >> 1);
                open |= at[j] < hi[j];
            }
            if (__ballot(open) == 0) break;
        }
    };
    uint32_t before = 0u;                             // entries of the columns before the block
    {
        const uint32_t c_first = block_first * block_cols;
        uint32_t mine = 0u, begin[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int r = tid + j * kBuildThreads;
            begin[j] = row_end[j] = 0u;
            if (r < rows) {
                begin[j] = (uint32_t)(clamp_i64(indptr[j0 + r], row_first, nnz) - row_first);
                row_end[j] = max(begin[j], (uint32_t)(clamp_i64(indptr[j0 + r + 1], row_first, nnz) - row_first));
            }
            cur[j] = begin[j];
        }
        if (block_first > 0u) find(cur, c_first, 0u);
#pragma unroll
        for (int j = 0; j < R; ++j) mine += cur[j] - begin[j];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mine += (uint32_t)__shfl_xor((int)mine, d);
        if (lane == 0) s_wave[wave] = mine;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < nw; ++w) before += s_wave[w];
    }
    // Where a block's piece begins in the tile's lists, `entries` before it.
    auto piece_of = [&](uint32_t entries, uint32_t block) {
        return (uint32_t)shape.room_of(entries) + (uint32_t)shape.dense_before((int32_t)block) * (uint32_t)shape.dense_room();
    };
    // Marks of the line's places where a row's stretch begins (its row, from 1 on), in LDS that the piece takes later: what lanes hold, or a window
    // behind the places that are staged then.
    uint16_t *const marks_behind = reinterpret_cast<uint16_t *>(s_value + (shape.stage - min(kBuildWindow, shape.stage) / 64u * 32u));
    const uint32_t held = min((uint32_t)(K * kBuildThreads), shape.stage * 2u) & ~63u, window = min(kBuildWindow, shape.stage) & ~63u;
    for (uint32_t block = block_first; block < block_last; ++block) {
        const uint32_t c0 = block * block_cols, range = min(block_cols, cols - c0);
        for (uint32_t i = 4u * (uint32_t)tid; i < block_cols; i += 4u * kBuildThreads) *reinterpret_cast<uint4 *>(s_count + i) = uint4{0u, 0u, 0u, 0u};
        uint32_t next[R], off[R], entries = 0u;
#pragma unroll
        for (int j = 0; j < R; ++j) next[j] = block + 1u < blocks ? cur[j] : row_end[j];
        if (block + 1u < blocks) find(next, c0 + block_cols, c0);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (j * kBuildThreads >= rows) continue;
            const int incl = wave_scan_add((int)(next[j] - cur[j]));
            if (lane == 63) s_lens[j][wave] = (uint32_t)incl;
            off[j] = (uint32_t)incl - (next[j] - cur[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (j * kBuildThreads >= rows) continue;
            off[j] += entries;
#pragma unroll
            for (int w = 0; w < nw; ++w) { off[j] += w < wave ? s_lens[j][w] : 0u; entries += s_lens[j][w]; }
            const int r = tid + j * kBuildThreads;
            if (r < rows) s_delta[r] = cur[j] - off[j];
        }
        const bool once = entries <= held;
        uint16_t *s_mark = once ? reinterpret_cast<uint16_t *>(s_raw) : marks_behind;
        // The line's places from w0 on, up to w1, an even share (`steps` times 64) to each wavefront.
        uint32_t w0 = 0u, w1 = 0u, steps = 0u, carry = 0u;
        auto mark = [&](uint32_t begin, uint32_t end) {
            w0 = begin;
            w1 = end;
            steps = (w1 - w0 + (uint32_t)(kWave * nw) - 1u) / (uint32_t)(kWave * nw);
            for (uint32_t i = 8u * (uint32_t)tid; i < w1 - w0; i += 8u * kBuildThreads) *reinterpret_cast<uint4 *>(s_mark + i) = uint4{0u, 0u, 0u, 0u};
            __syncthreads();
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const uint32_t r = (uint32_t)(tid + j * kBuildThreads), from = max(off[j], w0), to = min(off[j] + (next[j] - cur[j]), w1);
                if (j * kBuildThreads >= rows || from >= to) continue;
                if (from == off[j]) s_mark[from - w0] = (uint16_t)(r + 1u);
                const uint32_t share = steps * kWave;
                for (uint32_t w = (from - w0 + share - 1u) / share; w < (uint32_t)nw && w0 + w * share < to; ++w) s_first[w] = r + 1u;
            }
            __syncthreads();
            carry = s_first[wave];
        };
        // The wavefront's places, 64 after 64: the lane's row and its entry's position.
        auto place_of = [&](uint32_t step, uint32_t &row, uint32_t &e) {
            const uint32_t p = ((uint32_t)wave * steps + step) * kWave + (uint32_t)lane;
            const bool in = step < steps && p < w1 - w0;
            const int m = wave_scan_max(max(in ? (int)s_mark[p] : 0, (int)carry));
            carry = (uint32_t)__builtin_amdgcn_readlane(m, 63);
            row = (uint32_t)m - 1u;
            e = in ? s_delta[row] + w0 + p : 0u;
            return in;
        };
        // What a lane holds of an entry: column, row and rank (13, 12 and 6 bits; ~0: nothing), its value, and the entries of its list that were counted before
        // (16 bits each).
        uint32_t hold[K], hold_before[K / 2];
        float hold_value[K];
        auto hold_nothing = [&]() {
#pragma unroll
            for (int k = 0; k < K; ++k) { hold[k] = 0xFFFFFFFFu; hold_value[k] = 0.0f; hold_before[k / 2] = 0u; }
        };
        if (once) {
            mark(0u, entries);
            hold_nothing();
            constexpr int H = R == 5 ? K / 2 : K;               // entries whose loads are in flight together
#pragma unroll
            for (int h = 0; h < K; h += H) {
                uint32_t c[H], row[H];
#pragma unroll
                for (int x = 0; x < H; ++x) { c[x] = 0xFFFFFFFFu; row[x] = 0u; }
#pragma unroll
                for (int g = 0; g < H; g += 4) {
                    if ((uint32_t)(h + g) >= steps) continue;
#pragma unroll
                    for (int x = g; x < g + 4; ++x) {
                        uint32_t e;
                        if (place_of((uint32_t)(h + x), row[x], e)) {
                            c[x] = *reinterpret_cast<const uint32_t *>(tile_columns + e * 4u);
                            hold_value[h + x] = *reinterpret_cast<const float *>(tile_values + e * 4u);
                            if (ranks) row[x] |= (uint32_t)tile_ranks[e] << 16;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int g = 0; g < H; g += 4) {
                    if ((uint32_t)(h + g) >= steps) continue;
#pragma unroll
                    for (int x = g; x < g + 4; ++x) {
                        const uint32_t col = c[x] - c0;
                        if (col < range) {
                            hold[h + x] = col | (row[x] & 0xFFFu) << 13 | min(row[x] >> 16, 2u * kRanks - 1u) << 25;
                            hold_before[(h + x) / 2] |= atomicAdd(&s_count[col], 1u) << (16 * (x & 1));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            for (uint32_t w = 0u; w < entries; w += window) {
                mark(w, min(w + window, entries));
                for (uint32_t k = 0u; k < steps; k += kAgain) {
                    uint32_t c[kAgain];
#pragma unroll
                    for (int x = 0; x < kAgain; ++x) {
                        uint32_t row, e;
                        c[x] = 0xFFFFFFFFu;
                        if (place_of(k + (uint32_t)x, row, e)) c[x] = *reinterpret_cast<const uint32_t *>(tile_columns + e * 4u);
                    }
#pragma unroll
                    for (int x = 0; x < kAgain; ++x)
                        if (c[x] - c0 < range) atomicAdd(&s_count[c[x] - c0], 1u);
                }
                __syncthreads();
            }
            hold_nothing();                                     // (behind the loop: what it holds needs no registers there)
        }
        __syncthreads();
        // Which columns are dense: the first of the block that reach the mark, in column order (so that the same columns are dense in every
        // run).  A thread has some columns that follow one another.
        const uint32_t mine = ((block_cols + kBuildThreads - 1u) / kBuildThreads + 3u) & ~3u, mine_first = (uint32_t)tid * mine;
        auto columns = [&](auto &&each) {
            for (uint32_t i = mine_first; i < min(mine_first + mine, block_cols); i += 4u) {
                const uint4 v = *reinterpret_cast<const uint4 *>(s_count + i);
                each(i, v.x);
                each(i + 1u, v.y);
                each(i + 2u, v.z);
                each(i + 3u, v.w);
            }
        };
        // (as many as the block's share of their room holds; and half of its room for gaps, in a block that is gone through twice: where few columns have
        // most of the entries, they may lie in few blocks)
        const uint32_t whole = (uint32_t)T, dense_mark = (uint32_t)shape.dense_from, room_of_gaps = (uint32_t)(shape.room_of(before + entries) - shape.room_of(before)) - entries;
        const uint32_t most_dense = min(kBuildDense, (uint32_t)(shape.dense_before((int32_t)block + 1) - shape.dense_before((int32_t)block)) +
                                                         (!once && shape.dense_room() > 0 ? room_of_gaps / 2u / (uint32_t)shape.dense_room() : 0u));
        uint32_t rank = 0u, n_dense = 0u;                          // columns that reach the mark before the thread's, and all of them
        {
            uint32_t marked = 0u;
            columns([&](uint32_t, uint32_t v) { marked += v >= dense_mark ? 1u : 0u; });
            rank = (uint32_t)wave_scan_add((int)marked);
            if (lane == 63) s_wave[wave] = rank;
            __syncthreads();
            rank -= marked;
#pragma unroll
            for (int w = 0; w < nw; ++w) { rank += w < wave ? s_wave[w] : 0u; n_dense += s_wave[w]; }
            n_dense = min(n_dense, most_dense);
            __syncthreads();
        }
        // Counts -> starts, which count from a line's beginning in memory and in LDS, `phase` before the block's piece.  Long lists and dense columns
        // begin at a line; what they leave free before them is nobody's.  (A block whose gaps are more than its room has none.)
        const uint32_t base = piece_of(before, block), phase = (uint32_t)(first + base) & (kMatchLine - 1u);
        const uint32_t limit = phase + piece_of(before + entries, block + 1u) - base;
        uint32_t line = shape.aligned ? kMatchLine : 0xFFFFFFFFu, at = phase, total = phase;
        auto piece = [&](uint32_t v, bool dense) {
            return line <= whole && (dense || v >= line) ? Stretch{0u, (int32_t)(dense ? whole : v)} : Stretch{dense ? whole : v, -1};
        };
        for (;;) {
            Stretch incl{0u, -1};
            uint32_t r = rank;
            columns([&](uint32_t, uint32_t v) {
                incl = then(incl, piece(v, v >= dense_mark && r < most_dense));
                r += v >= dense_mark ? 1u : 0u;
            });
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const Stretch up{(uint32_t)__shfl_up((int)incl.before, d), __shfl_up(incl.after, d)};
                if (lane >= d) incl = then(up, incl);
            }
            const Stretch lower{(uint32_t)__shfl_up((int)incl.before, 1), __shfl_up(incl.after, 1)};
            if (lane == 63) { s_wave[wave] = incl.before; s_second[wave] = (uint32_t)incl.after; }
            __syncthreads();
            at = total = phase;
#pragma unroll
            for (int w = 0; w < nw; ++w) {
                total = end_of(total, Stretch{s_wave[w], (int32_t)s_second[w]});
                at = w + 1 == wave ? total : at;
            }
            if (lane > 0) at = end_of(at, lower);
            __syncthreads();
            if (total <= limit || line > whole) break;
            line = 0xFFFFFFFFu;
        }
        {
            uint32_t r = rank;
            columns([&](uint32_t i, uint32_t v) {
                const bool dense = v >= dense_mark && r < most_dense;
                const uint32_t flag = dense ? kMatchDense : 0u, end = end_of(at, piece(v, dense)), from = end - (dense ? whole : v);
                if (dense) s_dense[r] = from;
                r += v >= dense_mark ? 1u : 0u;
                s_count[i] = from | flag;
                if (i < range) ptr[c0 + block + i] = (base + from - phase) | (from - at) << kMatchGapShift | flag;
                at = end;
            });
        }
        if (tid == 0) ptr[c0 + block + range] = base + total - phase;
        __syncthreads();
        float *__restrict__ values_at = b.values + first + base - phase;   // the block's piece
        uint16_t *__restrict__ rows_at = b.rows + first + base - phase;
        const int64_t room = list_end - (first + base - phase);    // (never reached while the row pointers hold)
        // From the lanes where all of the piece is staged, else as the entries come again.
        const bool from_lanes = once && total <= shape.stage;
        const uint32_t stage = from_lanes ? shape.stage : shape.stage - window / 2u;
        s_mark = marks_behind;
        if (n_dense > 0u) {
            for (uint32_t d = 0; d < n_dense; ++d)
                for (uint32_t i = s_dense[d] + (uint32_t)tid; i < s_dense[d] + whole; i += kBuildThreads) {
                    if (i < stage) s_value[i] = 0.0f;
                    else if (i < room) values_at[i] = 0.0f;
                }
            __threadfence_block();
            __syncthreads();
        }
        // (a stored zero is absent: it goes to the spare row behind the tile's, and for the products of positive entries what is not positive)
        auto cell_of = [&](uint32_t row, uint32_t rank_in_row, float t) {
            return (uint16_t)(((positive ? t > 0.0f : t != 0.0f) ? row : (uint32_t)T) * (uint32_t)unit + (rank_in_row << kRankShift));
        };
        if (from_lanes) {
            if (transform != TR_ID) {
#pragma unroll
                for (int k = 0; k < K; ++k) hold_value[k] = transform_value(transform, hold_value[k]);
            }
#pragma unroll
            for (int g = 0; g < K; g += 4) {
                if ((uint32_t)g >= steps) continue;
#pragma unroll
                for (int k = g; k < g + 4; ++k) {
                    if (hold[k] == 0xFFFFFFFFu) continue;
                    const uint32_t start = s_count[hold[k] & 0x1FFFu], row = (hold[k] >> 13) & 0xFFFu;
                    const bool dense = (start & kMatchDense) != 0u;
                    const uint32_t at = (start & ~kMatchDense) + (dense ? row : (hold_before[k / 2] >> (16 * (k & 1))) & 0xFFFFu);
                    s_value[at] = hold_value[k];
                    s_row[at] = cell_of(row, hold[k] >> 25, hold_value[k]);          // (of a dense column nothing reads it)
                }
            }
        } else {
            for (uint32_t w = 0u; w < entries; w += window) {
                mark(w, min(w + window, entries));
                for (uint32_t k = 0u; k < steps; k += kAgain) {
                    uint32_t c[kAgain], row[kAgain];
                    float v[kAgain];
#pragma unroll
                    for (int x = 0; x < kAgain; ++x) {
                        uint32_t e;
                        c[x] = 0xFFFFFFFFu;
                        if (place_of(k + (uint32_t)x, row[x], e)) {
                            c[x] = *reinterpret_cast<const uint32_t *>(tile_columns + e * 4u);
                            v[x] = *reinterpret_cast<const float *>(tile_values + e * 4u);
                            if (ranks) row[x] |= min((uint32_t)tile_ranks[e], 2u * kRanks - 1u) << 16;
                        }
                    }
#pragma unroll
                    for (int x = 0; x < kAgain; ++x) {
                        const uint32_t col = c[x] - c0;
                        if (col >= range) continue;
                        const float t = transform_value(transform, v[x]);
                        const uint32_t start = s_count[col], r = row[x] & 0xFFFFu;
                        const bool dense = (start & kMatchDense) != 0u;
                        const uint32_t at = dense ? (start & ~kMatchDense) + r : atomicAdd(&s_count[col], 1u);
                        const uint16_t cell = cell_of(r, row[x] >> 16, t);
                        if (at < stage) {
                            s_value[at] = t;
                            s_row[at] = cell;
                        } else if (at < room) {
                            values_at[at] = t;
                            if (!dense) rows_at[at] = cell;
                        }
                    }
                }
                __syncthreads();
            }
        }
        __syncthreads();
        // (in memory as in LDS a piece begins `phase` entries behind a line)
        const uint32_t staged = (uint32_t)max((int64_t)0, min((int64_t)min(total, stage), room));
        const bool values_too = with_values || n_dense > 0u;
        for (uint32_t i = 8u * (uint32_t)tid; i < staged; i += 8u * kBuildThreads) {
            if (i >= phase && i + 8u <= staged) {
                *reinterpret_cast<Eight *>(rows_at + i) = *reinterpret_cast<const Eight *>(s_row + i);
            } else {
                for (uint32_t x = max(i, phase); x < min(i + 8u, staged); ++x) rows_at[x] = s_row[x];
            }
        }
        if (values_too)
            for (uint32_t i = 4u * (uint32_t)tid; i < staged; i += 4u * kBuildThreads) {
                if (i >= phase && i + 4u <= staged) {
                    *reinterpret_cast<Four *>(values_at + i) = *reinterpret_cast<const Four *>(s_value + i);
                } else {
                    for (uint32_t x = max(i, phase); x < min(i + 4u, staged); ++x) values_at[x] = s_value[x];
                }
            }
#pragma unroll
        for (int j = 0; j < R; ++j) cur[j] = next[j];
        before += entries;
        __syncthreads();
    }
}

// Lanes to a row.  A workgroup to the row where its own cost, one launch of many, counts less than the loads that it has in flight:
// with 256 / 64 lanes in us, L1: 300 rows of 3,700 8 / 18, 939 of 1,940 13 / 24, 4,096 of 1,870 18 / 26, 5,000 of 275 11 / 12, 20,000 of
// 280 35 / 30, 28,301 of 166 (power law, the longest 24,000) 50 / 35, 60,000 of 230 72 / 27, 65,536 of 1,760 128 / 109.  (With 16
// lanes to the row 10,000 rows of 38 take 17 to 20 us, with 64 11 to 15.)
int match_norm_lanes(int64_t n_rows, int64_t nnz) {
    const int64_t mean = nnz / n_rows;
    return mean >= 128 && n_rows <= 8192 ? 256 : (mean >= 16 ? 64 : 4);
}
hipError_t launch_match_norms(hipStream_t st, const int64_t *indptr, const float *values, int64_t n_rows, int64_t nnz,
                              int metric, int transform, int norm, float p, double k, const RowsVerdict &seen, double *norms, int16_t *scales) {
    if (n_rows <= 0) return hipSuccess;
    const NormArgs a{indptr, values, n_rows, nnz, metric, transform, norm, p, k, seen, norms, scales};
    auto go = [&](auto with_scales) {
        constexpr bool S = decltype(with_scales)::value;
        switch (match_norm_lanes(n_rows, nnz)) {
        case 256: hipLaunchKernelGGL(spd_match_norms_kernel<S>, dim3((unsigned)n_rows), dim3(256), 0, st, a); break;
        case 64: {
            // (as many rows as leave every place of the chip for a wavefront taken; one where a row has more entries than are loaded ahead)
            const int per_wave = nnz > 4 * kWave * n_rows ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(kNormRows, n_rows / 8192));
            hipLaunchKernelGGL(spd_match_norms_rows_kernel<S>, dim3((unsigned)((n_rows + 4 * per_wave - 1) / (4 * per_wave))), dim3(256), 0, st, a, per_wave);
            break;
        }
        default: hipLaunchKernelGGL(spd_match_norms_short_kernel<S>, dim3((unsigned)((n_rows + 63) / 64)), dim3(256), 0, st, a); break;
        }
    };
    if (scales) go(std::true_type{}); else go(std::false_type{});
    return hipGetLastError();
}

MatchShape match_shape(int64_t lds_budget, int op, int64_t n, int64_t n_cols, int64_t nnz) {
    MatchShape s{};
    const int cell = match_cell_bytes(op);
    if (cell == 0 || n <= 0 || n_cols <= 0) return s;
    s.waves = match_waves(cell);
    const int64_t strip = (lds_budget - match_static_lds(cell)) / s.waves;
    int64_t most = ((strip - 7) / cell - 1) / kWave * kWave;    // (a spare row behind them)
    if (op == OP_CHEB) most = std::min<int64_t>(most, kRankedRows);
    if (most < kWave) return s;
    const double per_cell = (double)nnz / (double)n / (double)n_cols;
    if (cell <= 8 && op != OP_JS) {
        // The lists of a tile that the workgroups of an XCD walk together: within twice its L2 (65,536 x 26,000 rows of 7 %,
        // L1: tiles of 256 rows 33.8 ms, 384 29.9, 512 28.6, 640 31.2, 768 34.0, 1,216 36.7), as long as a list is two
        // chunks of 16 on the mean; where tiles of all the LDS are within it, the largest (300,000 rows of 230, cosine:
        // 576 rows 9.0 ms, 832 7.0, 1,216 5.7).  (Jensen-Shannon is bound by its
        // arithmetic: on the 65,536 rows 512 rows to the tile 38.7, 1,216 37.3.)
        const int64_t within = (int64_t)((double)(2 * kMatchL2Bytes / 8) / std::max(per_cell * (double)n_cols, 1e-12)) / kWave * kWave;
        const int64_t least = ((int64_t)(32.0 / std::max(per_cell, 1e-9)) + kWave - 1) / kWave * kWave;
        most = std::max<int64_t>(kWave, std::min(most, std::max(within, least)));
    }
    const int64_t tiles = (n + most - 1) / most;
    if (tiles > (1 << 30)) return s;
    s.tile_rows = (int32_t)(((n + tiles - 1) / tiles + kWave - 1) / kWave * kWave);
    s.lds_bytes = (uint32_t)s.waves * match_strip_bytes(cell, s.tile_rows);
    // A block of columns: an eighth of the LDS for counters, or twice that, and entries for four fifths, on the mean,
    // of what counters and row positions leave for its piece of the lists, and of what the lanes hold (a fuller block is gone through
    // twice; narrower blocks read a row's lines more often).  Dense columns may take half as much again: so many to so many columns as
    // blocks have that take a compute unit each.
    // A step of 64 rows of a dense column costs half a list's step, and a third where that adds doubles.  (Dot products from a third / 0.4 / a
    // half of the rows on, us: 1,024 x 300,000 rows of 230, cosine, 5,385 / 5,344 / 5,519, k-NN of 2,048 of them, Hellinger, 7,304 /
    // 7,489 / 8,115; 10,000 x 10,000 rows of 38, cosine, 312 / 311 / 307.  From 0.3 / 0.4 / 0.5 / 0.6 on: the same rows of 38, L1, 336 /
    // 331 / 325 / 318; sets, Jaccard, 9,102 / 8,970 / 8,928 / 8,963.  Chebyshev: an entry has a rank, a column of values none.)
    s.dense_from = op == OP_CHEB ? s.tile_rows + 1 : std::max(1, s.tile_rows / (op == OP_DOT ? 3 : 2));
    const double per_col = per_cell * (double)s.tile_rows;
    const int64_t tiles_now = (n + s.tile_rows - 1) / s.tile_rows;
    auto blocks_of = [&](int at) { return (n_cols + (1 << at) - 1) >> at; };
    auto stage_of = [&](int64_t usable, int64_t rows_bytes, int shift) { return (usable - rows_bytes - ((int64_t)4 << shift)) / 48 * 8; };
    {
        const int64_t usable = lds_budget - 1024, rows_bytes = 12 * (int64_t)s.tile_rows;
        if (usable < rows_bytes + 4096) return s;
        int shift = 2;
        while ((4 << (shift + 1)) <= usable / 8 && (1 << shift) < n_cols) ++shift;
        const int narrow = shift;
        if ((n_cols >> shift) >= 16 && (4 << (shift + 1)) <= usable / 4) ++shift;
        while (shift > 2 && per_col * (double)(1 << shift) * 1.25 > (double)stage_of(usable, rows_bytes, shift)) --shift;
        // What the columns' share of the entries fills, once at least (of the halves of many columns, so that their number
        // does not cost memory: an index may keep lists that grow to its limit and no further).
        auto dense_of = [&](int at) {
            const int of = std::min(at, narrow);
            return (int32_t)std::min<double>(kBuildDensePer, std::max(1.0, std::floor(per_cell * (double)(1 << of))) * (double)(1 << (at - of)));
        };
        // (a workgroup for every compute unit, where there are columns enough, and so that dense columns take no more
        // than the entries do, and 512 KiB: 12,970 rows of 6 over 10,261 columns, with an index: 41 blocks took the lists over its limit,
        // and its calls 600 us by the scan instead of 240)
        while (shift > 8 && tiles_now * blocks_of(shift) < 256 &&
               tiles_now * blocks_of(shift - 1) * dense_of(shift - 1) * s.dense_room() * 6 <= 8 * nnz + (512 << 10)) --shift;
        s.dense_shift = shift;
        s.dense_per = dense_of(shift);
    }
    // Two workgroups to a compute unit, since what a block takes is mostly waiting for one thing after the other.
    const int64_t usable = lds_budget / kBuildPerCu - 1024, rows_bytes = 4 * (int64_t)s.tile_rows;
    if (usable < rows_bytes + 2048) return s;
    // A block as wide as its entries fit on the mean and a twelfth more (columns that are uniform fill the blocks of a tile alike: 60,000 rows of 1,820, KL, blocks of 64 columns
    // 1,671 us, of 128, 91 % full, 1,035; where they are not, wider blocks pay all the same: 300,000 rows of 230 899 / 699), and a quarter more where that leaves the chip less
    // than its two workgroups to a compute unit (8,000 of these 32 / 44).  Jensen-Shannon's 1,551 us are 1,087 with lanes that hold half as many again, and so twice the
    // columns; held for nothing these cost a tenth (KL 1,035 / 1,200, ratings 385 / 432).
    auto widest = [&](int64_t held, double spare) {
        int shift = s.dense_shift;
        while (shift > 2 && ((4 << shift) > usable / 4 ||
                             per_col * (double)(1 << shift) * spare > (double)std::min(stage_of(usable, rows_bytes, shift), held * kBuildThreads))) --shift;
        return shift;
    };
    const int lane_rows = build_rows(s.tile_rows);
    int held = build_held(lane_rows), shift = widest(held, 1.25);
    const int wider = widest(held, 1.08), more = lane_rows == 3 ? widest(kBuildHeldMore, 1.08) : wider;
    auto fills = [&](int at) { return tiles_now * blocks_of(at) >= 256 * kBuildPerCu; };
    if (wider > shift && fills(wider)) shift = wider;
    if (more > shift && fills(more)) { shift = more; held = kBuildHeldMore; }
    s.held = (int16_t)held;
    s.block_shift = shift;
    s.stage = (uint32_t)stage_of(usable, rows_bytes, shift);
    s.blocks = (int32_t)blocks_of(shift);
    s.ptr_stride = (n_cols + s.blocks + 3) / 4 * 4;
    s.tile_extra = (int64_t)s.dense_before(s.blocks) * s.dense_room();
    s.build_lds_bytes = s.stage * 6u + (4u << shift) + (uint32_t)rows_bytes;
    s.n_tiles = (int32_t)((n + s.tile_rows - 1) / s.tile_rows);
    if (op == OP_DOT && s.list_entries(nnz) >= (int64_t)1 << 29) {         // (positions end there: no more room than other products' columns take)
        s.dense_from = std::max(1, s.tile_rows / 2);
        s.tile_extra = (int64_t)s.dense_before(s.blocks) * s.dense_room();
    }
    // Lists at lines of memory, where a tile's positions and a gap fit a word and all positions their limit.
    s.aligned = 1;
    const double tile_most = 1.3125 * std::min((double)nnz, (double)s.tile_rows * (double)n_cols) + (double)s.tile_extra;
    if (tile_most >= (double)(s.position_bits() - 64u) || s.list_entries(nnz) >= (int64_t)1 << 29) s.aligned = 0;
    return s;
}

// Column blocks to a workgroup: some 2,048 workgroups (a run of blocks looks its rows' first entries up once).
static uint32_t match_build_blocks(const MatchShape &s) { return std::max(1u, (uint32_t)((uint64_t)s.blocks * (uint64_t)s.n_tiles / 2048u)); }
// (its workgroups in whole rounds of the eight XCDs)
static int64_t match_build_grid(const MatchShape &s) {
    const int64_t per_wg = match_build_blocks(s);
    return (s.n_tiles * ((s.blocks + per_wg - 1) / per_wg) + 7) / 8 * 8;
}
bool match_launches_fit(const MatchShape &s, int op, int64_t m, int64_t nnz_a, int64_t n, bool renumbered) {
    constexpr int64_t kMost = ((int64_t)1 << 32) - 1024;
    // (The build's launches lie a factor of two below that: the line stays where it was with workgroups of 1,024.  B's norms: of fewer than 2^30 rows and, from 16 entries to the row on, 2^25 of them, by its lists' positions)
    return (op == OP_CHEB ? match_ranks_grid(m + n) * 256 <= kMost : m * match_norm_lanes(std::max<int64_t>(m, 1), nnz_a) <= kMost) &&
           match_build_grid(s) * 2 * kBuildThreads <= kMost && (!renumbered || nnz_a <= kMost);
}

hipError_t launch_match_build(hipStream_t st, const int64_t *indptr, const int32_t *indices, const float *values,
                              int64_t n_rows, int64_t nnz, uint32_t k, const MatchB &b, int op, int transform, const RowsVerdict &seen) {
    if (n_rows <= 0) return hipSuccess;
    const MatchShape &s = b.shape;
    const uint32_t per_wg = match_build_blocks(s), wgs = ((uint32_t)s.blocks + per_wg - 1u) / per_wg;
    auto go = [&](auto rows, auto held) {
        auto kern = spd_match_build_kernel<decltype(rows)::value, decltype(held)::value>;
        static std::atomic<uint32_t> allowed[kMatchDevices];
        hipError_t err = allow_lds(kern, allowed, s.build_lds_bytes, 1024u);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(kern, dim3((unsigned)match_build_grid(s)), dim3(kBuildThreads), s.build_lds_bytes, st, indptr, indices, values, n_rows,
                           nnz, k, b, per_wg, wgs, op == OP_CHEB ? 1 : (match_cell_bytes(op) >= 8 ? 8 : 4), transform, op != OP_CNT, op == OP_JS || op == OP_KL, seen);
        return hipGetLastError();
    };
    constexpr std::integral_constant<int, kBuildHeld> few{};
    constexpr std::integral_constant<int, kBuildHeldMore> more{};
    switch (build_rows(s.tile_rows)) {
    case 1: return go(std::integral_constant<int, 1>{}, more);
    case 3: return s.held == kBuildHeld ? go(std::integral_constant<int, 3>{}, few) : go(std::integral_constant<int, 3>{}, more);
    default: return go(std::integral_constant<int, 5>{}, few);
    }
}

__global__ void __launch_bounds__(256) spd_match_knn_begin_kernel(unsigned long long *tau, int64_t *row_off, int32_t *row_lists,
                                                                  KnnEntry *part, int64_t m, int lists, int k) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, per = (int64_t)lists * k;
    if (i < m) {
        tau[i] = kKnnUnused;
        row_off[i] = i * per;
        row_lists[i] = lists;
    }
    for (int64_t e = i; e < m * per; e += (int64_t)gridDim.x * 256) part[e] = KnnEntry{__builtin_huge_valf(), 0x7fffffff};
}
hipError_t launch_match_knn_begin(hipStream_t st, unsigned long long *tau, int64_t *row_off, int32_t *row_lists, KnnEntry *part,
                                  int64_t m, int lists, int k) {
    if (m <= 0) return hipSuccess;
    const int64_t blocks = std::max<int64_t>((m + 255) / 256, std::min<int64_t>(2048, (m * lists * k + 255) / 256));
    hipLaunchKernelGGL(spd_match_knn_begin_kernel, dim3((unsigned)blocks), dim3(256), 0, st, tau, row_off, row_lists, part, m, lists, k);
    return hipGetLastError();
}

hipError_t launch_match_a(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes);
hipError_t launch_match_b(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes);

hipError_t launch_match(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes) {
    switch (op) {
    case OP_DOT: case OP_L1: case OP_HAMM: case OP_CNT: case OP_CANB: return launch_match_a(st, op, args, lds_bytes);
    case OP_KL: case OP_JS: case OP_MINK: case OP_MINK_ANY: case OP_CHEB: return launch_match_b(st, op, args, lds_bytes);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace spd
