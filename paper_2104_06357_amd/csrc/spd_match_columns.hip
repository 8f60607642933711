// The columns that A stores, renumbered, and copies of both operands over those columns alone.
//
// The list bounds take a word per tile and column, so over very many columns (n-grams: 858,000, sets over 2^20) they
// would outweigh the lists.  No list of a column that A does not store is ever walked: the columns are renumbered 0, 1, ...
// in ascending order of those in A, B's entries in other columns are dropped, and the lists are built from the copy.  Rows
// stay in their order and ascending in their columns.  Bound by memory: B's columns are read twice and its values
// once, what stays is written once (500,000 rows of 136 entries over 2^20 columns against 4,096 of 169: 79 % stay).
#include "spd_match.h"

namespace spd {

namespace {
constexpr int kRankBlock = 4096;          // words of a workgroup of the column kernels: 1,024 threads, 4 words each
constexpr int kEntryBlock = 4096;         // entries of a workgroup of the entry kernels: 64 masks

__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    return v;
}
// Exclusive sums over the wavefront's lanes.
__device__ __forceinline__ uint32_t wave_exclusive(uint32_t v, int lane) {
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)incl, d);
        if (lane >= d) incl += up;
    }
    return incl - v;
}
// ... and over a workgroup of 1,024 threads; `total` receives the sum.
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t *s_wave, uint32_t &total) {
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const uint32_t before = wave_exclusive(v, lane);
    if (lane == 63) s_wave[wave] = before + v;
    __syncthreads();
    uint32_t at = before;
    total = 0u;
#pragma unroll
    for (int w = 0; w < 16; ++w) { at += w < wave ? s_wave[w] : 0u; total += s_wave[w]; }
    __syncthreads();
    return at;
}
}  // namespace

__global__ void __launch_bounds__(256) spd_columns_clear_kernel(uint2 *words, uint32_t n_words) {
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n_words; i += gridDim.x * 256u) words[i] = make_uint2(0u, 0u);
}

__global__ void __launch_bounds__(256) spd_columns_mark_kernel(const int32_t *__restrict__ indices, int64_t nnz, uint32_t n_cols, uint2 *words) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    const uint32_t c = (uint32_t)indices[e];
    if (c >= n_cols) return;
    uint32_t *bits = &words[c >> 5].x;
    const uint32_t bit = 1u << (c & 31u);
    // (a popular column is marked already: no atomic for it)
    if (!(__atomic_load_n(bits, __ATOMIC_RELAXED) & bit)) atomicOr(bits, bit);
}

// words[i].y becomes the number of marked columns before word i's, in two steps around spd_columns_sums_kernel.
template <bool WRITE>
__global__ void __launch_bounds__(1024) spd_columns_rank_kernel(uint2 *words, uint32_t n_words, uint32_t *sums) {
    __shared__ uint32_t s_wave[16];
    const uint32_t i0 = blockIdx.x * (uint32_t)kRankBlock + 4u * threadIdx.x;
    uint32_t count[4], mine = 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u) { count[u] = i0 + u < n_words ? (uint32_t)__popc(words[i0 + u].x) : 0u; mine += count[u]; }
    uint32_t total, at = block_exclusive(mine, s_wave, total);
    if constexpr (!WRITE) {
        if (threadIdx.x == 0) sums[blockIdx.x] = total;
    } else {
        at += sums[blockIdx.x];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i0 + u < n_words) words[i0 + u].y = at;
            at += count[u];
        }
    }
}

// sums[0 .. n) become their exclusive sums, *total their sum.  One workgroup.
__global__ void __launch_bounds__(1024) spd_columns_sums_kernel(uint32_t *sums, uint32_t n, uint32_t *total) {
    __shared__ uint32_t s_wave[16];
    uint32_t carry = 0u;
    for (uint32_t i0 = 0; i0 < n; i0 += 1024u) {
        const uint32_t i = i0 + threadIdx.x;
        uint32_t sum;
        const uint32_t at = block_exclusive(i < n ? sums[i] : 0u, s_wave, sum);
        if (i < n) sums[i] = carry + at;
        carry += sum;
    }
    if (threadIdx.x == 0) *total = carry;
}

__device__ __forceinline__ uint32_t rank_in(const uint2 word, uint32_t c) {
    return word.y + (uint32_t)__popc(word.x & ((1u << (c & 31u)) - 1u));
}

__global__ void __launch_bounds__(256) spd_columns_renumber_kernel(const int32_t *__restrict__ indices, int64_t nnz, uint32_t n_cols,
                                                                   const uint2 *__restrict__ words, int32_t *__restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= nnz) return;
    const uint32_t c = (uint32_t)indices[e];
    out[e] = c < n_cols ? (int32_t)rank_in(words[c >> 5], c) : -1;          // (-1: a column of no list)
}

// Which of B's entries stay: a bit each in masks[entry / 64], and their number per workgroup.
__global__ void __launch_bounds__(1024) spd_columns_flag_kernel(const int32_t *__restrict__ indices, int64_t nnz, uint32_t n_cols,
                                                               const uint2 *__restrict__ words, uint64_t *__restrict__ masks,
                                                               uint32_t *__restrict__ sums) {
    __shared__ int s_wave[16];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int64_t e0 = (int64_t)blockIdx.x * kEntryBlock + threadIdx.x;
    uint32_t c[4];
    bool in[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = e0 + u * 1024 < nnz ? (uint32_t)indices[e0 + u * 1024] : 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < 4; ++u) in[u] = c[u] < n_cols && ((words[c[u] >> 5].x >> (c[u] & 31u)) & 1u) != 0u;
    int mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint64_t mask = __ballot(in[u]);
        mine += (int)__popcll(mask);
        if (lane == 0 && e0 + u * 1024 < nnz) masks[(e0 + u * 1024) >> 6] = mask;
    }
    if (lane == 0) s_wave[wave] = mine;
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int w = 0; w < 16; ++w) sum += s_wave[w];
        sums[blockIdx.x] = (uint32_t)sum;
    }
}

// The entries that stay, in their order; before[entry / 64] = how many stay before a mask's.
__global__ void __launch_bounds__(1024) spd_columns_keep_kernel(const int32_t *__restrict__ indices, const float *__restrict__ values,
                                                               int64_t nnz, const uint2 *__restrict__ words,
                                                               const uint64_t *__restrict__ masks, const uint32_t *__restrict__ sums,
                                                               uint32_t *__restrict__ before, int32_t *__restrict__ out_indices,
                                                               float *__restrict__ out_values) {
    __shared__ uint32_t s_before[64];
    const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
    const int64_t e0 = (int64_t)blockIdx.x * kEntryBlock, n_masks = (nnz + 63) >> 6;
    if (wave == 0) {
        const int64_t w = (e0 >> 6) + lane;
        const uint32_t n = w < n_masks ? (uint32_t)__popcll(masks[w]) : 0u;
        const uint32_t at = sums[blockIdx.x] + wave_exclusive(n, lane);
        s_before[lane] = at;
        if (w < n_masks) before[w] = at;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t e = e0 + u * 1024 + threadIdx.x;
        if (e >= nnz) continue;
        const uint64_t mask = masks[e >> 6];
        if (!((mask >> lane) & 1u)) continue;
        const uint32_t c = (uint32_t)indices[e];
        const uint32_t at = s_before[u * 16 + wave] + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        out_indices[at] = (int32_t)rank_in(words[c >> 5], c);
        out_values[at] = values[e];
    }
}

__global__ void __launch_bounds__(256) spd_columns_rows_kernel(const int64_t *__restrict__ indptr, int64_t n_rows, int64_t nnz,
                                                               const uint64_t *__restrict__ masks, const uint32_t *__restrict__ before,
                                                               const uint32_t *__restrict__ total, int64_t *__restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r > n_rows) return;
    int64_t p = indptr[r];
    p = p < 0 ? 0 : (p > nnz ? nnz : p);
    out[r] = p < nnz ? (int64_t)before[p >> 6] + (int64_t)__popcll(masks[p >> 6] & ((1ull << (p & 63)) - 1ull)) : (int64_t)*total;
}

hipError_t launch_match_columns(hipStream_t st, const int32_t *a_indices, int64_t a_nnz, const int64_t *b_indptr, const int32_t *b_indices,
                                const float *b_values, int64_t b_rows, int64_t b_nnz, uint32_t n_cols, const MatchColumns &c) {
    if (a_nnz <= 0 || b_nnz <= 0 || b_rows <= 0 || n_cols == 0u) return hipErrorInvalidValue;
    const uint32_t n_words = (n_cols + 31u) / 32u, word_blocks = (n_words + kRankBlock - 1u) / kRankBlock;
    const uint32_t entry_blocks = (uint32_t)((b_nnz + kEntryBlock - 1) / kEntryBlock);
    const uint32_t a_blocks = (uint32_t)((a_nnz + 255) / 256);
    hipLaunchKernelGGL(spd_columns_clear_kernel, dim3(std::min(1024u, (n_words + 255u) / 256u)), dim3(256), 0, st, c.words, n_words);
    hipLaunchKernelGGL(spd_columns_mark_kernel, dim3(a_blocks), dim3(256), 0, st, a_indices, a_nnz, n_cols, c.words);
    hipLaunchKernelGGL((spd_columns_rank_kernel<false>), dim3(word_blocks), dim3(1024), 0, st, c.words, n_words, c.sums);
    hipLaunchKernelGGL(spd_columns_sums_kernel, dim3(1), dim3(1024), 0, st, c.sums, word_blocks, c.totals);
    hipLaunchKernelGGL((spd_columns_rank_kernel<true>), dim3(word_blocks), dim3(1024), 0, st, c.words, n_words, c.sums);
    hipLaunchKernelGGL(spd_columns_renumber_kernel, dim3(a_blocks), dim3(256), 0, st, a_indices, a_nnz, n_cols, c.words, c.a_indices);
    hipLaunchKernelGGL(spd_columns_flag_kernel, dim3(entry_blocks), dim3(1024), 0, st, b_indices, b_nnz, n_cols, c.words, c.masks, c.sums);
    hipLaunchKernelGGL(spd_columns_sums_kernel, dim3(1), dim3(1024), 0, st, c.sums, entry_blocks, c.totals + 1);
    hipLaunchKernelGGL(spd_columns_keep_kernel, dim3(entry_blocks), dim3(1024), 0, st, b_indices, b_values, b_nnz, c.words, c.masks, c.sums,
                       c.before, c.b_indices, c.b_values);
    hipLaunchKernelGGL(spd_columns_rows_kernel, dim3((unsigned)((b_rows + 256) / 256)), dim3(256), 0, st, b_indptr, b_rows, b_nnz, c.masks,
                       c.before, c.totals + 1, c.b_indptr);
    return hipGetLastError();
}

}  // namespace spd
