// Small calls in one launch.
//
// Where the operands are a few thousand entries the plan, its uploads, the repack and their launches are all
// that a call costs (256 x 256 rows of 10, L1: 27 us a call, one after the other, of which the scan is 5).  Here a
// workgroup puts four rows of A into a strip of LDS, four values to a column, and a lane, or four where rows are longer, takes a
// row of B where the caller has it, looks its columns up and sums the row's norm on the way.  No scratch, no upload, no
// second launch.  Bound by the latency of a row's entries (four of a lane in flight) and by the launch itself: 7 x 194
// rows of 337, L1, 91 us with a lane to the row, 30 with four.
#include "spd_direct.h"
#include "spd_scan_impl.h"

namespace spd {

namespace {
constexpr int kDirectUnroll = 4;
__device__ __forceinline__ int64_t clamped(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }
}  // namespace

uint32_t direct_lds_bytes(int64_t n_cols, int64_t n, int knn_k) {
    return (uint32_t)(n_cols * (kDirectRows * 4) + (knn_k > 0 ? n * (kDirectRows * 4) : 0));
}

// G: lanes to a row of B.
template <int OP, bool KNN, int G>
__global__ void __launch_bounds__(kDirectRowsB * G) spd_direct_kernel(const DirectArgs args) {
    using O = Op<OP>;
    using Acc = typename O::Acc;
    constexpr int kThreads = kDirectRowsB * G;
    extern __shared__ __align__(16) float s_strip[];              // [column][row of A], then with k-NN [row of A][row of B]
    __shared__ double s_norm[kDirectRows][2];
    static_assert(kDirectRows * kWave <= kThreads && (G == 1 || G == kDirectRows), "a wavefront to a row of A, a lane of a row of B too");
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6), sub = tid % G;
    const int64_t i0 = (int64_t)blockIdx.x * kDirectRows, n = args.b.rows;
    for (uint32_t c = (uint32_t)tid; c < args.k; c += kThreads) reinterpret_cast<float4 *>(s_strip)[c] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    if (wave < kDirectRows) {
        const int64_t i = i0 + wave;
        double s0 = 0.0, s1 = 0.0;
        if (i < args.a.rows) {
            const int64_t begin = clamped(args.a.indptr[i], 0, args.a.nnz), end = clamped(args.a.indptr[i + 1], begin, args.a.nnz);
            for (int64_t e = begin + lane; e < end; e += kWave) {
                const uint32_t c = (uint32_t)args.a.indices[e];
                const float v = transform_value(args.transform, args.a.values[e]);
                norm_accumulate(args.norm, v, args.q.p, s0, s1);
                if (c < args.k) s_strip[c * kDirectRows + (uint32_t)wave] = v;
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) { s0 += __shfl_xor(s0, d); s1 += __shfl_xor(s1, d); }
        if (lane == 0) norm_derive(args.q.metric, args.q.k, s0, s1, s_norm[wave][0], s_norm[wave][1]);
    }
    __syncthreads();
    float *s_dist = s_strip + (size_t)args.k * kDirectRows;
    // (k-NN: every row of B passes through the workgroup; pairwise: 256 of them)
    const int64_t j_first = KNN ? 0 : (int64_t)blockIdx.y * kDirectRowsB, j_last = KNN ? n : min(n, j_first + kDirectRowsB);
    for (int64_t j = j_first + tid / G; j < j_last; j += kDirectRowsB) {
        const int64_t begin = clamped(args.b.indptr[j], 0, args.b.nnz), end = clamped(args.b.indptr[j + 1], begin, args.b.nnz);
        Acc acc[kDirectRows];
#pragma unroll
        for (int r = 0; r < kDirectRows; ++r) O::init(acc[r]);
        double s0 = 0.0, s1 = 0.0;
        for (int64_t e0 = begin + sub; e0 < end; e0 += kDirectUnroll * G) {
            uint32_t c[kDirectUnroll];
            float v[kDirectUnroll];
#pragma unroll
            for (int u = 0; u < kDirectUnroll; ++u) {
                c[u] = e0 + u * G < end ? (uint32_t)args.b.indices[e0 + u * G] : 0xFFFFFFFFu;
                v[u] = e0 + u * G < end ? args.b.values[e0 + u * G] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kDirectUnroll; ++u) {
                if (e0 + u * G >= end) break;
                const float b = transform_value(args.transform, v[u]);
                norm_accumulate(args.norm, b, args.q.p, s0, s1);
                if (c[u] < args.k) {
                    const float4 a = reinterpret_cast<const float4 *>(s_strip)[c[u]];
                    const typename O::Bv bv = O::prep(b, args.q);
                    O::visit(acc[0], a.x, bv, args.q);
                    O::visit(acc[1], a.y, bv, args.q);
                    O::visit(acc[2], a.z, bv, args.q);
                    O::visit(acc[3], a.w, bv, args.q);
                }
            }
        }
        if constexpr (G > 1) {                                    // (a row's lanes are neighbours and here together)
#pragma unroll
            for (int d = G / 2; d >= 1; d >>= 1) {
                s0 += __shfl_xor(s0, d);
                s1 += __shfl_xor(s1, d);
#pragma unroll
                for (int r = 0; r < kDirectRows; ++r) O::combine(acc[r], acc_shfl_xor<OP>(acc[r], d));
            }
        }
        double nb0, nb1;
        norm_derive(args.q.metric, args.q.k, s0, s1, nb0, nb1);
        for_metric_of<OP>(args.q.metric, [&](auto metric_tag) {
            constexpr int MT = decltype(metric_tag)::value;
            auto finish = [&](double v0, double v1, double v2, int r) {
                const float d = finish_as<MT>(args.q, v0, v1, v2, s_norm[r][0], s_norm[r][1], nb0, nb1);
                if constexpr (KNN) s_dist[(size_t)r * (size_t)n + (size_t)j] = MT == MT_INNER ? 0.0f - d : d;
                else if (i0 + r < args.a.rows) args.out[(size_t)(i0 + r) * (size_t)n + (size_t)j] = d;
            };
            if constexpr (G == 1) {
#pragma unroll
                for (int r = 0; r < kDirectRows; ++r) finish(O::v0(acc[r]), O::v1(acc[r]), O::v2(acc[r]), r);
            } else {
                double v0 = O::v0(acc[0]), v1 = O::v1(acc[0]), v2 = O::v2(acc[0]);       // (a lane to a row of A)
#pragma unroll
                for (int r = 1; r < kDirectRows; ++r) {
                    double w0 = O::v0(acc[r]), w1 = O::v1(acc[r]), w2 = O::v2(acc[r]);
                    asm volatile("" : "+v"(w0), "+v"(w1), "+v"(w2));          // (else the sums are indexed, in memory)
                    v0 = sub == r ? w0 : v0;
                    v1 = sub == r ? w1 : v1;
                    v2 = sub == r ? w2 : v2;
                }
                finish(v0, v1, v2, sub);
            }
        });
    }
    if constexpr (KNN) {
        __syncthreads();
        const int64_t i = i0 + wave;
        if (wave >= kDirectRows || i >= args.a.rows) return;
        // the k best of a wavefront's row, ascending over the lanes, 64 rows of B at a time
        const int k = args.knn_k;
        uint64_t best = kKnnUnused;
        float bar = __builtin_huge_valf();
        for (int64_t j0 = 0; j0 < n; j0 += kWave) {
            const int64_t j = j0 + lane;
            const float d = j < n ? s_dist[(size_t)wave * (size_t)n + (size_t)j] : __builtin_nanf("");
            const bool pass = d <= bar;                           // (later rows lose the ties)
            if (__ballot(pass) == 0) continue;
            const uint64_t c = wave_sort_desc(pass ? knn_key(d, (int)j) : kKnnUnused, lane);
            best = wave_merge_asc(c < best ? c : best, lane);
            if (lane >= k) best = kKnnUnused;
            bar = float_from_order_key((uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(best >> 32), k - 1));
        }
        if (lane < k) {
            const float d = float_from_order_key((uint32_t)(best >> 32));
            args.out_idx[(size_t)i * (size_t)k + (size_t)lane] = (int64_t)(uint32_t)best;
            args.out_dist[(size_t)i * (size_t)k + (size_t)lane] = args.q.metric == MT_INNER ? -d : d;
        }
    }
}

template <int OP, int G> static hipError_t launch_direct_op(hipStream_t st, const DirectArgs &args) {
    const uint32_t lds = direct_lds_bytes((int64_t)args.k, args.b.rows, args.knn_k);
    const unsigned groups = (unsigned)((args.a.rows + kDirectRows - 1) / kDirectRows);
    if (args.knn_k > 0) hipLaunchKernelGGL((spd_direct_kernel<OP, true, G>), dim3(groups), dim3(kDirectRowsB * G), lds, st, args);
    else
        hipLaunchKernelGGL((spd_direct_kernel<OP, false, G>), dim3(groups, (unsigned)((args.b.rows + kDirectRowsB - 1) / kDirectRowsB)),
                           dim3(kDirectRowsB * G), lds, st, args);
    return hipGetLastError();
}
template <int OP> static hipError_t launch_direct_by(hipStream_t st, const DirectArgs &args, int lanes) {
    return lanes == 1 ? launch_direct_op<OP, 1>(st, args) : launch_direct_op<OP, kDirectLanes>(st, args);
}

hipError_t launch_direct(hipStream_t st, int op, const DirectArgs &args, int lanes) {
    switch (op) {
    case OP_DOT: return launch_direct_by<OP_DOT>(st, args, lanes);
    case OP_L1: return launch_direct_by<OP_L1>(st, args, lanes);
    case OP_CANB: return launch_direct_by<OP_CANB>(st, args, lanes);
    case OP_HAMM: return launch_direct_by<OP_HAMM>(st, args, lanes);
    case OP_KL: return launch_direct_by<OP_KL>(st, args, lanes);
    case OP_JS: return launch_direct_by<OP_JS>(st, args, lanes);
    case OP_CNT: return launch_direct_by<OP_CNT>(st, args, lanes);
    case OP_MINK: return launch_direct_by<OP_MINK>(st, args, lanes);
    case OP_MINK_ANY: return launch_direct_by<OP_MINK_ANY>(st, args, lanes);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace spd
