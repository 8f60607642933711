// Column-list kernels of the products with several sums per pair or with logarithms (see spd_match_impl.h).
#include "spd_match_impl.h"

namespace spd {
hipError_t launch_match_b(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes) {
    switch (op) {
    case OP_KL: return launch_match_either<OP_KL>(st, args, lds_bytes);
    case OP_JS: return launch_match_either<OP_JS>(st, args, lds_bytes);
    case OP_MINK: return launch_match_either<OP_MINK>(st, args, lds_bytes);
    case OP_CHEB: return args.knn_k > 0 ? hipErrorInvalidValue : launch_match_op<OP_CHEB, false, false>(st, args, lds_bytes);
    case OP_MINK_ANY: return launch_match_either<OP_MINK_ANY>(st, args, lds_bytes);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace spd
