// Column-list kernels of the products with one sum per pair (see spd_match_impl.h).
#include "spd_match_impl.h"

namespace spd {
hipError_t launch_match_a(hipStream_t st, int op, const MatchArgs &args, uint32_t lds_bytes) {
    switch (op) {
    case OP_DOT: return launch_match_either<OP_DOT>(st, args, lds_bytes);
    case OP_L1: return launch_match_either<OP_L1>(st, args, lds_bytes);
    case OP_HAMM: return launch_match_either<OP_HAMM>(st, args, lds_bytes);
    case OP_CNT: return launch_match_either<OP_CNT>(st, args, lds_bytes);
    case OP_CANB: return launch_match_either<OP_CANB>(st, args, lds_bytes);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace spd
