// Calls of RNS exponentiation, moduli of up to 768 bits.
#include "rns_io.hpp"

namespace rsagpu {
#include "rns_tables_7.inc"

hipError_t rns_crt_u7(const RnsCrtArgs &a, hipStream_t stream) { return launch_rns_crt<7, 28, 4, 28, 4>(a, stream); }
hipError_t rns_exp_u7(const RnsExpArgs &a, hipStream_t stream) { return launch_rns_exp<7, 28, 4, 32, 16>(a, stream); }
hipError_t rns_ops_u7(const RnsOpsArgs &a, hipStream_t stream) { return launch_rns_ops<7, 28, 4>(a, stream); }
}  // namespace rsagpu
