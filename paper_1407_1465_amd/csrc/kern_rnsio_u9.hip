// Calls of RNS exponentiation, moduli of up to 1024 bits.
#include "rns_io.hpp"

namespace rsagpu {
#include "rns_tables_9.inc"

hipError_t rns_crt_u9(const RnsCrtArgs &a, hipStream_t stream) { return launch_rns_crt<9, 36, 4, 36, 4>(a, stream); }
hipError_t rns_exp_u9(const RnsExpArgs &a, hipStream_t stream) { return launch_rns_exp<9, 36, 2, 36, 4>(a, stream); }
hipError_t rns_ops_u9(const RnsOpsArgs &a, hipStream_t stream) { return launch_rns_ops<9, 36, 4>(a, stream); }
}  // namespace rsagpu
