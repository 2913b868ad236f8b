// Calls of RNS exponentiation, moduli of up to 1536 bits.
#include "rns_io.hpp"

namespace rsagpu {
#include "rns_tables_13.inc"

hipError_t rns_crt_u13(const RnsCrtArgs &a, hipStream_t stream) { return launch_rns_crt<13, 56, 8, 64, 16>(a, stream); }
hipError_t rns_exp_u13(const RnsExpArgs &a, hipStream_t stream) { return launch_rns_exp<13, 56, 8, 56, 8>(a, stream); }
hipError_t rns_ops_u13(const RnsOpsArgs &a, hipStream_t stream) { return launch_rns_ops<13, 56, 8>(a, stream); }
}  // namespace rsagpu
