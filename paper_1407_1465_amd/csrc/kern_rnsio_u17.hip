// Calls of RNS exponentiation, moduli of up to 2048 bits.
#include "rns_io.hpp"

namespace rsagpu {
#include "rns_tables_17.inc"

hipError_t rns_crt_u17(const RnsCrtArgs &a, hipStream_t stream) { return launch_rns_crt<17, 72, 8, 80, 16>(a, stream); }
hipError_t rns_exp_u17(const RnsExpArgs &a, hipStream_t stream) { return launch_rns_exp<17, 72, 4, 80, 16>(a, stream); }
hipError_t rns_ops_u17(const RnsOpsArgs &a, hipStream_t stream) { return launch_rns_ops<17, 72, 8>(a, stream); }
}  // namespace rsagpu
