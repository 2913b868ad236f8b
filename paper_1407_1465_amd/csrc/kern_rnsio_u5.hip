// Calls of RNS exponentiation, moduli of up to 512 bits.
#include "rns_io.hpp"

namespace rsagpu {
#include "rns_tables_5.inc"

hipError_t rns_crt_u5(const RnsCrtArgs &a, hipStream_t stream) { return launch_rns_crt<5, 18, 2, 20, 4>(a, stream); }
hipError_t rns_exp_u5(const RnsExpArgs &a, hipStream_t stream) { return launch_rns_exp<5, 18, 2, 20, 4>(a, stream); }
hipError_t rns_ops_u5(const RnsOpsArgs &a, hipStream_t stream) { return launch_rns_ops<5, 18, 2>(a, stream); }
}  // namespace rsagpu
