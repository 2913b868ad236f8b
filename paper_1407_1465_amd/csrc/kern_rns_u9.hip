// RNS exponentiation, moduli of up to 1024 bits: 9 residues per lane and base.
#include "rns_kernels.hpp"

namespace rsagpu {
#include "rns_tables_9.inc"

RSAGPU_INSTANTIATE_RNS(9)
}  // namespace rsagpu
