// RNS exponentiation, moduli of up to 2048 bits: 17 residues per lane and base.
#include "rns_kernels.hpp"

namespace rsagpu {
#include "rns_tables_17.inc"

RSAGPU_INSTANTIATE_RNS(17)
}  // namespace rsagpu
