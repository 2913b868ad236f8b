// RNS exponentiation, moduli of up to 512 bits: 5 residues per lane and base.
#include "rns_kernels.hpp"

namespace rsagpu {
#include "rns_tables_5.inc"

RSAGPU_INSTANTIATE_RNS(5)
}  // namespace rsagpu
