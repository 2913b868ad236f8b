// RNS exponentiation, moduli of up to 768 bits: 7 residues per lane and base.
#include "rns_kernels.hpp"

namespace rsagpu {
#include "rns_tables_7.inc"

RSAGPU_INSTANTIATE_RNS(7)
}  // namespace rsagpu
