// RNS exponentiation, moduli of up to 1536 bits: 13 residues per lane and base.
#include "rns_kernels.hpp"

namespace rsagpu {
#include "rns_tables_13.inc"

RSAGPU_INSTANTIATE_RNS(13)
}  // namespace rsagpu
