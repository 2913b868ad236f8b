// Resident keys and operation descriptors as the device sees them.
#pragma once

#include <stdint.h>

namespace rsagpu {

// Constants of one modulus m in one radix, S limbs each: one = R mod m,
// r2 = R^2 mod m, r3 = R^3 mod m and xr = x * R mod m for a multiplier x given
// at setup.  r3 and xr are null where no kernel needs them.
struct ModConsts {
    uint32_t *one;
    uint32_t *r2;
    uint32_t *r3;
    uint32_t *xr;
};

// Device view of one resident key.
struct KeyDev {
    int cls;                  // width class index
    int words;                // 32-bit words of n
    int hwords;               // 32-bit words of p and q
    int rns;                  // p and q have no factor in common with their class's RNS base A
    const uint32_t *n, *e, *p, *q, *dp, *dq, *qinv;
    ModConsts cn[2], cp[2], cq[2];     // [0]: radix 2^32, [1]: radix 2^29
};

// One operation descriptor (layout shared with include/rsagpu.h rsa_op).
struct OpDesc {
    uint32_t kind;            // 0: in^e mod n, 1: CRT decryption
    int32_t key_id;
    unsigned long long in_off, out_off;
};

}  // namespace rsagpu
