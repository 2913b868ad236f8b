// What the RNS exponentiation (rns_kernels.hpp) works on: tiles of 16 jobs, and
// where a call's jobs are found.
#pragma once

#include "launch.hpp"
#include "keyset_types.hpp"

namespace rsagpu {

// One exponentiation of a tile: io holds x * A mod n, then the result.
struct RnsJob {
    const uint32_t *n;
    const uint32_t *e;
    uint32_t *io;
    int words;                 // 32-bit words of n, io and e
    bool live;                 // false: no element (the pointers are another's)
};

// Limbs per reduction of a sum of limb * constant products: at most 7 keep
// 7 * 2^59 + 2^44 below 2^63 and the reduced word below 0.95 * 2^31.
template <int S>
constexpr int rns_chunk() { return S % 6 == 0 ? 6 : 7; }

// Jobs of a plain CRT call: tile t holds 16 slots of the processing order
// (kOrderHole: none; the identity without an order); blockIdx.y is the half
// (0: p, 1: q).
struct RnsCrtSource {
    const uint32_t *p, *q, *dp, *dq;
    const unsigned *order;
    uint32_t *out;
    unsigned long long slots;
    int hl;
    static constexpr bool kLoop = false, kExp = false;
    __device__ __forceinline__ unsigned long long tiles() const { return (slots + 15) / 16; }
    __device__ __forceinline__ bool idle() const { return false; }
    __device__ __forceinline__ RnsJob job(unsigned long long tile, int i) const
    {
        const unsigned long long first = tile * 16;
        auto at = [&](int k) -> unsigned {
            const unsigned long long s = first + (unsigned)k;
            return s >= slots ? kOrderHole : (order ? order[s] : (unsigned)s);
        };
        unsigned m = at(i);
        RnsJob j;
        j.live = m != kOrderHole;
        // an empty slot computes the tile's first message again
        const uint64_t any = __ballot(j.live);
        if (!j.live) m = any ? at(__builtin_ctzll(any) & 15) : 0u;
        const size_t hoff = (size_t)m * (size_t)hl;
        const bool second = blockIdx.y != 0;
        j.n = (second ? q : p) + hoff;
        j.e = (second ? dq : dp) + hoff;
        j.io = out + 2 * hoff + (second ? 0 : hl);
        j.words = hl;
        return j;
    }
};

// Jobs of a plain exponentiation call, elements in the given order.  Exponents
// of at most kRnsMinBits bits are k_rns_enter's, and so are even moduli.
// LOOP: a workgroup takes every gridDim.x-th tile; else there is one per tile.
template <bool LOOP>
struct RnsExpSource {
    const uint32_t *mod, *exp;
    uint32_t *out;
    unsigned long long count;
    int limbs;
    static constexpr bool kLoop = LOOP, kExp = true;
    RnsExpSource<true> looping() const { return {mod, exp, out, count, limbs}; }
    __device__ __forceinline__ unsigned long long tiles() const { return (count + 15) / 16; }
    // True where every exponent of the workgroup's tiles is short (all its
    // threads call it): the workgroups of a call of encryptions end at once.
    // No more than a latency of memory or two: 16 threads look at a word each
    // of the tile's 16 exponents.
    __device__ __forceinline__ bool idle() const
    {
        const int i = (int)threadIdx.x & 15, k0 = kRnsMinBits / 32 + ((int)threadIdx.x >> 4), dk = (int)blockDim.x >> 4;
        uint32_t any = 0;
        for (unsigned long long t = blockIdx.x; t < tiles(); t += gridDim.x) {
            const unsigned long long m = t * 16 + (unsigned)i;
            const uint32_t *e = exp + (m < count ? m : t * 16) * (unsigned long long)limbs;
#pragma unroll 8
            for (int k = k0; k < limbs; k += dk) any |= e[k];
        }
        return blockDim.x > 64 ? __syncthreads_or((int)any) == 0 : __ballot(any != 0u) == 0;
    }
    __device__ __forceinline__ RnsJob job(unsigned long long tile, int i) const
    {
        const unsigned long long first = tile * 16, at = first + (unsigned)i, m = at < count ? at : first;
        const size_t off = (size_t)m * (size_t)limbs;
        RnsJob j;
        j.n = mod + off;
        j.e = exp + off;
        j.io = out + off;
        j.words = limbs;
        bool wide = false;
        for (int k = kRnsMinBits / 32; k < limbs; ++k) wide = wide || j.e[k] != 0u;
        j.live = at < count && wide && (j.n[0] & 1u);
        return j;
    }
};

// Jobs of one CRT bucket of an ops batch (its list and size are on the device);
// blockIdx.y is the half.  The bucket is this launch's where its tiles number
// above `above` and at most `upto` (launches of several shapes follow each
// other, and the bucket's size picks one).
struct RnsOpsSource {
    const KeyDev *keys;
    const OpDesc *ops;
    const unsigned *list, *size;
    uint32_t *mid;
    unsigned above, upto;
    unsigned skip;                      // tiles before the launch's first
    static constexpr bool kLoop = false;
    __device__ __forceinline__ unsigned long long tiles() const
    {
        const unsigned t = (*size + 15u) / 16u;
        return t > above && t <= upto ? t : 0u;
    }
    __device__ __forceinline__ bool idle() const { return blockIdx.x + skip >= tiles(); }
    __device__ __forceinline__ RnsJob job(unsigned long long tile, int i) const
    {
        const unsigned first = ((unsigned)tile + skip) * 16u, idx = first + (unsigned)i;
        const unsigned at = idx < *size ? list[idx] : kOrderHole;
        RnsJob j;
        j.live = at != kOrderHole;
        const unsigned o = j.live ? at : list[first];            // a tile's first entry is never a hole
        const KeyDev &k = keys[ops[o].key_id];
        j.live = j.live && k.rns != 0;                           // (k_rns_enter_ops has done the others)
        const bool second = blockIdx.y != 0;
        j.n = second ? k.q : k.p;
        j.e = second ? k.dq : k.dp;
        j.words = k.hwords;
        // opaque: recomputed from the operation's number, the way out's address
        // cost the products' loop 1 to 2% (3000 2048-bit decryptions 1336 -> 1365
        // us; again 1332)
        unsigned long long off = (unsigned long long)o * kMidWords;
        asm volatile("" : "+v"(off));
        j.io = mid + off + (second ? 0 : k.hwords);
        return j;
    }
};

// k_rns_pow over `tiles` x `halves` tiles of a source, by configuration
// (residues per lane and base); defined in kern_rns_u*.hip.
template <int U>
hipError_t rns_pow(const RnsCrtSource &src, size_t tiles, unsigned halves, int cus, hipStream_t stream);
template <int U>
hipError_t rns_pow(const RnsExpSource<false> &src, size_t tiles, unsigned halves, int cus, hipStream_t stream);
// ... over a bucket of at most `tiles` tiles.
template <int U>
hipError_t rns_pow_bucket(const RnsOpsSource &src, size_t tiles, bool bulk, int cus, hipStream_t stream);

}  // namespace rsagpu
