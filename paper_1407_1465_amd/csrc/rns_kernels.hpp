// Exponentiation in RNS: out = x^e mod n for tiles of 16 integers.
//
// One of the kernels of a call (rns_io.hpp has the others): k_rns_pow takes
// x * A mod n from the caller's output words and leaves x^e mod n there.
#pragma once

#include "modexp_kernels.hpp"
#include "rns_arith.hpp"
#include "rns_jobs.hpp"

namespace rsagpu {

// ---- the exponentiation -------------------------------------------------------

// A table entry: 64 words per unit and base, those in A first.
template <int U>
constexpr size_t rns_slot_words() { return 2 * (size_t)U * 64; }
// LDS words outside the table: with W > 1 the three operand exchange buffers,
// and the flags of elements not to store.
template <int U, int W>
constexpr size_t rns_fixed_words() { return (W > 1 ? 3 * (size_t)Rns<U, W>::KS * 256 : 0) + 32; }
// The table's space also serves the way out (residues of 16 integers, then
// two positional integers each).
template <int U, int W>
constexpr size_t rns_lds_words(int w)
{
    const size_t slots = (size_t)1 << (w - 1);
    const size_t tab = slots * rns_slot_words<U>();
    const size_t need = 16 * (4 * U + 2) + 2 * 32 * (size_t)RnsTables<U>::LIMBS;
    return rns_fixed_words<U, W>() + (tab > need ? tab : need);
}

// x^e mod n of a tile by the left-to-right sliding window (Section 3.6.5)
// over the odd powers x^(2k+1), k < 2^(w-1), in LDS, where the tile's
// exponents are equal.  Otherwise the table holds x, x^2, ... and every
// integer takes a product after each w - 1 squarings, in windows of digits
// 1 .. 2^(w-1) (no zero digit, so that no integer has to sit one out): some
// 7% more products, in lockstep, where a schedule per integer multiplied each
// by itself or an entry as its turn came and kept the scans of 16 exponents
// in every step (200 2048-bit exponentiations with their own exponents: 4880
// us; now 2721).
//
// What bounds it: issue.  A product of a tile of 32-word integers (U = 9) on
// one wave is 57 matrix instructions (16 cycles each) and about 245 others in
// 1957 cycles: with one wave on a SIMD the two do not overlap (only a run of
// eight or more vector instructions hides a matrix instruction, and there are
// 4.3 for each; moving the next product's first half under the second
// extension, 1 matrix to 3 .. 5 vector instructions, 2333 -> 2344 .. 2601 us
// for 16384 2048-bit decryptions).  Both matrices, 228 registers of each
// lane, leave no room for a second wave on the SIMD; two waves a tile have it
// and pay two exchanges a product (3366 us).  16384 2048-bit decryptions,
// 2048 tiles: 3550 us positionally, now 2159; 1092 of 4096 bits 6277 -> 2304.
template <int U, int W, int OCC, typename Source>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(OCC))) void k_rns_pow(Source src, int w)
{
    using C = Rns<U, W>;
    using T = RnsTables<U>;
    constexpr int UW = C::UW, KS = C::KS, S = T::LIMBS, K = C::K, CH = rns_chunk<S>();
    uint32_t *lds = reinterpret_cast<uint32_t *>(rsagpu_lds);
    int wave = W == 1 ? 0 : (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // Two workgroups share a CU at W = 4, and wave 0 has a unit more than the
    // others where U = 13: turned by two in every other one, so that the long
    // waves are not on one SIMD (4096 3072-bit decryptions 2075 -> 2037 us).
    if constexpr (W == 4) wave = (wave + 2 * (int)((blockIdx.x ^ blockIdx.y) & 1)) & 3;
    // units wave, wave + W, ...: the last is past U in the later waves where W
    // does not divide U, and those pass over it (every wave worked on UW units
    // at first, padding too: with 9 waves for 17 units the SIMD with a third
    // wave had 6 units to do, now 5.  1092 4096-bit decryptions 2496 -> 2300
    // us, 4096 of 3072 bits, 13 units on 4 waves, 2319 -> 2075).
    constexpr bool kPadded = UW * W != U;
    const bool full = !kPadded || wave + W * (UW - 1) < U;
    auto unit_of = [&](int i) { return wave + W * i; };
    v4i *exch = reinterpret_cast<v4i *>(lds);            // [3][KS][64]
    uint32_t *nostore = lds + rns_fixed_words<U, W>() - 32;
    uint32_t *area = lds + rns_fixed_words<U, W>();
    constexpr int STRIDE = (int)rns_slot_words<U>();     // words between table entries
    constexpr int UNIT = W * 64, BASE_B = U * 64;        // and within one, between a wave's units, and to base B

    if (src.idle()) return;
    unsigned long long tile = blockIdx.x;
    do {
    int lane = (int)__lane_id();
    // opaque: what depends on the lane alone (the tables' words) is not
    // hoisted out of the loop over tiles, where it would not fit the registers
    if constexpr (Source::kLoop) asm volatile("" : "+v"(lane));
    const int g = lane >> 4;
    int *tab = reinterpret_cast<int *>(area) + wave * 64 + lane;
    const RnsJob job = src.job(tile, lane & 15);
    tile += gridDim.x;
    if (__ballot(job.live) == 0) continue;               // the same for every wave of the tile
    if constexpr (W > 1 && Source::kLoop) __syncthreads();       // the tile before has left LDS
    if (threadIdx.x < 16) nostore[threadIdx.x] = 0u;
    if constexpr (W > 1) {
        for (int i = (int)threadIdx.x; i < 3 * KS * 64; i += 64 * W) exch[i] = v4i{0, 0, 0, 0};
        __syncthreads();
    } else {
        lds_sync();
    }

    // ---- residues of n and x, and the products' constants
    int ma[UW], na[UW], mb[UW], nb[UW], kap[UW], c[UW], v[UW], v16[UW], xa[UW], xb[UW];
    int at[UW];
#pragma unroll
    for (int i = 0; i < UW; ++i) {
        const int u = unit_of(i) < U ? unit_of(i) : U - 1;       // padding repeats the last unit
        at[i] = g * U + u;
        ma[i] = (int)T::ma()[at[i]];
        na[i] = (int)T::na()[at[i]];
        mb[i] = (int)T::mb()[at[i]];
        nb[i] = (int)T::nb()[at[i]];
        c[i] = v[i] = xa[i] = xb[i] = 0;
    }
    {
        const uint32_t *ca = T::ca(), *cb = T::cb();
#pragma unroll 1
        for (int l0 = 0; l0 < S; l0 += CH) {
            int64_t tc[UW], tv[UW], ta[UW], tb[UW];
#pragma unroll
            for (int i = 0; i < UW; ++i) {
                const int ka = (int)(0u - 2u * (uint32_t)ma[i]), kb = (int)(0u - 2u * (uint32_t)mb[i]);   // 2^32 mod m
                tc[i] = (int64_t)c[i] * ka;
                ta[i] = (int64_t)xa[i] * ka;
                tv[i] = (int64_t)v[i] * kb;
                tb[i] = (int64_t)xb[i] * kb;
            }
#pragma unroll
            for (int l = 0; l < CH; ++l) {
                const int pos = 29 * (l0 + l), wd = pos >> 5, sh = pos & 31;
                auto limb = [&](const uint32_t *p) -> int {
                    const uint32_t lo = wd < job.words ? p[wd] : 0u, hi = wd + 1 < job.words ? p[wd + 1] : 0u;
                    return (int)((uint32_t)((((uint64_t)hi << 32) | lo) >> sh) & Radix<29>::MASK);
                };
                const int ln = limb(job.n), lx = limb(job.io);
#pragma unroll
                for (int i = 0; i < UW; ++i) {
                    const int ka = (int)ca[(l0 + l) * K + at[i]], kb = (int)cb[(l0 + l) * K + at[i]];
                    tc[i] += (int64_t)ln * ka;
                    ta[i] += (int64_t)lx * ka;
                    tv[i] += (int64_t)ln * kb;
                    tb[i] += (int64_t)lx * kb;
                }
            }
#pragma unroll
            for (int i = 0; i < UW; ++i) {
                c[i] = rns_red(tc[i], ma[i], na[i]);
                xa[i] = rns_red(ta[i], ma[i], na[i]);
                v[i] = rns_red(tv[i], mb[i], nb[i]);
                xb[i] = rns_red(tb[i], mb[i], nb[i]);
            }
        }
        // c = -n^-1 (A / a)^-1 (scaled): n^(a - 2) by squarings
        int inv[UW];
        bool zero = false;
#pragma unroll
        for (int i = 0; i < UW; ++i) {
            c[i] = rns_red((int64_t)c[i] * (int)T::r2a()[at[i]], ma[i], na[i]);    // n * 2^32
            zero = zero || c[i] == 0;
            inv[i] = c[i];
            xb[i] = rns_red((int64_t)xb[i] * (int)T::wr()[at[i]], mb[i], nb[i]);
            kap[i] = (int)T::kappa()[at[i]];
            v[i] = rns_red((int64_t)v[i] * (int)(0u - 2u * (uint32_t)mb[i]), mb[i], nb[i]);   // below b / 2 + 2^12
            v16[i] = rns_red((int64_t)v[i] * (int)T::v16()[at[i]], mb[i], nb[i]);
        }
#pragma unroll 1
        for (int bit = 29; bit >= 0; --bit) {            // a - 2 has 31 bits
#pragma unroll
            for (int i = 0; i < UW; ++i) {
                inv[i] = rns_red((int64_t)inv[i] * inv[i], ma[i], na[i]);
                const int m = rns_red((int64_t)inv[i] * c[i], ma[i], na[i]);
                inv[i] = ((ma[i] - 2) >> bit) & 1 ? m : inv[i];
            }
        }
#pragma unroll
        for (int i = 0; i < UW; ++i) c[i] = rns_red((int64_t)inv[i] * (int)T::cinv()[at[i]], ma[i], na[i]);
        if (zero) nostore[lane & 15] = 1u;
    }

    // ---- exponents
    int ebits = 0;
    bool uniform;
    {
        bool same = true;
        const int most = (int)wave_max((uint32_t)job.words);     // (an ops bucket's keys may differ in words)
        for (int k = 0; k < most; ++k) {
            const uint32_t ev = k < job.words ? job.e[k] : 0u;
            if (ev) ebits = 32 * k + 32 - __clz(ev);
            same = same && ev == (uint32_t)__builtin_amdgcn_readfirstlane((int)ev);
        }
        uniform = __ballot(!same) == 0;
    }
    const bool zero_exp = ebits == 0;
    ExpBits eb{job.e, job.words, 0, 0, 0};
    int pos = ebits - 1, sq = 0, mi = -1;
    auto next_window = [&]() {                           // as in group_modexp
        eb.seek(pos);
        if (((uint32_t)(eb.bits >> (pos - 32 * (eb.kw - 1))) & 1u) == 0u) {
            sq = 1;
            mi = -1;
            pos -= 1;
            return;
        }
        const int lo0 = pos - w + 1 > 0 ? pos - w + 1 : 0;
        uint32_t val = eb.field(pos, lo0);
        const int tz = __builtin_ctz(val);
        val >>= tz;
        sq = pos - (lo0 + tz) + 1;
        mi = (int)(val >> 1);
        pos = lo0 + tz - 1;
    };

    // ---- the extensions' matrices, held in registers
    v4i eab[UW][KS], eba[UW][KS], esum[W == 1 ? KS : 1];
#pragma unroll
    for (int i = 0; i < UW; ++i)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int u = unit_of(i) < U ? unit_of(i) : U - 1;
            eab[i][s] = C::matrix_word(T::eab(), u, s, lane);
            eba[i][s] = C::matrix_word(T::eba(), u, s, lane);
            asm volatile("" : "+a"(eab[i][s]), "+a"(eba[i][s]));
        }
    if constexpr (W == 1) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            esum[s] = C::matrix_word(T::eba(), U, s, lane);
            asm volatile("" : "+a"(esum[s]));
        }
    }

    // Operand of an extension from the digits of every wave's residues.  With
    // W > 1 they go through LDS: buffer 0 for A -> B, and for B -> A buffers
    // 1 and 2 in turn, since the sum of the top digits gathers (by LDS
    // atomics) in the word that becomes alpha and has to be cleared before
    // its next use: the product after does so between its two barriers.
    int alpha = 0, turn = 1;
    auto exchange = [&](v4i (&op)[KS], const int (&dig)[UW], bool back) {
        if constexpr (W == 1) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) op[s][j] = 4 * s + j < UW ? dig[(4 * s + j) % UW] : 0;
        } else {
            int *b = reinterpret_cast<int *>(exch + (back ? turn : 0) * KS * 64);
            int sum = 0;
#pragma unroll
            for (int i = 0; i < UW; ++i)
                if (i < UW - 1 || full) {
                    b[(unit_of(i) / 4 * 64 + lane) * 4 + unit_of(i) % 4] = dig[i];
                    sum += dig[i] >> 24;
                }
            constexpr int at_alpha = U % 4;
            if (back) atomicAdd(&b[(U / 4 * 64 + (lane & 15)) * 4 + at_alpha], sum);
            __syncthreads();
#pragma unroll
            for (int s = 0; s < KS; ++s) op[s] = reinterpret_cast<const v4i *>(b)[s * 64 + lane];
            if (back) {
                turn = 3 - turn;
            } else if (wave == 0 && lane < 16) {
                int *n = reinterpret_cast<int *>(exch + (3 - turn) * KS * 64);
                n[(U / 4 * 64 + lane) * 4 + at_alpha] = 0;
            }
        }
    };
    auto each_unit = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < UW - (kPadded ? 1 : 0); ++i) f(i);
        if constexpr (kPadded) {
            if (full) f(UW - 1);
        }
    };
    // x = x * y * A^-1 mod n, y = x (SQR) or the table entry at yt.
    auto product = [&](auto SQR, const int *yt) {
        constexpr bool kSqr = decltype(SQR)::value;
        // Opaque here, so that no 64-bit extension of a constant is made
        // outside the loop: a product with one is lowered as 64 by 32 bits.
#pragma unroll
        for (int i = 0; i < UW; ++i)
            asm volatile("" : "+v"(ma[i]), "+v"(na[i]), "+v"(mb[i]), "+v"(nb[i]), "+v"(c[i]), "+v"(v[i]), "+v"(v16[i]),
                         "+v"(kap[i]));
        int64_t bias = (int64_t)kDigitBias << 32;
        asm volatile("" : "+s"(bias));
        int dig[UW];
        each_unit([&](int i) {
            int y = xa[i];
            if constexpr (!kSqr) y = yt[i * UNIT];
            const int s = rns_red((int64_t)xa[i] * y, ma[i], na[i]);
            dig[i] = rns_digits(rns_red((int64_t)s * c[i] + bias, ma[i], na[i]));
        });
        v4i op[KS];
        exchange(op, dig, false);
        each_unit([&](int i) {
            const v4i q = C::tile(eab[i], op);
            int y = xb[i];
            if constexpr (!kSqr) y = yt[BASE_B + i * UNIT];
            const int s = rns_red((int64_t)xb[i] * y, mb[i], nb[i]);
            xb[i] = rns_red((int64_t)s * kap[i] + (int64_t)rns_lo(q) * v[i] + (int64_t)rns_hi(q) * v16[i], mb[i], nb[i]);
            dig[i] = rns_digits(xb[i] + kDigitBias);
        });
        exchange(op, dig, true);
        // alpha, in lanes 0 .. 15 (zero elsewhere): unit U of the operand
        if constexpr (W == 1) alpha = (C::tile(esum, op)[0] + 64) >> 7;
        else alpha = (op[KS - 1][U % 4] + 64) >> 7;
        op[KS - 1][U % 4] = alpha;
        v4i accs[UW];
#pragma unroll
        for (int i = 0; i < UW - (kPadded ? 1 : 0); ++i) accs[i] = C::tile(eba[i], op);
#pragma unroll
        for (int i = 0; i < UW - (kPadded ? 1 : 0); ++i) xa[i] = rns_red(rns_planes(accs[i]), ma[i], na[i]);
        if constexpr (kPadded) {
            if (full) xa[UW - 1] = rns_red(rns_planes(C::tile(eba[UW - 1], op)), ma[UW - 1], na[UW - 1]);
        }
    };
    auto put = [&](int slot) {
        each_unit([&](int i) {
            tab[slot * STRIDE + i * UNIT] = xa[i];
            tab[slot * STRIDE + BASE_B + i * UNIT] = xb[i];
        });
    };
    auto get = [&](int slot) {
        each_unit([&](int i) {
            xa[i] = tab[slot * STRIDE + i * UNIT];
            xb[i] = tab[slot * STRIDE + BASE_B + i * UNIT];
        });
    };

    constexpr std::true_type SQUARE{};
    constexpr std::false_type TIMES{};
    const int tsize = 1 << (w - 1);
    put(0);
    if (uniform) {
        // odd powers: entry 0 = x, entry k = entry k-1 times x^2, which waits
        // in the last entry
        if (tsize > 1) {
            product(SQUARE, tab);
            put(tsize - 1);
            get(0);
#pragma unroll 1
            for (int k = 1; k < tsize; ++k) {
                product(TIMES, tab + (tsize - 1) * STRIDE);
                put(k);
            }
        }
        eb = ExpBits{first_lane_ptr(job.e), __builtin_amdgcn_readfirstlane(job.words), 0, 0, 0};
        pos = __builtin_amdgcn_readfirstlane(ebits) - 1;
        if (pos >= 0) {
            eb.start(pos);
            next_window();                               // the leading window sets x
            get(__builtin_amdgcn_readfirstlane(mi));
        }
#pragma unroll 1
        while (__builtin_amdgcn_readfirstlane(pos) >= 0) {
            next_window();
            const int nsq = __builtin_amdgcn_readfirstlane(sq), ent = __builtin_amdgcn_readfirstlane(mi);
#pragma unroll 1
            for (int k = 0; k < nsq; ++k) product(SQUARE, tab);
            if (ent >= 0) product(TIMES, tab + ent * STRIDE);
        }
    } else {
        // all powers: entry k = x^(k+1)
#pragma unroll 1
        for (int k = 1; k < tsize; ++k) {
            product(TIMES, tab);
            put(k);
        }
        // e = sum of (d_i + 1) 2^(f i), i < len: d_i are the base-2^f digits of
        // e less a one in every window.  len is the windows of e, or one
        // less where that difference is negative; borrow bit k is what word
        // k - 1 of the subtraction takes from word k.
        const int f = w - 1;
        auto ones = [&](int k) -> uint32_t {             // the bits 32 k .. 32 k + 31 of the subtrahend
            if (f == 4) return 0x11111111u;
            const int r = k % 3;
            return r == 0 ? 0x49249249u : r == 1 ? 0x92492492u : 0x24924924u;
        };
        int len = (ebits + f - 1) / f;
        uint64_t borrows = 0;
        {
            uint32_t b = 0;
            for (int k = 0; k < job.words; ++k) {
                const int top = f * len - 32 * k;        // windows end here
                const uint32_t c = top >= 32 ? ones(k) : top > 0 ? ones(k) & ((1u << top) - 1u) : 0u;
                borrows |= (uint64_t)b << k;
                b = (uint32_t)(((uint64_t)job.e[k] - c - b) >> 63);
            }
            len -= (int)b;
        }
        int win = (int)wave_max((uint32_t)len) - 1;
        const int first = win;
#pragma unroll 1
        for (; win >= 0; --win) {
            const int p = f * win, k = p >> 5;
            const uint32_t e0 = k < job.words ? job.e[k] : 0u, e1 = k + 1 < job.words ? job.e[k + 1] : 0u;
            if (win != first) {
#pragma unroll 1
                for (int j = 0; j < f; ++j) product(SQUARE, tab);
            }
            const uint32_t lo = e0 - ones(k) - (uint32_t)((borrows >> k) & 1u);
            const uint32_t hi = k + 1 < job.words ? e1 - ones(k + 1) - (uint32_t)((borrows >> (k + 1)) & 1u) : 0u;
            const int d = (int)((uint32_t)((((uint64_t)hi << 32) | lo) >> (p & 31)) & (uint32_t)(tsize - 1));
            if (win != first) product(TIMES, tab + d * STRIDE);
            if (win == len - 1) get(d);                  // this integer's leading window
        }
    }
    // times one: leave the Montgomery domain
    each_unit([&](int i) {
        tab[i * UNIT] = 1;
        tab[BASE_B + i * UNIT] = (int)T::wone()[at[i]];
    });
    product(TIMES, tab);

    // ---- the way out: x = sum_j xb_j (B / b_j) - alpha B in 29-bit limbs,
    // made positive (terms xb_j + b_j, and 64 n), then reduced modulo n
    uint32_t *res = area, *pos_buf = area + 16 * (K + 1);
    if constexpr (W > 1) __syncthreads();
    else lds_sync();
#pragma unroll
    for (int i = 0; i < UW; ++i)
        if (i < UW - 1 || full) res[(lane & 15) * (K + 1) + 4 * unit_of(i) + g] = (uint32_t)(xb[i] + mb[i]);
    if (wave == 0 && lane < 16) res[lane * (K + 1) + K] = (uint32_t)(alpha + K);
    if constexpr (W > 1) __syncthreads();
    else lds_sync();
    if (wave != 0) continue;

    constexpr int G = S % 4 == 0 ? 4 : 2, L = S / G;
    using Ar = Arith<S, G, 29>;
    const int gi = (int)grp_index<G>() & 15, r = (int)grp_lane<G>();
    auto from = [&](const void *ptr) {
        const uint64_t a = reinterpret_cast<uint64_t>(ptr);
        const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)a, gi), hi = (uint32_t)__shfl((int)(uint32_t)(a >> 32), gi);
        return ((uint64_t)hi << 32) | lo;
    };
    const uint32_t *np = reinterpret_cast<const uint32_t *>(from(job.n));
    uint32_t *op = reinterpret_cast<uint32_t *>(from(job.io));
    const bool live = __shfl((int)job.live, gi) != 0 && (int)grp_index<G>() < 16 && nostore[gi] == 0u;
    const bool unit = __shfl((int)zero_exp, gi) != 0;
    const int words = __shfl(job.words, gi);
    uint32_t n[L], x[L];
    Ar::load(n, np, words, 0, true);
    {
        uint64_t acc[L], hi[L];
#pragma unroll
        for (int k = 0; k < L; ++k) {
            acc[k] = (uint64_t)n[k] << 6;
            hi[k] = 0;
        }
        const uint32_t *tp = T::pos() + r * L;
#pragma unroll 1
        for (int j0 = 0; j0 <= K; j0 += 6) {
#pragma unroll
            for (int j = j0; j < j0 + 6; ++j) {
                const int jj = j <= K ? j : K;
                const uint32_t m = j <= K ? res[gi * (K + 1) + jj] : 0u;
#pragma unroll
                for (int k = 0; k < L; ++k) acc[k] += (uint64_t)m * tp[jj * S + k];
            }
#pragma unroll
            for (int k = 0; k < L; ++k) {
                hi[k] += acc[k] >> 29;
                acc[k] &= Radix<29>::MASK;
            }
        }
        const uint32_t clo = grp_from_below<G>((uint32_t)hi[L - 1]), chi = grp_from_below<G>((uint32_t)(hi[L - 1] >> 32));
        acc[0] += ((uint64_t)chi << 32) | clo;
#pragma unroll
        for (int k = 1; k < L; ++k) acc[k] += hi[k - 1];
        (void)racc_normalise<S, G, 29>(x, acc);
    }
    const int bl = (int)Ar::bitlen(n);
    const double rn = 1.0 / rgrp_scaled<S, G, 29>(n, 0u, bl);
    rgrp_sub_multiple<S, G, 29>(x, 0u, n, rn, bl);
    if (unit) {
#pragma unroll
        for (int k = 0; k < L; ++k) x[k] = r == 0 && k == 0 ? 1u : 0u;
    }
    store_words<S, G, 29>(op, x, words, live, true, pos_buf);
    lds_sync();
    } while (Source::kLoop && tile < src.tiles());
}

// ---- launchers ------------------------------------------------------------------

template <int U, int W, int OCC, typename Source>
hipError_t launch_rns_pow(const Source &src, dim3 grid, int w, hipStream_t stream)
{
    const size_t lds = rns_lds_words<U, W>(w) * sizeof(uint32_t);
    if (lds > kMaxGroupLds) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_rns_pow<U, W, OCC, Source>), grid, dim3(64 * W), lds, stream, src, w);
    return hipGetLastError();
}

// Waves per tile for `tiles` x `halves` tiles on `cus` CUs.  A tile's chain of
// products is the same length however many waves share it, and each product
// costs two exchanges through LDS where they are more than one: many waves
// (one or two residues per lane and base each) where every tile has a CU of
// its own, and one wave, or the fewest whose matrices fit the registers,
// where the tiles fill the chip.  CRT decryptions, us: 2048-bit keys, 5
// messages 1153 with one wave, 828 with 3, 711 with 9; 4096 messages (512
// tiles) 1278 with one, 1103 with 3, 1099 with 4 and (9 waves) two rounds;
// 16384 messages 2159 with one and 3402 with 3.  3072-bit keys, 777 messages
// (114 tiles) 1454 with 13 waves, 1580 with 7, 1779 with 5; 4096 messages 2037
// with 4 waves (two tiles a CU; 3416 with one), 2492 with 2, 3357 with 5, 3889
// with 3; 16384 messages 8123 with 4 and 9678 with 2.  4096-bit keys, 1092
// messages 2301 with 9 waves, 2330 with 8, 2353 with 12; 4368 messages 6463,
// 6517 and 6643 (6 and 4 waves were 6 and 18% above 9).  The window is the
// widest whose table leaves LDS for the workgroups a CU is to hold.
template <int U, typename Source>
hipError_t launch_rns_tiles(const Source &src, size_t tiles, unsigned halves, int cus, hipStream_t stream)
{
    const size_t all = tiles * halves, cu = (size_t)(cus > 0 ? cus : 1);
    const dim3 grid((unsigned)tiles, halves);
    // the most resident workgroups (per_cu per CU), each taking several tiles
    // of a plain exponentiation call
    const auto resident = [&](size_t per_cu) {
        return dim3((unsigned)(tiles > per_cu * cu ? per_cu * cu : tiles));
    };
    if constexpr (U == 5) {
        return launch_rns_pow<U, 1, 1>(src, grid, 4, stream);
    } else if constexpr (U == 7) {
        if (all <= cu) return launch_rns_pow<U, 7, 4>(src, grid, 4, stream);
        if constexpr (Source::kExp) return launch_rns_pow<U, 1, 1>(src.looping(), resident(4), 4, stream);
        return launch_rns_pow<U, 1, 1>(src, grid, 4, stream);
    } else if constexpr (U == 9) {
        if (all <= cu) return launch_rns_pow<U, 9, 4>(src, grid, 5, stream);
        if (all <= 2 * cu) return launch_rns_pow<U, 3, 2>(src, grid, 4, stream);
        if constexpr (Source::kExp) return launch_rns_pow<U, 1, 1>(src.looping(), resident(4), 4, stream);
        return launch_rns_pow<U, 1, 1>(src, grid, 4, stream);
    } else if constexpr (U == 13) {
        if (all <= cu) return launch_rns_pow<U, 13, 4>(src, grid, 5, stream);
        if constexpr (Source::kExp) return launch_rns_pow<U, 4, 2>(src.looping(), resident(2), 4, stream);
        return launch_rns_pow<U, 4, 2>(src, grid, 4, stream);
    } else {
        static_assert(U == 17, "a configuration of rns_tables.py");
        return launch_rns_pow<U, 9, 2>(src, grid, 5, stream);
    }
}

// The halves of an ops batch's CRT bucket, whose size only the device knows:
// a workgroup for each tile it may have, of which those past the end leave at
// once (the resident workgroups taking several tiles each, in strides set
// before the others' speed is known, made three rounds out of two beside other
// buckets: mixed 32768-operation batch 6.2 ms, now 5.95).  A bulk batch takes
// the shape for many tiles, whatever a bucket holds.  For a smaller batch both
// shapes are launched, and the bucket's size decides which one's workgroups
// leave (beside other buckets' waves even those wait for a CU with room: in a
// bulk batch the empty launches of nine-wave workgroups held the 2048-bit
// bucket back by 3 ms).
constexpr size_t kBucketTiles = (size_t)1 << 20;     // a launch (2^32 threads a dimension at most)
template <int U>
hipError_t launch_rns_bucket(RnsOpsSource src, size_t tiles, bool bulk, int cus, hipStream_t stream)
{
    const size_t few = bulk ? 0 : (size_t)(cus > 1 ? cus : 2) / 2;
    hipError_t e = hipSuccess;
    if constexpr (U == 7 || U == 9 || U == 13) {
        constexpr int w = U == 7 ? 4 : 5;
        src.upto = (unsigned)few;
        if (few) e = launch_rns_pow<U, U, 4>(src, dim3((unsigned)(tiles < few ? tiles : few), 2), w, stream);
        if (e != hipSuccess || tiles <= few) return e;
        src.above = (unsigned)few;
        src.upto = ~0u;
    }
    for (size_t at = 0; at < tiles && e == hipSuccess; at += kBucketTiles) {
        const dim3 grid((unsigned)(tiles - at < kBucketTiles ? tiles - at : kBucketTiles), 2);
        src.skip = (unsigned)at;
        if constexpr (U == 17) e = launch_rns_pow<U, 9, 2>(src, grid, 5, stream);
        else if constexpr (U == 13) e = launch_rns_pow<U, 4, 2>(src, grid, 4, stream);
        else e = launch_rns_pow<U, 1, 1>(src, grid, 4, stream);
    }
    return e;
}

#define RSAGPU_INSTANTIATE_RNS(U_)                                                                              \
    template <>                                                                                                 \
    hipError_t rns_pow<U_>(const RnsCrtSource &src, size_t tiles, unsigned halves, int cus, hipStream_t stream) \
    {                                                                                                           \
        return launch_rns_tiles<U_>(src, tiles, halves, cus, stream);                                           \
    }                                                                                                           \
    template <>                                                                                                 \
    hipError_t rns_pow<U_>(const RnsExpSource<false> &src, size_t tiles, unsigned halves, int cus, hipStream_t stream) \
    {                                                                                                           \
        return launch_rns_tiles<U_>(src, tiles, halves, cus, stream);                                           \
    }                                                                                                           \
    template <>                                                                                                 \
    hipError_t rns_pow_bucket<U_>(const RnsOpsSource &src, size_t tiles, bool bulk, int cus,             \
                                  hipStream_t stream)                                                           \
    {                                                                                                           \
        return launch_rns_bucket<U_>(src, tiles, bulk, cus, stream);                                            \
    }

}  // namespace rsagpu
