// The ways into and out of RNS exponentiation, and the launchers of whole calls.
//
// A call runs up to three kernels on the same stream.  k_rns_enter_*
// (positional, lane groups of radix_bn.hpp) turns each input x into x * A
// mod n, the Montgomery form for base A, k_rns_pow (rns_kernels.hpp)
// exponentiates it in RNS, and for CRT k_rns_leave_crt recombines the halves.
// The intermediate integers of a plain call live in the caller's output words,
// so it needs no scratch memory; those of an ops batch, whose operations may
// name the same output, in its workspace.
//
// The positional kernels are bound by their own chains (a wave's Montgomery
// set-up, some 30 products), not by memory: of 2159 us for 16384 2048-bit
// decryptions the way in takes 72 and the way out 36, of 711 us for few
// messages 38 and 27.
//
// A modulus that shares a factor with base A has no inverse there (a random
// one, odds 2^-25); k_rns_enter_* finds such elements, exponentiates them
// positionally and leaves the result; k_rns_pow finds them again (a zero
// residue) and does not store.
#pragma once

#include "keyset_kernels.hpp"
#include "modexp_kernels.hpp"
#include "rns_arith.hpp"
#include "rns_jobs.hpp"

namespace rsagpu {

// True where the group's n (radix 2^29 limbs) has no common factor with base
// A.  buf: S words per group.
template <int S, int G, int U>
__device__ __forceinline__ bool rns_coprime(const uint32_t (&n)[S / G], uint32_t *buf)
{
    using T = RnsTables<U>;
    constexpr int L = S / G, K = 4 * U, CH = rns_chunk<T::LIMBS>();
    const int r = grp_lane<G>();
    uint32_t *q = buf + grp_index<G>() * S;
    lds_sync();
#pragma unroll
    for (int k = 0; k < L; ++k) q[r * L + k] = n[k];
    lds_sync();
    bool zero = false;
    for (int i = r; i < K; i += G) {
        const int m = (int)T::ma()[i], mi = (int)T::na()[i], k32 = (int)(0u - 2u * (uint32_t)m);
        int v = 0;
        for (int l0 = 0; l0 < T::LIMBS; l0 += CH) {
            int64_t t = (int64_t)v * k32;
#pragma unroll
            for (int l = 0; l < CH; ++l) t += (int64_t)(int)q[l0 + l] * (int)T::ca()[(l0 + l) * K + i];
            v = rns_red(t, m, mi);
        }
        zero = zero || v == 0 || v == m || v == -m;
    }
    lds_sync();
    return !grp_any<G>(zero);
}

// Waves per workgroup of the kernels here: one per SIMD of a CU.  One-wave
// workgroups have been measured to share SIMDs after a launch of larger ones
// (16384 2048-bit encryptions, 1024 waves: 289 us in one-wave workgroups
// between launches of k_rns_pow, 163 us in workgroups of four).
constexpr int kIoWaves = 4;

// The calling wave's LDS region, as of a workgroup at window w.
template <int S, int G>
__device__ __forceinline__ uint32_t *io_region(int w)
{
    return reinterpret_cast<uint32_t *>(rsagpu_lds) +
           (threadIdx.x >> 6) * (size_t)lds_entries(29, G, w) * Layout<S, G>::WORDS;
}

// First element of the calling wave where each wave takes 64 / G.
template <int G>
__device__ __forceinline__ unsigned long long io_first()
{
    return ((unsigned long long)blockIdx.x * kIoWaves + (threadIdx.x >> 6)) * (64 / G);
}

// y = x * A mod n from xt = x * R mod n (R = 2^(29 S)) and r2 = R^2 mod n:
// A = lo + hi * R with hi of a few limbs.
template <int S, int G, int U>
__device__ __forceinline__ void rns_times_a(uint32_t (&y)[S / G], const uint32_t (&xt)[S / G],
                                            const uint32_t (&r2)[S / G], const uint32_t (&n)[S / G], uint32_t n0inv,
                                            uint32_t *lds)
{
    using Ar = Arith<S, G, 29>;
    using T = RnsTables<U>;
    constexpr int L = S / G;
    constexpr int LA = T::LIMBS + 4;                     // limbs of A in the table
    const uint32_t *a = T::pos() + (4 * U + 1) * T::LIMBS;
    const int r = grp_lane<G>();
    uint32_t t[L];
#pragma unroll
    for (int k = 0; k < L; ++k) t[k] = S <= LA || r * L + k < LA ? a[r * L + k] : 0u;
    mont_mul_reg<S, G, 29>(y, t, xt, lds, n, n0inv);
    if constexpr (T::ABITS > 29 * S) {
        uint32_t u[L];
        mont_mul_reg<S, G, 29>(u, xt, r2, lds, n, n0inv);
#pragma unroll
        for (int k = 0; k < L; ++k) t[k] = r * L + k < LA - S ? a[S + r * L + k] : 0u;
        mont_mul_reg<S, G, 29>(u, t, u, lds, n, n0inv);
        const uint32_t ovf = Ar::add(y, u);
        Ar::cond_sub(y, ovf, n);
    }
}

// ---- entering: CRT halves ---------------------------------------------------
//
// A workgroup is two pairs of waves (kIoWaves), each over 64 / G messages as in
// k_crt: a pair's wave 0 the halves modulo p, its wave 1 those modulo q.  Writes c * A mod p to the
// upper hl words of the message's output and c * A mod q to the lower ones
// (invalid elements: zero).  Both waves have read c before either stores, so
// out may be c.
template <int S, int G, int U>
__global__ __launch_bounds__(64 * kIoWaves) void k_rns_enter_crt(
    const uint32_t *c, const uint32_t *__restrict__ p, const uint32_t *__restrict__ q,
    const uint32_t *__restrict__ dp, const uint32_t *__restrict__ dq, uint32_t *out, unsigned long long count, int hl)
{
    using Ar = Arith<S, G, 29>;
    constexpr int L = S / G, NG = 64 / G;
    const int wave = (int)(threadIdx.x >> 6), half = wave & 1;
    uint32_t *lds = io_region<S, G>(2);
    const unsigned long long msg =
        ((unsigned long long)blockIdx.x * (kIoWaves / 2) + (wave >> 1)) * NG + grp_index<G>();
    const bool live = msg < count;
    const size_t hoff = live ? (size_t)msg * (size_t)hl : 0, foff = 2 * hoff;

    uint32_t n[L], clo[L], chi[L];
    Ar::load(n, (half ? q : p) + hoff, hl, 0, live);
    Ar::load(clo, c + foff, 2 * hl, 0, live);
    Ar::load(chi, c + foff, 2 * hl, 29 * S, live);
    const uint32_t n0 = grp_bcast0<G>(n[0]);
    const bool valid = live && (n0 & 1u) && Ar::bitlen(n) > 1;
    const uint32_t n0inv = Ar::n0inv(n0 | 1u);
    uint32_t one[L], r2[L], xt[L], x[L], t[L];
    mont_setup<S, G, 29>(one, r2, n, n0inv, valid, lds);
    mont_mul_reg<S, G, 29>(xt, clo, r2, lds, n, n0inv);         // c * R = c_lo * R + c_hi * R * R
    mont_mul_reg<S, G, 29>(t, r2, r2, lds, n, n0inv);
    mont_mul_reg<S, G, 29>(t, chi, t, lds, n, n0inv);
    {
        const uint32_t ovf = Ar::add(xt, t);
        Ar::cond_sub(xt, ovf, n);
    }
    rns_times_a<S, G, U>(x, xt, r2, n, n0inv, lds);
    const bool rns = rns_coprime<S, G, U>(n, lds) || !valid;
    if (__ballot(!rns)) {       // exponentiate those elements here
        uint32_t m[L];
        group_modexp<S, G, 29>(m, xt, (half ? dq : dp) + hoff, hl, !rns, n, n0inv, one, lds, 2, xt);
        from_mont<S, G, 29>(m, lds, n, n0inv);
#pragma unroll
        for (int k = 0; k < L; ++k) x[k] = rns ? x[k] : m[k];
    }
    __syncthreads();
    store_words<S, G, 29>(out + foff + (half ? 0 : hl), x, hl, live, valid, lds);
}

// ---- entering: plain exponentiation -----------------------------------------
//
// A wave takes 64 / G elements: those with short exponents are exponentiated as
// in k_modexp, of the others x * A mod n is written to their output (or the
// result, where n shares a factor with base A).  Invalid elements give zero
// and are counted as k_modexp counts them; k_rns_pow takes no even modulus,
// and n = 1 gives zero there too.  out may be base.  The exponents' upper
// words are read first and looked at after the set-up, so that they cost a
// wave of encryptions no latency.
template <int S, int G, int U>
__global__ __launch_bounds__(64 * kIoWaves) RSAGPU_EXP_OCC(S / G) void k_rns_enter_exp(
    const uint32_t *base, const uint32_t *__restrict__ exp, const uint32_t *__restrict__ mod, uint32_t *out,
    unsigned long long count, int limbs, int w, unsigned long long *errs)
{
    using Ar = Arith<S, G, 29>;
    constexpr int L = S / G;
    uint32_t *lds = io_region<S, G>(w);
    const int r = grp_lane<G>();
    const unsigned long long msg = io_first<G>() + grp_index<G>();
    const bool live = msg < count;
    const size_t off = live ? (size_t)msg * (size_t)limbs : 0;
    uint32_t upper = 0;
    // unrolled, so that no load waits for another: 1000 2048-bit encryptions
    // 139 -> 131 us
#pragma unroll
    for (int i = 0; kRnsMinBits / 32 + i * G < S * 29 / 32; ++i) {
        const int k = kRnsMinBits / 32 + r + i * G;
        upper |= live && k < limbs ? exp[off + k] : 0u;
    }

    uint32_t n[L], x[L];
    Ar::load(n, mod + off, limbs, 0, live);
    Ar::load(x, base + off, limbs, 0, live);
    const uint32_t n0 = grp_bcast0<G>(n[0]);
    const uint32_t bl = Ar::bitlen(n);
    const bool valid = live && (n0 & 1u) && bl > 1;
    const uint32_t n0inv = Ar::n0inv(n0 | 1u);
    uint32_t one[L], r2[L], xt[L], A[L];
    mont_setup<S, G, 29, true, true>(one, r2, n, n0inv, valid, lds);
    mont_mul_reg<S, G, 29>(xt, x, r2, lds, n, n0inv);
    const bool wide = valid && grp_any<G>(upper != 0u);
    bool rns = false;
    if (__ballot(wide)) {
        uint32_t y[L];
        rns_times_a<S, G, U>(y, xt, r2, n, n0inv, lds);
        rns = wide && rns_coprime<S, G, U>(n, lds);
        store_words<S, G, 29>(out + off, y, limbs, rns, true, lds);
        if (__ballot(live && !rns) == 0) return;
    }
    if (!group_modexp<S, G, 29, true>(A, xt, exp + off, limbs, valid && !rns, n, n0inv, one, lds, w, x))
        from_mont<S, G, 29>(A, lds, n, n0inv);
    store_words<S, G, 29>(out + off, A, limbs, live && !rns, valid, lds);
    if (live && r == 0 && !valid && bl != 1) atomicAdd(errs, 1ull);
}

// ---- leaving: Garner ----------------------------------------------------------
//
// m = m_q + q * (qinv * (m_p - m_q) mod p), from m_p, m_q, qinv * R mod p and
// n = p, to `full` words at o (only when live; zeros when !valid).
template <int S, int G>
__device__ __forceinline__ void garner_store(uint32_t *o, uint32_t (&mp)[S / G], const uint32_t (&mq)[S / G],
                                             const uint32_t (&qv)[S / G], const uint32_t (&n)[S / G],
                                             const uint32_t (&qn)[S / G], uint32_t n0inv, int full, bool live,
                                             bool valid, uint32_t *lds)
{
    using Ar = Arith<S, G, 29>;
    using Ly = Layout<S, G>;
    constexpr int L = S / G;
    const int g = grp_index<G>(), r = grp_lane<G>();
    uint32_t d[L], e[L], hh[L], high[L];
    const uint32_t neg = Ar::sub(d, mp, mq);                     // m_p - m_q mod p  (m_q < q < p)
#pragma unroll
    for (int k = 0; k < L; ++k) e[k] = d[k];
    Ar::add(e, n);
#pragma unroll
    for (int k = 0; k < L; ++k) d[k] = neg ? e[k] : d[k];
    mont_mul_reg<S, G, 29>(hh, d, qv, lds, n, n0inv);
    lds_sync();
    lds_put<S, G>(lds, hh);
    lds_sync();
    uint32_t *stage = lds + Ly::WORDS + g * (2 * S);
    auto sink = [&](int i, uint32_t v) {
        if (r == 0) stage[i] = v;
    };
    Ar::mul_wide(high, mq, qn, lds, sink);
#pragma unroll
    for (int k = 0; k < L; ++k) stage[S + r * L + k] = high[k];
    lds_sync();
    if (live)
        for (int wd = r; wd < full; wd += G) o[wd] = valid ? rword<29>(stage, 2 * S, wd) : 0u;
}

// The recombination of the halves k_rns_pow left in the
// output, a wave over 64 / G messages; invalid elements give zero and are
// counted.
template <int S, int G>
__global__ __launch_bounds__(64 * kIoWaves) void k_rns_leave_crt(const uint32_t *__restrict__ p, const uint32_t *__restrict__ q,
                                                      const uint32_t *__restrict__ qinv, uint32_t *out,
                                                      unsigned long long count, int hl, unsigned long long *errs)
{
    using Ar = Arith<S, G, 29>;
    constexpr int L = S / G;
    uint32_t *lds = io_region<S, G>(2);
    const int r = grp_lane<G>();
    const unsigned long long msg = io_first<G>() + grp_index<G>();
    const bool live = msg < count;
    const size_t hoff = live ? (size_t)msg * (size_t)hl : 0, foff = 2 * hoff;

    uint32_t n[L], qn[L], A[L], mq[L], qv[L];
    Ar::load(n, p + hoff, hl, 0, live);
    Ar::load(qn, q + hoff, hl, 0, live);
    Ar::load(mq, out + foff, hl, 0, live);
    Ar::load(A, out + foff + hl, hl, 0, live);
    Ar::load(qv, qinv + hoff, hl, 0, live);
    const uint32_t n0 = grp_bcast0<G>(n[0]), q0 = grp_bcast0<G>(qn[0]);
    bool valid = live && (n0 & 1u) && (q0 & 1u) && Ar::bitlen(n) > 1 && Ar::bitlen(qn) > 1;
    {   // p > q
        uint32_t d[L];
        const uint32_t lt = Ar::sub(d, n, qn);
        bool nz = false;
#pragma unroll
        for (int k = 0; k < L; ++k) nz = nz || d[k] != 0u;
        valid = valid && !lt && grp_any<G>(nz);
    }
    const uint32_t n0inv = Ar::n0inv(n0 | 1u);
    uint32_t one[L], r2[L];
    mont_setup<S, G, 29>(one, r2, n, n0inv, valid, lds);
    mont_mul_reg<S, G, 29>(qv, qv, r2, lds, n, n0inv);          // qinv * R mod p
    garner_store<S, G>(out + foff, A, mq, qv, n, qn, n0inv, 2 * hl, live, valid, lds);
    if (live && r == 0 && !valid) atomicAdd(errs, 1ull);
}

// ---- ops batches: CRT buckets under resident keys ---------------------------------
//
// The same two ways for a bucket's operations, with the keys' constants in
// place of the set-up; workgroups take every gridDim.x-th run of the list.

// c * A mod p and mod q, as k_rns_enter_crt; keys whose p or q has no inverse
// for base A (KeyDev::rns) are exponentiated here.
template <int S, int G, int U>
__global__ __launch_bounds__(64 * kIoWaves) void k_rns_enter_ops(const KeyDev *__restrict__ keys,
                                                                 const OpDesc *__restrict__ ops,
                                                                 const unsigned *__restrict__ list,
                                                                 const unsigned *__restrict__ size,
                                                                 const uint32_t *__restrict__ in_pool,
                                                                 uint32_t *__restrict__ mid)
{
    using Ar = Arith<S, G, 29>;
    constexpr int L = S / G, NG = 64 / G;
    static_assert(standard_s29(S), "the limb count the keys' constants are stored with");
    const int wave = (int)(threadIdx.x >> 6), half = wave & 1;
    uint32_t *lds = io_region<S, G>(2);
    const unsigned count = *size;
#pragma unroll 1
    for (unsigned first = blockIdx.x * (kIoWaves / 2) * NG; first < count; first += gridDim.x * (kIoWaves / 2) * NG) {
        const unsigned idx = first + (wave >> 1) * NG + grp_index<G>();
        const unsigned at = idx < count ? list[idx] : kOrderHole;
        const bool live = at != kOrderHole;
        const unsigned o = live ? at : list[first];              // the first entry of a run of tiles is no hole
        const OpDesc &op = ops[o];
        const KeyDev &k = keys[op.key_id];
        const int hl = k.hwords;
        const ModConsts &mc = half ? k.cq[1] : k.cp[1];
        uint32_t n[L], clo[L], chi[L], r2[L], r3[L], xt[L], x[L], t[L];
        Ar::load(n, half ? k.q : k.p, hl, 0, live);
        Ar::load(clo, in_pool + op.in_off, 2 * hl, 0, live);
        Ar::load(chi, in_pool + op.in_off, 2 * hl, 29 * S, live);
        load_raw<S, G>(r2, mc.r2, live);
        load_raw<S, G>(r3, mc.r3, live);
        const uint32_t n0inv = Ar::n0inv(grp_bcast0<G>(n[0]) | 1u);
        mont_mul_reg<S, G, 29>(xt, clo, r2, lds, n, n0inv);      // c * R = c_lo * R + c_hi * R * R
        mont_mul_reg<S, G, 29>(t, chi, r3, lds, n, n0inv);
        {
            const uint32_t ovf = Ar::add(xt, t);
            Ar::cond_sub(xt, ovf, n);
        }
        rns_times_a<S, G, U>(x, xt, r2, n, n0inv, lds);
        const bool rns = !live || k.rns;
        if (__ballot(!rns)) {
            uint32_t m[L], one[L];
            load_raw<S, G>(one, mc.one, live);
            group_modexp<S, G, 29>(m, xt, half ? k.dq : k.dp, hl, !rns, n, n0inv, one, lds, 2, xt);
            from_mont<S, G, 29>(m, lds, n, n0inv);
#pragma unroll
            for (int i = 0; i < L; ++i) x[i] = rns ? x[i] : m[i];
        }
        store_words<S, G, 29>(mid + (size_t)o * kMidWords + (half ? 0 : hl), x, hl, live, true, lds);
        lds_sync();
    }
}

// Garner, as k_rns_leave_crt.
template <int S, int G>
__global__ __launch_bounds__(64 * kIoWaves) void k_rns_leave_ops(const KeyDev *__restrict__ keys,
                                                                 const OpDesc *__restrict__ ops,
                                                                 const unsigned *__restrict__ list,
                                                                 const unsigned *__restrict__ size,
                                                                 const uint32_t *__restrict__ mid, uint32_t *out_pool)
{
    using Ar = Arith<S, G, 29>;
    constexpr int L = S / G, NG = 64 / G;
    uint32_t *lds = io_region<S, G>(2);
    const unsigned count = *size;
#pragma unroll 1
    for (unsigned first = (unsigned)io_first<G>(); first < count; first += gridDim.x * kIoWaves * NG) {
        const unsigned idx = first + grp_index<G>();
        const unsigned at = idx < count ? list[idx] : kOrderHole;
        const bool live = at != kOrderHole;
        const uint64_t any = __ballot(live);
        if (any == 0) continue;
        const unsigned o = live ? at : list[first + (unsigned)__builtin_ctzll(any) / G];
        const OpDesc &op = ops[o];
        const KeyDev &k = keys[op.key_id];
        const int hl = k.hwords;
        const uint32_t *m = mid + (size_t)o * kMidWords;
        uint32_t n[L], qn[L], A[L], mq[L], qv[L];
        Ar::load(n, k.p, hl, 0, live);
        Ar::load(qn, k.q, hl, 0, live);
        Ar::load(mq, m, hl, 0, live);
        Ar::load(A, m + hl, hl, 0, live);
        load_raw<S, G>(qv, k.cp[1].xr, live);                    // qinv * R mod p
        const uint32_t n0inv = Ar::n0inv(grp_bcast0<G>(n[0]) | 1u);
        garner_store<S, G>(out_pool + op.out_off, A, mq, qv, n, qn, n0inv, 2 * hl, live, true, lds);
        lds_sync();
    }
}

// ---- launchers ----------------------------------------------------------------

// Plain CRT decryption, S-limb halves on G lanes at the way in and out.
template <int U, int S, int G>
hipError_t launch_rns_crt_on(const RnsCrtArgs &a, hipStream_t stream)
{
    static_assert(S >= RnsTables<U>::LIMBS, "limbs of the configuration");
    const size_t ng = 64 / G, lds = kIoWaves * lds_bytes_for(S, G, 29, 2);
    const auto blocks = [&](size_t per) { return dim3((unsigned)((a.count + per - 1) / per)); };
    hipLaunchKernelGGL((k_rns_enter_crt<S, G, U>), blocks(ng * kIoWaves / 2), dim3(64 * kIoWaves), lds, stream, a.c,
                       a.p, a.q, a.dp, a.dq, a.out, (unsigned long long)a.count, a.hl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const RnsCrtSource src{a.p, a.q, a.dp, a.dq, a.order, a.out, (unsigned long long)a.slots, a.hl};
    e = rns_pow<U>(src, (a.slots + 15) / 16, 2, a.cus, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rns_leave_crt<S, G>), blocks(ng * kIoWaves), dim3(64 * kIoWaves), lds, stream, a.p, a.q,
                       a.qinv, a.out, (unsigned long long)a.count, a.hl, a.errs);
    return hipGetLastError();
}

// Plain exponentiation, S limbs on G lanes at the way in.
template <int U, int S, int G>
hipError_t launch_rns_exp_on(const RnsExpArgs &a, int window, hipStream_t stream)
{
    static_assert(S >= RnsTables<U>::LIMBS, "limbs of the configuration");
    const size_t per = 64 / G * kIoWaves, lds = kIoWaves * lds_bytes_for(S, G, 29, window);
    if (lds > kMaxGroupLds) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_rns_enter_exp<S, G, U>), dim3((unsigned)((a.count + per - 1) / per)), dim3(64 * kIoWaves), lds,
                       stream, a.base, a.exp, a.mod, a.out, (unsigned long long)a.count, a.limbs, window, a.errs);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const RnsExpSource<false> src{a.mod, a.exp, a.out, (unsigned long long)a.count, a.limbs};
    return rns_pow<U>(src, (a.count + 15) / 16, 1, a.cus, stream);
}

// A CRT bucket of an ops batch, at most `most` entries.
template <int U, int S, int G>
hipError_t launch_rns_ops(const RnsOpsArgs &a, hipStream_t stream)
{
    const size_t ng = 64 / G, lds = kIoWaves * lds_bytes_for(S, G, 29, 2);
    const auto blocks = [&](size_t per) {
        const size_t b = (a.most + per - 1) / per, cap = 2 * (size_t)a.cus;
        return dim3((unsigned)(b < cap ? b : cap));
    };
    hipLaunchKernelGGL((k_rns_enter_ops<S, G, U>), blocks(ng * kIoWaves / 2), dim3(64 * kIoWaves), lds, stream, a.keys,
                       a.ops, a.list, a.size, a.in_pool, a.mid);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.entered && (e = hipEventRecord(a.entered, stream)) != hipSuccess) return e;
    const RnsOpsSource src{a.keys, a.ops, a.list, a.size, a.mid, 0, ~0u, 0};
    e = rns_pow_bucket<U>(src, (a.most + 15) / 16, a.bulk, a.cus, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rns_leave_ops<S, G>), blocks(ng * kIoWaves), dim3(64 * kIoWaves), lds, stream, a.keys, a.ops,
                       a.list, a.size, (const uint32_t *)a.mid, a.out_pool);
    return hipGetLastError();
}

// Narrow groups (S2 limbs on G2 lanes: a shorter chain of instructions per
// product, more of them in all) where the waves they take have a SIMD each.
// Plain exponentiation of 24 words, e = 65537, 64 .. 4096 elements: 43.5 .. 44.7
// us on 28 limbs and 4 lanes, the idle k_rns_pow included, 35.0 .. 36.8 on 32
// and 16 (k_modexp alone 42.7 .. 43.3).
template <int U, int S, int G, int S2, int G2>
hipError_t launch_rns_crt(const RnsCrtArgs &a, hipStream_t stream)
{
    if (2 * a.count * G2 <= (size_t)a.cus * 4 * 64) return launch_rns_crt_on<U, S2, G2>(a, stream);
    return launch_rns_crt_on<U, S, G>(a, stream);
}
template <int U, int S, int G, int S2, int G2>
hipError_t launch_rns_exp(const RnsExpArgs &a, hipStream_t stream)
{
    if (a.count * G2 <= (size_t)a.cus * 4 * 64) return launch_rns_exp_on<U, S2, G2>(a, 3, stream);
    return launch_rns_exp_on<U, S, G>(a, a.window, stream);
}

}  // namespace rsagpu
