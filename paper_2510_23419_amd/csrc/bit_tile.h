// bit_tile.h — the sweep of a cube or general graph with its spins as bits in LDS
// (device code shared by the per-instance kernel and the batched tiles).
//
// A workgroup holds RS replicas of every site: one 16-bit element per position, bit r
// = 1 where replica r's spin is -1, so that the two positions of a pair are one dword.
// A thread updates a pair (2 RS updates), a position (RS) or four replicas of a
// position, by the size of the update group.  The K slots of a position are XORed with
// their signs and counted by bit-sliced full adders, so a field costs about 30
// instructions for 32 updates instead of 2 to 5 per update bytewise.  The count's bits
// of two neighbouring replicas form the byte index of a pair of decision words in LDS
// (one 8-byte read for two updates): S(I) = Tm for I >= 0 and 2^32 - Tm for I < 0, and
// the new spin is -1 exactly when w + S(I) carries out of 32 bits, or when S(I) = 2^32
// (I < 0 with Tm = 0), which a bit-sliced comparison of the counts adds at the end.  The
// carries are shifted into the new element by v_addc: two instructions decide and store
// an update.
#pragma once

#include "bits.h"
#include "device.h"

namespace pbit {

namespace bit {

constexpr int kThreads = 1024;  // largest workgroup

// LDS layout, from address 0 (bytes).  Two buffers each, by the sweep's parity (rows:
// by the parity of the run of kRowRun sweeps).
constexpr int kPairs6 = 64, kPairs7 = 256, kWords15 = 32;
constexpr int kRowRun = 16;   // sweeps of threshold rows held at a time
constexpr int kRowWords = 16; // |I| <= 15
constexpr uint32_t kLdsPairs = 0;                                // pairs of decision words, index order
constexpr uint32_t kLdsWide = kLdsPairs + 2 * kPairs7 * 8;       // decision words of wide pairs
constexpr uint32_t kLdsSat = kLdsWide + 2 * kWords15 * 8;        // comparison masks of saturated counts
constexpr uint32_t kLdsRows = kLdsSat + 2 * 32;                  // threshold rows
constexpr uint32_t kLdsAcc = kLdsRows + 2 * kRowRun * kRowWords * 4;  // energy sums
constexpr uint32_t kLdsSlot = kLdsAcc + 64;                      // batched tiles: the taken item
static_assert(kLdsSlot + 16 <= kBitElBase, "tables below the elements");

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
// (a & m) | (b & ~m)
__device__ __forceinline__ uint32_t sel(uint32_t a, uint32_t b, uint32_t m)
{
    return __builtin_amdgcn_bitop3_b32(a, b, m, 0xE4);
}
// b << s, or b >> -s
template <int S>
__device__ __forceinline__ uint32_t shift(uint32_t b)
{
    return S >= 0 ? b << (S & 31) : b >> (-S & 31);
}

// Bit-sliced count of K one-bit inputs: n[w] holds bit w of every lane bit's count.
__device__ __forceinline__ void count7(const uint32_t *x, uint32_t *n)
{
    const uint32_t s1 = xor3(x[0], x[1], x[2]), c1 = maj(x[0], x[1], x[2]);
    const uint32_t s2 = xor3(x[3], x[4], x[5]), c2 = maj(x[3], x[4], x[5]);
    n[0] = xor3(s1, s2, x[6]);
    const uint32_t c3 = maj(s1, s2, x[6]);
    n[1] = xor3(c1, c2, c3);
    n[2] = maj(c1, c2, c3);
}
template <int K>
__device__ __forceinline__ void count(const uint32_t *x, uint32_t *n)
{
    if constexpr (K == 6) {
        const uint32_t s1 = xor3(x[0], x[1], x[2]), c1 = maj(x[0], x[1], x[2]);
        const uint32_t s2 = xor3(x[3], x[4], x[5]), c2 = maj(x[3], x[4], x[5]);
        n[0] = s1 ^ s2;
        const uint32_t c3 = s1 & s2;
        n[1] = xor3(c1, c2, c3);
        n[2] = maj(c1, c2, c3);
    } else if constexpr (K == 7) {
        count7(x, n);
    } else {
        static_assert(K == 15, "slot counts");
        uint32_t a[3], b[3];
        count7(x, a);
        count7(x + 7, b);
        n[0] = xor3(a[0], b[0], x[14]);
        const uint32_t k0 = maj(a[0], b[0], x[14]);
        n[1] = xor3(a[1], b[1], k0);
        const uint32_t k1 = maj(a[1], b[1], k0);
        n[2] = xor3(a[2], b[2], k1);
        n[3] = maj(a[2], b[2], k1);
    }
}

// LDS by byte address (the workgroup's LDS starts at 0; integer addresses let constant
// offsets go into the instructions).
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t a)
{
    return *(const __attribute__((address_space(3))) T *)(uintptr_t)a;
}
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t a, T v)
{
    *(__attribute__((address_space(3))) T *)(uintptr_t)a = v;
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// A load from memory that no kernel writes, at a wave-uniform address: a scalar load.
template <typename T>
__device__ __forceinline__ T load_const(const void *p)
{
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// 16-bit half of x, times two: the byte address of an element index.
__device__ __forceinline__ uint32_t addr_lo(uint32_t x)
{
    uint32_t r;
    const uint32_t one = 1u;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0"
        : "=v"(r) : "v"(one), "v"(x));
    return r;
}
__device__ __forceinline__ uint32_t addr_hi(uint32_t x)
{
    uint32_t r;
    const uint32_t one = 1u;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
        : "=v"(r) : "v"(one), "v"(x));
    return r;
}
// Byte B of x, times eight: the byte address of a pair of decision words (one SDWA shift).
template <int B>
__device__ __forceinline__ uint32_t addr_byte(uint32_t x)
{
    uint32_t r;
    const uint32_t three = 3u;
#define PBIT_BYTE_SHIFT(N)                                                                                        \
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_" #N      \
        : "=v"(r) : "v"(three), "v"(x))
    if constexpr (B == 0) PBIT_BYTE_SHIFT(0);
    else if constexpr (B == 1) PBIT_BYTE_SHIFT(1);
    else if constexpr (B == 2) PBIT_BYTE_SHIFT(2);
    else PBIT_BYTE_SHIFT(3);
#undef PBIT_BYTE_SHIFT
    return r;
}

// Four decisions shifted into acc: acc = 16 acc + 8 c3 + 4 c2 + 2 c1 + c0, c the carries of
// w + s.  A carry written to scalar registers may be read two instructions later at the
// earliest, so the four sums and the four shifts are interleaved.
__device__ __forceinline__ void decide_bits(uint32_t &acc, const Block4 &b, u32x2 s1, u32x2 s0)
{
    uint32_t t;
    uint64_t ca, cb, cc;
    asm("v_add_co_u32 %1, %2, %5, %9\n\t"
        "v_add_co_u32 %1, %3, %6, %10\n\t"
        "v_add_co_u32 %1, %4, %7, %11\n\t"
        "v_addc_co_u32 %0, %2, %0, %0, %2\n\t"
        "v_add_co_u32 %1, vcc, %8, %12\n\t"
        "v_addc_co_u32 %0, %3, %0, %0, %3\n\t"
        "v_addc_co_u32 %0, %4, %0, %0, %4\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(acc), "=&v"(t), "=&s"(ca), "=&s"(cb), "=&s"(cc)
        : "v"(b.w[3]), "v"(b.w[2]), "v"(b.w[1]), "v"(b.w[0]), "v"(s1.y), "v"(s1.x), "v"(s0.y), "v"(s0.x)
        : "vcc");
}

// Masks of the comparison u = 2 n + odd >= u_sat, u_sat the smallest u with I = K - u < 0
// and Tm(|I|) = 0: the start of the comparison (0 where there is none), and per bit of u
// ~0 where u_sat has a 0.
struct Saturated {
    uint32_t nm[4], low;
};

// Field of a pair table's entry e for replica r (0: the even one): bits 0-1, 2-3, 4-5 (6-7)
// of e hold bits 0, 1, 2 of the counts (and the odd bits) of two neighbouring replicas.
__device__ __forceinline__ int pair_field(int K, int e, int r)
{
    return K - 2 * (((e >> r) & 1) + 2 * ((e >> (2 + r)) & 1) + 4 * ((e >> (4 + r)) & 1)) - ((e >> (6 + r)) & 1);
}

// Philox4x32-10 of (site, sweep t, group, domain 0), split so that what depends on the
// group and sweep alone (three words, scalar registers) and on the site alone is computed
// once: rounds 0 and 1 of a block are two XORs, and a block is 34 vector instructions.
struct GroupKey {
    uint32_t a, b, c;
};
struct SiteKey {
    uint32_t hi, lo, l0;
};
__device__ __forceinline__ GroupKey group_key(uint32_t g, uint32_t t, uint32_t k0, uint32_t k1)
{
    const uint64_t q = (uint64_t)g * 0xCD9E8D57u;
    const uint64_t p = (uint64_t)((uint32_t)(q >> 32) ^ t ^ k0) * 0xD2511F53u;
    return GroupKey{(uint32_t)q ^ (k0 + 0x9E3779B9u), (uint32_t)(p >> 32) ^ (k1 + 0xBB67AE85u),
                    (uint32_t)p ^ (k1 + 2u * 0xBB67AE85u)};
}
__device__ __forceinline__ SiteKey site_key(uint32_t site, uint32_t k1)
{
    const uint64_t p = (uint64_t)site * 0xD2511F53u;
    const uint64_t q = (uint64_t)((uint32_t)(p >> 32) ^ k1) * 0xCD9E8D57u;
    return SiteKey{(uint32_t)(q >> 32), (uint32_t)q, (uint32_t)p};
}
__device__ __forceinline__ Block4 philox_sweep(const SiteKey &s, const GroupKey &g, uint32_t k0, uint32_t k1)
{
    uint32_t c0 = s.hi ^ g.a, c1 = s.lo, c2 = s.l0 ^ g.b, c3;
    k0 += 2u * 0x9E3779B9u;
    k1 += 2u * 0xBB67AE85u;
    {  // round 2: word 3 and the key are in g.c
        const uint64_t p = (uint64_t)c0 * 0xD2511F53u, q = (uint64_t)c2 * 0xCD9E8D57u;
        c0 = xor3((uint32_t)(q >> 32), c1, k0);
        c2 = (uint32_t)(p >> 32) ^ g.c;
        c1 = (uint32_t)q;
        c3 = (uint32_t)p;
    }
#pragma unroll
    for (int round = 3; round < 10; ++round) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        const uint64_t p = (uint64_t)c0 * 0xD2511F53u, q = (uint64_t)c2 * 0xCD9E8D57u;
        c0 = xor3((uint32_t)(q >> 32), c1, k0);
        c2 = xor3((uint32_t)(p >> 32), c3, k1);
        c1 = (uint32_t)q;
        c3 = (uint32_t)p;
    }
    return Block4{{c0, c1, c2, c3}};
}

// Four replica bytes (0x01 / 0xFF) <-> four bits (1: -1).
__device__ __forceinline__ uint32_t bits_of_bytes(uint32_t d)
{
    const uint32_t x = (d >> 7) & 0x01010101u;
    return (x | x >> 7 | x >> 14 | x >> 21) & 0xFu;
}
__device__ __forceinline__ uint32_t bytes_of_bits(uint32_t n)
{
    const uint32_t x = ((n & 0xFu) * 0x00204081u) & 0x01010101u;
    return 0x01010101u | (x * 0xFEu);
}

// Comparison of the counts with the saturated ones: bit = 1 where the new spin is -1
// whatever the random word.
template <int K>
__device__ __forceinline__ uint32_t saturated_bits(const uint32_t *n, const Saturated &sat)
{
    // without odd counts, u_sat is rounded up to an even one
    uint32_t ge = K == 7 ? maj(n[3], sat.low, sat.nm[0]) : sat.low & sat.nm[0];
    ge = maj(n[0], ge, sat.nm[1]);
    ge = maj(n[1], ge, sat.nm[2]);
    return maj(n[2], ge, sat.nm[3]);
}
// Index bytes of the pairs of decision words: byte B of the result belongs to replicas
// 8 B + 2 J and 8 B + 2 J + 1 of the counts n (3 planes, and the odd mask in n[3] if K = 7).
template <int K, int J>
__device__ __forceinline__ uint32_t pair_index(const uint32_t *n)
{
    const uint32_t x = sel(shift<-2 * J>(n[0]), shift<2 - 2 * J>(n[1]), 0x03030303u);
    if constexpr (K == 7)
        return sel(x, sel(shift<4 - 2 * J>(n[2]), shift<6 - 2 * J>(n[3]), 0x30303030u), 0x0F0F0F0Fu);
    else
        return sel(x, shift<4 - 2 * J>(n[2]), 0x0F0F0F0Fu) & 0x3F3F3F3Fu;
}
// Four decisions shifted into acc, replica 3 first: index bytes B of i0 (replicas 0, 1)
// and i1 (2, 3), tab the byte offset of the sweep's pair table.
template <int B, uint32_t TAB>
__device__ __forceinline__ void decide_four(uint32_t &acc, const Block4 &b, uint32_t i0, uint32_t i1)
{
    const u32x2 s1 = lds_get<u32x2>(TAB + addr_byte<B>(i1)), s0 = lds_get<u32x2>(TAB + addr_byte<B>(i0));
    decide_bits(acc, b, s1, s0);
}

// The new elements of P positions (bits 0 .. RS - 1 and 16 .. of the result).
template <int K, int RS, int P, uint32_t TAB>
__device__ __forceinline__ uint32_t decide(const uint32_t *n, uint32_t sites, const GroupKey *gk, uint32_t k0,
                                           uint32_t k1, const Saturated &sat)
{
    uint32_t idx[4];
    idx[0] = pair_index<K, 0>(n);
    idx[1] = pair_index<K, 1>(n);
    if constexpr (RS > 4) {
        idx[2] = pair_index<K, 2>(n);
        idx[3] = pair_index<K, 3>(n);
    }
    const uint32_t ge = saturated_bits<K>(n, sat);
    uint32_t acc = 0u;
    if constexpr (P == 2) {
        const SiteKey sk = site_key(sites >> 16, k1);
        if constexpr (RS == 16) {
            decide_four<3, TAB>(acc, philox_sweep(sk, gk[3], k0, k1), idx[2], idx[3]);
            decide_four<3, TAB>(acc, philox_sweep(sk, gk[2], k0, k1), idx[0], idx[1]);
        }
        if constexpr (RS >= 8) decide_four<2, TAB>(acc, philox_sweep(sk, gk[1], k0, k1), idx[2], idx[3]);
        decide_four<2, TAB>(acc, philox_sweep(sk, gk[0], k0, k1), idx[0], idx[1]);
        if constexpr (RS < 16) acc <<= 16 - RS;
    }
    const SiteKey sk = site_key(sites & 0xFFFFu, k1);
    if constexpr (RS == 16) {
        decide_four<1, TAB>(acc, philox_sweep(sk, gk[3], k0, k1), idx[2], idx[3]);
        decide_four<1, TAB>(acc, philox_sweep(sk, gk[2], k0, k1), idx[0], idx[1]);
    }
    if constexpr (RS >= 8) decide_four<0, TAB>(acc, philox_sweep(sk, gk[1], k0, k1), idx[2], idx[3]);
    decide_four<0, TAB>(acc, philox_sweep(sk, gk[0], k0, k1), idx[0], idx[1]);
    return acc | ge;
}
// Replicas 0 .. 3 of one position (n shifted to them): group g of the tile.
template <int K, uint32_t TAB>
__device__ __forceinline__ uint32_t decide_quad(const uint32_t *n, uint32_t site, uint32_t group, uint32_t t,
                                                uint32_t k0, uint32_t k1, const Saturated &sat)
{
    uint32_t acc = 0u;
    decide_four<0, TAB>(acc, philox(site, t, group, kDomainSweep, k0, k1), pair_index<K, 0>(n), pair_index<K, 1>(n));
    return (acc | saturated_bits<K>(n, sat)) & 0xFu;
}
// The same for a position of a wide pair: five-bit indices of single 64-bit words.
template <uint32_t WTAB>
__device__ __forceinline__ uint32_t decide_quad_wide(const uint32_t *n, uint32_t odd, uint32_t site, uint32_t group,
                                                     uint32_t t, uint32_t k0, uint32_t k1)
{
    const Block4 b = philox(site, t, group, kDomainSweep, k0, k1);
    uint32_t acc = 0u;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t e = ((odd >> p) & 1u) | ((n[0] >> p) & 1u) << 1 | ((n[1] >> p) & 1u) << 2 |
                           ((n[2] >> p) & 1u) << 3 | ((n[3] >> p) & 1u) << 4;
        const uint64_t S = lds_get<uint64_t>(WTAB + 8u * e);
        acc |= (uint32_t)(((uint64_t)b.w[p] + S) >> 32) << p;
    }
    return acc;
}

// A record of ordinary or wide pairs, and the slots of P positions read through it.
template <int FORM>
struct Rec {
    static constexpr int kSlots = FORM == kBitGeneral ? kBitSlots : 6;
    static constexpr int kWords = FORM == kBitCube4 ? 3 : 4;
    uint4 q[kWords];
    __device__ __forceinline__ void load(const uint4 *rec, int n_pairs, int p)
    {
#pragma unroll
        for (int w = 0; w < kWords; ++w) {
            typedef unsigned v4u __attribute__((ext_vector_type(4)));
            const v4u v = load_global<v4u>(rec + ((size_t)w * n_pairs + p));
            q[w] = make_uint4(v.x, v.y, v.z, v.w);
        }
    }
    // Brings one position's halves of a pair's record down: slots<FORM, 1> reads low halves.
    __device__ __forceinline__ void select(int hh)
    {
        if constexpr (FORM == kBitCube4) {
            const uint32_t both = (uint32_t)hh * 0x00010001u;
            q[0].x += both;
            q[0].y += both;
            q[0].z = ((q[0].z + (uint32_t)hh) & 0xFFFFu) | (hh ? q[0].w << 16 : q[0].z & 0xFFFF0000u);
        } else {
            q[0].x >>= 16 * hh; q[0].y >>= 16 * hh; q[0].z >>= 16 * hh; q[0].w >>= 16 * hh;
        }
#pragma unroll
        for (int w = 1; w < kWords; ++w) {
            q[w].x >>= 16 * hh; q[w].y >>= 16 * hh; q[w].z >>= 16 * hh; q[w].w >>= 16 * hh;
        }
    }
    // Keeps what is computed from the record from being hoisted out of the sweeps (it would
    // not fit the registers).
    __device__ __forceinline__ void pin()
    {
#pragma unroll
        for (int w = 0; w < kWords; ++w) asm volatile("" : "+v"(q[w].x), "+v"(q[w].y), "+v"(q[w].z), "+v"(q[w].w));
    }
    __device__ __forceinline__ uint32_t word(int w) const
    {
        const uint4 &v = q[w / 4];
        return w % 4 == 0 ? v.x : w % 4 == 1 ? v.y : w % 4 == 2 ? v.z : v.w;
    }
};

__device__ __forceinline__ uint32_t lds_u16(uint32_t a) { return lds_get<uint16_t>(a); }
__device__ __forceinline__ uint32_t lds_u32(uint32_t a) { return lds_get<uint32_t>(a); }

// x[u] = the negative products of slot u: of both positions of a pair (P = 2), or of the
// selected one in the low half (P = 1; the high half is undefined).
template <int FORM, int P>
__device__ __forceinline__ void slots(const Rec<FORM> &r, uint32_t *x)
{
    constexpr int K = Rec<FORM>::kSlots;
    if constexpr (FORM == kBitCube4) {
        uint32_t v[6];
#pragma unroll
        for (int u = 0; u < 5; ++u) {
            const uint32_t a = (u & 1) ? addr_hi(r.word(u / 2)) : addr_lo(r.word(u / 2));
            v[u] = P == 2 ? lds_u32(a) : lds_u16(a);
        }
        v[5] = lds_u16(addr_hi(r.word(2)));
        if constexpr (P == 2) v[5] |= lds_u16(addr_lo(r.word(3))) << 16;
#pragma unroll
        for (int u = 0; u < 6; ++u) x[u] = v[u] ^ r.word(4 + u);
    } else {
#pragma unroll
        for (int u = 0; u < K; ++u) {
            uint32_t v = lds_u16(addr_lo(r.word(u)));
            if constexpr (P == 2) v |= lds_u16(addr_hi(r.word(u))) << 16;
            x[u] = v ^ r.word(K + u);
        }
    }
}
// Counts of one position of a wide pair (low half), its odd bits and site.
__device__ __forceinline__ void wide_counts(const BitView &v, int pair, int hh, uint32_t *n,
                                            uint32_t &odd, uint32_t &site)
{
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    uint32_t w[32], x[kBitSlotsWide];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const v4u d = load_global<v4u>(v.wide + ((size_t)q * v.n_wide + pair));
        w[4 * q] = d.x; w[4 * q + 1] = d.y; w[4 * q + 2] = d.z; w[4 * q + 3] = d.w;
    }
#pragma unroll
    for (int u = 0; u < kBitSlotsWide; ++u)
        x[u] = lds_u16(addr_lo(w[u] >> (16 * hh))) ^ (w[15 + u] >> (16 * hh));
    count<kBitSlotsWide>(x, n);
    odd = w[30] >> (16 * hh);
    site = (w[31] >> (16 * hh)) & 0xFFFFu;
}

// The units of a group's ordinary pairs: whole pairs, positions, or four replicas of a
// position, the widest that still gives the workgroup's waves work (measured: see k_bit_slab).
enum Unit { kPair, kSite, kQuad, kByGroup };
__host__ __device__ __forceinline__ Unit unit_of(int rs, int pairs, int threads)
{
    if (pairs > threads / 2) return kPair;
    if (rs == 4 || 2 * pairs * (rs / 4) > threads) return kSite;
    return kQuad;
}

// One tile (RS replicas) of a job over local sweeps [s_begin, s_end): spins in from
// global memory (or drawn), the sweeps, optionally the energies, spins out.  All threads
// of the workgroup call it (a multiple of 64: at least 256, or 64 for the cube forms).
// UNIT: the units of both groups of a problem with two, whose first records a thread keeps
// in registers over all sweeps; kByGroup: any number of groups, the units by group.  The next sweep's decision words are written
// during the current one, from threshold rows loaded kRowRun sweeps at a time, so a sweep
// has one barrier per group and waits for no global load on small problems.
template <int FORM, int RS, int UNIT>
__device__ __forceinline__ void run(const BitJobDev &jb, int tile, int s_begin, int s_end, bool init)
{
    constexpr bool GEN = FORM == kBitGeneral, TWO = UNIT != kByGroup;
    constexpr int K = Rec<FORM>::kSlots;
    constexpr int NE = GEN ? kPairs7 : kPairs6;
    constexpr int RQ = RS / 4;
    auto el = [](int p) { return kBitElBase + 2u * (uint32_t)p; };  // element of a position
    const int tid = threadIdx.x, T = blockDim.x;
    const BitView &v = jb.v;
    const int width = jb.width;
    const uint32_t rg = jb.rq0 + (uint32_t)RQ * (uint32_t)tile;  // Philox counter word 2 of the first group
    const size_t stride = jb.row_stride ? (size_t)jb.row_stride : (size_t)RS;
    int8_t *gst = jb.state + (size_t)tile * (jb.row_stride ? (size_t)RS : (size_t)v.n * RS);

    // spins in
    for (int p = tid; p < v.n_pos + 2; p += T) {
        uint32_t bits = 0u;
        const uint32_t i = p < v.n_pos ? load_global<uint16_t>(v.pos_site + p) : kBitNoSite;
        if (i != kBitNoSite) {
#pragma unroll
            for (int k = 0; k < RQ; ++k) {
                if (init) {
                    const Block4 b = philox(i, 0u, rg + (uint32_t)k, kDomainInit, jb.k0, jb.k1);
#pragma unroll
                    for (int q = 0; q < 4; ++q) bits |= (b.w[q] >> 31) << (4 * k + q);
                } else {
                    bits |= bits_of_bytes(load_global<uint32_t>(gst + stride * i + 4 * k)) << (4 * k);
                }
            }
        }
        lds_put<uint16_t>(el(p), (uint16_t)bits);
    }

    // threshold rows of run q (sweeps s_begin + kRowRun q ..), entry |I| clamped to the last:
    // this thread's words in flight, then in LDS
    constexpr int kRowPer = GEN ? 1 : 4;  // words per thread (256 words)
    uint32_t rowp[kRowPer];
    auto rows_load = [&](int q) {
#pragma unroll
        for (int u = 0; u < kRowPer; ++u) {
            const int e = tid + T * u, s = s_begin + kRowRun * q + e / kRowWords;
            if (e < kRowRun * kRowWords && s < s_end)
                rowp[u] = load_global<uint32_t>(jb.table + (size_t)s * width + min(e % kRowWords, width - 1));
        }
    };
    auto rows_post = [&](int q) {
#pragma unroll
        for (int u = 0; u < kRowPer; ++u) {
            const int e = tid + T * u;
            if (e < kRowRun * kRowWords) lds_put(kLdsRows + 4u * (uint32_t)((q & 1) * kRowRun * kRowWords + e), rowp[u]);
        }
    };
    // this thread's decision words of sweep s, read from its row, then written to buffer buf
    auto absI = [](int I) { return I < 0 ? -I : I; };
    const int I0 = pair_field(K, tid, 0), I1 = pair_field(K, tid, 1), Iw = kBitSlotsWide - tid;
    const int a0 = min(absI(I0), kRowWords - 1), a1 = min(absI(I1), kRowWords - 1), aw = min(absI(Iw), kRowWords - 1);
    uint32_t p0 = 0u, p1 = 0u, pw = 0u, ps = 1u;
    auto fetch = [&](int s) {
        const int k = s - s_begin;
        const uint32_t row = kLdsRows + 4u * (uint32_t)((k & (2 * kRowRun - 1)) * kRowWords);
        if (tid < NE) {
            p0 = lds_u32(row + 4u * a0);
            p1 = lds_u32(row + 4u * a1);
            if (tid < 8) ps = lds_u32(row + 4u * (tid + 1));
            if (GEN && tid < kWords15) pw = lds_u32(row + 4u * aw);
        }
    };
    auto post = [&](int buf) {
        if (tid < NE)
            lds_put(kLdsPairs + 8u * (uint32_t)(buf * NE + tid),
                    u32x2{I0 >= 0 ? p0 : 0u - p0, I1 >= 0 ? p1 : 0u - p1});
        if (GEN && tid < kWords15)
            lds_put(kLdsWide + 8u * (uint32_t)(buf * kWords15 + tid),
                    Iw >= 0 ? (uint64_t)pw : ((uint64_t)1 << 32) - pw);
        if (tid < 64) {
            const uint64_t zero = __ballot(tid < 8 && ps == 0u);
            const int u = K + __builtin_ctzll(zero | 0x8000000000000000ull) + 1;  // u_sat, or beyond 15
            if (tid < 5)
                lds_put(kLdsSat + 4u * (uint32_t)(buf * 8 + tid),
                        u > 15 ? 0u : tid == 4 ? ~0u : ((u >> tid) & 1) ? 0u : ~0u);
        }
    };

    const int G = TWO ? 2 : v.n_groups;
    auto group = [&](int c) {
        const u32x4 g = load_const<u32x4>(v.groups + bit_group_at(c, G));
        return make_int4((int)g.x, (int)g.y, (int)g.z, (int)g.w);
    };
    auto pair_of = [&](Unit u, int j) { return u == kPair ? j : u == kSite ? j >> 1 : j / (2 * RQ); };
    auto units_of = [&](Unit u, const int4 &g) { return g.w * (u == kPair ? 1 : u == kSite ? 2 : 2 * RQ); };
    // record of unit j of a group, its position selected
    auto fetch_rec = [&](Unit u, const int4 &g, int j, Rec<FORM> &r) { r.load(v.rec, v.n_pairs, g.z + pair_of(u, j)); };
    auto select_rec = [&](Unit u, int j, Rec<FORM> &r) {
        if (u == kSite) r.select(j & 1);
        if (u == kQuad) r.select((j / RQ) & 1);
    };
    auto first = [&](const int4 &g, Rec<FORM> &r) {
        const Unit u = TWO ? (Unit)UNIT : unit_of(RS, g.w, T);
        if (tid < units_of(u, g)) fetch_rec(u, g, tid, r);
    };
    Rec<FORM> keep[TWO ? 2 : 1];  // the first record of each group, or of the next group
    int4 ga = group(0), gb = group(G > 1 ? 1 : 0);
    first(ga, keep[0]);
    if constexpr (TWO) {
        first(gb, keep[1]);
        select_rec((Unit)UNIT, tid, keep[0]);
        select_rec((Unit)UNIT, tid, keep[1]);
    }
    rows_load(0);
    rows_post(0);
    __syncthreads();
    if (s_begin < s_end) {
        fetch(s_begin);
        post(0);
    }
    __syncthreads();

    // one update group of one sweep: r holds this thread's first record
    auto class_pass = [&](const int4 &g, Rec<FORM> &r, uint32_t t, const GroupKey *gk, const Saturated &sat, auto bufc,
                          auto ahead) {
        constexpr int BUF = decltype(bufc)::value;
        constexpr uint32_t TAB = kLdsPairs + BUF * NE * 8, WTAB = kLdsWide + BUF * kWords15 * 8;
        const int base = g.x + g.z;  // first pair of the group by position
        const Unit unit = TWO ? (Unit)UNIT : unit_of(RS, g.w, T);
        const int work = units_of(unit, g);
        auto loop = [&](auto body) {
            // the first unit reads the kept record in place; later ones are loaded one ahead
            Rec<FORM> nx;
            int j = tid + T;
            if (j < work) fetch_rec(unit, g, j, nx);
            if constexpr (TWO)
                r.pin();
            else
                select_rec(unit, tid, r);
            if (tid < work) body(tid, r);
            ahead();
            while (j < work) {
                Rec<FORM> cur = nx;
                const int at = j;
                j += T;
                if (j < work) fetch_rec(unit, g, j, nx);
                select_rec(unit, at, cur);
                body(at, cur);
            }
        };
        auto sites_of = [&](const Rec<FORM> &c) {
            return FORM == kBitCube4 ? c.word(10) : FORM == kBitCube ? c.word(12) : c.word(15);
        };
        if (unit == kPair) {
            loop([&](int j, const Rec<FORM> &c) {
                uint32_t x[K], n[4];
                slots<FORM, 2>(c, x);
                count<K>(x, n);
                if constexpr (GEN) n[3] = c.word(14);
                lds_put(el(2 * (base + g.y + j)), decide<K, RS, 2, TAB>(n, sites_of(c), gk, jb.k0, jb.k1, sat));
            });
        } else if (unit == kSite) {
            loop([&](int j, const Rec<FORM> &c) {
                uint32_t x[K], n[4];
                slots<FORM, 1>(c, x);
                count<K>(x, n);
                if constexpr (GEN) n[3] = c.word(14);
                lds_put(el(2 * (base + g.y) + j),
                        (uint16_t)decide<K, RS, 1, TAB>(n, sites_of(c), gk, jb.k0, jb.k1, sat));
            });
        } else if constexpr (RS > 4) {
            loop([&](int j, const Rec<FORM> &c) {
                const int q = j % RQ, at = j / RQ;
                uint32_t x[K], n[4];
                slots<FORM, 1>(c, x);
                count<K>(x, n);
                if constexpr (GEN) n[3] = c.word(14);
#pragma unroll
                for (int w = 0; w < (GEN ? 4 : 3); ++w) n[w] >>= 4 * q;
                uint32_t o = decide_quad<K, TAB>(n, sites_of(c) & 0xFFFFu, rg + (uint32_t)q, t, jb.k0,
                                                 jb.k1, sat) << (4 * q);
#pragma unroll
                for (int off = 1; off < RQ; off *= 2) o |= __shfl_xor(o, off, 64);
                if (q == 0) lds_put(el(2 * (base + g.y) + at), (uint16_t)o);
            });
        }
        if constexpr (GEN) {
            // wide pairs, four replicas per thread, on the last threads (the first ones may
            // hold one more unit of the ordinary pairs)
            for (int j = T - 1 - tid; j < 2 * RQ * g.y; j += T) {
                const int q = (j % RQ) ^ (RQ - 1), at = j / RQ;
                uint32_t n[4], odd, site;
                wide_counts(v, g.x + (at >> 1), at & 1, n, odd, site);
#pragma unroll
                for (int w = 0; w < 4; ++w) n[w] >>= 4 * q;
                uint32_t o = decide_quad_wide<WTAB>(n, odd >> (4 * q), site, rg + (uint32_t)q, t, jb.k0, jb.k1)
                             << (4 * q);
#pragma unroll
                for (int off = 1; off < RQ; off *= 2) o |= __shfl_xor(o, off, 64);
                if (q == 0) lds_put(el(2 * base + at), (uint16_t)o);
            }
        }
    };

    auto sweep = [&](int s, auto bufc) {
        constexpr int BUF = decltype(bufc)::value;
        const int k = s - s_begin;
        const bool more = s + 1 < s_end;
        if (more) fetch(s + 1);
        if (k % kRowRun == 0) rows_load(k / kRowRun + 1);
        Saturated sat;
        {
            const u32x4 m = lds_get<u32x4>(kLdsSat + BUF * 32);
            sat = Saturated{{m.x, m.y, m.z, m.w}, lds_u32(kLdsSat + BUF * 32 + 16)};
        }
        const uint32_t t = jb.sweep0 + (uint32_t)s;
        GroupKey gk[RQ];
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            const GroupKey u = group_key(rg + (uint32_t)q, t, jb.k0, jb.k1);
            gk[q] = GroupKey{(uint32_t)__builtin_amdgcn_readfirstlane((int)u.a),
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)u.b),
                             (uint32_t)__builtin_amdgcn_readfirstlane((int)u.c)};
        }
        if constexpr (TWO) {
            class_pass(ga, keep[0], t, gk, sat, bufc, [] {});
            __syncthreads();
            class_pass(gb, keep[1], t, gk, sat, bufc, [] {});
        } else {
            for (int c = 0; c < G; ++c) {
                const int4 g = ga;
                ga = gb;
                gb = group(c + 2);
                class_pass(g, keep[0], t, gk, sat, bufc, [&] { first(ga, keep[0]); });
                if (c + 1 < G) __syncthreads();
            }
        }
        // the other buffers were last read a sweep (rows: more) ago
        if (more) post(BUF ^ 1);
        if (k % kRowRun == kRowRun / 2) rows_post(k / kRowRun + 1);
        __syncthreads();
    };
    for (int s = s_begin; s < s_end;) {
        sweep(s, std::integral_constant<int, 0>{});
        if (++s >= s_end) break;
        sweep(s++, std::integral_constant<int, 1>{});
    }

    // energies: sum_i m_i (I_i + h_i) counts every bond twice and every field twice
    if (jb.energy) {
                if (tid < RS) lds_put(kLdsAcc + 4u * tid, 0);
        __syncthreads();
        int32_t er[RS];
#pragma unroll
        for (int r = 0; r < RS; ++r) er[r] = 0;
        auto add = [&](const uint32_t *n, int planes, int Kx, uint32_t odd, uint32_t own, uint32_t site) {
            const int hv = v.h ? (int)load_global<int8_t>(v.h + site) : 0;
#pragma unroll
            for (int r = 0; r < RS; ++r) {
                int cnt = 0;
                for (int w = 0; w < planes; ++w) cnt += (int)((n[w] >> r) & 1u) << w;
                const int I = Kx - 2 * cnt - (int)((odd >> r) & 1u) + hv;
                er[r] += ((own >> r) & 1u) ? -I : I;
            }
        };
        for (int c = 0; c < G; ++c) {
            const int4 g = group(c);
            for (int j = tid; j < 2 * (g.y + g.w); j += T) {
                const int at = 2 * (g.x + g.z) + j, hh = j & 1;
                const uint32_t i = load_global<uint16_t>(v.pos_site + at);
                if (i == kBitNoSite) continue;
                const uint32_t own = lds_u16(el(at));
                uint32_t n[4], odd, site;
                if (GEN && j < 2 * g.y) {
                    wide_counts(v, g.x + (j >> 1), hh, n, odd, site);
                    add(n, 4, kBitSlotsWide, odd, own, i);
                } else {
                    Rec<FORM> r;
                    r.load(v.rec, v.n_pairs, g.z + (j >> 1) - g.y);
                    r.select(hh);
                    uint32_t x[K];
                    slots<FORM, 1>(r, x);
                    count<K>(x, n);
                    add(n, 3, K, GEN ? r.word(14) : 0u, own, i);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RS; ++r) {
            int e = er[r];
            for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
            if ((tid & 63) == 0)
                __hip_atomic_fetch_add((__attribute__((address_space(3))) int32_t *)(uintptr_t)(kLdsAcc + 4u * r), e, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        if (tid < RS) jb.energy[RS * tile + tid] = -lds_get<int32_t>(kLdsAcc + 4u * tid) / 2;
    }
    // spins out
    for (int p = tid; p < v.n_pos; p += T) {
        const uint32_t i = load_global<uint16_t>(v.pos_site + p);
        if (i == kBitNoSite) continue;
        const uint32_t bits = lds_u16(el(p));
#pragma unroll
        for (int k = 0; k < RQ; ++k)
            *reinterpret_cast<uint32_t *>(gst + stride * i + 4 * k) = bytes_of_bits(bits >> (4 * k));
    }
}

}  // namespace bit

}  // namespace pbit
