// device.h — device-side building blocks of the p-bit sweep for gfx950.
//
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) keyed by the anneal seed,
// and the integer heat-bath decision of the p-bit law m = sgn(tanh(beta I) - u)
// (paper Sec. 1.2.1, Eq. 2) through a per-sweep uint32 minority-threshold row.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pbit {

// Philox4x32-10 block function.  The key words are wave-uniform in every
// caller, so the key schedule runs on the scalar unit; each round is two
// 32x32->64 products (v_mad_u64_u32) and two three-way XORs.
struct Block4 {
    uint32_t w[4];
};

__device__ __forceinline__ Block4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                         uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p = (uint64_t)c0 * 0xD2511F53u;
        const uint64_t q = (uint64_t)c2 * 0xCD9E8D57u;
        // three-input XORs as single v_bitop3_b32 (truth table 0x96 = a ^ b ^ c)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(q >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p >> 32), c3, k1, 0x96);
        c1 = (uint32_t)q;
        c3 = (uint32_t)p;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    Block4 b;
    b.w[0] = c0; b.w[1] = c1; b.w[2] = c2; b.w[3] = c3;
    return b;
}

// Counter domains.
constexpr uint32_t kDomainSweep = 0;
constexpr uint32_t kDomainInit = 1;

// Heat-bath decision for field I, minority threshold T = Tm(beta, |I|) and
// uniform word w: -s if x < T else s, with s = sign(I) (+1 at I = 0) and
// x = ~w for I >= 0, w for I < 0.
__device__ __forceinline__ int8_t decide(int32_t I, uint32_t T, uint32_t w)
{
    const bool pos = I >= 0;
    const uint32_t x = pos ? ~w : w;
    const bool minority = x < T;
    return (pos != minority) ? (int8_t)1 : (int8_t)-1;
}

// v_writelane_b32: lane `lane` of `old` takes the wave-uniform `val` (the
// compiler's intrinsic, bound by name: hip exposes no builtin for it).
__device__ int lane_write(int val, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// q = n / d and r = n % d for 0 <= n < 2^22 and 1 <= d < 2^10 from a float
// reciprocal: the estimate is within one of the quotient and is corrected.
__device__ __forceinline__ int div_small(int n, int d, float inv, int &r)
{
    int q = (int)((float)n * inv);
    int rr = n - q * d;
    if (rr < 0) {
        q -= 1;
        rr += d;
    } else if (rr >= d) {
        q += 1;
        rr -= d;
    }
    r = rr;
    return q;
}

// A load from global memory through a pointer the compiler cannot place (one read
// out of a job descriptor, say): issued as a global load, counted by vmcnt alone.
// Through a generic pointer it would be a flat load, which also counts against
// lgkmcnt, so that every wait for an LDS read would wait for it as well.
template <typename T>
__device__ __forceinline__ T load_global(const void *p)
{
    return *(const __attribute__((address_space(1))) T *)p;
}

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v2i_t __attribute__((ext_vector_type(2)));
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef float v16f_t __attribute__((ext_vector_type(16)));

// ---- biclique fields on the FP4 matrix cores
//
// Spins (+-1 or bits) and couplings (-1, 0, 1) are exact E2M1 numbers, so their products
// are and a float sum of them is up to 2^24 in size.  Accumulators start at kFieldBase =
// 1.5 x 2^21, whose last place is 1/4: their bits are then kFieldBase + 4 sum while the sum
// stays within 2^20, and 4 |I|, the byte offset of a threshold, is a difference of bits.
constexpr uint32_t kFieldBase = 0x4A400000u;

// acc + A B over 64 K values, 32 (four registers) in each lane half; any K order that A and
// B share.
__device__ __forceinline__ v16f_t mfma_fp4(v4i_t a, v4i_t b, v16f_t acc)
{
    const v8i_t x = {a[0], a[1], a[2], a[3], 0, 0, 0, 0}, y = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, y, acc, 4, 4, 0, 127, 0, 127);  // both E2M1, scales 1
}

// 32 spin bits (set = -1) as E2M1 numbers +-1: bit 4 i + j to nibble i of dword j.
__device__ __forceinline__ v4i_t spin_nibbles(uint32_t w)
{
    constexpr uint32_t one = 0x22222222u, sign = 0x88888888u;
    return v4i_t{(int)(one | ((w << 3) & sign)), (int)(one | ((w << 2) & sign)), (int)(one | ((w << 1) & sign)),
                 (int)(one | (w & sign))};
}

// 32 spin bits for a product with couplings scaled to match: bit 4 i + j at nibble i of
// dword j, as 0 or (an E2M1 number) 1/2, 1, 2, 1/2 for j = 0 .. 3.
__device__ __forceinline__ v4i_t spin_bits_fp4(uint32_t w)
{
    return v4i_t{(int)(w & 0x11111111u), (int)(w & 0x22222222u), (int)(w & 0x44444444u), (int)((w >> 3) & 0x11111111u)};
}

// |a - b| + c
__device__ __forceinline__ uint32_t sad(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_sad_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}
__device__ __forceinline__ uint32_t lds_word(uint32_t address)
{
    return *(const __attribute__((address_space(3))) uint32_t *)(uintptr_t)address;
}

// The wave's heat-bath decisions as a mask, set where the new spin is -1: w + Tm(|I|)
// carries for I >= 0 (accumulator bits x from `mid` on), w >= Tm(|I|) for I < 0.
__device__ __forceinline__ uint64_t heat_bath(uint32_t w, uint32_t Tm, uint32_t x, uint32_t mid)
{
    constexpr int kUge = 35;  // wave-wide comparison
    uint32_t sum;
    uint64_t carry;  // as a mask, which the compiler would make of an add, a select and a test
    asm("v_add_co_u32 %0, %1, %2, %3" : "=v"(sum), "=s"(carry) : "v"(w), "v"(Tm));
    const uint64_t up = __builtin_amdgcn_uicmp(x, mid, kUge);
    return (up & carry) | (~up & __builtin_amdgcn_uicmp(w, Tm, kUge));
}

// Initial spin from a domain-1 word.
__device__ __forceinline__ int8_t init_spin(uint32_t w)
{
    return w < 0x80000000u ? (int8_t)1 : (int8_t)-1;
}

}  // namespace pbit
