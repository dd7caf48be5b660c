// fp6 (e2m3) operand packing shared by the load-time plane, the per-call activation planes and the quantizer that
// writes them directly (see mnnq_prefill6.hip for the operand layout).
#pragma once

#include "mnnq_common.h"

namespace mnnq {

// fp6 packing.  c[0..7]: 32 six-bit codes, one per byte (bits 6 and 7 clear), code j in byte j % 4 of c[j / 4].
// out[0..5]: the same codes at bits [6 j, 6 j + 6).  A dot product with 1 and 64 puts two codes side by side in one
// instruction, and shift-or brings eight such pairs into three dwords: 17 instructions for 16 codes.
__device__ __forceinline__ void pack_fp6_half(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t* out)
{
    constexpr uint32_t kLow = 0x00004001u, kHigh = 0x40010000u;   // bytes 0 and 1, bytes 2 and 3
    const uint32_t q0 = __builtin_amdgcn_udot4(c0, kLow, 0, false), q1 = __builtin_amdgcn_udot4(c0, kHigh, 0, false);
    const uint32_t q2 = __builtin_amdgcn_udot4(c1, kLow, 0, false), q3 = __builtin_amdgcn_udot4(c1, kHigh, 0, false);
    const uint32_t q4 = __builtin_amdgcn_udot4(c2, kLow, 0, false), q5 = __builtin_amdgcn_udot4(c2, kHigh, 0, false);
    const uint32_t q6 = __builtin_amdgcn_udot4(c3, kLow, 0, false), q7 = __builtin_amdgcn_udot4(c3, kHigh, 0, false);
    out[0] = (q2 << 24) | ((q1 << 12) | q0);
    out[1] = (q5 << 28) | ((q4 << 16) | ((q3 << 4) | (q2 >> 8)));
    out[2] = (q7 << 20) | ((q6 << 8) | (q5 >> 4));
}

__device__ __forceinline__ void pack_fp6(const uint32_t (&c)[8], uint32_t (&out)[6])
{
    pack_fp6_half(c[0], c[1], c[2], c[3], out);
    pack_fp6_half(c[4], c[5], c[6], c[7], out + 3);
}

// Sign-magnitude six-bit codes of four small integers held as bytes 0x80 + v (|v| <= 15).
__device__ __forceinline__ uint32_t signmag_from_biased(uint32_t b)
{
    const uint32_t neg = (~b >> 7) & 0x01010101u;             // 1 in the bytes of negative values
    const uint32_t v = b ^ 0x80808080u;                       // the values as two's complement bytes
    return ((v ^ (neg * 255u)) + neg) | (neg << 5);           // (|v| <= 15: no carry between bytes; zero has no sign)
}

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Load-time stores: nothing reads them back soon (see pack_kernel).
template <typename V>
__device__ __forceinline__ void store_once(uint8_t* p, V v) { __builtin_nontemporal_store(v, reinterpret_cast<V*>(p)); }

// One block (1536 B) of a plane: six dwords per lane, dwords 0..3 of lane l at 16 l, dwords 4..5 at
// 1024 + 8 l - a kilobyte of 16-byte units and half a kilobyte of 8-byte units, both read without
// bank conflicts.
__device__ __forceinline__ void store_block(uint8_t* block, int lane, const uint32_t (&d)[6])
{
    store_once(block + lane * 16, v4u{d[0], d[1], d[2], d[3]});
    store_once(block + 1024 + lane * 8, v2u{d[4], d[5]});
}

// One pair of blocks of the activation planes (3072 B, high and low parts of 32 rows and one group): twelve dwords per
// lane - six of the high part, six of the low part - as three kilobytes of 16-byte units, so that three 128-bit loads
// bring both operands into consecutive registers.  (The vector memory pipe takes as long for a 64-bit load as for a
// 128-bit one.)
__device__ __forceinline__ void store_pair(uint8_t* pair, int lane, const uint32_t (&hi)[6], const uint32_t (&lo)[6])
{
    uint4* p = reinterpret_cast<uint4*>(pair) + lane;
    p[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    p[64] = make_uint4(hi[4], hi[5], lo[0], lo[1]);
    p[128] = make_uint4(lo[2], lo[3], lo[4], lo[5]);
}

// Four int8 activations (bytes) -> six-bit codes of their high and low parts: xq = s (16 hi + lo) with s = +-1,
// hi = |xq| >> 4 (0..8), lo = |xq| & 15; the code of a part is its magnitude with the sign in bit 5.  (A zero part of
// a negative value is -0, whose products add nothing.)
__device__ __forceinline__ void split_act(uint32_t x, uint32_t& hi, uint32_t& lo)
{
    // 255 in the bytes with xq < 0: the permute's selectors 8..11 repeat the sign of bytes 1, 3 (of x) and 5, 7 (of
    // x << 8, i.e. bytes 0 and 2 of x)
    const uint32_t neg = __builtin_amdgcn_perm(x << 8, x, 0x090b080au);
    const uint32_t mag = (x ^ neg) + (neg & 0x01010101u);     // |xq| (at most 128: no carry between bytes)
    const uint32_t sign = neg & 0x20202020u;
    lo = (mag & 0x0f0f0f0fu) | sign;
    hi = ((mag >> 4) & 0x0f0f0f0fu) | sign;
}

}  // namespace mnnq
