// fp6 (e2m3) operand packing shared by the load-time plane, the per-call activation planes and the quantizer that
// writes them directly (see mnnq_prefill6.hip for the operand layout).
#pragma once

#include "mnnq_common.h"

namespace mnnq {

// fp6 packing.  c[0..7]: 32 six-bit codes, one per byte, code j in byte j % 4 of c[j / 4].
// out[0..5]: the same codes at bits [6 j, 6 j + 6).
__device__ __forceinline__ uint32_t pack24(uint32_t c)
{
    return (c & 0x3fu) | ((c >> 2) & 0xfc0u) | ((c >> 4) & 0x3f000u) | ((c >> 6) & 0xfc0000u);
}

__device__ __forceinline__ void pack_fp6(const uint32_t (&c)[8], uint32_t (&out)[6])
{
    const uint32_t p0 = pack24(c[0]), p1 = pack24(c[1]), p2 = pack24(c[2]), p3 = pack24(c[3]);
    const uint32_t p4 = pack24(c[4]), p5 = pack24(c[5]), p6 = pack24(c[6]), p7 = pack24(c[7]);
    out[0] = p0 | (p1 << 24);
    out[1] = (p1 >> 8) | (p2 << 16);
    out[2] = (p2 >> 16) | (p3 << 8);
    out[3] = p4 | (p5 << 24);
    out[4] = (p5 >> 8) | (p6 << 16);
    out[5] = (p6 >> 16) | (p7 << 8);
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
// hi = |xq| >> 4 (0..8), lo = |xq| & 15; the code of a part is its magnitude with the sign in bit 5, zero parts stay
// all-zero codes.
__device__ __forceinline__ void split_act(uint32_t x, uint32_t& hi, uint32_t& lo)
{
    const uint32_t neg = (x >> 7) & 0x01010101u;              // 1 in the bytes with xq < 0
    const uint32_t mag = (x ^ (neg * 255u)) + neg;            // |xq| (at most 128: no carry between bytes)
    const uint32_t ml = mag & 0x0f0f0f0fu, mh = (mag >> 4) & 0x0f0f0f0fu;
    const uint32_t nzl = ((ml + 0x0f0f0f0fu) >> 4) & 0x01010101u, nzh = ((mh + 0x0f0f0f0fu) >> 4) & 0x01010101u;
    lo = ml | ((neg & nzl) << 5);
    hi = mh | ((neg & nzh) << 5);
}

}  // namespace mnnq
