// Weight forms, their unpacking into matrix operands and the handling of int8 rows, shared by the few-token kernels
// (mnnq_skinny.hip), the GEMM with K split over the waves (mnnq_ksplit.hip) and the wide tiles (mnnq_prefill8w.hip,
// mnnq_prefill_f16w.hip).
#pragma once

#include "mnnq_common.h"

namespace mnnq {

namespace {

typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));

// Weights with an integer zero point or a float minimum, int8 weights as bytes; the first two with fp16 activations.
enum Form { kZp = 0, kMin = 1, kBytes = 2, kZpF16 = 3, kMinF16 = 4 };
constexpr bool is_f16(int form) { return form >= kZpF16; }
constexpr bool has_zero(int form) { return form == kZp || form == kZpF16; }
inline int form_of(const Layout& L, bool f16)
{
    if (f16) return L.minf ? kMinF16 : kZpF16;
    return L.native8 ? kBytes : L.minf ? kMin : kZp;
}

constexpr int kBufFlags = 0x00020000;     // raw buffer, 32-bit data format (gfx9 family)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufFlags);
}

// A lane's part of one chunk of a row tile.
template <int FORM>
struct Weights {
    v4i w[FORM == kBytes ? 2 : 1];   // .x,.y group 2c, .z,.w group 2c + 1; byte form: one register quad per group
    v2f s;                           // scales of the lane's weight row for both groups
    int z;                           // zero points of both groups of two weight rows, the lane's and its neighbour (kZp)
    v2f mn;                          // group minima of both groups                    (kMin, kBytes)
};

// The B operands of a group: one register quad of int8, or two of halves.
template <int FORM>
struct Operand {
    v4i q[is_f16(FORM) ? 2 : 1];
};

// q - z per byte for four codes in the bytes of v (c4 = 0x80 - z in every byte).
__device__ __forceinline__ int sub_zero(uint32_t v, uint32_t c4) { return (int)((v + c4) ^ 0x80808080u); }

// Eight codes (dword w) as halves q - z in natural order: a byte c under the high byte 0x64 is the half 1024 + c, and
// subtracting the half 1024 + z (zb, twice) leaves c - z exactly (float minimum: 1024, the codes stay as they are).
__device__ __forceinline__ v4i halves8(uint32_t w, h2 zb)
{
    const uint32_t lo = w & 0x0f0f0f0fu, hi = (w >> 4) & 0x0f0f0f0fu;
    auto pair = [&](uint32_t v, uint32_t sel) {
        return __builtin_bit_cast(int, __builtin_bit_cast(h2, __builtin_amdgcn_perm(0x64646464u, v, sel)) - zb);
    };
    return v4i{pair(lo, 0x04010400u), pair(lo, 0x04030402u), pair(hi, 0x04010400u), pair(hi, 0x04030402u)};
}

// Group h of a chunk.  zsel: the byte of the lane's row and first group in Weights::z, in every byte.
// CENTERED (float minima with fp16 activations): codes less the middle of their range, see Centered.
template <int FORM, bool CENTERED = false>
__device__ __forceinline__ Operand<FORM> unpack(const Weights<FORM>& r, int h, uint32_t zsel)
{
    Operand<FORM> o;
    if (FORM == kBytes) {
        o.q[0] = r.w[FORM == kBytes ? h : 0];
        return o;
    }
    const uint32_t w0 = (uint32_t)(h ? r.w[0].z : r.w[0].x), w1 = (uint32_t)(h ? r.w[0].w : r.w[0].y);
    const uint32_t sel = h ? zsel + 0x01010101u : zsel;
    if (is_f16(FORM)) {
        // (bytes 1 and 3 of the selector pick 0x64)
        const h2 zb = __builtin_bit_cast(h2, has_zero(FORM) ? __builtin_amdgcn_perm(0x64646464u, (uint32_t)r.z, (sel & 0x00ff00ffu) | 0x04000400u)
                                                            : CENTERED ? 0x64086408u : 0x64006400u);
        o.q[0] = halves8(w0, zb);
        o.q[is_f16(FORM) ? 1 : 0] = halves8(w1, zb);
        return o;
    }
    const uint32_t n0 = w0 & 0x0f0f0f0fu, n1 = (w0 >> 4) & 0x0f0f0f0fu;
    const uint32_t n2 = w1 & 0x0f0f0f0fu, n3 = (w1 >> 4) & 0x0f0f0f0fu;
    if (FORM == kMin) {
        o.q[0] = v4i{(int)n0, (int)n1, (int)n2, (int)n3};
        return o;
    }
    const uint32_t c4 = 0x80808080u - __builtin_amdgcn_perm(0u, (uint32_t)r.z, sel);
    o.q[0] = v4i{sub_zero(n0, c4), sub_zero(n1, c4), sub_zero(n2, c4), sub_zero(n3, c4)};
    return o;
}

__device__ __forceinline__ v4f mfma_f16(v4i a, v4i b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, a), __builtin_bit_cast(h8, b), c, 0, 0, 0);
}

// float(I) from a matrix instruction that accumulated on the bit pattern of 1.5 * 2^23: the register holds
// 0x4B400000 + I, i.e. the float 12582912 + I (|I| < 2^22), and one exact subtraction - full rate, unlike a convert -
// leaves I.
constexpr int kMagicBits = 0x4B400000;
__device__ __forceinline__ float from_magic(int v) { return __int_as_float(v) - 12582912.0f; }

// Float minima on the matrix cores (the GEMMs).  A group's term  scale * sum x q + min * sum x  is taken as
//     scale * sum x (q - mid) + (min + mid * scale) * sum x,   mid = 8 of 4-bit codes (fp16 activations), 128 of bytes:
// the second part is a contraction over the groups, one v_mfma_f32_16x16x4_f32 per tile and four groups (xs: lane l holds the sum
// of token l % 16 in group l / 16 of the four; mn: the coefficient of weight row l % 16), and costs no vector instruction per
// output.  Around the middle of the codes both parts are as small as the term itself; with q as it is they are large and of
// opposite sign, four groups of one before the other, and the sums' error was 13 - 34 % larger than that of scale and minimum group by group.
// A group whose codes are all 0 (a constant one: scale 1, whatever its value) is the minimum alone: its scale counts as 0, so
// that nothing large cancels.  One more matrix instruction per column and group tells: with an all-ones operand it sums the
// group's codes, in every lane of the column.
template <int FORM>
struct Centered {
    static constexpr float mid = FORM == kMinF16 ? 8.0f : 128.0f;

    float lanes;      // mid in the lanes of the group at hand, 0 in the others
    __device__ __forceinline__ Centered(int group, int kb) : lanes(kb == group ? mid : 0.0f) {}

    static __device__ __forceinline__ v4i column_sum(const Operand<FORM>& o)
    {
        const v4i one = is_f16(FORM) ? v4i{0x3c003c00, 0x3c003c00, 0x3c003c00, 0x3c003c00} : v4i{0x01010101, 0x01010101, 0x01010101, 0x01010101};
        if constexpr (is_f16(FORM))
            return __builtin_bit_cast(v4i, mfma_f16(one, o.q[1], mfma_f16(one, o.q[0], v4f{0.0f, 0.0f, 0.0f, 0.0f})));
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(one, o.q[0], v4i{0, 0, 0, 0}, 0, 0, 0);
    }
    // s: the group's scale, mn: minimum -> coefficient, in the lanes of the group.
    __device__ __forceinline__ void operator()(v4i sum, float& s, float& mn) const
    {
        const bool lowest = is_f16(FORM) ? __int_as_float(sum[0]) == -64.0f * mid : sum[0] == (int)(-64.0f * mid);
        s *= lowest ? 0.0f : 1.0f;      // (an infinite scale stays a NaN)
        mn = fmaf(lanes, s, mn);
    }
};

// A lane's four results of a 16 x 16 tile, y[m + r][n] = f[r] * scale[r] + shift, as fp32 or binary16; rows past M lie past the
// end of y, columns past N are sent there.
__device__ __forceinline__ void store_tile(__amdgpu_buffer_rsrc_t rs_y, const Layout& L, int m, int n, v4f f, const float (&scale)[4],
                                           float shift)
{
    const int N = (int)L.N;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float o = fmaf(f[r], scale[r], shift);
        const int at = n < N ? ((m + r) * N + n) * (L.out16 ? 2 : 4) : 0x7fff0000;
        if (L.out16) {
            const _Float16 q = (_Float16)o;
            __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, q), rs_y, at, 0, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(o), rs_y, at, 0, 0);
        }
    }
}

// Centred sums of a weight row cannot express a group whose scale or minimum is infinite or NaN, or whose coefficient overflows
// (imported parameters; the quantizer makes none): infinity around the middle of the codes and infinity times the
// activations' sum meet as NaN, and the zeros of the other groups' lanes do as well.  The row's sums are then not finite for any
// token, so that one token per tile tells and the loops need no check; a wave that sees it computes its tiles again, one by one,
// with the codes as they are: scale * (sum x q) + minimum * (sum x), group by group.
// first: cell (chunk of a row tile) that the tile's weights start at; load_a(c, h): the A operand of group h of chunk c.
template <int FORM, typename LoadA>
__device__ __forceinline__ v4f tile_by_definition(__amdgpu_buffer_rsrc_t packed, const Layout& L, int lane, int first, LoadA load_a)
{
    constexpr int WB = FORM == kBytes ? 2048 : 1024, X = is_f16(FORM) ? 1 : 0;
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101}, onesh = {0x3c003c00, 0x3c003c00, 0x3c003c00, 0x3c003c00};
    const v4i zero4 = {0, 0, 0, 0};
    const v4f zerof = {0.0f, 0.0f, 0.0f, 0.0f};
    v4f y = zerof;
#pragma unroll 1
    for (int c = 0; c < (int)L.C; ++c) {
        const int at = (lane & 15) * 8;
        Weights<FORM> w;
#pragma unroll
        for (int h = 0; h < (FORM == kBytes ? 2 : 1); ++h)
            w.w[h] = __builtin_amdgcn_raw_buffer_load_b128(packed, lane * 16 + h * 1024, (first + c) * WB, 0);
        w.s = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(packed, at, (int)L.scales_off() + (first + c) * 128, 0));
        w.mn = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(packed, at, (int)L.zeros_off() + (first + c) * 128, 0));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const Operand<FORM> a = load_a(c, h), b = unpack<FORM>(w, h, 0);
            v4f d, x;
            if constexpr (is_f16(FORM)) {
                d = mfma_f16(a.q[X], b.q[X], mfma_f16(a.q[0], b.q[0], zerof));
                x = mfma_f16(a.q[X], onesh, mfma_f16(a.q[0], onesh, zerof));
            } else {
                const v4i di = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.q[0], b.q[0], zero4, 0, 0, 0);
                const v4i xi = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.q[0], ones, zero4, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) d[r] = (float)(di[r] + xi[r] * (FORM == kBytes ? 128 : 0)), x[r] = (float)xi[r];
            }
            const float s = h ? w.s.y : w.s.x, mn = h ? w.mn.y : w.mn.x;
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = fmaf(mn, x[r], fmaf(s, d[r], y[r]));
        }
    }
    return y;
}

// Rows of int8 codes (calls that bring their codes).  Read in the operand's order - lane l: token l % 16, k block l / 16 -
// four neighbouring lanes ask for 16 bytes of four tokens each, and the calls lost to the tiled GEMM wherever the token
// blocks won; here they take 64 consecutive bytes of one token (lane l: token l / 4, k block l % 4), the two groups of a
// chunk - one line - are requested together, and the operand's order is made in registers, through the LDS crossbar, a row
// of tiles ahead (1024 tokens of 3584 x 18944 183 -> 141 us, 128 of 3584 x 3584 24.6 -> 13.6 us, int8 bytes 1024 tokens of
// 3584 x 18944 216 -> 172 us; whole lines staged through LDS instead: the same within 2 %).
struct RowExchange {
    int from;       // byte address of the lane that holds this lane's piece
    __device__ __forceinline__ explicit RowExchange(int lane) : from((4 * (lane & 15) + (lane >> 4)) * 4) {}
    __device__ __forceinline__ void operator()(v4i& v) const
    {
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = __builtin_amdgcn_ds_bpermute(from, v[d]);
    }
};

}  // namespace

}  // namespace mnnq
