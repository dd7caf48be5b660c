// Shared definitions of the mnnq HIP library (gfx950 only).
//
// Packed weight layout ("chunk layout").  The paper rearranges weights once at
// load so that the inner loop reads exactly what one instruction consumes
// (Section 5.1); on CDNA4 the unit is one 128-bit load per lane of a 64-wide
// wavefront:
//
//   row tile  t = n / 16            (16 output rows)
//   chunk     c = g / 2             (two quantization groups = 128 values of K)
//   C = ceil(G / 2) chunks per row tile; an odd G gets one zero padding group.
//
//   codes  : [T][C][64 lanes][16 B]   at byte 0
//            lane l serves row 16 t + (l % 16), k-block kb = l / 16;
//            bytes 0..7  = its 16 codes of group 2c   (k = 64 (2c)   + 16 kb + j),
//            bytes 8..15 = its 16 codes of group 2c+1 (k = 64 (2c+1) + 16 kb + j).
//            Inside 8 bytes, dword d, byte b holds code j = 8 d + b in the low
//            nibble and code j = 8 d + 4 + b in the high nibble, so that
//            `w & 0x0f0f0f0f` and `(w >> 4) & 0x0f0f0f0f` give codes 8d..8d+3
//            and 8d+4..8d+7 in byte order.
//   scales : [T][C][16 rows][2] fp32  at byte T*C*1024
//   zeros  : [T][C][16 rows][2] u8    at byte T*C*1024 + T*C*128        (mode MNNQ_W4_ZP_INT)
//   mins   : [T][C][16 rows][2] fp32  at the same place                 (mode MNNQ_W4_MIN_FLOAT:
//            the group minimum of Eq. 1 as a float offset instead of an integer zero point)
//
// One chunk is exactly one wave-wide 128-bit load (1 KiB) for the decode GEMV,
// and lane l's 16 bytes are exactly its B operands of two 16x16x64 int8 MFMAs
// (one per group) for the prefill GEMM.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/mnnq.h"

namespace mnnq {

constexpr int kGroup = 64;
constexpr int kTileN = 16;
constexpr int kChunkBytes = 1024;

// int8 weights (mode MNNQ_W8_MIN_FLOAT) reuse this layout and the int4 kernels: a code
// q8 = 16 hi + lo is stored as two 4-bit planes along a doubled reduction axis - groups
// 0..G-1 hold the high nibbles with step 16 s and the group minimum, groups G..2G-1 the low
// nibbles with step s and minimum 0 - so that q8 s + min = hi (16 s) + min + lo s.  The
// activation row is not doubled: chunk c of the packed matrix meets chunk c % Cx of the row.
// Byte form of int8 weights (mode flag MNNQ_NATIVE_8BIT): the reduction axis is not doubled; chunk
// (t, c) is two kilobytes, one per group - lane l of kilobyte h holds the 16 codes k = 64 (2 c + h) +
// 16 (l / 16) + j of row 16 t + l % 16 as bytes q8 - 128, i.e. the B operand of v_mfma_i32_16x16x64_i8 and
// of four v_dot4_i32_i8 as it stands; scales (the step s) and minima [T][C][16][2] fp32 as in the float
// minimum form.  With D = sum xq (q8 - 128) and xs = sum xq a group's term is  s D + (min + 128 s) xs.
// Matrix-core plane (mode flag MNNQ_WITH_MATRIX_PLANE): a second copy of the int4 weights behind the
// chunk layout, as the B operand of the fp6 matrix instruction v_mfma_scale_f32_32x32x64_f8f6f4 -
// every q - zero (|q - zero| <= 15) is the e2m3 value (q - zero) / 8 exactly, and its code is the
// sign-magnitude form of q - zero.  Unit: column tile tn = n / 32 and group g (64 values of K):
//   codes  [G][T32p][1536 B]: lane l (0..63) holds column 32 tn + l % 32 and the 32 values
//          k = 64 g + 32 (l / 32) + j, j = 0..31, code j at bits [6 j, 6 j + 6) of its 192 bits;
//          dwords 0..3 of lane l at byte 16 l, dwords 4..5 at byte 1024 + 8 l of the block;
//   scales [G][T32p][32] fp32 behind the codes.
// T32p = column tiles rounded up to a multiple of 8 (zero codes and scales in the padding), so that a
// workgroup's tile of up to 256 columns is one contiguous, in-range piece per group.
constexpr int kPlaneBlockBytes = 1536;
constexpr int kPlaneTilePad = 8;

struct Layout {
    int64_t N, K;   // K: length of the packed reduction axis (2 x the row length for int8 weights)
    int64_t Kx;     // length of an activation row
    int64_t Cx;     // chunks of an activation row
    int mode;       // mnnq_mode
    bool minf;      // groups carry an fp32 minimum instead of a one-byte zero point
    bool out16;     // the output array holds IEEE binary16 values (set per call, not a property of the packing)
    int64_t T;  // row tiles
    int64_t G;  // groups per row
    int64_t C;  // chunks per row tile
    size_t codes_bytes, scales_bytes, zeros_bytes;
    bool native8;     // int8 weights as bytes: a chunk is two kilobytes, one per group (see below)
    bool plane;       // the packed buffer carries the matrix-core plane behind the chunk layout
    int64_t T32p;     // column tiles of 32 in the plane (padded to a multiple of 8)
    int64_t Gx;       // quantization groups of an activation row (= groups of the plane)
    __host__ __device__ size_t scales_off() const { return codes_bytes; }
    __host__ __device__ size_t zeros_off() const { return codes_bytes + scales_bytes; }
    // bytes of the chunk layout (what the decode kernels and the int8 GEMM read)
    __host__ __device__ size_t total() const { return codes_bytes + scales_bytes + zeros_bytes; }
    __host__ __device__ size_t plane_off() const { return (total() + 255) / 256 * 256; }
    __host__ __device__ size_t plane_codes_bytes() const { return (size_t)Gx * T32p * kPlaneBlockBytes; }
    __host__ __device__ size_t plane_scales_bytes() const { return (size_t)Gx * T32p * 32 * sizeof(float); }
    __host__ __device__ size_t plane_bytes() const { return plane_codes_bytes() + plane_scales_bytes(); }
    // bytes of the whole packed buffer
    __host__ __device__ size_t full_total() const { return plane ? plane_off() + plane_bytes() : total(); }
};

constexpr int kModeMask = 15;

inline __host__ __device__ Layout make_layout(int64_t N, int64_t K, int mode_and_flags = MNNQ_W4_ZP_INT)
{
    Layout L;
    const int mode = mode_and_flags & kModeMask;
    L.plane = (mode_and_flags & MNNQ_WITH_MATRIX_PLANE) != 0;
    L.T32p = ((N + 31) / 32 + kPlaneTilePad - 1) / kPlaneTilePad * kPlaneTilePad;
    L.Gx = K / kGroup;
    L.N = N;
    L.native8 = mode == MNNQ_W8_MIN_FLOAT && (mode_and_flags & MNNQ_NATIVE_8BIT) != 0;
    L.Kx = K;
    L.K = (mode == MNNQ_W8_MIN_FLOAT && !L.native8) ? 2 * K : K;
    L.mode = mode;
    L.minf = (mode != MNNQ_W4_ZP_INT);
    L.out16 = false;
    L.T = N / kTileN;
    L.G = L.K / kGroup;
    L.C = (L.G + 1) / 2;
    L.Cx = (K / kGroup + 1) / 2;
    L.codes_bytes = (size_t)L.T * L.C * kChunkBytes * (L.native8 ? 2 : 1);
    L.scales_bytes = (size_t)L.T * L.C * 32 * sizeof(float);
    L.zeros_bytes = (size_t)L.T * L.C * 32 * (L.minf ? sizeof(float) : 1);
    return L;
}

#if defined(__HIPCC__)
// One output value: fp32, or rounded once (nearest even) to binary16 when the call asked for it.
__device__ __forceinline__ void store_out(float* y, int64_t i, float v, bool out16)
{
    if (out16) reinterpret_cast<_Float16*>(y)[i] = (_Float16)v;
    else y[i] = v;
}

// Activation codes (Section 4.2, per-token symmetric int8): the definition is
// clamp(rint(fl(x / scale)), -127, 127) with IEEE binary32 operations, but
// a correctly rounded division per element is expensive (about ten vector
// instructions).  The exact product r = x * fl(1 / scale) differs from fl(x / scale) by
// less than 3 * 2^-24 * 127.5 < 2.3e-5, so both round to the same integer unless
// r is within that distance of a half-integer, i.e. unless |r - rint(r)| exceeds
// 0.5 - 6e-5 (a fused multiply-add gives it with one rounding of at most 2^-25); only then
// (about one element in ten thousand) the division is done, for the four elements of a dword
// together.  |r| <= 127 (1 + 2^-22) in this path, so rint(r) needs no clamp.
// (lim is 0.5 - 6e-5 normally; negative - "always divide" - when 1 / scale is not
// a normal number; the division path clamps as the definition does.)
// rint(r) itself is taken from the fused sum x * fl(1 / scale) + 1.5 * 2^23 (round to nearest even
// happens in it), not from a rounding and a convert instruction per element - converts run at a
// fraction of the rate of the other vector instructions.
__device__ __forceinline__ int quant4_fast(float4 v, float scale, float inv, float lim)
{
    // Round to nearest even by adding 1.5 * 2^23: for |r| < 2^22 the sum is exactly 12582912 + rint(r),
    // and its bit pattern is 0x4B400000 + rint(r), i.e. the low byte already is the int8 code.
    constexpr float kMagic = 12582912.0f;
    float m0 = __builtin_fmaf(v.x, inv, kMagic), m1 = __builtin_fmaf(v.y, inv, kMagic);
    float m2 = __builtin_fmaf(v.z, inv, kMagic), m3 = __builtin_fmaf(v.w, inv, kMagic);
    const float d0 = fabsf(__builtin_fmaf(v.x, inv, kMagic - m0)), d1 = fabsf(__builtin_fmaf(v.y, inv, kMagic - m1));
    const float d2 = fabsf(__builtin_fmaf(v.z, inv, kMagic - m2)), d3 = fabsf(__builtin_fmaf(v.w, inv, kMagic - m3));
    if (!(fmaxf(fmaxf(d0, d1), fmaxf(d2, d3)) <= lim)) {
        m0 = fminf(fmaxf(rintf(v.x / scale), -127.0f), 127.0f) + kMagic;
        m1 = fminf(fmaxf(rintf(v.y / scale), -127.0f), 127.0f) + kMagic;
        m2 = fminf(fmaxf(rintf(v.z / scale), -127.0f), 127.0f) + kMagic;
        m3 = fminf(fmaxf(rintf(v.w / scale), -127.0f), 127.0f) + kMagic;
    }
    // low bytes of the four patterns into one dword
    const uint32_t lo = __builtin_amdgcn_perm(__float_as_uint(m1), __float_as_uint(m0), 0x0c0c0400u);
    const uint32_t hi = __builtin_amdgcn_perm(__float_as_uint(m3), __float_as_uint(m2), 0x04000c0cu);
    return (int)(lo | hi);
}

// Lane exchange inside a row of 16 lanes as an operand modifier of the vector ALU (a general shuffle
// goes through the LDS pipe and costs a round trip each).  CTRL: 0xB1 / 0x4E = lanes xor 1 / xor 2
// of a quad, 0x141 / 0x140 = mirror of 8 / of 16 lanes.
template <int CTRL>
__device__ __forceinline__ int row_exchange(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

// Maximum of a non-negative, non-NaN value over the wave (as integers: the order of such floats),
// the same in all lanes.
__device__ __forceinline__ float wave_max_nonneg(float a)
{
    int v = __float_as_int(a);
    v = max(v, row_exchange<0xB1>(v));
    v = max(v, row_exchange<0x4E>(v));
    v = max(v, row_exchange<0x141>(v));
    v = max(v, row_exchange<0x140>(v));     // every lane: maximum of its row of 16
    const int m = max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                      max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
    return __int_as_float(m);
}

// Sum over each row of 16 lanes, the same in all of its lanes.
__device__ __forceinline__ int row_sum16(int v)
{
    v += row_exchange<0xB1>(v);
    v += row_exchange<0x4E>(v);
    v += row_exchange<0x141>(v);     // the quads hold equal values: the mirrored lane is in the other quad
    v += row_exchange<0x140>(v);
    return v;
}

__device__ __forceinline__ float quant_fast_limit(float scale, float inv)
{
    return (inv < 1.0e37f && scale > 1.0e-30f) ? 0.5f - 6.0e-5f : -1.0f;   // largest |r - rint(r)| of the fast path
}

#endif

// Test and tuning switches (mnnq_debug_set): nullptr unless set by that call.  The launch plans depend
// on the shapes alone otherwise; the environment is never read.
enum DebugKey {
    kDbgDecodeKsplit, kDbgDecodeWaves, kDbgDecodeEarly, kDbgPrefillTile, kDbgNoSkinny, kDbgSkinnyStaged,
    kDbgW8Planes, kDbgFusedTwoKernelMib, kDbgPrefill6Plan, kDbgPrefill6Stages, kDbgCount
};
const char* debug_option(DebugKey key);

// Records a failing HIP call for mnnq_last_hip_error() and maps it to a status.
int record_hip_error(hipError_t e);

#define MNNQ_HIP_TRY(expr)                                   \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return ::mnnq::record_hip_error(e_); \
    } while (0)

// Kernel launchers (one translation unit each).  All return a status.
int launch_pack(const float* W, const Layout& L, uint8_t* packed, hipStream_t st);
// zero: uint8 zero points (mode MNNQ_W4_ZP_INT) or fp32 group minima (mode MNNQ_W4_MIN_FLOAT), [N, G].
int launch_repack(const uint8_t* q, const float* scale, const void* zero, const Layout& L, uint8_t* packed,
                  hipStream_t st);
int launch_unpack(const uint8_t* packed, const Layout& L, uint8_t* q, float* scale, void* zero,
                  hipStream_t st);
int launch_quant_act(const float* x, int64_t M, int64_t K, int8_t* xq, float* sx, int32_t* xsum,
                     hipStream_t st);
// The same quantizer with the codes in the order of the kernel behind it (fused prefill): token blocks for
// launch_skinny, activation planes for launch_prefill6 (TMp: prefill6_row_tiles(M)).  possible: the row length fits.
bool quant_packed_possible(int64_t K);
int launch_quant_token_blocks(const float* x, int64_t M, int64_t K, int8_t* xq, float* sx, hipStream_t st);
int launch_quant_planes(const float* x, int64_t M, int64_t K, int TMp, void* planes, float* sx, hipStream_t st);
int launch_decode(const uint8_t* packed, const Layout& L, const int8_t* xq, const float* sx,
                  const float* bias, float* y, hipStream_t st);
bool decode_fused_splits(const Layout& L);   // the quantizer of a one-token fused call in a kernel of its own
int launch_decode_fused(const uint8_t* packed, const Layout& L, const float* x, const float* bias, float* y,
                        hipStream_t st);
int launch_decode_acc(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq,
                      int32_t* acc, hipStream_t st);
int launch_prefill(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq,
                   const float* sx, const float* bias, float* y, int32_t* acc_debug, hipStream_t st);
// GEMM on the fp6 matrix instructions (mnnq_prefill6.hip): needs the matrix-core plane in the packed
// buffer and `planes_ws`, prefill6_ws_bytes(M, K) bytes of scratch for the activation planes.
int launch_plane_build(uint8_t* packed, const Layout& L, hipStream_t st);
// planes: the activation planes launch_act_planes wrote for the same M and K.
int launch_act_planes(const int8_t* xq, int64_t M, int64_t K, void* planes, hipStream_t st);
int launch_prefill6(const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx,
                    const float* bias, float* y, int32_t* acc_debug, hipStream_t st);
size_t prefill6_ws_bytes(int64_t M, int64_t K);
// possible: the plane is there, more than 32 tokens, sizes within the kernels' 32-bit offsets.
bool prefill6_possible(const Layout& L, int64_t M);
void describe_prefill6(const Layout& L, int64_t M, int32_t out[8]);
int prefill6_row_tiles(int64_t M);
// The same product with K split over the waves of a workgroup (mnnq_ksplit6.hip), for shapes with few output tiles.
size_t ksplit6_lds_bytes(int form);
int launch_ksplit6(int form, const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx,
                   const float* bias, float* y, hipStream_t st);
// The same product on tiles of 64 tokens x 384 columns whose waves share the tokens (mnnq_prefill6w.hip); ks: K parts (1, 2).
size_t prefill6_wide_lds_bytes(int ks);
int launch_prefill6_wide(int ks, const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx,
                         const float* bias, float* y, hipStream_t st);
// A few tokens sharing one pass over the weights; token_blocks: xq as launch_quant_token_blocks writes it.
bool skinny_wanted(const Layout& L, int64_t M);
int launch_skinny(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, bool token_blocks, const float* sx,
                  const float* bias, float* y, hipStream_t st);
// The same with fp16 activations.
bool skinny_f16_wanted(const Layout& L, int64_t M);
int launch_skinny_f16(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16, const float* bias, float* y,
                      hipStream_t st);
// The GEMMs with K split over the waves of a workgroup (mnnq_ksplit.hip); token_blocks as for launch_skinny.
bool ksplit8_wanted(const Layout& L, int64_t M);
int launch_ksplit8(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, bool token_blocks, const float* sx,
                   const float* bias, float* y, hipStream_t st);
bool ksplit_f16_wanted(const Layout& L, int64_t M);
int launch_ksplit_f16(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16, const float* bias, float* y,
                      hipStream_t st);
int launch_decode_f16(const uint8_t* packed, const Layout& L, const uint16_t* x16, const float* bias,
                      float* y, hipStream_t st);
// rs: optional per-row factor applied to the fp32 sums before the bias (NULL = none).
int launch_prefill_f16(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16,
                       const float* rs, const float* bias, float* y, hipStream_t st);
// What the tiled GEMM with int4 zero-point weights, and the one with K split over waves, are expected to take (microseconds).
float prefill_f16_us(const Layout& L, int64_t M);
float ksplit_f16_us(const Layout& L, int64_t M);
// The same on tiles of 128 tokens x 256, 192 or 128 columns (mnnq_prefill_f16w.hip): int4 weights with a zero point; ks: K parts
// (1 or 2; of 128 columns 4).
int launch_prefill_f16_wide(int columns, int ks, const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16,
                            const float* rs, const float* bias, float* y, hipStream_t st);
// The int8 GEMM on tiles of 128 tokens x 256 or 192 columns (mnnq_prefill8w.hip): int4 with a zero point, int8 bytes; ks: K
// parts (1, 2).
// prefill8_us: what the tiled int8 GEMM is expected to take where it has more than one tile per CU, else 0.
float prefill8_us(const Layout& L, int64_t M);
size_t prefill8_wide_lds_bytes(int columns, int ks);
int launch_prefill8_wide(int columns, int ks, const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, const float* sx,
                         const float* bias, float* y, hipStream_t st);

// The largest operand of a prefill call (32-bit byte offsets; operands are multiples of 16 bytes).
constexpr int64_t kMaxBufferBytes = ((int64_t)1 << 31) - 1;

// Compute units of the current device (cached per thread and device).
int num_cus();

// Output tiles of a GEMM by XCD: workgroup b runs on XCD b % 8, and each XCD takes an even run of the tiles in column order,
// so that a column of weights is fetched into one L2 (two where a run ends inside it) and the rules that count tiles per
// CU hold.  Whole columns per XCD - 36 columns are five for four of them, four for the others - left a CU of the fuller
// XCDs with a second tile where there was one per CU: fp16 activations, 1792 tokens of 4608 x 3584, 252 tiles, 119 us; fp6,
// 1328 tokens of 2256 x 5504, 198 tiles, 63 against 35 us.  Where whole columns cost no round they fetch less (1024 tokens of 37888 x 3584
// in fp6 268 against 305 MB) but are no faster: 187.2 / 186.4 us there, 2048 x 28672 x 4096 304.1 / 303.0, 1.006 : 1 over 85 fp6 shapes
// and 1.001 : 1 over 107 int8 ones, so that there is one way.
constexpr int kXcdCount = 8;
inline int64_t xcd_tile_grid(int64_t MT, int64_t NT) { return (MT * NT + kXcdCount - 1) / kXcdCount * kXcdCount; }
__device__ __forceinline__ bool xcd_tile(int MT, int NT, int& tile_m, int& tile_n)
{
    const int tiles = MT * NT, run = (tiles + kXcdCount - 1) / kXcdCount;
    const int t = (int)(blockIdx.x % kXcdCount) * run + (int)(blockIdx.x / kXcdCount);
    tile_m = t % MT;
    tile_n = t / MT;
    return t < tiles;
}

// LDS of a workgroup on gfx950, and the amount a kernel may use without asking.
constexpr size_t kLdsPerWorkgroup = 160 * 1024;
constexpr size_t kLdsDefault = 64 * 1024;

// Allows `kern` more than 64 KiB of dynamic LDS (needed once per kernel and device; remembered per
// thread in `allowed_dev`, which starts at -1).  Returns a status.
template <typename Kernel>
int allow_large_lds(Kernel kern, size_t bytes, int& allowed_dev)
{
    if (bytes <= kLdsDefault) return MNNQ_OK;
    if (bytes > kLdsPerWorkgroup) return MNNQ_ERR_UNSUPPORTED;
    int dev = 0;
    MNNQ_HIP_TRY(hipGetDevice(&dev));
    if (allowed_dev != dev) {
        MNNQ_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)kLdsPerWorkgroup));
        allowed_dev = dev;
    }
    return MNNQ_OK;
}

// Launch configuration the launchers above would choose (host logic only, nothing is launched).
// prefill: {tile rows, tile columns, K parts in the workgroup, K split over workgroups, waves per
// workgroup, LDS bytes, workgroups, 1 if the nibble planes of int8 weights are merged};
// decode: {waves per workgroup, waves per row tile, chunks held in registers, 1 if the wave loops with
// a prefetch, LDS bytes, workgroups, row tiles per workgroup, 0}.
void describe_prefill(const Layout& L, int64_t M, int32_t out[8]);
// few tokens, K split and fp16 tiles: {family (mnnq_plan_debug, what = 4), tile tokens, tile weight rows, waves, waves the
// kernel is built for, chunks held in registers, workgroups (not for few tokens)}
void describe_skinny(const Layout& L, int64_t M, bool f16, int32_t out[8]);
void describe_ksplit(const Layout& L, int64_t M, bool f16, int32_t out[8]);
void describe_prefill_f16(const Layout& L, int64_t M, int32_t out[8]);
void describe_decode(const Layout& L, bool fused, int32_t out[8]);

}  // namespace mnnq
