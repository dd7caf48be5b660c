// Load-time step: quantize fp32 weights to asymmetric int4 (Section 4.2, Eq. 1,
// groups of 64 along K; with an integer zero point or, as the equation is
// printed, with the group minimum as a float offset) and store them in the chunk layout
// described in mnnq_common.h; plus the inverse view used by tests and export,
// and the import of already quantized weights into the same layout.
//
// This file is compiled with -ffp-contract=off: the quantizer is a fixed
// sequence of IEEE binary32 operations (subtract, divide, round-to-nearest-even,
// add, clamp) and must not be fused.
#include "mnnq_common.h"
#include "mnnq_fp6.h"

namespace mnnq {

namespace {

constexpr int kPackThreads = 256;
constexpr int kPackRows = 32;       // rows of a workgroup

enum PackForm { kPackZp = 0, kPackZpPlane = 1, kPackMin = 2, kPackBytes = 3, kPackNibbles = 4 };

// Four codes (0 .. MAX, one per byte) of the weights v of a group with the given scale: rint(x / scale) with IEEE
// operations, x = v (integer zero point, which is added to the rounded quotient) or v - mn (float minimum), clamped.
// The correctly rounded divisions are replaced as in quant4_fast: r = x * rcp(scale) differs from fl(x / scale) by less
// than |x / scale| * 2^-22 (one unit of the reciprocal, two roundings), i.e. 4e-6 for 4-bit and 6.1e-5 for 8-bit codes,
// so both round to the same integer unless r lies within that of a half-integer; only then - one value in 50000 (4 bits)
// or 5000 (8 bits) - the divisions are done.  The integer is the low part of r + 1.5 * 2^23.  (A scale near the ends of
// the exponent range, where the reciprocal is no normal number, always divides.)
template <int FORM>
__device__ __forceinline__ uint32_t quant_group(const float4 v, float scale, float mn, int& zero)
{
    constexpr bool ZP = FORM == kPackZp || FORM == kPackZpPlane;
    constexpr int MAX = FORM >= kPackBytes ? 255 : 15;
    constexpr float LIM = 0.5f - (FORM >= kPackBytes ? 1.0e-4f : 1.0e-5f), MAGIC = 12582912.0f;
    const float inv = __builtin_amdgcn_rcpf(scale);
    const float lim = (scale > 1.0e-30f && scale < 1.0e30f) ? LIM : -1.0f;
    const float x[4] = {ZP ? v.x : v.x - mn, ZP ? v.y : v.y - mn, ZP ? v.z : v.z - mn, ZP ? v.w : v.w - mn};
    float m[4], dmax = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float r = x[i] * inv;
        m[i] = r + MAGIC;
        dmax = fmaxf(dmax, fabsf(r - (m[i] - MAGIC)));
    }
    float mz = MAGIC;
    if (ZP) {
        const float r = -mn * inv;
        mz = r + MAGIC;
        dmax = fmaxf(dmax, fabsf(r - (mz - MAGIC)));
    }
    float base = MAGIC - (mz - MAGIC);     // the sum that stands for code 0: MAGIC less the zero point
    zero = ZP ? __float_as_int(mz) - __float_as_int(MAGIC) : 0;
    // (fmaxf drops a NaN: the limit is negative where the reciprocal gives one; of a NaN weight see below)
    if (!(dmax <= lim)) {
        // the definition itself, its clamp included: a range that rounds to scale 0 or overflows gives quotients and zero
        // points that no integer holds (NaN: code 0, as below; a zero point past the byte: 255)
        const float zf = ZP ? rintf(-mn / scale) : 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = fminf(fmaxf(rintf(x[i] / scale) + zf, 0.0f), (float)MAX) + MAGIC;
        zero = (int)fminf(fmaxf(zf, 0.0f), 255.0f);
        base = MAGIC;
    }
    // clamped as floats, in one instruction: the median, with a NaN the smallest of the other two, i.e. code 0 (minimum and
    // maximum instead: 37888 x 3584 with the plane 138.3 -> 139.7 us)
    uint32_t c[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        c[i] = (uint32_t)(__float_as_int(__builtin_amdgcn_fmed3f(m[i], base, base + (float)MAX)) - __float_as_int(base));
    return c[0] | (c[1] << 8) | (c[2] << 16) | (c[3] << 24);
}

// (the weights pass once: they need not stay in the caches)
__device__ __forceinline__ float4 load_once(const float* p)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

// A workgroup takes 32 rows (two row tiles, one column tile of the matrix-core plane) and CH consecutive chunks of 128
// weights (four; two where that leaves CUs without a workgroup).  A wave reads a kilobyte of one row per load - sixteen lanes, one float4 each, are a group -
// and issues all its loads before it uses the first.  Minimum and maximum of a group are DPP exchanges in its row of
// sixteen lanes.  The codes are put together in LDS in the layout's lane order and leave as whole consecutive kilobytes
// (Section 5.1: consecutive lanes on consecutive addresses), and with the plane flag the operand blocks of the matrix
// instructions are built from the same image: the weights are read once, the plane is not built from a second pass over
// the chunk layout.  Loads and stores are marked as passing once, which is worth 15 % (37888 x 3584,
// int4: 125 -> 107 - 115 us).  Bound by HBM: 37888 x 3584 with the plane, 543 MB in and 189 MB out, 187 us as two kernels
// with one group per team of lanes -> 137 us = 5.35 TB/s (a large copy: 4.85); int8 bytes 210 -> 122 us.
template <int FORM, int CH>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const float* __restrict__ W, Layout L,
                                                            uint8_t* __restrict__ packed, int chunk_blocks)
{
    constexpr bool ZP = FORM == kPackZp || FORM == kPackZpPlane, MINF = !ZP, BYTES = FORM == kPackBytes;
    // chunk images: [plane of codes][row tile][chunk] of four k-blocks (eight in the byte form: two halves), 16 rows of
    // 16 bytes each, padded by 16 bytes so that a wave's writes fall into different banks
    constexpr int IMAGES = FORM == kPackNibbles ? 2 : 1, KBS = BYTES ? 8 : 4, KB_DW = 68;
    __shared__ __align__(16) uint32_t img[IMAGES * 2 * CH * KBS * KB_DW];
    __shared__ float sc_s[2 * CH * 32], mn_s[2 * CH * 32];
    __shared__ uint8_t z_s[2 * CH * 32];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t tn = blockIdx.x / chunk_blocks;
    const int c0 = (int)(blockIdx.x % chunk_blocks) * CH;     // first chunk of the activation row
    const int G = (int)L.Gx;

    constexpr int RPW = kPackRows / 4;       // rows of a wave
    float4 w[RPW][CH / 2];
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int64_t n = tn * kPackRows + wave * RPW + j;
#pragma unroll
        for (int h = 0; h < CH / 2; ++h) {
            const int g = c0 * 2 + h * 4 + (lane >> 4);
            w[j][h] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (n < L.N && g < G) w[j][h] = load_once(W + n * L.Kx + g * kGroup + li * 4);
        }
    }
#pragma unroll
    for (int j = 0; j < RPW; ++j) {
        const int rr = wave * RPW + j, rt = rr >> 4, r = rr & 15;
        const bool row_ok = tn * kPackRows + rr < L.N;
#pragma unroll
        for (int h = 0; h < CH / 2; ++h) {
            const float4 v = w[j][h];
            const int cl = h * 2 + (lane >> 5), half = (lane >> 4) & 1;
            const bool ok = row_ok && c0 * 2 + h * 4 + (lane >> 4) < G;
            float mn = fminf(fminf(v.x, v.y), fminf(v.z, v.w)), mx = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
#define MNNQ_STEP(CTRL)                                                                        \
    mn = fminf(mn, __int_as_float(row_exchange<CTRL>(__float_as_int(mn))));                    \
    mx = fmaxf(mx, __int_as_float(row_exchange<CTRL>(__float_as_int(mx))));
            MNNQ_STEP(0xB1) MNNQ_STEP(0x4E) MNNQ_STEP(0x141) MNNQ_STEP(0x140)
#undef MNNQ_STEP
            if (ZP) {
                // Integer zero point: a group that does not straddle zero gets its range widened to contain it.
                mn = fminf(mn, 0.0f);
                mx = fmaxf(mx, 0.0f);
            }
            // (a constant group: scale 1, codes 0; outside the matrix, and the half that pads an odd row: all zero)
            float scale = 1.0f;
            int zero = 0;
            uint32_t codes = 0;
            if (mx != mn) {
                scale = (mx - mn) / (FORM >= kPackBytes ? 255.0f : 15.0f);
                codes = quant_group<FORM>(v, scale, mn, zero);
            }
            if (!ok) scale = mn = 0.0f;

            const int kb = li >> 2, image = rt * CH + cl;
            if (BYTES) {
                img[((image * 2 + half) * 4 + kb) * KB_DW + r * 4 + (li & 3)] = ok ? codes ^ 0x80808080u : 0u;
            } else {
                // Lane li holds codes j = 4 (li % 4) .. +3 of the k-block.  Codes j % 8 < 4 go to low nibbles, the others
                // to high nibbles of the same bytes.
#pragma unroll
                for (int p = 0; p < IMAGES; ++p) {
                    uint32_t x = FORM != kPackNibbles ? codes : p == 0 ? (codes >> 4) & 0x0f0f0f0fu : codes & 0x0f0f0f0fu;
                    if (li & 1) x <<= 4;
                    x |= (uint32_t)row_exchange<0xB1>((int)x);
                    if ((li & 1) == 0)
                        img[((p * 2 * CH + image) * 4 + kb) * KB_DW + r * 4 + half * 2 + ((li & 3) >> 1)] = x;
                }
            }
            if (li == 0) {
                sc_s[image * 32 + r * 2 + half] = scale;
                if (MINF) mn_s[image * 32 + r * 2 + half] = mn;
                else z_s[image * 32 + r * 2 + half] = (uint8_t)zero;
            }
        }
    }
    __syncthreads();

    // Chunk layout: the images of a row tile are consecutive in all three arrays.
    const int Cx = (int)L.Cx;
    const int live = Cx - c0 < CH ? Cx - c0 : CH;
#pragma unroll
    for (int p = 0; p < IMAGES; ++p) {
        constexpr int UNITS = BYTES ? 128 : 64;       // 16-byte units of a chunk
#pragma unroll
        for (int u0 = 0; u0 < 2 * CH * UNITS; u0 += kPackThreads) {
            const int u = u0 + tid, image = u / UNITS, v = u % UNITS, rt = image / CH, cl = image % CH;
            const int64_t t = tn * 2 + rt;
            if (t < L.T && cl < live)
                store_once(packed + ((t * L.C + p * Cx + c0 + cl) * UNITS + v) * 16,
                           *reinterpret_cast<const v4u*>(img + ((p * 2 * CH + image) * KBS + v / 16) * KB_DW + (v % 16) * 4));
        }
        const int image = tid / 32, rt = image / CH, cl = image % CH;
        const int64_t t = tn * 2 + rt, at = (t * L.C + p * Cx + c0 + cl) * 32 + tid % 32;
        if (tid < 2 * CH * 32 && t < L.T && cl < live) {
            const float s = sc_s[tid];
            // int8 weights as nibbles: high nibbles with step 16 s and the minimum, low nibbles with step s and minimum 0
            reinterpret_cast<float*>(packed + L.scales_off())[at] = FORM == kPackNibbles && p == 0 ? 16.0f * s : s;
            if (MINF) reinterpret_cast<float*>(packed + L.zeros_off())[at] = p == 0 ? mn_s[tid] : 0.0f;
            else (packed + L.zeros_off())[at] = z_s[tid];
        }
    }

    if (FORM == kPackZpPlane) {
        // The plane's blocks of these 32 columns: eight groups of 64 lanes.
        uint8_t* plane = packed + L.plane_off();
#pragma unroll
        for (int k = 0; k < CH / 2; ++k) {
            const int u = k * kPackThreads + tid, gl = u / 64, ln = u % 64, cl = gl >> 1, half = gl & 1;
            const int col = ln & 31, image = (col >> 4) * CH + cl, r = col & 15;
            const int64_t g = c0 * 2 + gl;
            if (g < G) {
                const uint32_t bias4 = 0x80808080u - z_s[image * 32 + r * 2 + half] * 0x01010101u;   // 0x80 - zero per byte
                uint32_t c[8], d[6];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint2 x = *reinterpret_cast<const uint2*>(img + (image * 4 + 2 * (ln >> 5) + q) * KB_DW + r * 4 + half * 2);
                    c[q * 4 + 0] = signmag_from_biased((x.x & 0x0f0f0f0fu) + bias4);
                    c[q * 4 + 1] = signmag_from_biased(((x.x >> 4) & 0x0f0f0f0fu) + bias4);
                    c[q * 4 + 2] = signmag_from_biased((x.y & 0x0f0f0f0fu) + bias4);
                    c[q * 4 + 3] = signmag_from_biased(((x.y >> 4) & 0x0f0f0f0fu) + bias4);
                }
                pack_fp6(c, d);
                const int64_t blk = g * L.T32p + tn;
                store_block(plane + blk * kPlaneBlockBytes, ln, d);
                if (ln < 32)
                    *reinterpret_cast<float*>(plane + L.plane_codes_bytes() + blk * 128 + ln * 4) = sc_s[image * 32 + r * 2 + half];
            }
        }
        // (the few bytes between the chunk layout and the plane's 256-byte boundary: zero, so that equal weights give
        // equal buffers)
        if (blockIdx.x == 0)
            for (size_t i = L.total() + tid; i < L.plane_off(); i += kPackThreads) packed[i] = 0;
    }
}

// Byte form of int8 weights (Layout::native8): the 16 bytes of row n, group g, k-block kb.
__device__ __forceinline__ size_t native8_codes_off(const Layout& L, int64_t n, int64_t g, int kb)
{
    const int64_t chunk = (n / kTileN) * L.C + g / 2;
    return (size_t)chunk * (2 * kChunkBytes) + (size_t)(g & 1) * kChunkBytes + (16 * kb + (int)(n % kTileN)) * 16;
}

// Index of the per-group parameters (scale, zero / minimum) of group g, row n.
__device__ __forceinline__ int64_t param_index(const Layout& L, int64_t n, int64_t g)
{
    return (((n / kTileN) * L.C + g / 2) * 16 + n % kTileN) * 2 + (g & 1);
}

// 16 codes (one per byte) of k-block kb of group g of the packed axis, row n.
__device__ __forceinline__ uint4 read_codes(const uint8_t* __restrict__ packed, const Layout& L, int64_t n, int64_t g,
                                            int kb)
{
    const int64_t chunk = (n / kTileN) * L.C + g / 2;
    const int r = (int)(n % kTileN);
    const uint2 w = *reinterpret_cast<const uint2*>(packed + chunk * kChunkBytes + (16 * kb + r) * 16 + (g & 1) * 8);
    uint4 o;
    o.x = w.x & 0x0f0f0f0fu;
    o.y = (w.x >> 4) & 0x0f0f0f0fu;
    o.z = w.y & 0x0f0f0f0fu;
    o.w = (w.y >> 4) & 0x0f0f0f0fu;
    return o;
}


__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t* __restrict__ packed, Layout L,
                                                     uint8_t* __restrict__ q, float* __restrict__ scale,
                                                     void* __restrict__ zero)
{
    // One thread per (row, group of the weight matrix, k-block): 16 codes.
    const int64_t G = L.Kx / kGroup;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= L.N * G * 4) return;
    const int kb = (int)(idx % 4);
    const int64_t g = (idx / 4) % G;
    const int64_t n = idx / (4 * G);
    if (L.native8) {   // byte form: q8 - 128 as stored, step and minimum of the group itself
        if (q) {
            uint4 o = *reinterpret_cast<const uint4*>(packed + native8_codes_off(L, n, g, kb));
            o.x ^= 0x80808080u; o.y ^= 0x80808080u; o.z ^= 0x80808080u; o.w ^= 0x80808080u;
            *reinterpret_cast<uint4*>(q + n * L.Kx + g * kGroup + 16 * kb) = o;
        }
        if (kb == 0) {
            if (scale) scale[n * G + g] = reinterpret_cast<const float*>(packed + L.scales_off())[param_index(L, n, g)];
            if (zero) static_cast<float*>(zero)[n * G + g] =
                          reinterpret_cast<const float*>(packed + L.zeros_off())[param_index(L, n, g)];
        }
        return;
    }
    const bool w8 = (L.mode == MNNQ_W8_MIN_FLOAT);   // high nibbles in group g, low nibbles in group G + g
    if (q) {
        uint4 o = read_codes(packed, L, n, g, kb);
        if (w8) {
            const uint4 lo = read_codes(packed, L, n, G + g, kb);
            o.x = (o.x << 4) | lo.x; o.y = (o.y << 4) | lo.y; o.z = (o.z << 4) | lo.z; o.w = (o.w << 4) | lo.w;
        }
        *reinterpret_cast<uint4*>(q + n * L.Kx + g * kGroup + 16 * kb) = o;
    }
    if (kb == 0) {
        const float* sc = reinterpret_cast<const float*>(packed + L.scales_off());
        // int8: the low plane carries the step itself, the high plane the minimum
        if (scale) scale[n * G + g] = sc[param_index(L, n, w8 ? G + g : g)];
        if (zero) {
            if (L.minf)
                static_cast<float*>(zero)[n * G + g] =
                    reinterpret_cast<const float*>(packed + L.zeros_off())[param_index(L, n, g)];
            else
                static_cast<uint8_t*>(zero)[n * G + g] = (packed + L.zeros_off())[param_index(L, n, g)];
        }
    }
}

// Writes 16 codes (one per byte, 0..15) of k-block kb of group g of the packed axis and,
// from the thread with kb == 0, the group's parameters.
__device__ __forceinline__ void write_codes(uint8_t* __restrict__ packed, const Layout& L, int64_t n, int64_t g,
                                            int kb, uint4 o, float scale, float mn, uint8_t z)
{
    const int64_t chunk = (n / kTileN) * L.C + g / 2;
    const int r = (int)(n % kTileN);
    const int half = (int)(g & 1);
    uint2 w;
    w.x = (o.x & 0x0f0f0f0fu) | ((o.y & 0x0f0f0f0fu) << 4);
    w.y = (o.z & 0x0f0f0f0fu) | ((o.w & 0x0f0f0f0fu) << 4);
    uint2* slot = reinterpret_cast<uint2*>(packed + chunk * kChunkBytes + (16 * kb + r) * 16);
    slot[half] = w;
    float* sc = reinterpret_cast<float*>(packed + L.scales_off()) + (chunk * 16 + r) * 2;
    uint8_t* zp = packed + L.zeros_off() + (chunk * 16 + r) * 2;
    float* mp = reinterpret_cast<float*>(packed + L.zeros_off()) + (chunk * 16 + r) * 2;
    if (kb == 0) {
        sc[half] = scale;
        if (L.minf) mp[half] = mn;
        else zp[half] = z > 15 ? (uint8_t)15 : z;
    }
    if ((L.G & 1) && g == L.G - 1) {   // padding group of an odd G
        slot[1] = make_uint2(0u, 0u);
        if (kb == 0) {
            sc[1] = 0.0f;
            if (L.minf) mp[1] = 0.0f;
            else zp[1] = 0;
        }
    }
}

// Import of weights that are already quantized (Section 4.2: quantized weights,
// e.g. from GPTQ, can be imported): canonical arrays -> chunk layout, the exact
// inverse of unpack_kernel.  One thread per (row, group, k-block).  int4 codes are
// taken modulo 16, zero points above 15 are stored as 15.
__global__ __launch_bounds__(256) void repack_kernel(const uint8_t* __restrict__ q, const float* __restrict__ scale,
                                                     const void* __restrict__ zero, Layout L,
                                                     uint8_t* __restrict__ packed)
{
    const int64_t G = L.Kx / kGroup;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= L.N * G * 4) return;
    const int kb = (int)(idx % 4);
    const int64_t g = (idx / 4) % G;
    const int64_t n = idx / (4 * G);
    const uint4 o = *reinterpret_cast<const uint4*>(q + n * L.Kx + g * kGroup + 16 * kb);
    const float s = scale[n * G + g];
    if (L.native8) {
        uint4 v = o;
        v.x ^= 0x80808080u; v.y ^= 0x80808080u; v.z ^= 0x80808080u; v.w ^= 0x80808080u;
        *reinterpret_cast<uint4*>(packed + native8_codes_off(L, n, g, kb)) = v;
        if (kb == 0) {
            reinterpret_cast<float*>(packed + L.scales_off())[param_index(L, n, g)] = s;
            reinterpret_cast<float*>(packed + L.zeros_off())[param_index(L, n, g)] = static_cast<const float*>(zero)[n * G + g];
        }
    } else if (L.mode == MNNQ_W8_MIN_FLOAT) {
        const float mn = static_cast<const float*>(zero)[n * G + g];
        uint4 hi;
        hi.x = o.x >> 4; hi.y = o.y >> 4; hi.z = o.z >> 4; hi.w = o.w >> 4;
        write_codes(packed, L, n, g, kb, hi, 16.0f * s, mn, 0);
        write_codes(packed, L, n, G + g, kb, o, s, 0.0f, 0);
    } else if (L.minf) {
        write_codes(packed, L, n, g, kb, o, s, static_cast<const float*>(zero)[n * G + g], 0);
    } else {
        write_codes(packed, L, n, g, kb, o, s, 0.0f, static_cast<const uint8_t*>(zero)[n * G + g]);
    }
}

}  // namespace

int launch_repack(const uint8_t* q, const float* scale, const void* zero, const Layout& L, uint8_t* packed,
                  hipStream_t st)
{
    const int64_t total = L.N * (L.Kx / kGroup) * 4;
    const int64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL(repack_kernel, dim3((unsigned)blocks), dim3(256), 0, st, q, scale, zero, L, packed);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

template <int FORM>
static int launch_pack_form(const float* W, const Layout& L, uint8_t* packed, hipStream_t st)
{
    const int64_t row_blocks = L.plane ? L.T32p : (L.T + 1) / 2;     // (the plane's padding tiles are written as zeros)
    auto go = [&](auto kern, int ch) -> int {
        const int chunk_blocks = (int)((L.Cx + ch - 1) / ch);
        hipLaunchKernelGGL(kern, dim3((unsigned)(row_blocks * chunk_blocks)), dim3(kPackThreads), 0, st, W, L, packed,
                           chunk_blocks);
        MNNQ_HIP_TRY(hipGetLastError());
        return MNNQ_OK;
    };
    if (row_blocks * ((L.Cx + 3) / 4) < 8 * (int64_t)num_cus()) return go(pack_kernel<FORM, 2>, 2);
    return go(pack_kernel<FORM, 4>, 4);
}

int launch_pack(const float* W, const Layout& L, uint8_t* packed, hipStream_t st)
{
    if (L.native8) return launch_pack_form<kPackBytes>(W, L, packed, st);
    if (L.mode == MNNQ_W8_MIN_FLOAT) return launch_pack_form<kPackNibbles>(W, L, packed, st);
    if (L.minf) return launch_pack_form<kPackMin>(W, L, packed, st);
    return L.plane ? launch_pack_form<kPackZpPlane>(W, L, packed, st) : launch_pack_form<kPackZp>(W, L, packed, st);
}

int launch_unpack(const uint8_t* packed, const Layout& L, uint8_t* q, float* scale, void* zero,
                  hipStream_t st)
{
    const int64_t total = L.N * (L.Kx / kGroup) * 4;
    const int64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)blocks), dim3(256), 0, st, packed, L, q, scale, zero);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

}  // namespace mnnq
