// Run-time activation quantizer (Section 4.2: activations are quantized to int8
// during calculation): per token, symmetric, scale = max|x| / 127.
//
// Compiled with -ffp-contract=off.  The codes are those of the fixed sequence of
// IEEE binary32 operations divide, round-to-nearest-even, clamp; they are computed
// with a multiply by fl(1 / scale) and the division only next to a tie, which gives
// the same integers (quant4_fast) at a fraction of the vector instructions.
#include "mnnq_common.h"
#include "mnnq_fp6.h"

namespace mnnq {

namespace {

constexpr int kQThreads = 256;

__global__ __launch_bounds__(kQThreads) void quant_act_kernel(const float* __restrict__ x, int64_t K,
                                                              int8_t* __restrict__ xq,
                                                              float* __restrict__ sx,
                                                              int32_t* __restrict__ xsum)
{
    __shared__ float s_part[kQThreads / 64];
    const int64_t m = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t K4 = K / 4;  // a multiple of 16: teams of 16 lanes cover whole groups
    const float4* xr = reinterpret_cast<const float4*>(x + m * K);
    // With few rows (decode) a row is split over gridDim.y workgroups: each finds the
    // row maximum itself and quantizes its own slice of the row.
    const int64_t per = (K4 + gridDim.y - 1) / gridDim.y;
    const int64_t per16 = (per + 15) / 16 * 16;          // slices hold whole groups
    const int64_t i0 = per16 * blockIdx.y;
    const int64_t i1 = (i0 + per16 < K4) ? i0 + per16 : K4;

    float amax = 0.0f;
    for (int64_t i = tid; i < K4; i += kQThreads) {
        const float4 v = xr[i];
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
    amax = wave_max_nonneg(amax);
    if ((tid & 63) == 0) s_part[tid >> 6] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(s_part[0], s_part[1]), fmaxf(s_part[2], s_part[3]));

    const bool zero_row = (amax == 0.0f);
    const float scale = zero_row ? 0.0f : amax / 127.0f;
    if (tid == 0 && blockIdx.y == 0) sx[m] = scale;

    uint32_t* out = reinterpret_cast<uint32_t*>(xq + m * K);
    const int64_t G = K / kGroup;
    const float inv = zero_row ? 0.0f : 1.0f / scale;
    const float lim = quant_fast_limit(scale, inv);
    for (int64_t i = i0 + tid; i < i1; i += kQThreads) {
        int codes = 0;
        if (!zero_row) codes = quant4_fast(xr[i], scale, inv, lim);
        out[i] = (uint32_t)codes;
        if (xsum) {
            const int s = row_sum16(__builtin_amdgcn_sdot4(codes, 0x01010101, 0, false));
            if ((tid & 15) == 0) xsum[m * G + i / 16] = s;
        }
    }
}

// Many rows (prefill): the row is held in registers between the maximum and the
// quantization, so it crosses the memory system once and all of a thread's loads
// are in flight together.  NV float4 per thread; K <= NV * 4 * kQThreads.
template <int NV>
__global__ __launch_bounds__(kQThreads) void quant_act_rows_kernel(const float* __restrict__ x, int64_t K,
                                                                   int8_t* __restrict__ xq,
                                                                   float* __restrict__ sx,
                                                                   int32_t* __restrict__ xsum)
{
    __shared__ float s_part[kQThreads / 64];
    const int64_t m = blockIdx.x;
    const int tid = threadIdx.x;
    const int K4 = (int)(K / 4);
    const float4* xr = reinterpret_cast<const float4*>(x + m * K);

    float4 v[NV];
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = tid + j * kQThreads;
        v[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (i < K4) v[j] = xr[i];
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[j].x), fabsf(v[j].y)), fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
    }
    amax = wave_max_nonneg(amax);
    if ((tid & 63) == 0) s_part[tid >> 6] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(s_part[0], s_part[1]), fmaxf(s_part[2], s_part[3]));

    const bool zero_row = (amax == 0.0f);
    const float scale = zero_row ? 0.0f : amax / 127.0f;
    if (tid == 0) sx[m] = scale;

    uint32_t* out = reinterpret_cast<uint32_t*>(xq + m * K);
    const int64_t G = K / kGroup;
    const float inv = zero_row ? 0.0f : 1.0f / scale;
    const float lim = quant_fast_limit(scale, inv);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = tid + j * kQThreads;
        int codes = 0;
        if (!zero_row) codes = quant4_fast(v[j], scale, inv, lim);
        if (i < K4) out[i] = (uint32_t)codes;
        if (xsum) {
            // K4 is a multiple of 16, so a team of 16 lanes is inside the row or outside it as a whole
            const int s = row_sum16(__builtin_amdgcn_sdot4(codes, 0x01010101, 0, false));
            if ((tid & 15) == 0 && i < K4) xsum[m * G + i / 16] = s;
        }
    }
}

// The fused prefill call: the quantizer writes the codes in the order in which the contraction kernel behind it reads
// them, so that no pass over the codes rearranges them (Section 5.1) and the kernel's loads are whole lines.
//   kTokenBlocks - the few-token kernels: [group][token block of 16][k block of 16][token][16 codes], the last block as
//                  narrow as its tokens (M K bytes in all);
//   kPlanes      - the fp6 GEMM: the activation planes [group][TMp][3072 B] (see planes_kernel).
// A workgroup of 512 threads quantizes R rows, each in the registers of 512 / R threads (NV float4 per thread) between
// the maximum and the codes, collects the codes in LDS and stores them from there: R tokens lie side by side in the
// output, i.e. pieces of 16 R bytes.
//
// Bound: latency for few rows (load, maximum, codes, store in a row), HBM for many.  A line of the output holds the
// pieces of eight tokens, so eight rows in a row go to workgroups of one XCD (workgroup b runs on XCD b % 8), whose L2
// puts the line together; spread over the XCDs every line left the chip in pieces, and small workgroups - several per CU,
// one storing while another loads - did not pay.  Planes, one row per workgroup: 1024 x 18944 38.6 -> 26.6 us; against
// 1024 threads with one, two or four rows and no such order: 5 x 4096 (token blocks) 3.0 -> 2.2 us, 512 x 3584 7.9 -> 6.8,
// 512 x 18944 14.5 -> 13.7, 2048 x 18944 48.3 -> 44.8 us (4.7 TB/s; a large copy reaches 5.0 TB/s).
// Vector issue is the next share: codes and tie check by fused multiply-adds and the packing by dot products took an
// activation of the planes from about 16 instructions to 9.5; a pass over the four layers of a block, 512 tokens of width
// 1536 and 1024 of 3584, 93.4 -> 92.2 and 407.8 -> 404.9 us.
enum ActOrder { kTokenBlocks = 0, kPlanes = 1 };
constexpr int kPackThreads = 512;
constexpr int kPackMaxVec = 10 * kPackThreads;   // float4 of the longest row: ten registers quads per thread with R = 1
constexpr int kLineRows = 8;                     // tokens that share a 128-byte line of the output
constexpr int kXcds = 8;

template <int R, int NV, int ORDER>
__global__ __launch_bounds__(kPackThreads) void quant_pack_kernel(const float* __restrict__ x, int M, int K, int TMp,
                                                                  int rows, uint8_t* __restrict__ out,
                                                                  float* __restrict__ sx)
{
    extern __shared__ __align__(16) uint8_t lds_codes[];   // [R][K + 16]: rows 16 bytes apart in the banks; maxima
    constexpr int TPR = kPackThreads / R, WPR = TPR / 64;
    const int tid = threadIdx.x;
    const int r = __builtin_amdgcn_readfirstlane(tid / TPR), i0 = tid % TPR;
    // (the grid covers whole sets of kXcds * kLineRows rows)
    constexpr int per_line = kLineRows / R;
    const int set = blockIdx.x / kXcds, xcd = blockIdx.x % kXcds;
    const int first = (set / per_line * kXcds + xcd) * kLineRows + set % per_line * R;
    if (first >= rows) return;
    const int m = first + r;
    const int K4 = K / 4, stride = K + 16;
    float* const s_part = reinterpret_cast<float*>(lds_codes + R * stride);
    const float4* xr = reinterpret_cast<const float4*>(x + (int64_t)m * K);

    float4 v[NV];
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = i0 + j * TPR;
        v[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (i < K4 && m < M) v[j] = xr[i];
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[j].x), fabsf(v[j].y)), fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
    amax = wave_max_nonneg(amax);
    if ((tid & 63) == 0) s_part[tid >> 6] = amax;
    __syncthreads();
    amax = s_part[r * WPR];
#pragma unroll
    for (int w = 1; w < WPR; ++w) amax = fmaxf(amax, s_part[r * WPR + w]);

    const bool zero_row = (amax == 0.0f);
    const float scale = zero_row ? 0.0f : amax / 127.0f;
    if (i0 == 0 && m < M) sx[m] = scale;
    const float inv = zero_row ? 0.0f : 1.0f / scale;
    const float lim = quant_fast_limit(scale, inv);
    int* codes = reinterpret_cast<int*>(lds_codes + r * stride);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = i0 + j * TPR;
        int c = 0;
        if (!zero_row) c = quant4_fast(v[j], scale, inv, lim);
        if (i < K4) codes[i] = c;
    }
    __syncthreads();

    if (ORDER == kTokenBlocks) {
        const int units = R * (K / 16);      // 16 codes of one token
        for (int u = tid; u < units; u += kPackThreads) {
            const int rr = u % R, kk = u / R, mm = first + rr;
            const int tb = mm >> 4, left = M - tb * 16, width = left < 16 ? left : 16;
            const uint4 c = *reinterpret_cast<const uint4*>(lds_codes + rr * stride + kk * 16);
            if (mm < M)
                *reinterpret_cast<uint4*>(out + ((int64_t)(kk >> 2) * M * 4 + tb * 64 + (kk & 3) * width + (mm & 15)) * 16) = c;
        }
    } else {
        const int units = R * (K / 32);      // 32 codes of one token: a lane of two blocks
        for (int u = tid; u < units; u += kPackThreads) {
            const int rr = u % R, kk = u / R, mm = first + rr;
            const uint4* p = reinterpret_cast<const uint4*>(lds_codes + rr * stride + kk * 32);
            const uint4 a = p[0], b = p[1];
            const uint32_t q[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            uint32_t hi[8], lo[8], dh[6], dl[6];
#pragma unroll
            for (int i = 0; i < 8; ++i) split_act(q[i], hi[i], lo[i]);
            pack_fp6(hi, dh);
            pack_fp6(lo, dl);
            uint8_t* pair = out + ((int64_t)(kk >> 1) * TMp + (mm >> 5)) * (2 * kPlaneBlockBytes);
            store_pair(pair, (mm & 31) + 32 * (kk & 1), dh, dl);
        }
    }
}

template <int R, int ORDER>
int launch_quant_pack(const float* x, int64_t M, int64_t K, int TMp, int64_t rows, uint8_t* out, float* sx, hipStream_t st)
{
    const int nv = (int)((K / 4 + kPackThreads / R - 1) / (kPackThreads / R));
    const size_t smem = (size_t)R * (K + 16) + kPackThreads / 64 * sizeof(float);
    constexpr int set_rows = kXcds * kLineRows;
    const unsigned grid = (unsigned)((rows + set_rows - 1) / set_rows * (set_rows / R));
#define MNNQ_PACK(NV)                                                                                             \
    if (nv <= NV) {                                                                                               \
        static thread_local int allowed = -1;                                                                     \
        auto kern = quant_pack_kernel<R, NV, ORDER>;                                                              \
        if (int s = allow_large_lds(kern, smem, allowed)) return s;                                               \
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kPackThreads), smem, st, x, (int)M, (int)K, TMp, (int)rows, out, sx); \
        MNNQ_HIP_TRY(hipGetLastError());                                                                          \
        return MNNQ_OK;                                                                                           \
    }
    MNNQ_PACK(R) MNNQ_PACK(2 * R) MNNQ_PACK(4 * R) MNNQ_PACK(5 * R) MNNQ_PACK(7 * R) MNNQ_PACK(10 * R)
#undef MNNQ_PACK
    return MNNQ_ERR_UNSUPPORTED;
}

}  // namespace

// The row stays in registers.
bool quant_packed_possible(int64_t K) { return K / 4 <= kPackMaxVec; }

// One row per workgroup fills more CUs, two rows make larger stores (measured, one / two rows: 256 x 3584 4.7 / 5.0 us,
// 256 x 18944 9.9 / 11.1, 352 x 3584 5.9 / 5.6, 1024 x 3584 8.4 / 8.0, 1024 x 18944 26.6 / 23.8 us).
constexpr int64_t kOneRowMax = 256;

int launch_quant_token_blocks(const float* x, int64_t M, int64_t K, int8_t* xq, float* sx, hipStream_t st)
{
    uint8_t* out = reinterpret_cast<uint8_t*>(xq);
    if (M <= kOneRowMax) return launch_quant_pack<1, kTokenBlocks>(x, M, K, 0, M, out, sx, st);
    return launch_quant_pack<2, kTokenBlocks>(x, M, K, 0, M, out, sx, st);
}

int launch_quant_planes(const float* x, int64_t M, int64_t K, int TMp, void* planes, float* sx, hipStream_t st)
{
    // (rows up to the next whole block of 32 are written as zeros; the blocks behind are not read for results)
    const int64_t rows = (M + 31) / 32 * 32;
    uint8_t* out = static_cast<uint8_t*>(planes);
    if (rows <= kOneRowMax) return launch_quant_pack<1, kPlanes>(x, M, K, TMp, rows, out, sx, st);
    return launch_quant_pack<2, kPlanes>(x, M, K, TMp, rows, out, sx, st);
}

int launch_quant_act(const float* x, int64_t M, int64_t K, int8_t* xq, float* sx, int32_t* xsum,
                     hipStream_t st)
{
    // Decode-sized calls are latency bound: spread a row over several workgroups.
    unsigned slices = 1;
    if (M <= 16) {
        slices = (unsigned)((K / 4 + kQThreads - 1) / kQThreads);
        if (slices > 32) slices = 32;
    }
    if (M > 16 && K <= 20 * 4 * kQThreads) {
        const int nv = (int)((K / 4 + kQThreads - 1) / kQThreads);
#define MNNQ_ROWS(NV)                                                                                          \
    if (nv <= NV) {                                                                                            \
        hipLaunchKernelGGL(quant_act_rows_kernel<NV>, dim3((unsigned)M), dim3(kQThreads), 0, st, x, K, xq, sx, \
                           xsum);                                                                              \
        MNNQ_HIP_TRY(hipGetLastError());                                                                       \
        return MNNQ_OK;                                                                                        \
    }
        MNNQ_ROWS(2) MNNQ_ROWS(4) MNNQ_ROWS(8) MNNQ_ROWS(12) MNNQ_ROWS(20)
#undef MNNQ_ROWS
    }
    hipLaunchKernelGGL(quant_act_kernel, dim3((unsigned)M, slices), dim3(kQThreads), 0, st, x, K, xq, sx, xsum);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

}  // namespace mnnq
