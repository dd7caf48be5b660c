// What the GEMMs on wide tiles (mnnq_prefill8w.hip, mnnq_prefill_f16w.hip) do behind their loops: WAVES waves share the tokens of a
// workgroup's tile and own 16 TN columns each, TM x TN tiles of 16 x 16 in acc[i * TN + j]; KS parts of K, one behind the other.
#pragma once

#include "mnnq_forms.h"

namespace mnnq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

// LDS of a K part's sums, and of the patches that the output passes through.
template <int WAVES, int TM, int TN, int KS>
struct WideOut {
    static constexpr int sum_bytes = KS > 1 ? WAVES * TM * TN * 4 * 64 * 4 : 0;
    static constexpr int patch_bytes = WAVES * 16 * (16 * TN + 4) * 4;      // (rows padded by four floats)
};

// A part > 0 leaves its sums in LDS (one conflict-free float per lane and accumulator), part 0 adds them, in order.  All waves call
// it; false: the wave belongs to another part and is done.  Ends with LDS free for the output.
template <int TM, int TN, int KS>
__device__ __forceinline__ bool sum_parts(uint8_t* lds, int wave, int part, int lane, v4f (&acc)[TM * TN])
{
    if (KS > 1) {
        float* red = reinterpret_cast<float*>(lds) + wave * (TM * TN * 4 * 64) + lane;
#pragma unroll
        for (int p = 1; p < KS; ++p) {
            __syncthreads();                         // the stages are dead, the previous part's sums are read
            if (part == p) {
#pragma unroll
                for (int t = 0; t < TM * TN; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) red[(t * 4 + r) * 64] = acc[t][r];
            }
            __syncthreads();
            if (part == 0) {
#pragma unroll
                for (int t = 0; t < TM * TN; ++t)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[t][r] += red[(t * 4 + r) * 64];
            }
        }
        __syncthreads();
        return part == 0;
    }
    __syncthreads();                                 // (a load past the end may still be writing to a stage)
    return true;
}

// y = acc * factor[m] + bias[n] (either NULL: 1, 0).  Rows past M fall outside the buffers (loads give 0, stores are dropped), a
// NULL bias is an empty buffer.  The 16 x 16 TN block of a row of tiles goes through a private LDS patch and leaves as
// 128-bit (binary16: 64-bit) stores of whole row segments; LDS operations of a wave complete in order.
// rt0: the wave's first row tile of the layout (16 columns).
template <int TM, int TN>
__device__ __forceinline__ void store_wide(uint8_t* lds, int wave, int lane, const Layout& L, int64_t M, int m0, int rt0,
                                           const float* factor, const float* bias, float* y, const v4f (&acc)[TM * TN])
{
    const int row = lane & 15, kb = lane >> 4;
    const __amdgpu_buffer_rsrc_t rs_f = rsrc(factor, factor ? M * 4 : 0);
    const __amdgpu_buffer_rsrc_t rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
    const int out_size = L.out16 ? 2 : 4, row_bytes = (int)L.N * out_size, y_bytes = (int)(uint32_t)(M * L.N * out_size);
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(y, (uint32_t)y_bytes);
    float bj[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bj[j] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, row * 4, (rt0 + j) * 64, 0));
    constexpr int RS = 16 * TN + 4;
    float* patch = reinterpret_cast<float*>(lds) + wave * (16 * RS);
    float* wr = patch + (kb * 4) * RS + row;
    // sixteen rows of 4 TN units of 16 bytes (four values), TN units per lane; units past N are sent out of range
    int rd[TN], y_voff[TN];
#pragma unroll
    for (int p = 0; p < TN; ++p) {
        const int u = p * 64 + lane, ur = u / (4 * TN), uc = u % (4 * TN);
        rd[p] = ur * RS + uc * 4;
        y_voff[p] = rt0 + (uc >> 2) < (int)L.T ? ur * row_bytes + uc * 4 * out_size : y_bytes;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float f[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f[r] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_f, kb * 16, (m0 + i * 16 + r) * 4, 0));
            if (!factor) f[r] = 1.0f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < TN; ++j) wr[r * RS + j * 16] = fmaf(acc[i * TN + j][r], f[r], bj[j]);
#pragma unroll
        for (int p = 0; p < TN; ++p) {
            const float4 v = *reinterpret_cast<const float4*>(patch + rd[p]);
            const int at = (m0 + i * 16) * row_bytes + rt0 * 16 * out_size;
            if (L.out16) {
                const v2i o = {__builtin_bit_cast(int, h2{(_Float16)v.x, (_Float16)v.y}), __builtin_bit_cast(int, h2{(_Float16)v.z, (_Float16)v.w})};
                __builtin_amdgcn_raw_buffer_store_b64(o, rs_y, y_voff[p], at, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), rs_y, y_voff[p], at, 0);
            }
        }
    }
}

}  // namespace

}  // namespace mnnq
