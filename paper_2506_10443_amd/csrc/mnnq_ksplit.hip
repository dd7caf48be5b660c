// Prefill GEMM on the int8 and fp16 matrix instructions with K split over the waves of a workgroup: for the weight forms
// without a matrix-core plane (int4 with a zero point or a float minimum, int8 bytes; int4 and nibble planes with fp16
// activations) wherever the tiled GEMMs of mnnq_prefill.hip and mnnq_prefill_f16.hip leave the chip partly idle.
//
// The tiled GEMM works on 128 x 128 outputs per workgroup: 333 tokens of a 4096-wide projection are 96 such tiles on 256
// CUs.  Here a wave owns 64 x 64 outputs (48, 32 or 16 x 64: tile_height) and a part of K, the KS waves of a workgroup share the tile and add their parts
// through LDS at the end, in a fixed order.  The waves share no operand, so everything goes from L2 straight into
// registers, refilled for the next chunk of 128 values as soon as it has been used, with no LDS and no barrier in the loop.
// What bounds it is vector issue: per group of a 16 x 16 tile two instructions per output for the scale (three with a
// float minimum) behind one matrix instruction - with fp16 activations one behind two, and twice the unpacking -;
// unpacking a column tile is shared by the row tiles.
//
// Operand layout and arithmetic as in mnnq_skinny.hip (A: 16 tokens x 64 k, B: 64 k x 16 weight rows, D: lane l holds
// weight row l % 16, tokens 4 (l / 16) + r).
#include "mnnq_forms.h"

namespace mnnq {

namespace {

constexpr int kOutOfRange = 0x7fff0000;   // a byte offset beyond every buffer (ksplit8_wanted): loads give 0, stores are dropped

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

constexpr int TN = 4;   // 16 x 16 tiles of a wave: 16 TM tokens x 64 weight rows

template <int FORM, int KS, int TM, bool BLOCKS>
__global__ __launch_bounds__(64 * KS, 2) void ksplit_kernel(const uint8_t* __restrict__ packed, Layout L, int M,
                                                          const void* __restrict__ xq,
                                                          const float* __restrict__ sx, const float* __restrict__ bias,
                                                          float* __restrict__ y, int MT, int NT)
{
    constexpr int T = TM * TN;
    // the minima's part on the matrix cores (Centered), or with the scale on the vector ALU: unpacking centred 4-bit codes costs
    // int8 activations more than it saves (1024 tokens of 3584 x 18944 170 / 167, 100 of 4096 x 14336 27.3 / 26.0 us)
    constexpr bool CENTER = FORM == kBytes || FORM == kMinF16, PAIRS = FORM == kMin;
    extern __shared__ __align__(16) float4 lds_sum[];   // [KS][T][64]
    const int lane = threadIdx.x & 63, row = lane & 15, kb = lane >> 4;
    const int ks = uniform(threadIdx.x >> 6);
    int tile_m, tile_n;
    if (!xcd_tile(MT, NT, tile_m, tile_n)) return;
    const int C = (int)L.C, m0 = tile_m * (16 * TM);
    const int c0 = C * ks / KS, c1 = C * (ks + 1) / KS;
    const int odd_last = (L.G & 1) ? C - 1 : -1;

    // activations: int8 or fp16 rows, or the token blocks of launch_quant_token_blocks; chunk c of the packed axis meets
    // chunk c % Cx of the row
    constexpr int E = is_f16(FORM) ? 2 : 1;
    const int Cx = (int)L.Cx;
    const __amdgpu_buffer_rsrc_t rs_x = rsrc(xq, (int64_t)M * L.Kx * E);
    const int x_step = BLOCKS ? M * 64 : 64 * E;        // bytes from group to group
    constexpr bool XCH = !BLOCKS && !is_f16(FORM);
    const RowExchange exchange(lane);
    int x_voff[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int first = m0 + i * 16, left = M - first, width = left < 16 ? left : 16;
        const int m = XCH ? lane >> 2 : row, k = XCH ? lane & 3 : kb;
        x_voff[i] = m < width ? (BLOCKS ? first * 64 + (k * width + m) * 16 : (first + m) * (int)L.Kx * E + k * 16 * E)
                              : kOutOfRange;
    }
    // weights: column tile j of this workgroup is row tile t0 + j of the layout (past the matrix: outside the buffers)
    constexpr int WB = FORM == kBytes ? 2048 : 1024, ZB = has_zero(FORM) ? 32 : 128;
    const int t0 = tile_n * TN;
    const int live = (int)L.T - t0 < TN ? (int)L.T - t0 : TN;
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(packed + (int64_t)t0 * C * WB, (int64_t)live * C * WB);
    const __amdgpu_buffer_rsrc_t rs_s = rsrc(packed + L.scales_off() + (int64_t)t0 * C * 128, (int64_t)live * C * 128);
    const __amdgpu_buffer_rsrc_t rs_z = rsrc(packed + L.zeros_off() + (int64_t)t0 * C * ZB, (int64_t)live * C * ZB);
    const uint32_t zsel = (row & 1) * 0x02020202u;

    v4i a[2][TM][E];
    // weights two chunks ahead (they come from HBM), activations one (from L2)
    Weights<FORM> w[2][TN];
    float mn[TN], mn_next[TN], xs[TM];      // operands of the minima's part (Centered), the next two chunks' on their way
    auto load_a = [&](int h, int i, int c) {
        const int cx = c >= Cx ? c - Cx : c;
        const int off = uniform(c < c1 && (h == 0 || c != odd_last) ? (2 * cx + h) * x_step : kOutOfRange);
#pragma unroll
        for (int e = 0; e < E; ++e) a[h][i][e] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, x_voff[i] + e * 16, off, 0);
    };
    auto load_codes = [&](int u, int j, int h, int c) {   // (the byte form: a kilobyte per group; else both groups with h = 0)
        const int off = uniform(c < c1 ? (j * C + c) * WB : kOutOfRange);
        w[u][j].w[FORM == kBytes ? h : 0] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, lane * 16 + h * 1024, off, 0);
    };
    auto load_params = [&](int u, int j, int c) {
        const int cell = uniform(j * C + c);
        const bool have = c < c1;
        w[u][j].s = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(rs_s, row * 8, uniform(have ? cell * 128 : kOutOfRange), 0));
        if (has_zero(FORM))
            w[u][j].z = __builtin_amdgcn_raw_buffer_load_b32(rs_z, (row >> 1) * 4, uniform(have ? cell * ZB : kOutOfRange), 0);
        if (PAIRS)
            w[u][j].mn = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(rs_z, row * 8, uniform(have ? cell * ZB : kOutOfRange), 0));
    };
    auto load_min = [&](int j, int c) {      // (chunks past the wave's: zeros)
        const int off = c + (kb >> 1) < c1 ? (kb >> 1) * ZB + row * 8 + (kb & 1) * 4 : kOutOfRange;
        mn_next[j] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_z, off, uniform((j * C + c) * ZB), 0));
    };
    // In the order of the loop's refills: the waits are counts.  (Not so with group minima: they are requested last here and first in
    // the loop, whose head waits for the smaller count, all but three loads, once per turn of two chunks.)
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (u == 1) {
#pragma unroll
                for (int i = 0; i < TM; ++i) load_a(h, i, c0);
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (FORM == kBytes || h == 1) load_codes(u, j, FORM == kBytes ? h : 0, c0 + u);
                if (h == 1) load_params(u, j, c0 + u);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    if (CENTER) {
#pragma unroll
        for (int j = 0; j < TN; ++j) load_min(j, c0);
    }

    v4f acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    const v4i magic = {kMagicBits, kMagicBits, kMagicBits, kMagicBits};
    const v4i zero4 = {0, 0, 0, 0};
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const v4i onesh = {0x3c003c00, 0x3c003c00, 0x3c003c00, 0x3c003c00};
    const v4f zerof = {0.0f, 0.0f, 0.0f, 0.0f};
    int c = c0;
    do {
      if (CENTER) {
#pragma unroll
          for (int i = 0; i < TM; ++i) xs[i] = 0.0f;
          // (copies: the loads' registers stay where they are)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
              asm volatile("v_mov_b32 %0, %1" : "=v"(mn[j]) : "v"(mn_next[j]));
              load_min(j, c + 2);
          }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (u == 1 && c + 1 >= c1) break;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            Operand<FORM> b[TN];
            float s[TN], pm[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                b[j] = unpack<FORM, CENTER>(w[u][j], h, zsel);
                if (PAIRS) pm[j] = h ? w[u][j].mn.y : w[u][j].mn.x;
                s[j] = h ? w[u][j].s.y : w[u][j].s.x;
            }
            if (h == 1) {      // the second group is unpacked: the chunk's registers take the next chunk
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    // (copies: the refilled registers stay where they are)
                    asm volatile("v_mov_b32 %0, %1" : "=v"(s[j]) : "v"(w[u][j].s.y));
                    if (PAIRS) asm volatile("v_mov_b32 %0, %1" : "=v"(pm[j]) : "v"(w[u][j].mn.y));
                    if (FORM != kBytes) load_codes(u, j, 0, c + u + 2);
                    load_params(u, j, c + u + 2);
                }
            }
            const Centered<FORM> center(2 * u + h, kb);
            v4i sum[2];
            float xf[2][4];
            if (XCH && h == 0) exchange(a[0][0][0]);
            v4i d[2];
#pragma unroll
            for (int t = 0; t <= T; ++t) {
                if (t < T) {
                    const int i = t / TN, j = t % TN;
                    constexpr int X = E - 1;
                    if (PAIRS && j == 0) {      // sums of the group's activations, tokens in the rows
                        const v4i x = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[h][i][0], ones, zero4, 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < 4; ++r) xf[i & 1][r] = (float)x[r];
                    }
                    if (CENTER && j == 0) {
                        // ... tokens in the lanes (all rows of the product are equal)
                        if (is_f16(FORM)) {
                            const v4f x = mfma_f16(onesh, a[h][i][X], mfma_f16(onesh, a[h][i][0], zerof));
                            xs[i] = kb == 2 * u + h ? x[0] : xs[i];
                        } else {
                            const v4i x = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, a[h][i][0], zero4, 0, 0, 0);
                            xs[i] = kb == 2 * u + h ? (float)x[0] : xs[i];
                        }
                    }
                    if (is_f16(FORM))
                        d[t & 1] = __builtin_bit_cast(v4i, mfma_f16(a[h][i][X], b[j].q[X], mfma_f16(a[h][i][0], b[j].q[0], zerof)));
                    else
                        d[t & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[h][i][0], b[j].q[0], magic, 0, 0, 0);
                    if constexpr (CENTER) {
                        if (i == 0) sum[j & 1] = Centered<FORM>::column_sum(b[j]);
                    }
                    if (!XCH && j == TN - 1) load_a(h, i, c + u + 1);
                    if (XCH && h == 1 && j == TN - 1) {      // (both groups of a line)
                        load_a(0, i, c + u + 1);
                        load_a(1, i, c + u + 1);
                    }
                    if (FORM == kBytes && i == TM - 1) load_codes(u, j, h, c + u + 2);
                    // the next operand, a row of tiles ahead
                    if (XCH && j == 0 && i + 1 < TM) exchange(a[h][(i + 1) % TM][0]);
                    if (XCH && j == 0 && i + 1 == TM && h == 0) exchange(a[1][0][0]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (t > 0) {
                    const int p = t - 1, i = p / TN, j = p % TN;
                    if constexpr (CENTER) {
                        if (p < TN) center(sum[j & 1], s[j], mn[j]);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float v = is_f16(FORM) ? __int_as_float(d[p & 1][r]) : from_magic(d[p & 1][r]);
                        acc[p][r] = fmaf(s[j], v, acc[p][r]);
                        if (PAIRS) acc[p][r] = fmaf(pm[j], xf[i & 1][r], acc[p][r]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
      }
      if (CENTER) {
#pragma unroll
          for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[t / TN], mn[t % TN], acc[t], 0, 0, 0);
      }
      c += 2;
    } while (c < c1);
    // Sum over the waves in a fixed order, the tiles dealt to the waves; their scales and biases are requested before the
    // exchange, which their latency would follow.
    constexpr int NP = (T + KS - 1) / KS;
    const __amdgpu_buffer_rsrc_t rs_sx = rsrc(sx, (int64_t)M * 4);
    const __amdgpu_buffer_rsrc_t rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(y, (int64_t)M * L.N * (L.out16 ? 2 : 4));
    float bn[NP], sm[NP][4];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int t = ks + k * KS, m = m0 + (t / TN) * 16 + 4 * kb, n = (t0 + t % TN) * 16 + row;
        bn[k] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, n * 4, 0, 0));
#pragma unroll
        for (int r = 0; r < 4; ++r) sm[k][r] = sx ? __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_sx, (m + r) * 4, 0, 0)) : 1.0f;
    }
    uint64_t bad = 0;      // (CENTER) lanes with a sum that is not finite
#pragma unroll
    for (int t = 0; t < T; ++t)
        lds_sum[(ks * T + t) * 64 + lane] = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int t = ks + k * KS;
        if (T % KS != 0 && t >= T) break;
        float4 v = lds_sum[t * 64 + lane];
#pragma unroll
        for (int p = 1; p < KS; ++p) {
            const float4 o = lds_sum[(p * T + t) * 64 + lane];
            v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
        }
        store_tile(rs_y, L, m0 + (t / TN) * 16 + 4 * kb, (t0 + t % TN) * 16 + row, v4f{v.x, v.y, v.z, v.w}, sm[k], bn[k]);
        if (CENTER) bad |= t % TN < live ? __ballot(v.x * 0.0f != 0.0f) : 0;
    }
    if constexpr (CENTER) {
        if (__builtin_expect(bad == 0, 1)) return;
        // Groups that centred sums cannot express: the wave's tiles again by the definition.  Behind everything else, with the
        // buffers described anew, so that neither registers nor instruction fetches of the usual way pay for it (inside the
        // loop over the tiles 0.7 us of 17).
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): the stores above are done
        const uint8_t* wp = packed;
        const void* xp = xq;
        int l = lane;
        asm volatile("" : "+s"(wp), "+s"(xp), "+v"(l));
        const int row = l & 15, kb = l >> 4;
        const __amdgpu_buffer_rsrc_t rx = rsrc(xp, (int64_t)M * L.Kx * E), rw = rsrc(wp, (int64_t)L.total());
#pragma unroll 1
        for (int t = ks; t < T; t += KS) {
            if (t % TN >= live) continue;
            const int first = m0 + (t / TN) * 16, left = M - first, width = left < 16 ? left : 16;
            const int voff = row < width ? (BLOCKS ? first * 64 + (kb * width + row) * 16 : (first + row) * (int)L.Kx * E + kb * 16 * E)
                                         : kOutOfRange;
            const auto operand_a = [&](int cc, int h) {
                const int off = uniform(h == 0 || cc != odd_last ? (2 * (cc >= Cx ? cc - Cx : cc) + h) * x_step : kOutOfRange);
                Operand<FORM> o;
#pragma unroll
                for (int e = 0; e < E; ++e) o.q[e] = __builtin_amdgcn_raw_buffer_load_b128(rx, voff + e * 16, off, 0);
                return o;
            };
            const int cell = uniform((t0 + t % TN) * C);
            const v4f f = tile_by_definition<FORM>(rw, L, l, cell, operand_a);
            const int m = first + 4 * kb, n = (t0 + t % TN) * 16 + row;
            float scale[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) scale[r] = sx ? __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_sx, (m + r) * 4, 0, 0)) : 1.0f;
            store_tile(rs_y, L, m, n, f, scale, __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, n * 4, 0, 0)));
        }
    }
}

template <int FORM, int KS, int TM, bool BLOCKS>
int launch(const uint8_t* packed, const Layout& L, int64_t M, const void* xq, const float* sx, const float* bias, float* y,
           hipStream_t st)
{
    constexpr int T = TM * TN;
    const int MT = (int)((M + 16 * TM - 1) / (16 * TM)), NT = (int)((L.T + TN - 1) / TN);
    constexpr size_t smem = (size_t)KS * T * 64 * 16;
    static_assert(smem <= kLdsPerWorkgroup, "partial tiles in LDS");
    auto kern = ksplit_kernel<FORM, KS, TM, BLOCKS>;
    static thread_local int allowed_dev = -1;
    if (int s = allow_large_lds(kern, smem, allowed_dev)) return s;
    const int64_t grid = xcd_tile_grid(MT, NT);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * KS), smem, st, packed, L, (int)M, xq, sx, bias, y, MT, NT);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

// The height of the tiles, 16 tm tokens: a launch takes as many rounds as its busiest CU has tiles, and a round as long as
// a tile's tm row tiles and a part that does not depend on them (weights, minima).  The tallest of the cheapest is taken,
// so that 333 tokens of 4096 columns, 384 tiles of 64 x 64 - two rounds -, run as 448 tiles of 48 x 64, two shorter ones.
// Measured rounds at K = 4096 with tm = 4 / 3 / 2 / 1: int8 bytes 11.4 / 9.5 / 7.4 / 6 us, int4 9.3 / 7.9 / 5.8 / 4.3, with
// fp16 activations 17.0 / 13.4 / 10.0 / 5.7.  Over 314 shapes of the listed layers, 80 - 2048 tokens, the choice is within
// 1 % (geometric mean) of the best of tm = 1 .. 4 and the tiled GEMM, and 12 % faster than tm = 4 alone up to three (fp16
// activations: two) tiles per CU: 333 tokens of 4096 x 14336 65 -> 58 us (int8 bytes), 130 tokens of 1536 x 8960
// 27 -> 19 us, 1500 tokens of 4096 x 14336 253 -> 206 us.
// (With a float minimum and fp16 activations tm = 4 spills 17 registers of 256; at most three rows there is no faster: 441
// shapes within 0.3 % in the geometric mean, 0.82 - 0.90 on short rows, 1.03 - 1.06 on long ones.)
struct Height {
    int tm;
    float rounds;      // in rounds of tm = 4
};

Height tile_height(const Layout& L, int64_t M, int form)
{
    const float fixed = is_f16(form) ? 0.65f : form == kBytes ? 2.3f : 1.4f;   // in row tiles
    const int64_t NT = (L.T + TN - 1) / TN, cus = num_cus();
    Height best{4, 0.0f};
    for (int tm = 4; tm >= 1; --tm) {
        const int64_t tiles = (M + 16 * tm - 1) / (16 * tm) * NT;
        const float cost = (float)((tiles + cus - 1) / cus) * (tm + fixed) / (4 + fixed);
        if (tm == 4 || cost < 0.97f * best.rounds) best = Height{tm, cost};
    }
    return best;
}

// Rounds of the tiled GEMM (128 x 128 tiles) in the same unit; the constants are fitted to the same measurements.  The
// first round weighs more than the next ones, with a CU's second workgroup beside it.
float tiled_rounds(const Layout& L, int64_t M, int form)
{
    // (int8: whole columns per XCD, as the fit saw them and as the tiles were dealt then; this side is asked up to one tile per CU,
    // and for 65 - 128 tokens of any number of columns)
    const int64_t columns = (L.T + 7) / 8, cus = num_cus();
    const int64_t tiles = (M + 127) / 128 * (is_f16(form) ? columns : (columns + kXcdCount - 1) / kXcdCount * kXcdCount);
    const float n = (float)((tiles + cus - 1) / cus);
    // (two tiles per CU run as one of 256 x 128, split: 1300 tokens of 3072 x 4096 66 us, in four rounds here 74 us)
    if (is_f16(form)) return n == 2.0f ? 3.8f : 1.8f * n + 0.4f;
    return form == kBytes ? 3.1f * n + 0.75f : form == kMin ? 2.6f * n + 1.5f : 2.25f * n + 1.8f;
}

// Waves that share a tile: eight where there is one tile per CU, else four, and a CU holds two workgroups.
int waves_of(const Layout& L, int64_t M, int tm)
{
    return (M + 16 * tm - 1) / (16 * tm) * ((L.T + TN - 1) / TN) <= num_cus() ? 8 : 4;
}

template <int FORM, int TM>
int launch_height(const uint8_t* packed, const Layout& L, int64_t M, const void* xq, bool blocks, const float* sx,
                  const float* bias, float* y, hipStream_t st)
{
    const bool eight = waves_of(L, M, TM) == 8;
    if constexpr (!is_f16(FORM)) {
        if (blocks && eight) return launch<FORM, 8, TM, true>(packed, L, M, xq, sx, bias, y, st);
        if (blocks) return launch<FORM, 4, TM, true>(packed, L, M, xq, sx, bias, y, st);
    }
    if (eight) return launch<FORM, 8, TM, false>(packed, L, M, xq, sx, bias, y, st);
    return launch<FORM, 4, TM, false>(packed, L, M, xq, sx, bias, y, st);
}

template <int FORM>
int launch_form(const uint8_t* packed, const Layout& L, int64_t M, const void* xq, bool blocks, const float* sx,
                const float* bias, float* y, hipStream_t st)
{
    switch (tile_height(L, M, FORM).tm) {
        case 1: return launch_height<FORM, 1>(packed, L, M, xq, blocks, sx, bias, y, st);
        case 2: return launch_height<FORM, 2>(packed, L, M, xq, blocks, sx, bias, y, st);
        case 3: return launch_height<FORM, 3>(packed, L, M, xq, blocks, sx, bias, y, st);
        default: return launch_height<FORM, 4>(packed, L, M, xq, blocks, sx, bias, y, st);
    }
}

}  // namespace

// Where its rounds cost less than the tiled GEMM's: 1024 tokens of 6144 x 4096 in int8 bytes (six rounds against two) 68
// against 76 us, 512 tokens of 17920 x 1536 (nine against three) 48 against 52 us; int4 57 against 60 and 41 against 39 us -
// with the chip full, the tiled form's sharing of operands through LDS counts.
//
// Where the tiled GEMM has more than one tile per CU both are weighed in microseconds fitted to the same calls (K-split / tiled,
// us: float minimum 2048 tokens of 6144 x 4096 129 / 103, 427 of 24288 x 3456 102 / 84, 342 of 36688 x 1216 49 / 72; bytes 1220
// of 14720 x 3456 173 / 154).  A call on rows and a fused one take the same kernel, so that their results are the same bits.
// Else a round costs as much again as two chunks of it, which the measured rounds (32 chunks) hold already: the exchange of the
// partial sums.  Over 595 shapes of 65 - 2048 tokens, calls on int8 rows and fused ones, the choice costs 0.25 % against the
// better of the two kernels at each shape, 8 % at most where the call is fused and 12 % on rows; without the round's own part
// and with the byte form's constant at 1.0 it had been 0.53 % and 20 % (int8 bytes on rows, K-split / tiled, 377 tokens of
// 17920 x 1536 41 / 34 us, 113 tokens of 28672 x 4096 55 / 49; int4 256 tokens of 15952 x 1664 24.3 / 20.3).
bool ksplit8_wanted(const Layout& L, int64_t M)
{
    if (debug_option(kDbgPrefillTile) || debug_option(kDbgNoSkinny)) return false;   // tests and tuning: the tiled GEMM
    if (L.mode == MNNQ_W8_MIN_FLOAT && !L.native8) return false;     // (nibble planes: the tiled GEMM merges them)
    const int64_t lim = kOutOfRange;                                 // 32-bit offsets
    const int form = form_of(L, false);
    const float rounds = tile_height(L, M, form).rounds, C = (float)L.C;
    bool faster;
    if (const float tiled = prefill8_us(L, M); tiled > 0.0f) {
        // microseconds against microseconds (of a call on rows; M Kx: what the quantizer in token-block order costs less)
        const float us = -0.3e-6f * (float)(M * L.Kx) + (form == kBytes ? 6.25f + (1.5f + 0.275f * C) * rounds
                       : form == kMin ? 6.6f + (1.41f + 0.252f * C) * rounds : 6.45f + (1.35f + 0.216f * C) * rounds);
        faster = us <= tiled * (form == kZp ? 1.03f : 1.02f);      // (within the fits, the side that the fused call gains by)
    } else {
        const float own = (1.0f + 2.0f / C) / (1.0f + 2.0f / 32.0f);
        faster = rounds * own <= tiled_rounds(L, M, form);
    }
    return faster && (M + 64) * L.Kx < lim &&
           (M + 64) * L.N * (L.out16 ? 2 : 4) < lim && TN * L.C * 2048 < lim;
}

void describe_ksplit(const Layout& L, int64_t M, bool f16, int32_t out[8])
{
    const int tm = tile_height(L, M, form_of(L, f16)).tm;
    out[0] = 3;
    out[1] = 16 * tm;
    out[2] = 16 * TN;
    out[3] = out[4] = waves_of(L, M, tm);
    out[6] = (int32_t)xcd_tile_grid((M + 16 * tm - 1) / (16 * tm), (L.T + TN - 1) / TN);
}

int launch_ksplit8(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, bool blocks, const float* sx,
                   const float* bias, float* y, hipStream_t st)
{
    if (L.native8) return launch_form<kBytes>(packed, L, M, xq, blocks, sx, bias, y, st);
    if (L.minf) return launch_form<kMin>(packed, L, M, xq, blocks, sx, bias, y, st);
    return launch_form<kZp>(packed, L, M, xq, blocks, sx, bias, y, st);
}

// fp16 activations: microseconds of a launch, from its rounds; over 8000 measured shapes of 17 - 2048 tokens, either form, nine
// in ten are within 10 %.
float ksplit_f16_us(const Layout& L, int64_t M)
{
    const float C = (float)L.C, rounds = tile_height(L, M, form_of(L, true)).rounds;
    return L.minf ? 5.0f + (1.1f + 0.55f * C) * rounds : 4.7f + (1.0f + 0.515f * C) * rounds;
}

// Against the expected time of the wide tiles (float minimum: the rounds of 128 x 128 ones): 333 tokens of 4096 x 14336 (two
// rounds of 48 rows) 93 against 120 us tiled, 512 tokens (two of 64) 119 against 119 us; 700 tokens (three) 176 against 115 us.
bool ksplit_f16_wanted(const Layout& L, int64_t M)
{
    if (debug_option(kDbgPrefillTile) || debug_option(kDbgNoSkinny)) return false;   // tests and tuning: the tiled GEMM
    const int64_t lim = kOutOfRange;                                 // 32-bit offsets
    const bool faster = L.minf ? tile_height(L, M, kMinF16).rounds <= tiled_rounds(L, M, kMinF16)
                               : ksplit_f16_us(L, M) <= 1.04f * prefill_f16_us(L, M);
    return faster && (M + 64) * L.Kx * 2 < lim && (M + 64) * L.N * (L.out16 ? 2 : 4) < lim && TN * L.C * 1024 < lim;
}

int launch_ksplit_f16(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16, const float* bias, float* y,
                      hipStream_t st)
{
    if (L.minf) return launch_form<kMinF16>(packed, L, M, x16, false, nullptr, bias, y, st);
    return launch_form<kZpF16>(packed, L, M, x16, false, nullptr, bias, y, st);
}

}  // namespace mnnq
