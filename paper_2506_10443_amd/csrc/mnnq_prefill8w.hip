// Prefill GEMM on the int8 matrix instruction on wide tiles: 128 tokens x 256 or 192 columns per workgroup, for the
// weight forms without a matrix-core plane (int4 with a zero point, int8 bytes; a float minimum of 4-bit codes gained nothing).  Arithmetic and operand
// order are those of mnnq_ksplit.hip.
//
// The waves of a workgroup share the tokens and own 16 TN columns each:
//   * activations (int8 rows) reach LDS with direct loads, a ring of NS chunks (128 values of K), NS - 1 of them in flight or in
//     use; one barrier per chunk makes a stage visible and frees the one before;
//   * weights, scales, zero points and minima go from L2 straight into registers, refilled as soon as they have been used: no
//     wave reads another one's columns;
//   * tiles are walked row by row, the operands of the next group unpacked beside the tiles of this one, the multiply-adds of a
//     tile behind the matrix instruction of the next.
// A tile and group costs eight instructions for the scale.  The minima's part, min[n,g] * (sum of the token's codes in g), is a
// contraction over the groups on v_mfma_f32_16x16x4_f32 (Centered, mnnq_forms.h), with one more matrix instruction per 16 tokens and
// group for the sums.
#include "mnnq_wide.h"

namespace mnnq {

namespace {

#define MNNQ_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kOutOfRange = 0x7ffffff0;   // a byte offset beyond every buffer: loads give 0
static_assert((int64_t)kOutOfRange >= kMaxBufferBytes / 16 * 16, "beyond every buffer that the calls accept");

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

constexpr int kStageBytes = 128 * 128;    // 128 rows of a chunk

// vmcnt(n), the other counters left alone
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

template <int WAVES, int TM, int TN, int KS>
struct Tile8 {
    static constexpr int NS = 3;
    static constexpr int part_bytes = NS * kStageBytes;
    using Out = WideOut<WAVES, TM, TN, KS>;
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int lds_bytes = most(KS * part_bytes, most(Out::sum_bytes, Out::patch_bytes));
};

template <int FORM, int WAVES, int TM, int TN, int KS>
__global__ __launch_bounds__(64 * WAVES * KS, KS > 1 ? 1 : 2) void prefill8_wide_kernel(
    const uint8_t* __restrict__ packed, Layout L, int64_t M, const int8_t* __restrict__ xq, const float* __restrict__ sx,
    const float* __restrict__ bias, float* __restrict__ y, int MT, int NT)
{
    using Cfg = Tile8<WAVES, TM, TN, KS>;
    constexpr int NS = Cfg::NS, T = TM * TN;
    constexpr int NA = 16 / WAVES;                   // direct loads of a stage per wave
    constexpr int NU = has_zero(FORM) ? 1 : 2;       // chunks per turn of the loop: the minima go two at a time
    constexpr int NW = 3 * TN;      // loads into registers per chunk, at least
    extern __shared__ __align__(16) uint8_t lds_all[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = uniform(tid >> 6);
    const int wave = wave_id % WAVES, part = wave_id / WAVES;
    uint8_t* const lds = lds_all + part * Cfg::part_bytes;
    const int row = lane & 15, kb = lane >> 4;
    const int C = (int)L.C, K = (int)L.Kx;
    int tile_m, tile_n;
    if (!xcd_tile(MT, NT, tile_m, tile_n)) return;
    const int m0 = tile_m * 16 * TM;
    const int rt0 = (tile_n * WAVES + wave) * TN;    // first row tile of the layout (16 columns) of this wave
    const int cb = C * part / KS, ce = C * (part + 1) / KS, n_iter = (C + KS - 1) / KS;

    // Activations of a chunk: unit u = 4 h + kb (16 bytes) of a row lies at place u ^ (row % 8).  (The padding group of an odd
    // G reads the next row's first group or past the end: its weights, scales and minima are zero.)
    const __amdgpu_buffer_rsrc_t rs_x = rsrc(xq, M * L.Kx);
    const int a_voff = (lane >> 3) * K + (((lane & 7) ^ (lane >> 3)) << 4);
    auto issue_a = [&](int c, int slot) {            // (rows past the tile and chunks past the part: zeros)
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int q = wave * NA + i;
            const int off = uniform(c < ce && q < 2 * TM ? (m0 + q * 8) * K + c * 128 : kOutOfRange);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, MNNQ_LDS(lds + slot * kStageBytes + q * 1024), 16, a_voff, off, 0, 0);
        }
    };
    const int a_off = row * 128;
    auto read_a = [&](int i, int h, int slot) {
        return *reinterpret_cast<const v4i*>(lds + slot * kStageBytes + i * 2048 + a_off + (((4 * h + kb) ^ (row & 7)) << 4));
    };

    // Weights (what the loads bring for row tiles past the matrix is not stored).
    constexpr int WB = FORM == kBytes ? 2048 : 1024, ZB = has_zero(FORM) ? 32 : 128;
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(packed, (int64_t)L.total());
    const int scales_off = (int)L.scales_off(), zeros_off = (int)L.zeros_off();
    const uint32_t zsel = (row & 1) * 0x02020202u;
    Weights<FORM> w[TN];
    float mn[TN], mn_next[TN], xs[TM];      // operands of the minima's part (Centered), the next two chunks' on their way
    auto load_codes = [&](int j, int h, int c) {     // (the byte form: a kilobyte per group; else both groups with h = 0)
        const int off = uniform(c < ce ? ((rt0 + j) * C + c) * WB : kOutOfRange);
        w[j].w[FORM == kBytes ? h : 0] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, lane * 16 + h * 1024, off, 0);
    };
    auto load_params = [&](int j, int c) {
        const int cell = (rt0 + j) * C + c;
        const int off_s = uniform(c < ce ? scales_off + cell * 128 : kOutOfRange), off_z = uniform(c < ce ? zeros_off + cell * ZB : kOutOfRange);
        w[j].s = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(rs_w, row * 8, off_s, 0));
        if (has_zero(FORM)) w[j].z = __builtin_amdgcn_raw_buffer_load_b32(rs_w, (row >> 1) * 4, off_z, 0);
    };
    auto load_min = [&](int j, int c) {              // of chunks c and c + 1
        const int off = c + (kb >> 1) < ce ? (kb >> 1) * ZB + row * 8 + (kb & 1) * 4 : kOutOfRange;
        mn_next[j] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_w, off, uniform(zeros_off + ((rt0 + j) * C + c) * ZB), 0));
    };

    v4f acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const v4i magic = {kMagicBits, kMagicBits, kMagicBits, kMagicBits};
    const v4i zero4 = {0, 0, 0, 0};
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};

#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue_a(cb + s, s);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        load_params(j, cb);
        load_codes(j, 0, cb);
        if (FORM == kBytes) load_codes(j, 1, cb);
        if (FORM != kZp) load_min(j, cb);
    }
    // (landed here: inside the loop the waits are counts of its own loads)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        asm volatile("" : "+v"(w[j].w[0]), "+v"(w[j].s));
        if (FORM == kBytes) asm volatile("" : "+v"(w[j].w[FORM == kBytes ? 1 : 0]));
        if (FORM != kZp) asm volatile("" : "+v"(mn_next[j]));
    }
    // operands of a group (the byte form takes the loaded registers as they are) and its scales
    Operand<FORM> b[2][FORM == kBytes ? 1 : TN];
    float s[2][TN];
    auto prepare = [&](int j, int h) {
        if (FORM != kBytes) b[h][FORM == kBytes ? 0 : j] = unpack<FORM>(w[j], h, zsel);
        s[h][j] = h ? w[j].s.y : w[j].s.x;
    };
#pragma unroll
    for (int j = 0; j < TN; ++j) prepare(j, 0);

    int slot = 0;                                    // stage of the chunk being contracted
    for (int it = 0; it < n_iter; it += NU) {
        if (!has_zero(FORM)) {
#pragma unroll
            for (int i = 0; i < TM; ++i) xs[i] = 0.0f;
            // (copies: the loads' registers stay where they are)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                asm volatile("v_mov_b32 %0, %1" : "=v"(mn[j]) : "v"(mn_next[j]));
                load_min(j, cb + it + 2);
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int c = cb + it + u;
            // This wave's pieces of the chunk's stage have landed (in order behind them, at least: a stage's loads and a chunk's
            // weights) and its reads of the stage before are done.
            __builtin_amdgcn_s_waitcnt(wait_vm(NA + NW) & ~0x0F00);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            issue_a(c + NS - 1, slot == 0 ? NS - 1 : slot - 1);
            v4i a[2];
            a[0] = read_a(0, 0, slot);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                auto operand = [&](int j) {
                    Operand<FORM> o;
                    o.q[0] = FORM == kBytes ? w[j].w[FORM == kBytes ? h : 0] : b[h][FORM == kBytes ? 0 : j].q[0];
                    return o;
                };
                const Centered<FORM> center(2 * u + h, kb);
                v4i sum[2];
                v4i d[2];
#pragma unroll
                for (int t = 0; t <= T; ++t) {
                    if (t < T) {
                        const int i = t / TN, j = t % TN;
                        if (j == 0) {
                            if (i + 1 < TM) a[(i + 1) & 1] = read_a(i + 1, h, slot);
                            else if (h == 0) a[0] = read_a(0, 1, slot);
                            static_assert(TM % 2 == 0, "the first operand of the second group takes the free slot");
                        }
                        const v4i av = a[i & 1];
                        if (!has_zero(FORM) && j == 0) {     // tokens in the lanes; all rows of the product are equal
                            const v4i x = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, av, zero4, 0, 0, 0);
                            xs[i] = kb == 2 * u + h ? (float)x[0] : xs[i];
                        }
                        d[t & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, operand(j).q[0], magic, 0, 0, 0);
                        if constexpr (!has_zero(FORM)) {
                            if (i == 0) sum[j & 1] = Centered<FORM>::column_sum(operand(j));
                        }
                        if (FORM == kBytes && i == TM - 1) load_codes(j, h, c + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (t > 0) {
                        const int p = t - 1, i = p / TN, j = p % TN;
                        if constexpr (!has_zero(FORM)) {
                            if (i == 0) center(sum[j & 1], s[h][j], mn[j]);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[p][r] = fmaf(s[h][j], from_magic(d[p & 1][r]), acc[p][r]);
                        // the next group's operands, a column in every second row of tiles
                        if (i % 2 == 1 && j == 0 && i / 2 < TN) {
                            const int jn = i / 2;
                            if (h == 1) {            // (both groups are unpacked: the registers have the next chunk)
                                prepare(jn, 0);
                            } else {
                                prepare(jn, 1);
                                if (FORM != kBytes) load_codes(jn, 0, c + 1);
                                load_params(jn, c + 1);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            slot = slot + 1 == NS ? 0 : slot + 1;
        }
        if (!has_zero(FORM)) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i * TN + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[i], mn[j], acc[i * TN + j], 0, 0, 0);
            }
        }
    }

    if (!sum_parts<TM, TN, KS>(lds_all, wave, part, lane, acc)) return;
    store_wide<TM, TN>(lds_all, wave, lane, L, M, m0, rt0, sx, bias, y, acc);
    if constexpr (!has_zero(FORM)) {
        float probe = 0.0f;      // NaN: a column's sums are not finite
#pragma unroll
        for (int j = 0; j < TN; ++j) probe = rt0 + j < (int)L.T ? fmaf(acc[j][0], 0.0f, probe) : probe;
        if (__builtin_expect(__ballot(probe != 0.0f) == 0, 1)) return;
        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the stores above are done
        const __amdgpu_buffer_rsrc_t rs_sx = rsrc(sx, M * 4), rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
        const __amdgpu_buffer_rsrc_t rs_y = rsrc(y, M * L.N * (L.out16 ? 2 : 4));
#pragma unroll 1
        for (int t = 0; t < TM * TN; ++t) {          // (rows past M: past the ends of the buffers)
            const int rt = rt0 + t % TN, first = m0 + (t / TN) * 16;
            if (rt >= (int)L.T) continue;
            const auto operand_a = [&](int c, int h) {
                Operand<FORM> o;
                o.q[0] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, (first + row) * K + kb * 16, uniform(c * 128 + h * 64), 0);
                return o;
            };
            const v4f f = tile_by_definition<FORM>(rs_w, L, lane, uniform(rt * C), operand_a);
            float scale[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) scale[r] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_sx, (first + 4 * kb + r) * 4, 0, 0));
            store_tile(rs_y, L, first + 4 * kb, rt * 16 + row, f, scale,
                       __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, (rt * 16 + row) * 4, 0, 0)));
        }
    }
}

template <int FORM, int WAVES, int TM, int TN, int KS>
int launch(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, const float* sx, const float* bias, float* y,
           hipStream_t st)
{
    const int MT = (int)((M + 16 * TM - 1) / (16 * TM)), NT = (int)((L.T + WAVES * TN - 1) / (WAVES * TN));
    constexpr size_t smem = Tile8<WAVES, TM, TN, KS>::lds_bytes;
    static_assert(smem <= kLdsPerWorkgroup && 2 * TN <= TM, "LDS; a column of the next group per two rows of tiles");
    auto kern = prefill8_wide_kernel<FORM, WAVES, TM, TN, KS>;
    static thread_local int allowed_dev = -1;
    if (int s = allow_large_lds(kern, smem, allowed_dev)) return s;
    hipLaunchKernelGGL(kern, dim3((unsigned)xcd_tile_grid(MT, NT)), dim3(64 * WAVES * KS), smem, st, packed, L, M, xq, sx, bias, y,
                       MT, NT);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

template <int FORM>
int launch_form(int columns, int ks, const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, const float* sx,
                const float* bias, float* y, hipStream_t st)
{
    if (columns == 192 && ks == 2) return launch<FORM, 4, 8, 3, 2>(packed, L, M, xq, sx, bias, y, st);
    if (columns == 192) return launch<FORM, 4, 8, 3, 1>(packed, L, M, xq, sx, bias, y, st);
    if (ks == 2) return launch<FORM, 4, 8, 4, 2>(packed, L, M, xq, sx, bias, y, st);
    return launch<FORM, 4, 8, 4, 1>(packed, L, M, xq, sx, bias, y, st);
}

}  // namespace

size_t prefill8_wide_lds_bytes(int columns, int ks)
{
    if (columns == 192) return ks == 2 ? Tile8<4, 8, 3, 2>::lds_bytes : Tile8<4, 8, 3, 1>::lds_bytes;
    return ks == 2 ? Tile8<4, 8, 4, 2>::lds_bytes : Tile8<4, 8, 4, 1>::lds_bytes;
}

int launch_prefill8_wide(int columns, int ks, const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, const float* sx,
                         const float* bias, float* y, hipStream_t st)
{
    if (L.native8) return launch_form<kBytes>(columns, ks, packed, L, M, xq, sx, bias, y, st);
    return launch_form<kZp>(columns, ks, packed, L, M, xq, sx, bias, y, st);
}

}  // namespace mnnq
