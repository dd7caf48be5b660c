// Prefill GEMM with fp16 activations on wide tiles: 128 tokens x 256 columns per workgroup, int4 weights with a zero
// point.  Arithmetic and operand order are those of mnnq_prefill_f16.hip (two v_mfma_f32_16x16x32_f16 per group and
// 16 x 16 tile on the exact halves q - z, the group scale once per group in fp32).
//
// What moves per group is 16 KB of activations and 8 KB of weights for 128 x 256 outputs; a 256 x 128 tile moves 32 + 4.
// The four waves share the tokens and own 64 columns each, so a weight is unpacked by one wave of the workgroup only:
//   * activations reach LDS with direct loads, a ring of NS groups, two of them in flight; a group's operands (sixteen
//     128-bit reads per wave) stay in registers while it is contracted and are replaced, in its last column of tiles, by
//     the next group's - one barrier per group, in its middle, frees a stage and makes another one visible;
//   * weight codes go from L2 straight into registers, replaced by the next chunk's as soon as their second group is
//     unpacked; scales and zero points through a wave's own LDS, no barrier;
//   * tiles are walked column by column: the eight matrix instruction pairs of a column run beside the unpacking of the
//     next one and the multiply-adds of the tile before.
//
// Bound: issue.  Per pair of matrix instructions (32 cycles) come four multiply-adds and three instructions of unpacking; a
// loop of just these on registers, two waves per SIMD, reaches 1430 TFLOP/s on this card, the kernel 1320 while its CUs are
// full (2048 tokens of 28672 x 4096; 1.75 waves per SIMD over the launch: seven tiles per CU).  32 x 32 matrix instructions
// were 8 % slower in that loop.  Measured, 256 x 128 tiles -> these, us: 2048 tokens of 28672 x 4096 436 -> 417, of
// 4096 x 14336 228 -> 206, of 6144 x 4096 120 -> 97 (192 columns), 1024 tokens of 4096 x 14336 136 -> 119 (four K parts).
#include "mnnq_wide.h"

namespace mnnq {

namespace {

#define MNNQ_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kOutOfRange = 0x7ffffff0;   // a byte offset beyond every buffer: loads give 0
static_assert((int64_t)kOutOfRange >= kMaxBufferBytes / 16 * 16, "beyond every buffer that the calls accept");

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

constexpr int BM = 128;
constexpr int TM = BM / 16;                          // 16 x 16 tiles of a wave: TM x TN, 128 tokens x 64 or 48 columns
constexpr int kStageBytes = BM * 128;
constexpr int kParamBytes = 1024;                    // a wave's scales and zero points of a chunk: one direct load
constexpr int kParamRing = 2;

// WAVES share the tokens, TN columns of tiles each; KS: K parts in the workgroup; NS: stages (groups) of activations.
template <int WAVES, int TN, int KS>
struct Tile {
    static constexpr int NS = WAVES * KS == 8 && WAVES == 2 ? 2 : 3;
    static constexpr int part_bytes = NS * kStageBytes + kParamRing * WAVES * kParamBytes;
    using Out = WideOut<WAVES, TM, TN, KS>;
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int lds_bytes = most(KS * part_bytes, most(Out::sum_bytes, Out::patch_bytes));
};

// vmcnt(n), the other counters left alone
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

template <int WAVES, int TN, int KS>
__global__ __launch_bounds__(64 * WAVES * KS, KS > 1 ? 1 : 2) void prefill_f16_wide_kernel(
    const uint8_t* __restrict__ packed, Layout L, int64_t M, const uint16_t* __restrict__ x16,
    const float* __restrict__ rs, const float* __restrict__ bias, float* __restrict__ y, int MT, int NT)
{
    using Cfg = Tile<WAVES, TN, KS>;
    constexpr int NS = Cfg::NS;
    constexpr int NA = BM / 8 / WAVES;               // direct loads of a stage per wave
    extern __shared__ __align__(16) uint8_t lds_all[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = uniform(tid >> 6);
    const int wave = wave_id % WAVES, part = wave_id / WAVES;
    uint8_t* const lds = lds_all + part * Cfg::part_bytes;
    const int row = lane & 15, kb = lane >> 4;
    const int C = (int)L.C, G = (int)L.G;
    const int K2 = (int)L.Kx * 2;                    // bytes per activation row
    int tile_m, tile_n;
    if (!xcd_tile(MT, NT, tile_m, tile_n)) return;
    const int m0 = tile_m * BM;
    const int rt0 = (tile_n * WAVES + wave) * TN;  // first row tile of the layout (16 columns) of this wave
    const int cb = C * part / KS, ce = C * (part + 1) / KS, n_iter = (C + KS - 1) / KS;

    const __amdgpu_buffer_rsrc_t rs_x = rsrc(x16, M * L.Kx * 2);
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(packed, (int64_t)L.total());

    // Activations of a group: unit u = 2 kb + e (16 bytes) of a row lies at place (kb + 4 e) ^ (row % 8), so that the
    // sixteen lanes which a 128-bit LDS read serves together - 0-3, 12-15 and 20-27 of every 32 - touch every bank once.
    const int place = (lane & 7) ^ (lane >> 3);
    const int a_voff = (lane >> 3) * K2 + ((2 * (place & 3) + (place >> 2)) << 4);
    auto issue_a = [&](int g, int slot) {            // (the padding group of an odd G and groups past the part's: zeros)
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int q = wave * NA + i;
            const int off = uniform(g < G && g < 2 * ce ? (m0 + q * 8) * K2 + g * 128 : kOutOfRange);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, MNNQ_LDS(lds + slot * kStageBytes + q * 1024), 16, a_voff, off, 0, 0);
        }
    };
    // Scales (lanes 0-31: 16 bytes of the 128 of a row tile each) and zero points (lanes 32-39, two per row tile) of a chunk.
    const int p_lane = lane < 32 ? (int)L.scales_off() + (rt0 + (lane >> 3)) * C * 128 + (lane & 7) * 16
                     : lane < 40 ? (int)L.zeros_off() + (rt0 + ((lane - 32) >> 1)) * C * 32 + (lane & 1) * 16 : kOutOfRange;
    const int p_step = lane < 32 ? 128 : lane < 40 ? 32 : 0;
    auto param_slot = [&](int c) { return lds + NS * kStageBytes + ((c & 1) * WAVES + wave) * kParamBytes; };
    auto issue_p = [&](int c) {
        const int off = c < ce ? p_lane + c * p_step : kOutOfRange;
        uint8_t* const at = param_slot(c);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, MNNQ_LDS(at), 16, off, 0, 0, 0);
    };
    v2i w[TN];                                       // a lane's sixteen codes of a group, per column of tiles
    auto load_w = [&](int j, int c, int h) {
        const int off = uniform(c < ce ? ((rt0 + j) * C + c) * 1024 + h * 8 : kOutOfRange);
        w[j] = __builtin_amdgcn_raw_buffer_load_b64(rs_w, lane * 16, off, 0);
    };

    v4f acc[TM * TN];
#pragma unroll
    for (int t = 0; t < TM * TN; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const v4f zerof = {0.0f, 0.0f, 0.0f, 0.0f};

    v4i a[TM][2];
    const int a0_off = row * 128 + ((kb ^ (row & 7)) << 4), a1_off = row * 128 + (((kb + 4) ^ (row & 7)) << 4);
    auto read_a = [&](int i, int slot) {
        const uint8_t* st = lds + slot * kStageBytes + i * 2048;
        a[i][0] = *reinterpret_cast<const v4i*>(st + a0_off);
        a[i][1] = *reinterpret_cast<const v4i*>(st + a1_off);
    };
    float sc[2];
    uint32_t z;
    auto read_scale = [&](int j, int c, int h) {
        sc[(h * TN + j) & 1] = *reinterpret_cast<const float*>(param_slot(c) + j * 128 + row * 8 + h * 4);
    };
    auto read_zero = [&](int j, int c, int h) { z = *(param_slot(c) + 512 + j * 32 + row * 2 + h); };

    // Operands of a column of tiles, sixteen halves per lane; built a dword at a time (step 0 .. 7) beside the column before.
    uint32_t b[2][8];
    uint32_t nib = 0;
    h2 zb = {};
    auto unpack_step = [&](int j, int h, int s) {
        const uint32_t codes = (uint32_t)(s < 4 ? w[j].x : w[j].y);
        if (s == 0) zb = __builtin_bit_cast(h2, (z << 16 | z) | 0x64006400u);
        if (s % 4 == 0) nib = codes & 0x0f0f0f0fu;
        if (s % 4 == 2) nib = (codes >> 4) & 0x0f0f0f0fu;
        // (a byte c under the high byte 0x64 is the half 1024 + c)
        const uint32_t p = __builtin_amdgcn_perm(0x64646464u, nib, (s & 1) ? 0x04030402u : 0x04010400u);
        b[(h * TN + j) & 1][s] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(h2, p) - zb);
    };
    auto operand = [&](int slot, int e) {
        return v4i{(int)b[slot][4 * e], (int)b[slot][4 * e + 1], (int)b[slot][4 * e + 2], (int)b[slot][4 * e + 3]};
    };

    issue_p(cb);
#pragma unroll
    for (int s = 0; s < NS; ++s) issue_a(2 * cb + s, s);
#pragma unroll
    for (int j = 0; j < TN; ++j) load_w(j, cb, 0);
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) read_a(i, 0);
    read_zero(0, cb, 0);
    read_scale(0, cb, 0);
#pragma unroll
    for (int s = 0; s < 8; ++s) unpack_step(0, 0, s);
    load_w(0, cb, 1);
    read_zero(1, cb, 0);

    // The multiply-adds of tile p run behind the matrix instructions of the next one.
    v4f d[2] = {zerof, zerof};
    sc[1] = 0.0f;                                    // (the first one has no tile before it)
    auto fold = [&](int p, int h) {
        const int j = p / TM, i = p % TM;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i * TN + j][r] = fmaf(sc[(h * TN + j) & 1], d[p & 1][r], acc[i * TN + j][r]);
    };
    int slot = 0;                                    // stage of the group being contracted
    for (int it = 0; it < n_iter; ++it) {
        const int c = cb + it;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int next = slot + 1 == NS ? 0 : slot + 1;
#pragma unroll
            for (int t = 0; t < TM * TN; ++t) {
                const int j = t / TM, i = t % TM;
                if (t == TN / 2 * TM) {
                    // This wave's pieces of the next group's stage and (h = 1) of the next chunk's parameters have landed -
                    // in order behind the one, with three stages: a group's w, a stage's loads, a group's w; behind the
                    // other: a stage's, a group's w; with two stages: a group's w - and its operands of this group are in
                    // registers.
                    if (h == 0) __builtin_amdgcn_s_waitcnt(wait_vm(NS == 2 ? TN : 2 * TN + NA));
                    else __builtin_amdgcn_s_waitcnt(wait_vm(NS == 2 ? TN : TN + NA));
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    if (h == 0) issue_p(c + 1);
                    issue_a(2 * c + h + NS, slot);
                }
                d[t & 1] = mfma_f16(a[i][0], operand((h * TN + j) & 1, 0), zerof);
                d[t & 1] = mfma_f16(a[i][1], operand((h * TN + j) & 1, 1), d[t & 1]);
                if (j == TN - 1) read_a(i, next);
                if (i == 1) read_scale((j + 1) % TN, j + 1 < TN || h == 0 ? c : c + 1, j + 1 < TN ? h : 1 - h);
                __builtin_amdgcn_sched_barrier(0);
                unpack_step((j + 1) % TN, j + 1 < TN ? h : 1 - h, i);
                fold((t + TM * TN - 1) % (TM * TN), t > 0 ? h : 1 - h);   // (t = 0: the last tile of the group before)
                // the zero point two columns on; the codes of the column just unpacked, of the next group
                if (i == TM - 3) read_zero((j + 2) % TN, j + 2 < TN || h == 0 ? c : c + 1, j + 2 < TN ? h : 1 - h);
                if (i == TM - 1) {
                    if (j + 1 < TN) load_w(j + 1, h == 0 ? c : c + 1, 1 - h);
                    else load_w(0, c + 1, h);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            slot = next;
        }
    }
    fold(TM * TN - 1, 1);

    if (!sum_parts<TM, TN, KS>(lds_all, wave, part, lane, acc)) return;
    store_wide<TM, TN>(lds_all, wave, lane, L, M, m0, rt0, rs, bias, y, acc);
}

template <int WAVES, int TN, int KS>
int launch(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16, const float* rs, const float* bias, float* y,
           hipStream_t st)
{
    const int MT = (int)((M + BM - 1) / BM), NT = (int)((L.T + WAVES * TN - 1) / (WAVES * TN));
    constexpr size_t smem = Tile<WAVES, TN, KS>::lds_bytes;
    auto kern = prefill_f16_wide_kernel<WAVES, TN, KS>;
    static thread_local int allowed_dev = -1;
    if (int s = allow_large_lds(kern, smem, allowed_dev)) return s;
    hipLaunchKernelGGL(kern, dim3((unsigned)xcd_tile_grid(MT, NT)), dim3(64 * WAVES * KS), smem, st, packed, L, M, x16, rs, bias, y,
                       MT, NT);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

}  // namespace

int launch_prefill_f16_wide(int columns, int ks, const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16,
                            const float* rs, const float* bias, float* y, hipStream_t st)
{
    if (columns == 128) return launch<2, 4, 4>(packed, L, M, x16, rs, bias, y, st);
    if (columns == 192 && ks == 2) return launch<4, 3, 2>(packed, L, M, x16, rs, bias, y, st);
    if (columns == 192) return launch<4, 3, 1>(packed, L, M, x16, rs, bias, y, st);
    if (ks == 2) return launch<4, 4, 2>(packed, L, M, x16, rs, bias, y, st);
    return launch<4, 4, 1>(packed, L, M, x16, rs, bias, y, st);
}

}  // namespace mnnq
