// Prefill GEMM on the fp6 matrix instructions on wide tiles: 64 tokens x 384 columns per workgroup, four waves per K part.
// Operands and arithmetic are those of mnnq_prefill6.hip, the split of the work is that of mnnq_prefill8w.hip:
//   * the waves share the tokens: the activation planes of two groups (a chunk) reach LDS with direct loads, a ring of three chunks;
//   * each wave owns 96 columns, whose weights and scales go from L2 straight into registers (refilled after the last use in a
//     group: a chunk ahead), so that they cross neither LDS nor a barrier;
//   * one barrier per chunk, ahead of its last row of tiles, makes the next chunk's stage visible and frees this one's, whose
//     fragments have been read by then; the multiply-adds of a tile run behind the matrix instructions of the next one, across groups too.
//
// Bound: matrix and vector issue, as in mnnq_prefill6.hip.  A tile is three quarters of what a CU contracts as two tiles of
// 128 x 128, and one of them keeps a CU as busy as those two: it is for layers that are one wide tile per CU and more than one
// 128 x 128 tile (the rule and what it measured: choose_tiled6).
#include "mnnq_common.h"

namespace mnnq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

#define MNNQ_LDS(p) ((__attribute__((address_space(3))) void*)(p))

constexpr int kBufFlags = 0x00020000;     // raw buffer, 32-bit data format (gfx9 family)
constexpr int kOutOfRange = 0x7ffffff0;   // a byte offset beyond every buffer: loads give 0, stores are dropped
static_assert((int64_t)kOutOfRange >= kMaxBufferBytes / 16 * 16, "beyond every buffer that the calls accept");

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufFlags);
}

constexpr int kPairBytes = 2 * kPlaneBlockBytes;     // both parts of 32 tokens and a group
constexpr int kWaves = 4;                            // of a K part

template <int TM, int TN, int KS>
struct Tile6 {
    static constexpr int NS = 3;
    static constexpr int pieces = 2 * TM * kPairBytes / 1024;                // direct loads of a stage
    static constexpr int NA = (pieces + kWaves - 1) / kWaves;                // ... of each wave (the last ones may bring zeros)
    static constexpr int stage_bytes = NA * kWaves * 1024;
    static constexpr int part_bytes = NS * stage_bytes;
    static constexpr int sum_bytes = KS > 1 ? kWaves * TM * TN * 16 * 64 * 4 : 0;
    static constexpr int patch_floats = 8 * (32 * TN + 4);                   // of a wave: eight rows, padded by four floats
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    static constexpr int lds_bytes = most(KS * part_bytes, most(sum_bytes, kWaves * patch_floats * 4));
};

// vmcnt(n) lgkmcnt(0)
constexpr int wait_loads(int n) { return 0x0070 | (n & 15) | ((n >> 4) << 14); }

__device__ __forceinline__ v16f mfma6(v8i a, v8i b, v16f c, int scale_a, int scale_b)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, scale_a, 0, scale_b);
}

template <int TM, int TN, int KS>
__global__ __launch_bounds__(64 * kWaves * KS, 2) void prefill6_wide_kernel(
    const uint8_t* __restrict__ plane, const uint8_t* __restrict__ a6, Layout L, int64_t M, int TMp, const float* __restrict__ sx,
    const float* __restrict__ bias, float* __restrict__ y, int MT, int NT)
{
    using Cfg = Tile6<TM, TN, KS>;
    constexpr int NS = Cfg::NS, T = TM * TN, BLK = kPlaneBlockBytes;
    extern __shared__ __align__(16) uint8_t lds_all[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = uniform(tid >> 6);
    const int wave = wave_id % kWaves, part = wave_id / kWaves;
    uint8_t* const lds = lds_all + part * Cfg::part_bytes;
    int tile_m, tile_n;
    if (!xcd_tile(MT, NT, tile_m, tile_n)) return;
    const int G = (int)L.Gx, C = (G + 1) / 2;
    const int cb = C * part / KS, ce = C * (part + 1) / KS, n_iter = (C + KS - 1) / KS;
    const int g_end = 2 * ce < G ? 2 * ce : G;       // (groups past it: zeros)

    // Activations: a group's TM pairs of blocks are consecutive in memory and in the stage.
    const int a_step = TMp * kPairBytes, a_base = tile_m * TM * kPairBytes;
    const __amdgpu_buffer_rsrc_t rs_a = rsrc(a6, (int64_t)G * a_step);
    const int off16 = lane * 16;
    // (offsets are formed without branches: they would part the loop's instructions)
    int a_off[Cfg::NA];                              // of this wave's pieces in chunk 0
#pragma unroll
    for (int i = 0; i < Cfg::NA; ++i) {
        const int q = wave * Cfg::NA + i, h = q >= 3 * TM ? 1 : 0;
        a_off[i] = uniform(h * a_step + a_base + (q - 3 * TM * h) * 1024);
    }
    auto issue_a = [&](int c, uint8_t* stage) {
        const int at = 2 * c * a_step;
#pragma unroll
        for (int i = 0; i < Cfg::NA; ++i) {
            const int q = wave * Cfg::NA + i, last = q < 3 * TM ? g_end : q < 6 * TM ? g_end - 1 : -1;
            const int off = uniform(2 * c < last ? at + a_off[i] : kOutOfRange);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_a, MNNQ_LDS(stage + q * 1024), 16, off16, off, 0, 0);
        }
    };
    struct Pair {
        v8i hi, lo;
    };
    auto read_a = [&](const uint8_t* stage, int i, int h) {
        const uint8_t* p = stage + (h * TM + i) * kPairBytes + off16;
        const v4i p0 = *reinterpret_cast<const v4i*>(p), p1 = *reinterpret_cast<const v4i*>(p + 1024);
        const v4i p2 = *reinterpret_cast<const v4i*>(p + 2048);
        return Pair{v8i{p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, 0, 0}, v8i{p1.z, p1.w, p2.x, p2.y, p2.z, p2.w, 0, 0}};
    };

    // Weights of the wave's columns (tiles past the plane's end of a group: another group's, or zeros; they are not stored).
    const int ct0 = (tile_n * kWaves + wave) * TN;
    const int T32p = (int)L.T32p;
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(plane, (int64_t)L.plane_codes_bytes());
    const __amdgpu_buffer_rsrc_t rs_s = rsrc(plane + L.plane_codes_bytes(), (int64_t)L.plane_scales_bytes());
    const int off8 = 1024 + lane * 8, off4 = (lane & 31) * 4;
    v4i wa[2][TN];                                   // both groups of a chunk
    v2i wb[2][TN];
    int s[2][TN];
    int w_off[2], s_off[2];                          // of the groups of the chunk to load
    const int w_step = 2 * T32p * BLK, s_step = 2 * T32p * 128;
    int w_at = uniform((2 * cb * T32p + ct0) * BLK), s_at = uniform((2 * cb * T32p + ct0) * 128);
    auto next_offsets = [&](int c) {                 // chunk c is w_at's and s_at's
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            w_off[h] = 2 * c + h < g_end ? w_at + h * (w_step / 2) : kOutOfRange;
            s_off[h] = 2 * c + h < g_end ? s_at + h * (s_step / 2) : kOutOfRange;
        }
        w_at += w_step;
        s_at += s_step;
    };
    auto load_codes = [&](int j, int h) {
        const int off = (int)((uint32_t)w_off[h] + j * BLK);
        wa[h][j] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, off16, off, 0);
        wb[h][j] = __builtin_amdgcn_raw_buffer_load_b64(rs_w, off8, off, 0);
    };
    auto load_scale = [&](int j, int h) {
        s[h][j] = __builtin_amdgcn_raw_buffer_load_b32(rs_s, off4, (int)((uint32_t)s_off[h] + j * 128), 0);
    };

    float acc[T][16];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

    // operand scales (one byte per lane, 2^(b - 127)): operands are value / 8 each, the high parts weigh 16
    int scale_hi = 127 + 10, scale_lo = 127 + 6, scale_b = 127;
    asm volatile("" : "+v"(scale_hi), "+v"(scale_lo), "+v"(scale_b));
    const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int n = 0; n < NS; ++n) issue_a(cb + n, lds + n * Cfg::stage_bytes);
    next_offsets(cb);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            load_codes(j, h);
            load_scale(j, h);
        }
    // (landed here, the stages too: inside the loop the waits are counts of its own loads)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(wa[n][j]), "+v"(wb[n][j]), "+v"(s[n][j]));
    __builtin_amdgcn_s_waitcnt(wait_loads(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    uint8_t* stage = lds;                            // of the chunk being contracted
    Pair a[2];
    a[0] = read_a(stage, 0, 0);
    v16f d[2] = {zero16, zero16};
    int s_last = 0;                                  // scale of the tile before
    auto scale_add = [&](int t, int scale, v16f v) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[t][r] = fmaf(__int_as_float(scale), v[r], acc[t][r]);
            asm volatile("" : "+v"(acc[t][r]));
        }
    };
    next_offsets(cb + 1);
    for (int it = 0; it < n_iter; ++it) {
        const int c = cb + it;
        uint8_t* const next = stage + Cfg::stage_bytes == lds + Cfg::part_bytes ? lds : stage + Cfg::stage_bytes;
#pragma unroll
        for (int u = 0; u < 2 * T; ++u) {
            const int h = u / T, i = u % T / TN, j = u % TN, row = h * TM + i;
            if (j == 0) {
                if (row == 2 * TM - 1) {
                    // All of this wave's reads of the stage are done, and its pieces of the next one have landed: the loads younger
                    // than those are NS - 2 stages and a chunk's weights and scales per chunk in between.  The count holds only while
                    // a chunk issues exactly those loads and the direct ones ahead of the codes that follow them: what other waves
                    // read rests on it, so the order is fixed below and checked in the compiled kernel (test_generated_code_cpu.py).
                    constexpr int kYounger = (NS - 2) * Cfg::NA + (NS - 1) * 6 * TN;
                    __builtin_amdgcn_s_waitcnt(wait_loads(kYounger < 63 ? kYounger : 63));
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    issue_a(c + NS, stage);
                    __builtin_amdgcn_sched_barrier(0);
                    a[(row + 1) & 1] = read_a(next, 0, 0);
                } else {
                    a[(row + 1) & 1] = read_a(stage, (row + 1) % TM, (row + 1) / TM);
                }
            }
            const v4i x = wa[h][j];
            const v2i z = wb[h][j];
            const v8i b = {x.x, x.y, x.z, x.w, z.x, z.y, 0, 0};
            d[u & 1] = mfma6(a[row & 1].hi, b, zero16, scale_hi, scale_b);
            d[u & 1] = mfma6(a[row & 1].lo, b, d[u & 1], scale_lo, scale_b);
            if (i == TM - 1) load_codes(j, h);
            __builtin_amdgcn_sched_barrier(0);
            // the tile before (of the chunk before, for the first one)
            if (u == 0) {
                scale_add(T - 1, s_last, d[1]);
            } else {
                const int hp = (u - 1) / T, tp = (u - 1) % T, jp = tp % TN;
                scale_add(tp, s[hp][jp], d[(u - 1) & 1]);
                if (tp / TN == TM - 1) load_scale(jp, hp);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // (a copy that the register allocator cannot merge with the register that is loaded again)
        asm volatile("v_mov_b32 %0, %1" : "=v"(s_last) : "v"(s[1][TN - 1]));
        load_scale(TN - 1, 1);
        next_offsets(c + 2);
        stage = next;
    }
    scale_add(T - 1, s_last, d[1]);

    __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0) lgkmcnt(0): no direct load may still land in LDS
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (KS > 1) {
        // A part > 0 leaves its sums in LDS, part 0 adds them, in order.
        float* red = reinterpret_cast<float*>(lds_all) + wave * (T * 16 * 64) + lane;
#pragma unroll
        for (int p = 1; p < KS; ++p) {
            if (p > 1) __syncthreads();
            if (part == p) {
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[(t * 16 + r) * 64] = acc[t][r];
            }
            __syncthreads();
            if (part == 0) {
#pragma unroll
                for (int t = 0; t < T; ++t)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[t][r] += red[(t * 16 + r) * 64];
            }
        }
        __syncthreads();                             // LDS is free for the output
        if (part != 0) return;
    }

    // Output: y = acc * sx[m] + bias[n].  Rows past M fall outside the buffers (loads give 0, stores are dropped), columns past N
    // are sent out of range, a NULL bias is an empty buffer.  Eight rows x 32 TN columns at a time go through a private LDS patch
    // and leave as 128-bit (binary16: 64-bit) stores of whole row segments; LDS operations of a wave complete in order.
    const __amdgpu_buffer_rsrc_t rs_sx = rsrc(sx, M * 4);
    const __amdgpu_buffer_rsrc_t rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
    const int esz = L.out16 ? 2 : 4, N = (int)L.N;
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(y, (int64_t)(uint32_t)(M * L.N * esz));
    const int row0 = tile_m * TM * 32, col0 = ct0 * 32;
    constexpr int RS = 32 * TN + 4;                  // floats per patch row
    constexpr int UPR = TN * 8;                      // 16-byte units per row segment
    float* patch = reinterpret_cast<float*>(lds_all) + wave * Cfg::patch_floats;
    float* wr = patch + (4 * (lane >> 5)) * RS + (lane & 31);
    float bj[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
        bj[j] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, off4, (col0 + j * 32) * 4, 0));
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int mrow = row0 + i * 32 + 8 * q;  // the patch's first row; this lane writes rows + 4 (lane / 32) + r
            const v4i s4 = __builtin_amdgcn_raw_buffer_load_b128(rs_sx, (lane >> 5) * 16, mrow * 4, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int j = 0; j < TN; ++j) wr[r * RS + j * 32] = fmaf(acc[i * TN + j][q * 4 + r], __int_as_float(s4[r]), bj[j]);
#pragma unroll
            for (int p = 0; p < TN; ++p) {
                const int unit = p * 64 + lane, r = unit / UPR, c4 = unit % UPR;
                // (read as a struct of floats: the same scalar type as the writes for alias analysis)
                const float4 f = *reinterpret_cast<const float4*>(patch + r * RS + c4 * 4);
                const int voff = col0 + c4 * 4 < N ? (r * N + c4 * 4) * esz : kOutOfRange;
                const int soff = (mrow * N + col0) * esz;
                if (L.out16) {
                    const _Float16 h[4] = {(_Float16)f.x, (_Float16)f.y, (_Float16)f.z, (_Float16)f.w};
                    v2i v;
                    __builtin_memcpy(&v, h, 8);
                    __builtin_amdgcn_raw_buffer_store_b64(v, rs_y, voff, soff, 0);
                } else {
                    const v4i v = {__float_as_int(f.x), __float_as_int(f.y), __float_as_int(f.z), __float_as_int(f.w)};
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs_y, voff, soff, 0);
                }
            }
        }
    }
}

template <int TM, int TN, int KS>
int launch(const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx, const float* bias, float* y,
           hipStream_t st)
{
    const int MT = (int)((M + 32 * TM - 1) / (32 * TM)), NT = (int)((L.N + 32 * kWaves * TN - 1) / (32 * kWaves * TN));
    constexpr size_t smem = Tile6<TM, TN, KS>::lds_bytes;
    static_assert(smem <= kLdsPerWorkgroup, "LDS of a workgroup");
    auto kern = prefill6_wide_kernel<TM, TN, KS>;
    static thread_local int allowed_dev = -1;
    if (int s = allow_large_lds(kern, smem, allowed_dev)) return s;
    hipLaunchKernelGGL(kern, dim3((unsigned)xcd_tile_grid(MT, NT)), dim3(64 * kWaves * KS), smem, st, packed + L.plane_off(),
                       static_cast<const uint8_t*>(planes), L, M, prefill6_row_tiles(M), sx, bias, y, MT, NT);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

}  // namespace

size_t prefill6_wide_lds_bytes(int ks) { return ks == 2 ? Tile6<2, 3, 2>::lds_bytes : Tile6<2, 3, 1>::lds_bytes; }

int launch_prefill6_wide(int ks, const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx,
                         const float* bias, float* y, hipStream_t st)
{
    if (ks == 2) return launch<2, 3, 2>(packed, L, M, planes, sx, bias, y, st);
    return launch<2, 3, 1>(packed, L, M, planes, sx, bias, y, st);
}

}  // namespace mnnq
