// Prefill GEMM on the fp6 matrix instructions for shapes with few output tiles: the operands of mnnq_prefill6.hip (weight
// plane and activation planes, see there for the arithmetic), another split of the work.
//
// The tiled GEMM gives a 128 x 128 output tile to a workgroup; 512 tokens of a 1536-wide layer are 48 such tiles on 256
// CUs.  Here a wave owns a tile of 32 TM x 32 TN outputs and a part of K, and the KS waves of a workgroup share the tile:
// four to eight times the parallelism per output.  No operand is shared between the waves of a workgroup (each meets its
// own groups), so fragments go straight from L2 into registers, up to DEPTH groups ahead, with no LDS and no barrier in
// the loop (a wave may leave it after any of the DEPTH stages: where those paths meet again, at the loop's head, the
// 64 x 64 forms wait for all loads in flight, once per DEPTH groups); the KS partial tiles are added through LDS in a fixed
// order at the end.  What bounds it is the vector memory pipe: a group of a 64 x 64 tile is 9 KiB, 144 cycles at 64 bytes
// per cycle and CU, against about 100 cycles of matrix and vector issue (four pairs of matrix instructions and 64
// multiply-adds on four SIMDs).
#include "mnnq_common.h"

namespace mnnq {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kBufFlags = 0x00020000;     // raw buffer, 32-bit data format (gfx9 family)
constexpr int kOutOfRange = 0x7fff0000;   // a byte offset beyond every buffer (prefill6_possible and the limits on y): loads give 0, stores are dropped

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kBufFlags);
}

struct PairFrag {  // the two activation operands of 32 rows and a group (store_pair): twelve registers per lane
    v4i p[3];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int lane, int off)   // off: uniform
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) p[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + i * 1024, off, 0);
    }
    __device__ __forceinline__ v8i hi() const { return v8i{p[0].x, p[0].y, p[0].z, p[0].w, p[1].x, p[1].y, 0, 0}; }
    __device__ __forceinline__ v8i lo() const { return v8i{p[1].z, p[1].w, p[2].x, p[2].y, p[2].z, p[2].w, 0, 0}; }
};

struct Frag {      // a weight operand: six registers per lane
    v4i a;
    v2i b;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, int lane, int off)   // off: uniform
    {
        a = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, off, 0);
        b = __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8 + 1024, off, 0);
    }
    __device__ __forceinline__ v8i operand() const { return v8i{a.x, a.y, a.z, a.w, b.x, b.y, 0, 0}; }
};

__device__ __forceinline__ v16f mfma6(v8i a, v8i b, v16f c, int scale_a, int scale_b)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 2, 2, 0, scale_a, 0, scale_b);
}

template <int TM, int TN, int KS, int DEPTH>
__global__ __launch_bounds__(64 * KS) void ksplit6_kernel(const uint8_t* __restrict__ plane,
                                                          const uint8_t* __restrict__ a6, Layout L, int64_t M, int TMp,
                                                          const float* __restrict__ sx, const float* __restrict__ bias,
                                                          float* __restrict__ y, int MT, int NT)
{
    extern __shared__ __align__(16) float4 lds_sum[];   // [KS][TM * TN * 4][64]
    constexpr int T = TM * TN, BLK = kPlaneBlockBytes;
    const int lane = threadIdx.x & 63;
    const int ks = uniform(threadIdx.x >> 6);
    int tile_m, tile_n;
    if (!xcd_tile(MT, NT, tile_m, tile_n)) return;
    const int G = (int)L.Gx;
    const int g0 = G * ks / KS, g1 = G * (ks + 1) / KS;

    const int a_step = TMp * 2 * BLK, w_step = (int)L.T32p * BLK, s_step = (int)L.T32p * 128;
    const __amdgpu_buffer_rsrc_t rs_a = rsrc(a6, (int64_t)G * a_step);
    const __amdgpu_buffer_rsrc_t rs_w = rsrc(plane, (int64_t)L.plane_codes_bytes());
    const __amdgpu_buffer_rsrc_t rs_s = rsrc(plane + L.plane_codes_bytes(), (int64_t)L.plane_scales_bytes());
    const int a_base = tile_m * TM * 2 * BLK, w_base = tile_n * TN * BLK, s_base = tile_n * TN * 128;
    const int s_voff = (TN == 1 ? lane & 31 : lane) * 4;
    static_assert(TN <= 2, "the scales of a group fit the wave's lanes");

    // operand scales (one byte per lane, 2^(b - 127)): operands are value / 8 each, the high parts weigh 16
    int scale_hi = 127 + 10, scale_lo = 127 + 6, scale_b = 127;
    asm volatile("" : "+v"(scale_hi), "+v"(scale_lo), "+v"(scale_b));
    const v16f zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    PairFrag a[DEPTH][TM];
    Frag b[DEPTH][TN];
    int sc[DEPTH];
    // (a group past the wave's own: outside the buffers, zeros)
    auto load_a = [&](int u, int i, int g) {
        a[u][i].load(rs_a, lane, uniform(g < g1 ? g * a_step + a_base + i * 2 * BLK : kOutOfRange));
    };
    auto load_b = [&](int u, int j, int g) {
        b[u][j].load(rs_w, lane, uniform(g < g1 ? g * w_step + w_base + j * BLK : kOutOfRange));
        if (j == TN - 1)      // one load for the scales of up to two column tiles, one per half of the wave
            sc[u] = __builtin_amdgcn_raw_buffer_load_b32(rs_s, s_voff, uniform(g < g1 ? g * s_step + s_base : kOutOfRange), 0);
    };
    // in the order of the loop's refills: within an iteration the waits are counts
    auto refill = [&](int u, int t, int g) {     // after tile t of stage u's group
        const int i = t / TN, j = t % TN;
        if (j == TN - 1) load_a(u, i, g);
        if (i == TM - 1) load_b(u, j, g);
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            refill(u, t, g0 + u);
            __builtin_amdgcn_sched_barrier(0);
        }

    float acc[T][16];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;
    // The multiply-adds of a tile run behind the matrix instructions of the next one (of the next group, for the last).
    v16f d[2] = {zero16, zero16};
    float s_last = 0.0f;
    int g = g0;
    do {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (u > 0 && g + u >= g1) break;      // (T is even: the last result is in d[1] either way)
            float s[TN];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int i = t / TN, j = t % TN;
                const int cur = (u * T + t) & 1;
                d[cur] = mfma6(a[u][i].hi(), b[u][j].operand(), zero16, scale_hi, scale_b);
                d[cur] = mfma6(a[u][i].lo(), b[u][j].operand(), d[cur], scale_lo, scale_b);
                if (t == 0) {
                    if (TN == 1) {
                        asm("v_mov_b32 %0, %1" : "=v"(s[0]) : "v"(sc[u]));
                    } else {   // lower half of the wave to both halves, upper half to both
                        // (copies the register allocator cannot merge with the refilled register: it would have
                        // to move that one at the end of the loop, and wait for its load there)
                        int lo, hi;
                        asm("v_mov_b32 %0, %1" : "=v"(lo) : "v"(sc[u]));
                        asm("v_mov_b32 %0, %1" : "=v"(hi) : "v"(sc[u]));
                        const auto p = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                        s[0] = __int_as_float(p[0]);
                        s[TN - 1] = __int_as_float(p[1]);
                    }
                }
                refill(u, t, g + u + DEPTH);
                __builtin_amdgcn_sched_barrier(0);
                const int tp = (t + T - 1) % T;
                const float sp = t == 0 ? s_last : s[(t - 1) % TN];
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[tp][r] = fmaf(sp, d[cur ^ 1][r], acc[tp][r]);
                __builtin_amdgcn_sched_barrier(0);
            }
            s_last = s[TN - 1];
        }
        g += DEPTH;
    } while (g < g1);
    static_assert((DEPTH * T) % 2 == 0, "the two result registers alternate over the whole loop body");
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[T - 1][r] = fmaf(s_last, d[1][r], acc[T - 1][r]);

    // Sum over the waves in a fixed order: piece p = four rows per half of a tile (a float4 per lane), dealt to the waves.
    // The scales and biases of a wave's pieces are requested before the exchange, which their latency would follow.
    constexpr int NP = T * 4 / KS;
    const __amdgpu_buffer_rsrc_t rs_sx = rsrc(sx, M * 4);
    const __amdgpu_buffer_rsrc_t rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
    const __amdgpu_buffer_rsrc_t rs_y = rsrc(y, M * L.N * (L.out16 ? 2 : 4));
    const int N = (int)L.N;
    float bn[NP], sm[NP][4];
    int m[NP], n[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int p = ks * NP + k, t = p / 4, q = p % 4;
        m[k] = (tile_m * TM + t / TN) * 32 + 8 * q + 4 * (lane >> 5);   // the lane's four rows
        n[k] = (tile_n * TN + t % TN) * 32 + (lane & 31);
        bn[k] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, n[k] * 4, 0, 0));
#pragma unroll
        for (int r = 0; r < 4; ++r) sm[k][r] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_sx, (m[k] + r) * 4, 0, 0));
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            lds_sum[(ks * T * 4 + t * 4 + q) * 64 + lane] =
                make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int p = ks * NP + k;
        float4 v = lds_sum[p * 64 + lane];
#pragma unroll
        for (int w = 1; w < KS; ++w) {
            const float4 o = lds_sum[(w * T * 4 + p) * 64 + lane];
            v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
        }
        const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float o = fmaf(f[r], sm[k][r], bn[k]);
            // rows past M lie past the end of y
            const int at = n[k] < N ? ((m[k] + r) * N + n[k]) * (L.out16 ? 2 : 4) : kOutOfRange;
            if (L.out16) {
                const _Float16 h = (_Float16)o;
                __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, h), rs_y, at, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(o), rs_y, at, 0, 0);
            }
        }
    }
}

template <int TM, int TN, int KS, int DEPTH>
int launch(const uint8_t* packed, const Layout& L, int64_t M, const uint8_t* a6, const float* sx, const float* bias,
           float* y, hipStream_t st)
{
    const int MT = (int)((M + 32 * TM - 1) / (32 * TM));
    const int NT = (int)((L.N + 32 * TN - 1) / (32 * TN));
    constexpr size_t smem = (size_t)KS * TM * TN * 4 * 64 * 16;
    static_assert(smem <= kLdsPerWorkgroup && (TM * TN * 4) % KS == 0, "partial tiles in LDS");
    auto kern = ksplit6_kernel<TM, TN, KS, DEPTH>;
    static thread_local int allowed_dev = -1;
    if (int s = allow_large_lds(kern, smem, allowed_dev)) return s;
    const int64_t blocks = xcd_tile_grid(MT, NT);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * KS), smem, st, packed + L.plane_off(), a6, L, M,
                       prefill6_row_tiles(M), sx, bias, y, MT, NT);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

}  // namespace

// Forms: 0 = 64 x 64 tiles of eight waves, 1 = 64 x 64 of four waves (two workgroups per CU), 2 = 64 x 32 of eight waves.
// Groups in flight per wave: more did not help where the registers allow it (3584 x 18944, 128 tokens: two 44.3 us, three
// 44.8 us; each iteration's wait for all of them may be why), so the forms take what their registers leave at two waves per SIMD.
size_t ksplit6_lds_bytes(int form) { return (size_t)(form == 0 ? 8 * 4 : form == 1 ? 4 * 4 : 8 * 2) * 4 * 64 * 16; }

int launch_ksplit6(int form, const uint8_t* packed, const Layout& L, int64_t M, const void* planes, const float* sx,
                   const float* bias, float* y, hipStream_t st)
{
    const uint8_t* a6 = static_cast<const uint8_t*>(planes);
    switch (form) {
        case 0: return launch<2, 2, 8, 2>(packed, L, M, a6, sx, bias, y, st);
        case 1: return launch<2, 2, 4, 3>(packed, L, M, a6, sx, bias, y, st);
        default: return launch<2, 1, 8, 4>(packed, L, M, a6, sx, bias, y, st);
    }
}

}  // namespace mnnq
