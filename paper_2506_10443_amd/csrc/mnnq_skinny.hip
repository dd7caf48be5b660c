// A few tokens at once (batched or speculative decoding).  The step is still memory-bound (Section 2.1), so the
// weights are streamed exactly once, as in the one-token GEMV, and every chunk meets all M activation rows in the
// matrix cores: one v_mfma_i32_16x16x64_i8 per quantization group contracts the 16 weight rows of a row tile with up
// to 16 tokens; up to TM = 4 blocks of 16 tokens share one unpacking of the weights.
//
//   y[m,n] = sx[m] * sum_g scale[n,g] * sum_{k in g} xq[m,k] * (q[n,k] - zero[n,g]) (+ bias[n])
//
// (float-minimum forms: sx[m] * sum_g (scale * sum xq q + min * sum xq), the row sums from one more matrix
// instruction with an all-ones operand.)
//
// Work split: the K range of a row tile is dealt to the KS waves of a workgroup, whose partial sums are added in a
// fixed order through LDS.  Every wave meets its own part of K only, so nothing of the activations is shared
// between the waves of a workgroup and they go straight from L2 into registers:
//   resident form (few_resident_kernel): a wave's part is at most NCH chunks; its A operands stay in registers while
//     the workgroup walks over row tiles (grid-stride), so that the loop streams weights and nothing else.  The
//     registers of a chunk are refilled with the same chunk of the next row tile as soon as it has been contracted, by loads
//     that no branch guards: only then does the compiler wait by count, with the refills in flight.  (The waves that store a
//     row tile wait for all of their refills before the store.)  The last row tile of a workgroup stands behind the loop.
//   streaming form (few_stream_kernel): longer rows; weights and activations of a chunk are requested together, DEPTH
//     chunks ahead.
//
// MFMA lane mapping (A: 16 x 64 tokens x k, B: 64 x 16 k x weight rows, D: 16 x 16):
//   A: lane l holds token l % 16, k block l / 16;  B: lane l holds weight row l % 16, the same k block - exactly the
//   lane's 8 bytes of the chunk, unpacked (16 bytes in the byte form of int8 weights, as they are);
//   D: lane l holds weight row l % 16, tokens 4 (l / 16) + r, r = 0..3.
#include "mnnq_forms.h"

#include <stdlib.h>

#include <type_traits>

namespace mnnq {

namespace {

// Memory is read through buffer descriptors whose sizes are exact: a chunk that is not the wave's own, a row tile past
// the matrix, a token past M or the missing half of an odd row lies outside and arrives as zeros without a branch and
// without traffic.  (Plain loads in a loop that refills its registers are no alternative: the compiler moves a load
// whose value crosses the back edge down to its use.)
constexpr int kOutOfRange = 0x7ffffff0;   // a byte offset beyond every buffer

// The chunks of one row tile (an empty buffer past the last one).
template <int FORM>
struct TileBuffers {
    __amdgpu_buffer_rsrc_t w, s, z;
    __device__ __forceinline__ TileBuffers(const uint8_t* __restrict__ packed, const Layout& L, int64_t tile)
    {
        const bool have = tile < L.T;
        const int64_t first = have ? tile * L.C : 0, n = have ? L.C : 0;   // (K <= 2^24: under 2^28 bytes)
        constexpr int WB = FORM == kBytes ? 2048 : 1024, ZB = has_zero(FORM) ? 32 : 128;
        w = rsrc(packed + first * WB, n * WB);
        s = rsrc(packed + L.scales_off() + first * 128, n * 128);
        z = rsrc(packed + L.zeros_off() + first * ZB, n * ZB);
    }
    __device__ __forceinline__ Weights<FORM> load(int c, int lane, int row) const   // c: chunk (uniform)
    {
        Weights<FORM> r;
        const int off = __builtin_amdgcn_readfirstlane(c);
        // (aux 2: the weights pass once and need not stay in the caches)
        r.w[0] = __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16, off * (FORM == kBytes ? 2048 : 1024), 2);
        if (FORM == kBytes)
            r.w[FORM == kBytes ? 1 : 0] = __builtin_amdgcn_raw_buffer_load_b128(w, lane * 16 + 1024, off * 2048, 2);
        r.s = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(s, row * 8, off * 128, 0));
        if (has_zero(FORM)) r.z = __builtin_amdgcn_raw_buffer_load_b32(z, (row >> 1) * 4, off * 32, 0);
        else r.mn = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(z, row * 8, off * 128, 0));
        return r;
    }
};

// The vector side runs one group behind the matrix side: while a group's matrix instructions execute (a result is
// readable 32 cycles after its issue, and at two waves per SIMD nothing else covers that), the results of the group
// before are scaled and added.
template <int TM, int FORM>
struct Pending {
    v4i d[TM], xs[has_zero(FORM) ? 1 : TM];     // (fp16 activations: the bits of floats)
    float s, mn;
    __device__ __forceinline__ Pending() : s(0.0f), mn(0.0f)   // (nothing yet: zeros, whatever the form makes of them)
    {
        const int z = FORM == kZp || FORM == kMin ? kMagicBits : 0;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            d[t] = v4i{z, z, z, z};
            if (!has_zero(FORM)) xs[t] = v4i{0, 0, 0, 0};
        }
    }
    __device__ __forceinline__ void add(int t, float (&acc)[TM][4]) const
    {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int v = d[t][rr], x = has_zero(FORM) ? 0 : xs[has_zero(FORM) ? 0 : t][rr];
            // byte form: sum xq q8 = D + 128 xs as an integer (below 2^22) before it meets the step
            const float i = is_f16(FORM) ? __int_as_float(v) : FORM == kBytes ? (float)(v + (x << 7)) : from_magic(v);
            acc[t][rr] = fmaf(s, i, acc[t][rr]);
            if (!has_zero(FORM)) acc[t][rr] = fmaf(mn, is_f16(FORM) ? __int_as_float(x) : (float)x, acc[t][rr]);
        }
    }
};

// A operands of one chunk: per group and token block 16 consecutive k of a token per lane - one register quad of int8
// codes, or two of halves (for the two matrix instructions of 32 k a group takes; the weights follow suit).
template <int TM, int FORM>
using ActRegs = v4i[2][TM][is_f16(FORM) ? 2 : 1];

// Resident int4 chunks: the codes enter the matrix instruction as q - z + 64 (positive bytes, one addition each; q - z takes an
// addition and an exclusive or), and its accumulator starts at the pattern of 1.5 * 2^23 less 64 times the sum of the token's group,
// which leaves the same integers.  The starts come from one matrix instruction per group when the activations arrive and stay in
// registers for all row tiles.
constexpr int kShift = 64;
template <int TM>
using Starts = v4i[2][TM];

__device__ __forceinline__ v4i shifted_start(v4i a)
{
    const v4i magic = {kMagicBits, kMagicBits, kMagicBits, kMagicBits};
    constexpr int minus = (int)(0x01010101u * (256 - kShift));
    return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, v4i{minus, minus, minus, minus}, magic, 0, 0, 0);
}

__device__ __forceinline__ v4i unpack_shifted(const Weights<kZp>& r, int h, uint32_t zsel)
{
    const uint32_t w0 = (uint32_t)(h ? r.w[0].z : r.w[0].x), w1 = (uint32_t)(h ? r.w[0].w : r.w[0].y);
    const uint32_t c4 = 0x01010101u * kShift - __builtin_amdgcn_perm(0u, (uint32_t)r.z, h ? zsel + 0x01010101u : zsel);
    return v4i{(int)((w0 & 0x0f0f0f0fu) + c4), (int)(((w0 >> 4) & 0x0f0f0f0fu) + c4), (int)((w1 & 0x0f0f0f0fu) + c4),
               (int)(((w1 >> 4) & 0x0f0f0f0fu) + c4)};
}

// One chunk: both groups of 16 weight rows against TM blocks of 16 tokens.  start: of shifted codes, or NULL.
template <int TM, int FORM>
__device__ __forceinline__ void contract(const Weights<FORM>& r, const ActRegs<TM, FORM>& a, uint32_t zsel,
                                         Pending<TM, FORM>& p, float (&acc)[TM][4], const Starts<TM>* start = nullptr)
{
    const v4i magic = {kMagicBits, kMagicBits, kMagicBits, kMagicBits};
    const v4i zero = {0, 0, 0, 0};
    const v4f zerof = {0.0f, 0.0f, 0.0f, 0.0f};
    const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const v4i onesh = {0x3c003c00, 0x3c003c00, 0x3c003c00, 0x3c003c00};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        Operand<FORM> o;
        if constexpr (FORM == kZp) o.q[0] = start ? unpack_shifted(r, h, zsel) : unpack<FORM>(r, h, zsel).q[0];
        else o = unpack<FORM>(r, h, zsel);
        const v4i b = o.q[0], b1 = o.q[is_f16(FORM) ? 1 : 0];
        Pending<TM, FORM> n;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            constexpr int X = is_f16(FORM) ? 1 : 0;
            const int tx = has_zero(FORM) ? 0 : t;
            if (is_f16(FORM)) {
                n.d[t] = __builtin_bit_cast(v4i, mfma_f16(a[h][t][X], b1, mfma_f16(a[h][t][0], b, zerof)));
                if (!has_zero(FORM)) n.xs[tx] = __builtin_bit_cast(v4i, mfma_f16(a[h][t][X], onesh, mfma_f16(a[h][t][0], onesh, zerof)));
            } else {
                n.d[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[h][t][0], b, FORM == kBytes ? zero : start ? (*start)[h][t] : magic, 0, 0, 0);
                if (!has_zero(FORM)) n.xs[tx] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[h][t][0], ones, zero, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            p.add(t, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
        n.s = h ? r.s.y : r.s.x;
        if (!has_zero(FORM)) n.mn = h ? r.mn.y : r.mn.x;
        p = n;
    }
}

// The activations of one slice of tokens.  A operand of group g, token block t: 16 consecutive k of one token per lane,
// from int8 rows or from the token blocks the fused call's quantizer writes ([group][block of 16 tokens][k block][token],
// the last block as narrow as its tokens): there a wave reads one contiguous piece per group and block, and the
// few-token kernels, which are bound by this traffic from L2 where K is long, gain a third (48 tokens, 3584 x 18944:
// 32 -> 22 us).  Chunk c of the packed axis meets chunk c % Cx of the row; an odd row's last chunk has one group only.
template <int TM, int FORM, bool BLOCKS>
struct Acts {
    static constexpr int E = is_f16(FORM) ? 2 : 1;     // bytes of a value
    static constexpr bool XCH = !BLOCKS && !is_f16(FORM);
    const RowExchange exchange;
    __amdgpu_buffer_rsrc_t x;
    int voff[TM];
    int Cx, odd_last, step;     // step: bytes from group to group
    __device__ __forceinline__ Acts(const void* __restrict__ xp, const Layout& L, int M, int m0, int lane)
        : exchange(lane), x(rsrc(xp, (int64_t)M * L.Kx * E)), Cx((int)L.Cx), odd_last((L.G & 1) ? (int)L.C - 1 : -1),
          step(BLOCKS ? M * 64 : 64 * E)
    {
        const int kb = XCH ? lane & 3 : lane >> 4, m = XCH ? lane >> 2 : lane & 15;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            const int first = m0 + t * 16, left = M - first, width = left < 16 ? left : 16;
            const int at = BLOCKS ? first * 64 + (kb * width + m) * 16 : (first + m) * (int)L.Kx * E + kb * 16 * E;
            voff[t] = m < width ? at : kOutOfRange;      // (tokens past M: zeros, no traffic)
        }
    }
    __device__ __forceinline__ void load(ActRegs<TM, FORM>& a, int c, bool have) const
    {
        const int cx = c >= Cx ? c - Cx : c;
        const int o0 = __builtin_amdgcn_readfirstlane(have ? 2 * cx * step : kOutOfRange);
        const int o1 = __builtin_amdgcn_readfirstlane(have && c != odd_last ? (2 * cx + 1) * step : kOutOfRange);
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                a[0][t][e] = __builtin_amdgcn_raw_buffer_load_b128(x, voff[t] + e * 16, o0, 0);
                a[1][t][e] = __builtin_amdgcn_raw_buffer_load_b128(x, voff[t] + e * 16, o1, 0);
            }
    }
    // what load brought -> the operands
    __device__ __forceinline__ void arrange(ActRegs<TM, FORM>& a) const
    {
        if (!XCH) return;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < TM; ++t) exchange(a[h][t][0]);
    }
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sum of the KS waves' partial results of a row tile and its output, token block t by wave (t + turn) % KS - the turn
// passes on from tile to tile, so that the same waves are not always the late ones.
template <int TM>
struct Output {
    __amdgpu_buffer_rsrc_t y;
    const float* sx;     // scales of the slice's tokens, in LDS
    int ks, KS, lane, m0, N;
    bool out16;
    __device__ __forceinline__ Output(float* __restrict__ yp, const float* lds_sx, const Layout& L, int M, int m0_, int ks_,
                                      int KS_, int lane_)
        : y(rsrc(yp, (int64_t)M * L.N * (L.out16 ? 2 : 4))), sx(lds_sx), ks(ks_), KS(KS_), lane(lane_), m0(m0_),
          N((int)L.N), out16(L.out16)
    {
    }
    // Requests the slice's scales (first wave; a lane per token, tokens past M: zeros), to be stored before a barrier.
    static __device__ __forceinline__ float fetch_sx(const float* __restrict__ sxp, int M, int m0, int lane)
    {
        if (!sxp) return 1.0f;      // (fp16 activations have no scales)
        return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc(sxp, (int64_t)M * 4), (m0 + lane) * 4, 0, 0));
    }
    __device__ __forceinline__ void store(const float4* part, int turn, int64_t tile, float bias) const
    {
        for (int t = ks >= turn ? ks - turn : ks - turn + KS; t < TM; t += KS) {
            float4 v = part[t * 64 + lane];
            for (int j = 1; j < KS; ++j) {
                const float4 p = part[(j * TM + t) * 64 + lane];
                v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
            }
            const float o[4] = {v.x, v.y, v.z, v.w};
            const int mt = t * 16 + (lane >> 4) * 4;
            const float4 s4 = *reinterpret_cast<const float4*>(sx + mt);
            const float s[4] = {s4.x, s4.y, s4.z, s4.w};
            const int n = (int)tile * kTileN + (lane & 15);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float f = fmaf(o[r], s[r], bias);
                const int at = (m0 + mt + r) * N + n;   // tokens past M: past the end of y, dropped
                if (out16) {
                    const _Float16 h = (_Float16)f;
                    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(short, h), y, at * 2, 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(f), y, at * 4, 0, 0);
                }
            }
        }
    }
};

// Chunks of a wave with shifted codes: as many as the registers hold starts of (8 TM each) without spilling.  A row tile is 179 vector
// instructions of a wave instead of 214 (one block of tokens, four chunks), 243 instead of 275 (two), 325 instead of 341 (three); 24 tokens of
// 28672 x 4096 19.5 -> 19.2 us, 40 of 37888 x 3584 26.2 -> 25.8, 9 of 37888 x 3584 19.2 -> 18.9.
constexpr int shifted_chunks(int tm, int nch, int form)
{
    if (form != kZp || tm * nch == 16 || (tm == 3 && nch == 2)) return 0;
    return tm == 3 ? 2 : nch;
}

template <int TM, int NCH, int FORM, int MAXW, bool BLOCKS>
__global__ __launch_bounds__(MAXW * 64) void few_resident_kernel(const uint8_t* __restrict__ packed, Layout L, int M,
                                                                const void* __restrict__ xq,
                                                                const float* __restrict__ sx,
                                                                const float* __restrict__ bias, float* __restrict__ y)
{
    extern __shared__ __align__(16) float4 lds_part[];   // [2][KS][TM][64], then the tokens' scales
    const int KS = blockDim.x >> 6;
    float* const lds_sx = reinterpret_cast<float*>(lds_part + 2 * KS * TM * 64);
    const int lane = threadIdx.x & 63;
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15;
    const uint32_t zsel = (row & 1) * 0x02020202u;
    const int C = (int)L.C;
    const int c0 = C * ks / KS, own = C * (ks + 1) / KS - c0;   // 1 .. NCH chunks
    const int m0 = blockIdx.y * (16 * TM);

    const Output<TM> out(y, lds_sx, L, M, m0, ks, KS, lane);
    const float sx_own = out.fetch_sx(sx, M, m0, lane);
    const __amdgpu_buffer_rsrc_t rs_bias = rsrc(bias, bias ? L.N * 4 : 0);
    const Acts<TM, FORM, BLOCKS> acts(xq, L, M, m0, lane);
    ActRegs<TM, FORM> a[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) acts.load(a[u], c0 + u, u < own);

    int64_t tile = blockIdx.x;
    Weights<FORM> cur[NCH];
    const TileBuffers<FORM> first(packed, L, tile);
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
        cur[u] = first.load(u < own ? c0 + u : C, lane, row);
        __builtin_amdgcn_sched_barrier(0);      // (the order of the loop: the waits are counts)
    }
    auto bias_of = [&](int64_t t) {
        return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_bias, ((int)t * kTileN + row) * 4, 0, 0));
    };
    float b = bias_of(tile);
    asm volatile("" ::: "memory");              // (all requested here: else the weights sink into the loop, behind the activations)
#pragma unroll
    for (int u = 0; u < NCH; ++u) acts.arrange(a[u]);
    constexpr int SH = shifted_chunks(TM, NCH, FORM);
    Starts<TM> start[SH > 0 ? SH : 1];
#pragma unroll
    for (int u = 0; u < SH; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < TM; ++t) start[u][h][t] = shifted_start(a[u][h][t][0]);

    int buf = 0, turn = 0;
    auto row_tile = [&](auto refill) {
        constexpr bool REFILL = decltype(refill)::value;
        const float b_next = REFILL ? bias_of(tile + gridDim.x) : 0.0f;
        const TileBuffers<FORM> next(packed, L, REFILL ? tile + gridDim.x : tile);
        float acc[TM][4];
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) acc[t][rr] = 0.0f;
        Pending<TM, FORM> pend;
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
            // A chunk that is not the wave's own is passed over, and the refills go on: without the branches the compiler moves the
            // chunks' scales together, at the top of the loop, and waits there for all but the last two loads (24 tokens of 28672 x 4096
            // 20.8 -> 19.2 us, 9 of 37888 x 3584 with fp16 activations 21.0 -> 19.4).  Four blocks of the other forms spill with
            // them; there, and in the last row tile, the chunk is zero.
            if (u == 0 || !REFILL || (TM * NCH == 16 && FORM != kZp) || u < own)
                contract<TM, FORM>(cur[u], a[u], zsel, pend, acc, u < SH ? &start[u < SH ? u : 0] : nullptr);
            if (REFILL) {
                cur[u] = next.load(u < own ? c0 + u : C, lane, row);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        float4* part = lds_part + buf * KS * TM * 64;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            pend.add(t, acc);
            part[(ks * TM + t) * 64 + lane] = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
        }
        if (ks == 0) lds_sx[lane] = sx_own;
        // One barrier per row tile: the buffer written now was read two tiles ago, before the barrier in between.
        lds_barrier();
        out.store(part, turn, tile, b);
        turn = turn + TM < KS ? turn + TM : 0;
        b = b_next;
        buf ^= 1;
        tile += gridDim.x;
    };
    // (The grid has no more workgroups than there are row tiles.)  The last row tile requests nothing and has no branches: with both it
    // cost the launches of one row tile per workgroup, or little more, up to 9 % over the straight loop before them - requests past the
    // matrix bring nothing but take their turn, and the stores wait for them.  us, straight loop / branches / branches, last tile apart:
    // 9 tokens of 10720 x 2240, float minima 8.2 / 8.9 / 6.8; 5 of 10864 x 1152, nibble planes 8.2 / 8.9 / 6.8; 5 of 4032 x 2688,
    // bytes 5.3 / 5.5 / 5.2; 31 of 5056 x 3584, float minima 7.7 / 7.9 / 7.5; over 560 shapes of 2 - 64 tokens 1 / 0.99 / 0.953,
    // with fp16 activations 1 / 0.984 / 0.971.
    while (tile + gridDim.x < L.T) row_tile(std::true_type{});
    row_tile(std::false_type{});
}

template <int TM, int DEPTH, int FORM, int MAXW, bool BLOCKS>
__global__ __launch_bounds__(MAXW * 64) void few_stream_kernel(const uint8_t* __restrict__ packed, Layout L, int M,
                                                              const void* __restrict__ xq,
                                                              const float* __restrict__ sx,
                                                              const float* __restrict__ bias, float* __restrict__ y)
{
    extern __shared__ __align__(16) float4 lds_part[];   // [KS][TM][64], then the tokens' scales
    const int KS = blockDim.x >> 6;
    float* const lds_sx = reinterpret_cast<float*>(lds_part + KS * TM * 64);
    const int lane = threadIdx.x & 63;
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15;
    const uint32_t zsel = (row & 1) * 0x02020202u;
    const int C = (int)L.C;
    const int c0 = C * ks / KS, c1 = C * (ks + 1) / KS;   // at least one chunk
    const int m0 = blockIdx.y * (16 * TM);
    const int64_t tile = blockIdx.x;

    const Output<TM> out(y, lds_sx, L, M, m0, ks, KS, lane);
    const float sx_own = out.fetch_sx(sx, M, m0, lane);
    const float b = __int_as_float(
        __builtin_amdgcn_raw_buffer_load_b32(rsrc(bias, bias ? L.N * 4 : 0), ((int)tile * kTileN + row) * 4, 0, 0));
    const Acts<TM, FORM, BLOCKS> acts(xq, L, M, m0, lane);
    const TileBuffers<FORM> weights(packed, L, tile);
    ActRegs<TM, FORM> a[DEPTH];
    Weights<FORM> cur[DEPTH];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        const int c = c0 + u;
        cur[u] = weights.load(c < c1 ? c : C, lane, row);
        acts.load(a[u], c, c < c1);
        __builtin_amdgcn_sched_barrier(0);      // (the order of the loop: the waits are counts)
    }
    float acc[TM][4];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) acc[t][rr] = 0.0f;
    Pending<TM, FORM> pend;
    int c = c0;
    do {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            // (past the wave's chunks nothing is contracted, but the loads go on - outside the buffers, so that they cost
            // nothing: the waits stay counts)
            if (u == 0 || c + u < c1) {
                acts.arrange(a[u]);
                contract<TM, FORM>(cur[u], a[u], zsel, pend, acc);
            }
            const int next = c + u + DEPTH;
            cur[u] = weights.load(next < c1 ? next : C, lane, row);
            acts.load(a[u], next, next < c1);
            __builtin_amdgcn_sched_barrier(0);
        }
        c += DEPTH;
    } while (c < c1);
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        pend.add(t, acc);
        lds_part[(ks * TM + t) * 64 + lane] = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
    }
    if (ks == 0) lds_sx[lane] = sx_own;
    lds_barrier();
    out.store(lds_part, 0, tile, b);
}

struct FewPlan {
    bool resident;
    int nch;     // chunks of a wave held in registers (resident form)
    int ks;      // waves of a workgroup
};

// Waves a CU holds, by registers: sixteen (128 registers each) or eight (256); 0: the operands do not fit.
constexpr int resident_waves(int tm, int nch, int form)
{
    if (is_f16(form)) {     // 16 TM registers per chunk
        if (tm * nch > 8) return 0;
        return tm * nch <= 2 || (tm * nch <= 4 && form == kZpF16 && tm == 2) ? 16 : 8;
    }
    return tm == 1 || (nch == 2 && (tm == 2 || (tm == 3 && form == kZp))) ? 16 : 8;
}
constexpr int stream_waves(int tm, int form) { return tm == 1 && !(form == kMinF16) ? 16 : 8; }
// chunks in flight in the streaming form: what the registers hold without spilling
constexpr int stream_depth(int tm, int form) { return is_f16(form) ? (tm == 1 ? 3 : tm <= 2 ? 4 : 2) : (tm <= 3 ? 4 : 3); }

// Waves that share a row tile in the streaming form.  One block of tokens: the chunks a wave takes one after the other are
// read ahead, further waves on the tile bring no more bytes in flight at once than that, and each adds its partial sums -
// four, eight where half the CUs have no tile.  Two tokens with 4 / 8 / 16 waves: 4096 x 14336 int4 9.9 / 10.8 / 11.1 us,
// float minimum 9.6 / 10.4 / 11.8, int8 nibble planes 16.4 / 16.9 / 19.2; 5120 x 13824 float minimum 15.4 / 18.0 / 21.5;
// 1536 x 8960 (96 tiles) int4 7.2 / 6.5 / 7.6.  (The kernel stays built for sixteen: two to four workgroups on a CU.)
int stream_split(const Layout& L, int tm, int form)
{
    if (tm > 1 || is_f16(form)) return stream_waves(tm, form);
    return 2 * L.T < num_cus() ? 8 : 4;
}

FewPlan few_plan(const Layout& L, int tm, int form)
{
    FewPlan p{};
    const int64_t C = L.C;
    auto fits = [&](int nch) { return (C + nch - 1) / nch <= resident_waves(tm, nch, form); };
    // short rows of layers with few row tiles: two chunks per wave, twice the waves
    int nch = 4;
    if (L.T <= 2 * (int64_t)num_cus() && (C + 1) / 2 <= 8) nch = 2;
    if (!fits(nch) && fits(2)) nch = 2;
    int64_t ks = (C + nch - 1) / nch;
    // (One block of tokens, one row tile per workgroup and more than eight waves on it: resident operands serve one tile, and
    // every wave adds its partial sums.  2 - 16 tokens, resident / streaming / the kernel before: 4096 x 4096 int8 nibble planes
    // 10.0 / 8.7 / 9.3 us, 1728 x 4096 9.2 / 8.5 / 8.1; 4096 x 8192 float minimum 1.15 : 1 : 1.10, int4 1.10 : 1 : 1.25; from
    // 4608 columns on - the second tile - the other way round, 0.93 : 1 and less.)
    const bool one_tile = tm == 1 && !is_f16(form) && ks > 8 && L.T <= num_cus();
    p.resident = fits(nch) && !one_tile;
    if (const char* e = debug_option(kDbgSkinnyStaged)) p.resident = fits(nch) && e[0] == '1';   // tests
    if (!p.resident) {
        ks = stream_split(L, tm, form);
        if (C < ks) ks = C;
    }
    if (const char* e = debug_option(kDbgDecodeKsplit)) {   // tests and tuning: force the split
        const int v = atoi(e);
        if (v >= 1 && v <= stream_waves(tm, form) && v <= C) {
            // (the resident kernel is built for its own number of waves, which may be the smaller one)
            p.resident = p.resident && (C + v - 1) / v <= nch && v <= resident_waves(tm, nch, form);
            ks = v;
        }
    }
    p.nch = nch;
    p.ks = (int)ks;
    return p;
}

template <int TM, int FORM, bool BLOCKS>
int launch_form(const uint8_t* packed, const Layout& L, int M, const void* xq, const float* sx, const float* bias, float* y,
                hipStream_t st)
{
    const FewPlan p = few_plan(L, TM, FORM);
    const unsigned slices = (unsigned)((M + 16 * TM - 1) / (16 * TM));
    if (p.resident) {
        // as many workgroups as the chip holds at once
        const int per_cu = resident_waves(TM, p.nch, FORM) / p.ks;
        const int64_t slots = (int64_t)num_cus() * (per_cu > 0 ? per_cu : 1);
        const int64_t grid = L.T < slots ? L.T : slots;
        const size_t smem = (size_t)2 * p.ks * TM * 64 * 16 + 256;
        static thread_local int allowed[2] = {-1, -1};
        auto go = [&](auto kern, int& dev) -> int {
            if (int s = allow_large_lds(kern, smem, dev)) return s;
            hipLaunchKernelGGL(kern, dim3((unsigned)grid, slices), dim3(64 * p.ks), smem, st, packed, L, M, xq, sx, bias, y);
            MNNQ_HIP_TRY(hipGetLastError());
            return MNNQ_OK;
        };
        if constexpr (resident_waves(TM, 4, FORM) != 0)
            if (p.nch == 4) return go(few_resident_kernel<TM, 4, FORM, resident_waves(TM, 4, FORM), BLOCKS>, allowed[1]);
        return go(few_resident_kernel<TM, 2, FORM, resident_waves(TM, 2, FORM), BLOCKS>, allowed[0]);
    }
    const size_t smem = (size_t)p.ks * TM * 64 * 16 + 256;
    hipLaunchKernelGGL((few_stream_kernel<TM, stream_depth(TM, FORM), FORM, stream_waves(TM, FORM), BLOCKS>),
                       dim3((unsigned)L.T, slices), dim3(64 * p.ks), smem, st, packed, L, M, xq, sx, bias, y);
    MNNQ_HIP_TRY(hipGetLastError());
    return MNNQ_OK;
}

// Token blocks per workgroup: all of them up to 64 tokens, beyond that an even share of at most four.
int blocks_of(int64_t M)
{
    const int n = (int)(M + 15) / 16;
    const int slices = (n + 3) / 4;
    return (n + slices - 1) / slices;
}

template <int FORM, bool BLOCKS>
int launch_tokens(const uint8_t* packed, const Layout& L, int M, const void* xq, const float* sx, const float* bias, float* y,
                  hipStream_t st)
{
    switch (blocks_of(M)) {
        case 1: return launch_form<1, FORM, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
        case 2: return launch_form<2, FORM, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
        case 3: return launch_form<3, FORM, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
        default: return launch_form<4, FORM, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
    }
}

}  // namespace

// int8 activations, from rows or token blocks (the same line for both, so that the fused call stays bit for bit the two calls).
// Up to 16 tokens always.  Up to 64 tokens:
//   * where the activations stay in registers, but for the tallest operands (49 tokens and more) on layers of many row tiles.
//     64 tokens, the fused call, few-token / the GEMM behind it: int4 from six tiles per CU where a row takes three or five
//     waves of four chunks, which leave a quarter of a CU's eight empty or more (28672 x 1152 16.2 / 14.5, x 2560
//     23.3 / 21.2; four, six and seven waves 28672 x 2048 19.1 / 19.4, 24576 x 3072 22.7 / 23.5, 28672 x 3584
//     26.2 / 28.5 us); with a float minimum, twice the matrix instructions, from three (37888 x 3584 39.4 / 38.5, 25424 x
//     2304 27.1 / 21.1; 8192 x 2048 9.1 / 9.8); never in the byte form, half the unpacking (28672 x 4096 33.2 / 36.9), nor
//     with the matrix-core plane, whose GEMM has tiles of 64 tokens for few row tiles only (28672 x 4096 27.6 / 32.6,
//     37888 x 3584 33.7 / 49.7, 40960 x 2304 30.7 / 33.7 us);
//   * where both operands stream, while the row tiles are one round of workgroups (a CU holds one): 33 tokens, few-token /
//     K-split / tiled, int4 4096 x 14336 (256 tiles) 16.1 / 16.7 / 26.0, 5120 x 5120 (320) 17.9 / 8.4 / 16.6, 13824 x 5120
//     (864) 34.4 / 13.6 / 18.5 us;
//   * int8 nibble planes run twice the chunks here, which the tiled GEMM - the only other kernel - merges: what decides is
//     the time of the rounds in us, fitted to 330 shapes (17 - 64 tokens; few-token / tiled, 33 tokens: 8192 x 8192 34 / 48,
//     13824 x 5120 50 / 53, 28672 x 4096 75 / 46, 37888 x 3584 100 / 67).
// Up to 128 tokens, in two slices, where the slices of all row tiles are one round of workgroups and the rows not too long
// (row tiles x chunks up to 7000; 128 tokens, few-token / K-split / tiled: 2048 x 1536 (128 tiles) 4.7 / 5.3 / 8.5, 1104 x 4096
// 7.7 / 7.3 / 14.4, 1536 x 8960 13.0 / 11.4 / 19.7, with the quantizer's call before 15.8 / 16.1; beyond one round 2560 x 2560
// (160 tiles) 11.7 / 7.8 / 10.8, 3584 x 3584 13.6 / 8.9 / 13.2 us; nibble planes, tiled only, 2560 x 2560 17.4 / - / 29.3).
bool skinny_wanted(const Layout& L, int64_t M)
{
    constexpr int64_t kFewTokens = 64, kTwoSlices = 128, kSmallCells = 7000;
    if (debug_option(kDbgNoSkinny)) return false;
    if (M <= 16) return true;
    if (debug_option(kDbgPrefillTile) || debug_option(kDbgPrefill6Plan)) return false;   // tests and tuning: the tiled GEMMs
    const int64_t cus = num_cus();
    const bool planes8 = L.mode == MNNQ_W8_MIN_FLOAT && !L.native8;
    if (M > kFewTokens) return M <= kTwoSlices && L.T * L.C <= kSmallCells && (planes8 || 2 * L.T <= cus);
    if (debug_option(kDbgSkinnyStaged) || debug_option(kDbgDecodeKsplit)) return true;   // tests and tuning
    const int tm = blocks_of(M), form = form_of(L, false);
    const FewPlan plan = few_plan(L, tm, form);
    if (plan.resident) {
        if (tm < 4 || form == kBytes || L.plane) return true;
        if (form == kMin) return L.T < (planes8 ? 6 : 3) * cus;
        return L.T < 6 * cus || (plan.ks != 3 && plan.ks != 5);
    }
    if (!planes8) return L.T <= cus;
    const float C = (float)L.Cx;
    const int64_t tiles = (L.T + 7) / 8, rounds = (tiles + cus - 1) / cus;      // of 128 x 128
    const bool halved = 2 * tiles <= cus && L.Cx >= 64 && !L.out16;             // (K split over two workgroups)
    const float tiled = rounds == 1 ? 5.6f + (halved ? 0.6f : 1.2f) * C : (float)rounds * (3.4f + 1.07f * C);
    const float few = (float)((L.T + cus - 1) / cus) * (4.4f + (0.033f + 0.0715f * (float)tm) * C);
    return few <= tiled;
}

template <bool BLOCKS>
static int launch_int8(const uint8_t* packed, const Layout& L, int M, const int8_t* xq, const float* sx, const float* bias,
                       float* y, hipStream_t st)
{
    if (L.native8) return launch_tokens<kBytes, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
    if (L.minf) return launch_tokens<kMin, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
    return launch_tokens<kZp, BLOCKS>(packed, L, M, xq, sx, bias, y, st);
}

int launch_skinny(const uint8_t* packed, const Layout& L, int64_t M, const int8_t* xq, bool blocks, const float* sx,
                  const float* bias, float* y, hipStream_t st)
{
    return blocks ? launch_int8<true>(packed, L, (int)M, xq, sx, bias, y, st)
                  : launch_int8<false>(packed, L, (int)M, xq, sx, bias, y, st);
}

// fp16 activations.  Up to 16 tokens always.  Up to 64 by the time expected of either kernel, where the activation operands
// stay in registers: the few-token kernel takes fixed + chunk C + n (tile + tile_chunk C) with n row tiles on the busiest CU, the
// GEMM with K split over waves whole rounds of 64-column tiles (its formula, fitted up to 2048 tokens, is 10 % short here; us,
// few-token / K-split: int4 32 tokens of 7040 x 1984 11.6 / 7.3, 24 of 16448 x 4096 - a second round - 17.9 / 23.2, 56 of
// 19264 x 1664 16.9 / 20.3; float minimum 54 of 10480 x 1088 12.7 / 15.9, 24 of 36224 x 3840 32.0 / 37.7, 42 of 31888 x 1152
// 20.0 / 16.5).  Over 3000 shapes of 17 - 64 tokens that costs 0.3 % (int4) and 0.6 % (float minimum) against the better kernel;
// the time of 32 tokens and a limit on the cells beyond, fitted to int4, had cost 1.1 %, up to 29 % on float minima of short rows.
// Where the operands are streamed the K-split kernel wins (few-token : K-split at one row tile per CU, by tokens: int4 17
// 0.93, 18 1.03, 22 1.09; float minima 17 0.90, 18 0.96, 19 0.99, 20 1.01, 24 1.08, 32 1.18; at more tiles 1.7 - 3) but for the first of a second block of
// tokens, whose 16-row tiles there are nearly empty.  More tokens only on the smallest layers (68 of 1152 x 1024 6.1 / 7.5, 77 of 2800 x 2048 in
// two slices 14.3 / 7.2 us).
struct FewCost {
    float fixed, chunk, tile, tile_chunk;
};
constexpr FewCost kFewF16[2][3] = {      // [float minimum][blocks of 16 tokens, from two on]
    {{2.53f, 0.202f, 1.21f, 0.029f}, {2.62f, 0.327f, 1.19f, 0.023f}, {2.49f, 0.428f, 1.37f, 0.025f}},
    {{2.48f, 0.212f, 1.18f, 0.046f}, {2.15f, 0.355f, 1.52f, 0.024f}, {2.27f, 0.42f, 1.8f, 0.02f}}};

bool skinny_f16_wanted(const Layout& L, int64_t M)
{
    if (debug_option(kDbgNoSkinny) || debug_option(kDbgPrefillTile)) return false;   // tests and tuning: the tiled GEMM
    if (M <= 16) return true;
    const int64_t cus = num_cus();
    if (M > 128) return false;
    if (!few_plan(L, blocks_of(M), form_of(L, true)).resident) return M <= (L.minf ? 19 : 17) && L.T <= cus;
    if (M > 64) return L.C <= 10 && L.T * L.C <= 600;
    const FewCost& f = kFewF16[L.minf ? 1 : 0][blocks_of(M) - 2];
    const float C = (float)L.C, n = (float)((L.T + cus - 1) / cus);
    return f.fixed + f.chunk * C + n * (f.tile + f.tile_chunk * C) <= 1.1f * ksplit_f16_us(L, M);
}

void describe_skinny(const Layout& L, int64_t M, bool f16, int32_t out[8])
{
    const int tm = blocks_of(M), form = form_of(L, f16);
    const FewPlan p = few_plan(L, tm, form);
    const int waves = p.resident ? resident_waves(tm, p.nch, form) : stream_waves(tm, form);
    out[0] = p.resident ? 1 : 2;
    out[1] = 16 * tm;
    out[2] = kTileN;
    out[3] = p.ks;
    out[4] = waves;
    out[5] = p.resident ? p.nch : 0;
}

int launch_skinny_f16(const uint8_t* packed, const Layout& L, int64_t M, const uint16_t* x16, const float* bias, float* y,
                      hipStream_t st)
{
    if (L.minf) return launch_tokens<kMinF16, false>(packed, L, (int)M, x16, nullptr, bias, y, st);
    return launch_tokens<kZpF16, false>(packed, L, (int)M, x16, nullptr, bias, y, st);
}

}  // namespace mnnq
