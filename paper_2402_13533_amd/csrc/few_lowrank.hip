// The factorised layer with at most 64 tokens: two launches forward, two backward.
//
//     launch 1   H = X A                     (forward)      launch 2   Y = H B
//     launch 1   dH = dY B^T                 (backward)     launch 2   dX = dH A^T,  dA = X^T dH,  dB = H^T dY
//
// The factors are read once and there are few operations, so what counts is the number of launches in the chain (an empty
// one takes 2.5 microseconds, and a call's host side 4 per launch) and, inside each, the trips to memory.  On the GEMM tiles the chain was
// nine launches: every product cut into slices, each with a launch that summed its slabs.  Here operands go from memory
// straight into registers, a wave's whole share of the reduction requested at once, and a byte permute per register pair
// transposes what is stored reduction-major; the eight waves of a workgroup split the reduction and meet in LDS.  A long reduction into
// the rank is cut further, over workgroups: the last slice to arrive at a tile (a ticket in the workspace header) adds the slabs in
// their order, which takes 2.6 microseconds where a launch of its own took 3.5 and a gap.  (Slabs added up by every workgroup of
// launch 2 instead: 7.0 + 7.0 microseconds against 8.2 + 5.3 at 16 tokens, r = 512, but 9.4 + 18 against 9.0 + 5.7 at 64.)
// GPU time of a layer, forward / backward, microseconds, before -> now: 4096 -> 512 -> 4096 at 16 tokens 15.7 / 24.0 -> 13.5 / 16.5,
// at 64 21.2 / 34.0 -> 15 / 18; 1664 -> 80 -> 800 at 3 11.9 / 15.5 -> 11.5 / 11; 4096 -> 1024 -> 11008 at 64 29 / 41 -> 24 / 38 (67 MB of factors and
// gradients in 62 microseconds).
#include "few_lowrank.h"
#include "gemm_ring.h"
#include "profile.h"

namespace fhpc {
namespace few {

using ring::bf16x8;
using ring::f32x4;
using ring::u32x2;
using ring::u32x4;

constexpr int WAVES = 8, NT = WAVES * 64;
constexpr int STEP = 32;                      // reduction of a matrix instruction
constexpr int IN_COLS = 32;                   // ranks of a workgroup of the rank products
constexpr uint32_t NONE = 0x80000000u;        // an offset beyond any operand: reads as zeros
constexpr int SC1 = 16;                       // cache policy of accesses that other compute units' accesses must meet
constexpr int ahead(int v, int mt) { return v * mt == 2 ? 8 : v * mt == 4 ? 6 : 4; }      // steps a wave has in flight
constexpr int red_floats(int v, int mt) { return WAVES * 16 * mt * (16 * v + 4); }

struct Product {
    const uint16_t* left;   // bf16 [M][K]
    const uint16_t* right;  // bf16 [K][N] or [N][K]
    uint16_t* out;          // bf16 [M][N]
    float* part;            // slabs of the slices, a workgroup's 16 MT x 32 floats contiguous: [row block][tile][slice]
    uint32_t* tickets;      // one per [row block][tile]
    int M, N, K, chunk, tiles, splits, items;
};
// out[b][a] = sum_m P[m][a] Q[m][b], a < na, b < nb
struct Outer {
    const uint16_t *p, *q;
    float* out;
    int na, nb, tiles_a, tiles;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
// 16-bit halves (low or high) of eight words as one operand
__device__ __forceinline__ bf16x8 halves(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t a4, uint32_t a5, uint32_t a6, uint32_t a7,
                                         bool high)
{
    const uint32_t pick = high ? 0x07060302u : 0x05040100u;
    const u32x4 w = {__builtin_amdgcn_perm(a1, a0, pick), __builtin_amdgcn_perm(a3, a2, pick), __builtin_amdgcn_perm(a5, a4, pick),
                     __builtin_amdgcn_perm(a7, a6, pick)};
    return __builtin_bit_cast(bf16x8, w);
}

// One workgroup's part of a product: 16 MT rows x 16 V columns x a slice of the reduction.
template <bool KC, int V, int MT>
__device__ __forceinline__ void product_body(const Product& a, int item, float* red, uint32_t* s_ticket)
{
    constexpr int ROWS = 16 * MT, COLS = 16 * V, LD = COLS + 4, AHEAD = ahead(V, MT);
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row_block = item / (a.tiles * a.splits), in_block = item - row_block * a.tiles * a.splits;
    const int split = in_block / a.tiles, tile = in_block - split * a.tiles;
    const int n0 = tile * COLS, m0 = row_block * ROWS;
    const int kb = split * a.chunk, ke = kb + a.chunk < a.K ? kb + a.chunk : a.K;
    const int steps = (ke - kb + STEP - 1) / STEP, per = (steps + WAVES - 1) / WAVES;
    const int k0 = kb + wave * per * STEP;
    const __amdgpu_buffer_rsrc_t rR = rsrc(a.right, (int64_t)a.K * a.N * 2), rL = rsrc(a.left, (int64_t)a.M * a.K * 2);

    // Step u of the wave: reduction indices k0 + 32 u + 8 g .. + 7 of this lane, inside or outside as a whole.
    struct Right {
        uint32_t w[4 * V];      // eight reduction rows x V columns, or V columns x eight of the reduction
    };
    auto fetch_right = [&](Right& x, int u) __attribute__((always_inline)) {
        const int k = k0 + STEP * u + 8 * g;
        const bool in = u < per && k < ke;
        if constexpr (KC) {
#pragma unroll
            for (int i = 0; i < V; i++) {
                const int n = n0 + 16 * i + c;
                const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rR, (in && n < a.N) ? ((uint32_t)n * a.K + k) * 2u : NONE, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; e++) x.w[4 * i + e] = t[e];
            }
        } else {
            const int n = n0 + V * c;
            const uint32_t at = ((uint32_t)k * a.N + n) * 2u;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t o = (in && n < a.N) ? at + (uint32_t)e * a.N * 2u : NONE;
                if constexpr (V == 2) {
                    x.w[e] = __builtin_amdgcn_raw_buffer_load_b32(rR, o, 0, 0);
                } else {
                    const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rR, o, 0, 0);
                    x.w[e] = t.x;
                    x.w[8 + e] = t.y;
                }
            }
        }
    };
    auto operand = [&](const Right& x, int i) __attribute__((always_inline)) -> bf16x8 {
        if constexpr (KC) return __builtin_bit_cast(bf16x8, (u32x4){x.w[4 * i], x.w[4 * i + 1], x.w[4 * i + 2], x.w[4 * i + 3]});
        else {
            const int b = i / 2 * 8;
            return halves(x.w[b], x.w[b + 1], x.w[b + 2], x.w[b + 3], x.w[b + 4], x.w[b + 5], x.w[b + 6], x.w[b + 7], i & 1);
        }
    };
    auto fetch_left = [&](u32x4 (&x)[MT], int u) __attribute__((always_inline)) {
        const int k = k0 + STEP * u + 8 * g;
#pragma unroll
        for (int t = 0; t < MT; t++) {
            const int m = m0 + 16 * t + c;
            x[t] = __builtin_amdgcn_raw_buffer_load_b128(rL, (u < per && k < ke && m < a.M) ? ((uint32_t)m * a.K + k) * 2u : NONE, 0, 0);
        }
    };

    f32x4 acc[MT][V];
#pragma unroll
    for (int t = 0; t < MT; t++)
#pragma unroll
        for (int i = 0; i < V; i++) acc[t][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    Right rv[AHEAD];
    u32x4 lv[AHEAD][MT];
#pragma unroll
    for (int u = 0; u < AHEAD; u++) {
        fetch_right(rv[u], u);
        fetch_left(lv[u], u);
    }
    for (int u0 = 0; u0 < per; u0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; u++) {
            if (u0 + u >= per) break;
#pragma unroll
            for (int i = 0; i < V; i++) {
                const bf16x8 b = operand(rv[u], i);
#pragma unroll
                for (int t = 0; t < MT; t++)
                    acc[t][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, lv[u][t]), b, acc[t][i], 0, 0, 0);
            }
            if (u0 + u + AHEAD < per) {
                fetch_right(rv[u], u0 + u + AHEAD);
                fetch_left(lv[u], u0 + u + AHEAD);
            }
        }
    }
    // The waves' sums meet in LDS.  A lane holds rows 4 g .. 4 g + 3 of column V c + i (right reduction-major) or 16 i + c.
#pragma unroll
    for (int t = 0; t < MT; t++)
#pragma unroll
        for (int i = 0; i < V; i++)
#pragma unroll
            for (int v = 0; v < 4; v++) red[(wave * ROWS + 16 * t + 4 * g + v) * LD + (KC ? 16 * i + c : V * c + i)] = acc[t][i][v];
    __syncthreads();
    constexpr int QUADS = ROWS * COLS / 4;
    const auto sum_waves = [&](int e) __attribute__((always_inline)) -> f32x4 {        // four columns of a row
        const float* const at = red + e / (COLS / 4) * LD + e % (COLS / 4) * 4;
        f32x4 x = *reinterpret_cast<const f32x4*>(at);
#pragma unroll
        for (int w = 1; w < WAVES; w++) x += *reinterpret_cast<const f32x4*>(at + w * (ROWS * LD));
        return x;
    };
    const auto store = [&](int e, const f32x4& x) __attribute__((always_inline)) {
        const int m = m0 + e / (COLS / 4), n = n0 + e % (COLS / 4) * 4;
        const u32x2 p = {ring::pack_bf16(x.x, x.y), ring::pack_bf16(x.z, x.w)};
        if (m < a.M && n < a.N) *reinterpret_cast<u32x2*>(a.out + (int64_t)m * a.N + n) = p;          // (N is a multiple of 8)
    };
    if (a.splits == 1) {
#pragma unroll
        for (int e0 = 0; e0 < QUADS; e0 += NT) {
            const int e = e0 + threadIdx.x;
            if (QUADS >= NT || e < QUADS) store(e, sum_waves(e));
        }
        return;
    }
    if constexpr (QUADS > NT) return;                       // (not launched: the tiles that are cut have at most NT quads)
    else {
    // The slice's sums go to its slab; the last slice to arrive adds the slabs up, in their order.
    const int own = row_block * a.tiles + tile;
    const __amdgpu_buffer_rsrc_t rP = rsrc(a.part + (int64_t)own * a.splits * (ROWS * COLS), (int64_t)a.splits * (ROWS * COLS) * 4);
    const int e = threadIdx.x % QUADS;
    if ((int)threadIdx.x < QUADS)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, sum_waves(e)), rP, (uint32_t)(split * (ROWS * COLS) + 4 * e) * 4u, 0, SC1);
    FHPC_WAIT_VM(0);                                        // (the slab is where every compute unit finds it before the ticket is drawn)
    __syncthreads();
    if (threadIdx.x == 0) *s_ticket = __hip_atomic_fetch_add(a.tickets + own, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*s_ticket != (uint32_t)(a.splits - 1)) return;
    if (threadIdx.x == 0) __hip_atomic_store(a.tickets + own, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    constexpr int SETS = NT / QUADS;                        // threads that share an output quad
    const int set = threadIdx.x / QUADS;
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = set; s0 < a.splits; s0 += 4 * SETS) {
        u32x4 y[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int s = s0 + i * SETS;
            y[i] = __builtin_amdgcn_raw_buffer_load_b128(rP, s < a.splits ? (uint32_t)(s * (ROWS * COLS) + 4 * e) * 4u : NONE, 0, SC1);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) x += __builtin_bit_cast(f32x4, y[i]);
    }
    if constexpr (SETS > 1) {
        *reinterpret_cast<f32x4*>(red + threadIdx.x * 4) = x;
        __syncthreads();
#pragma unroll
        for (int i = 1; i < SETS; i++) x += *reinterpret_cast<const f32x4*>(red + ((i * QUADS + e) * 4));
    }
    if ((int)threadIdx.x < QUADS) store(e, x);
    }
}

template <bool KC, int MT>
__global__ __launch_bounds__(NT) void few_in_kernel(Product a)
{
    __shared__ __attribute__((aligned(16))) float red[red_floats(2, MT)];
    __shared__ uint32_t s_ticket;
    product_body<KC, 2, MT>(a, ring::xcd_contiguous((int)blockIdx.x, (int)gridDim.x), red, &s_ticket);
}

// A wave's 64 x 64 tile of an outer product over the tokens.  A lane reads eight consecutive tokens of four columns of either
// operand; a byte permute per register pair makes them matrix operands, whose reduction index is the token.  Bound by writing the
// gradients.  Lane c takes column block 4 (c % 4) + c / 4 of P, so that the four lane groups of a store write 64 contiguous bytes
// (blocks in lane order, 16 bytes in every 64: 16 MB of gradients 11.4 microseconds against 7.9).
__device__ __forceinline__ void outer_body(const Outer& o, int t, int M)
{
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    const int a0 = t % o.tiles_a * 64, b0 = t / o.tiles_a * 64;
    const __amdgpu_buffer_rsrc_t rp = rsrc(o.p, (int64_t)M * o.na * 2), rq = rsrc(o.q, (int64_t)M * o.nb * 2);
    const int ca = a0 + 4 * (4 * (c & 3) + (c >> 2)), cb = b0 + 4 * c;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int m0 = 0; m0 < M; m0 += STEP) {
        u32x2 p[8], q[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int m = m0 + 8 * g + e;
            p[e] = __builtin_amdgcn_raw_buffer_load_b64(rp, (m < M && ca < o.na) ? ((uint32_t)m * o.na + ca) * 2u : NONE, 0, 0);
            q[e] = __builtin_amdgcn_raw_buffer_load_b64(rq, (m < M && cb < o.nb) ? ((uint32_t)m * o.nb + cb) * 2u : NONE, 0, 0);
        }
        bf16x8 fp[4], fq[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            fp[i] = halves(p[0][i / 2], p[1][i / 2], p[2][i / 2], p[3][i / 2], p[4][i / 2], p[5][i / 2], p[6][i / 2], p[7][i / 2], i & 1);
            fq[i] = halves(q[0][i / 2], q[1][i / 2], q[2][i / 2], q[3][i / 2], q[4][i / 2], q[5][i / 2], q[6][i / 2], q[7][i / 2], i & 1);
        }
#pragma unroll
        for (int i = 0; i < 4; i++)
#pragma unroll
            for (int j = 0; j < 4; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp[i], fq[j], acc[i][j], 0, 0, 0);
    }
    // register v of acc[i][j]: a = a0 + 4 (4 v + g) + i, b = b0 + 4 c + j
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int b = cb + j;
        if (b >= o.nb) break;
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int at = a0 + 4 * (4 * v + g);
            if (at < o.na) *reinterpret_cast<f32x4*>(o.out + (int64_t)b * o.na + at) = f32x4{acc[0][j][v], acc[1][j][v], acc[2][j][v], acc[3][j][v]};
        }
    }
}

// The products that follow: out = T right, and the weight gradients beside it.
template <bool KC, int V, int MT>
__global__ __launch_bounds__(NT) void few_out_kernel(Product a, Outer o0, Outer o1)
{
    __shared__ __attribute__((aligned(16))) float red[red_floats(V, MT)];
    if ((int)blockIdx.x < a.items) {
        product_body<KC, V, MT>(a, ring::xcd_contiguous((int)blockIdx.x, a.items), red, nullptr);
        return;
    }
    const int t = ((int)blockIdx.x - a.items) * WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (t < o0.tiles) outer_body(o0, t, a.M);
    else if (t < o0.tiles + o1.tiles) outer_body(o1, t - o0.tiles, a.M);
}

}  // namespace few

FewPlan plan_few(int64_t M, int64_t Kred, int64_t r, int units)
{
    FewPlan p;
    // (17 to 64 tokens, microseconds in blocks of 16 / 32 / 64 rows: 64 x 512 from 4096 9.1 / 9.0 / 9.9, 64 x 1024 from 11008 21.4 / 16.2 /
    // 15.0, 20 x 1024 from 11008 15.7 / 13.5 / -, 33 x 64 from 11008 8.4 / 9.0 / 10.0)
    p.row_frags = M <= 16 ? 1 : 2;
    p.tiles = (int)((r + few::IN_COLS - 1) / few::IN_COLS);
    p.row_blocks = (int)((M + 16 * p.row_frags - 1) / (16 * p.row_frags));
    // Slices of 512 at least (of 256 / 512 / 768: 16 x 512 from 4096 9.5 / 8.2 / 8.3, 64 x 64 from 11008 11.4 / 9.0 / 9.9), and none up to
    // 1536, where a workgroup's eight steps per wave cost less than the tickets (whole / cut: 80 from 1664 5.4 / 6.9 and 6.7 / 6.4 with the
    // reduction contiguous, 128 from 1024 5.6 / 6.8, from 2048 7.8 / 6.5).
    const int64_t steps = (Kred + 63) / 64;
    int64_t s = 1;
    if (Kred > 1536) {
        s = units / (p.tiles * p.row_blocks);
        if (s > steps / 8) s = steps / 8;
        if (s < 1) s = 1;
    }
    const int64_t per = (steps + s - 1) / s;
    p.chunk = (int)(per * 64);
    p.splits = (int)((steps + per - 1) / per);
    p.part_bytes = p.splits > 1 ? (int64_t)p.row_blocks * p.tiles * p.splits * (16 * p.row_frags * few::IN_COLS) * 4 : 0;
    return p;
}

hipError_t launch_few_in(const void* left, const void* right, bool right_kc, void* T, int64_t M, int64_t Kred, int64_t r, const FewPlan& p,
                         float* part, uint32_t* tickets, hipStream_t s)
{
    using namespace few;
    if (M < 1 || M > FEW_MMAX || r < 8 || r > FEW_RMAX || (r % 8) || (Kred % 8) || p.splits < 1 || p.chunk < 64 || (p.chunk % 64)) return hipErrorInvalidValue;
    if ((int64_t)(p.splits - 1) * p.chunk >= Kred || (int64_t)p.splits * p.chunk < Kred) return hipErrorInvalidValue;
    if ((int64_t)p.row_blocks * p.row_frags * 16 < M || (int64_t)p.tiles * IN_COLS < r) return hipErrorInvalidValue;
    Product a = {static_cast<const uint16_t*>(left), static_cast<const uint16_t*>(right), static_cast<uint16_t*>(T), part, tickets,
                 (int)M, (int)r, (int)Kred, p.chunk, p.tiles, p.splits, p.tiles * p.splits * p.row_blocks};
    const int slot = prof_begin("few_in", 2.0 * M * r * (double)Kred, 2.0 * Kred * (double)(M + r), s);
    const dim3 grid((unsigned)a.items), block(NT);
    if (p.row_frags == 1) {
        if (right_kc) hipLaunchKernelGGL((few_in_kernel<true, 1>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((few_in_kernel<false, 1>), grid, block, 0, s, a);
    } else if (p.row_frags == 2) {
        if (right_kc) hipLaunchKernelGGL((few_in_kernel<true, 2>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((few_in_kernel<false, 2>), grid, block, 0, s, a);
    } else {
        return hipErrorInvalidValue;
    }
    prof_end(slot, s);
    return hipGetLastError();
}

hipError_t launch_few_out(const void* T, const void* right, bool right_kc, void* out, int64_t M, int64_t r, int64_t n, const FewGrads* grads, int units, hipStream_t s)
{
    using namespace few;
    if (M < 1 || M > FEW_MMAX || r < 8 || (r % 8) || (out && (n < 8 || (n % 8)))) return hipErrorInvalidValue;
    Product a = {};
    a.M = (int)M;
    // All tokens in one block of rows, so that the factor is read once; 32 columns per workgroup while that gives at most one workgroup
    // per compute unit, else 64 (microseconds, 32 / 64: 64 x 11008 from 1024 17.9 / 12.2, 64 x 4096 from 512 5.6 / 7.0, 16 x 4096 from 1024 7.9 / 8.6).
    const int mt = M <= 16 ? 1 : M <= 32 ? 2 : 4, v = (n + 31) / 32 > units ? 4 : 2;
    if (out) {
        a.left = static_cast<const uint16_t*>(T); a.right = static_cast<const uint16_t*>(right); a.out = static_cast<uint16_t*>(out);
        a.N = (int)n; a.K = (int)r; a.chunk = (int)((r + 63) / 64 * 64); a.splits = 1;
        a.tiles = (int)((n + 16 * v - 1) / (16 * v));
        a.items = a.tiles * (int)((M + 16 * mt - 1) / (16 * mt));
    }
    Outer o[2] = {};
    double cols = 0.0;
    if (grads) {
        const auto job = [](const void* p, int64_t na, const void* q, int64_t nb, float* to) {
            Outer j = {static_cast<const uint16_t*>(p), static_cast<const uint16_t*>(q), to, (int)na, (int)nb, (int)((na + 63) / 64), 0};
            j.tiles = to ? j.tiles_a * (int)((nb + 63) / 64) : 0;
            return j;
        };
        if ((grads->K % 8) || (grads->N % 8)) return hipErrorInvalidValue;
        o[0] = job(grads->dH, r, grads->X, grads->K, grads->dA);
        o[1] = job(grads->dY, grads->N, grads->H, r, grads->dB);
        cols = (double)((grads->dA ? grads->K : 0) + (grads->dB ? grads->N : 0));
    }
    const unsigned blocks = (unsigned)(a.items + (o[0].tiles + o[1].tiles + WAVES - 1) / WAVES);
    if (blocks == 0) return hipSuccess;
    const int slot = prof_begin("few_out", 2.0 * M * r * ((out ? n : 0) + cols), 2.0 * (out ? n : 0) * (double)(M + r) + 4.0 * r * cols, s);
    const dim3 grid(blocks), block(NT);
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, a, o[0], o[1]); };
    if (right_kc) {
        if (v == 2) mt == 1 ? go(few_out_kernel<true, 2, 1>) : mt == 2 ? go(few_out_kernel<true, 2, 2>) : go(few_out_kernel<true, 2, 4>);
        else mt == 1 ? go(few_out_kernel<true, 4, 1>) : mt == 2 ? go(few_out_kernel<true, 4, 2>) : go(few_out_kernel<true, 4, 4>);
    } else {
        if (v == 2) mt == 1 ? go(few_out_kernel<false, 2, 1>) : mt == 2 ? go(few_out_kernel<false, 2, 2>) : go(few_out_kernel<false, 2, 4>);
        else mt == 1 ? go(few_out_kernel<false, 4, 1>) : mt == 2 ? go(few_out_kernel<false, 4, 2>) : go(few_out_kernel<false, 4, 4>);
    }
    prof_end(slot, s);
    return hipGetLastError();
}

}  // namespace fhpc
