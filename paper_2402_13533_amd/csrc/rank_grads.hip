// Weight gradients of a rank of at most 32 over up to a few thousand tokens, both products in one launch:
//     dA[k][j] = alpha sum_m X[m][k] dH[m][j],    dB[j][n] = alpha sum_m H[m][j] dY[m][n]
//
// Both are sums over the tokens of a wide operand against a narrow one, bound by streaming X and dY once and, at a few
// hundred tokens, by launches.  On the GEMM tiles they took three: one per product, cut over the tokens so that enough
// workgroups run, and the sum of their slabs.  Here a workgroup owns a panel of 64 or 128 columns and all tokens: its
// eight waves take steps of 32 tokens in turn and add their sums through LDS at the end, so nothing leaves the chip but
// the gradients, and the panels of both products share the launch.  Operands go from memory straight into registers: a
// lane reads eight consecutive tokens of its columns (128 or 256 contiguous bytes per row of a 16-lane group), and a byte
// permute per register pair turns them into matrix operands, whose reduction index is the token.  Both gradients,
// microseconds, before / now: int8 4096 x 4096 r 16 at 65 / 300 / 1100 / 4096 tokens 11.8 / 4.3, 13.2 / 5.0, 14.9 / 7.5,
// 25.4 / 18.8; int4 5120 x 13824 r 16 13.7 / 5.4, 17.6 / 6.7, 25.1 / 15.9, 58 / 48; 13824 x 5120 r 32 16 / 5, 24 / 7,
// 31 / 15, 54 / 39.
#include "rank_grads.h"
#include "gemm_ring.h"
#include "profile.h"

namespace fhpc {
namespace rg {

using ring::bf16x8;
using ring::f32x4;
using ring::u32x4;

constexpr int WAVES = 8, NT = WAVES * 64;
constexpr int STEP = 32;                      // tokens per matrix instruction

struct Job {
    const uint16_t* U;      // the wide operand, bf16 [M][cols]
    const uint16_t* T;      // the rank operand, bf16 [M][rp]
    float* out;             // fp32, [cols][r] (`by_col`) or [r][cols]
    int cols, panels, by_col;
};

template <int V, int JF>
struct Rows {
    uint32_t u[8][V / 2];
    uint32_t t[8];
};

// Eight tokens of a lane's group: V columns of the wide operand and JF of the rank operand.
template <int V, int JF>
__device__ __forceinline__ void load_rows(Rows<V, JF>& x, const uint16_t* U, int64_t cols, const uint16_t* T, int rp, int m0, int M)
{
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int64_t m = m0 + e < M ? m0 + e : M - 1;
        if constexpr (V == 4) {
            const uint2 w = *reinterpret_cast<const uint2*>(U + m * cols);
            x.u[e][0] = w.x; x.u[e][1] = w.y;
        } else {
            const u32x4 w = *reinterpret_cast<const u32x4*>(U + m * cols);
#pragma unroll
            for (int i = 0; i < 4; i++) x.u[e][i] = w[i];
        }
        if constexpr (JF == 1) x.t[e] = T[m * rp];
        else x.t[e] = *reinterpret_cast<const uint32_t*>(T + m * rp);
    }
    if (m0 + 8 > M) {                          // tokens past the end count as zero on both sides
#pragma unroll
        for (int e = 0; e < 8; e++)
            if (m0 + e >= M) {
                x.t[e] = 0u;
#pragma unroll
                for (int i = 0; i < V / 2; i++) x.u[e][i] = 0u;
            }
    }
}

// 16-bit halves (low or high) of eight words as one operand
__device__ __forceinline__ bf16x8 halves(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t a4, uint32_t a5, uint32_t a6, uint32_t a7,
                                         uint32_t pick)
{
    const u32x4 w = {__builtin_amdgcn_perm(a1, a0, pick), __builtin_amdgcn_perm(a3, a2, pick), __builtin_amdgcn_perm(a5, a4, pick),
                     __builtin_amdgcn_perm(a7, a6, pick)};
    return __builtin_bit_cast(bf16x8, w);
}

// V columns of the wide operand and JF of the rank operand per lane
template <int V, int JF>
__global__ __launch_bounds__(NT) void rank_grads_kernel(Job j0, Job j1, int M, int r, int rp, float alpha)
{
    constexpr int COLS = 16 * V, RT = 16 * JF, LDR = RT + 1;
    __shared__ float red[WAVES][COLS][LDR];
    const bool first = (int)blockIdx.x < j0.panels;
    const Job j = first ? j0 : j1;
    const int c0 = (first ? (int)blockIdx.x : (int)blockIdx.x - j0.panels) * COLS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, g = lane >> 4;
    const int col = c0 + c * V, jc = c * JF;
    // (a lane outside the matrix repeats another's columns: its sums are not stored)
    const uint16_t* const U = j.U + (col < j.cols ? col : 0);
    const uint16_t* const T = j.T + (jc < rp ? jc : 0);
    const int nsteps = (M + STEP - 1) / STEP;
    f32x4 acc[V][JF];
#pragma unroll
    for (int i = 0; i < V; i++)
#pragma unroll
        for (int f = 0; f < JF; f++) acc[i][f] = (f32x4){0.f, 0.f, 0.f, 0.f};
    Rows<V, JF> x;
    int s = wave;
    if (s < nsteps) load_rows<V, JF>(x, U, j.cols, T, rp, s * STEP + g * 8, M);
    while (s < nsteps) {
        const Rows<V, JF> y = x;
        s += WAVES;
        if (s < nsteps) load_rows<V, JF>(x, U, j.cols, T, rp, s * STEP + g * 8, M);
        bf16x8 b[JF];
#pragma unroll
        for (int f = 0; f < JF; f++)
            b[f] = halves(y.t[0], y.t[1], y.t[2], y.t[3], y.t[4], y.t[5], y.t[6], y.t[7], f ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int i = 0; i < V; i++) {
            const int d = i / 2;
            const bf16x8 a = halves(y.u[0][d], y.u[1][d], y.u[2][d], y.u[3][d], y.u[4][d], y.u[5][d], y.u[6][d], y.u[7][d],
                                    (i & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int f = 0; f < JF; f++) acc[i][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[f], acc[i][f], 0, 0, 0);
        }
    }
    // register v of acc[i][f]: column (4 g + v) V + i of the panel, rank index c JF + f
#pragma unroll
    for (int i = 0; i < V; i++)
#pragma unroll
        for (int f = 0; f < JF; f++)
#pragma unroll
            for (int v = 0; v < 4; v++) red[wave][(4 * g + v) * V + i][jc + f] = acc[i][f][v];
    __syncthreads();
    for (int e = threadIdx.x; e < COLS * RT; e += NT) {
        const int cc = j.by_col ? e / RT : e % COLS, jj = j.by_col ? e % RT : e / COLS;
        if (c0 + cc >= j.cols || jj >= r) continue;
        float a = red[0][cc][jj];
#pragma unroll
        for (int w = 1; w < WAVES; w++) a += red[w][cc][jj];
        j.out[j.by_col ? (int64_t)(c0 + cc) * r + jj : (int64_t)jj * j.cols + c0 + cc] = alpha * a;
    }
}

template <int V>
static void launch(const Job (&j)[2], int M, int r, int rp, float alpha, hipStream_t s)
{
    Job a = j[0], b = j[1];
    a.panels = a.out ? (a.cols + 16 * V - 1) / (16 * V) : 0;
    b.panels = b.out ? (b.cols + 16 * V - 1) / (16 * V) : 0;
    const dim3 grid((unsigned)(a.panels + b.panels));
    if (rp <= 16) hipLaunchKernelGGL((rank_grads_kernel<V, 1>), grid, dim3(NT), 0, s, a, b, M, r, rp, alpha);
    else hipLaunchKernelGGL((rank_grads_kernel<V, 2>), grid, dim3(NT), 0, s, a, b, M, r, rp, alpha);
}

}  // namespace rg

// A panel's workgroup walks all the tokens: from some thousands on, slices over more workgroups are ahead (both gradients and dH,
// microseconds, slices / one launch: 5120 x 13824 r 16 at 2500 / 4096 / 8192 tokens 53 / 45, 65 / 55, 120 / 123; 2048 x 2048 r 8
// 17.9 / 15.5, 21.3 / 20.2, 29 / 34).
bool rank_grads_pay(int64_t M, int64_t rp) { return rp <= 32 && M <= 4096; }

hipError_t launch_rank_grads(const void* X, const void* dH, float* dA, const void* H, const void* dY, float* dB, int64_t M, int64_t K,
                             int64_t r, int64_t rp, int64_t N, float alpha, hipStream_t s)
{
    using namespace rg;
    if (M < 1 || r < 1 || rp < r || rp > 32 || (rp % 8) || (K % 8) || (N % 8)) return hipErrorInvalidValue;
    if (!dA && !dB) return hipSuccess;
    const Job j[2] = {{static_cast<const uint16_t*>(X), static_cast<const uint16_t*>(dH), dA, (int)K, 0, 1},
                      {static_cast<const uint16_t*>(dY), static_cast<const uint16_t*>(H), dB, (int)N, 0, 0}};
    const int64_t cols = (dA ? K : 0) + (dB ? N : 0);
    const int slot = prof_begin("rank_grads", 2.0 * M * r * (double)cols, 2.0 * M * (double)cols, s);
    // 128 columns per workgroup once such panels still give half the compute units work and there are tokens to stream (64 / 128
    // columns, microseconds with dH: 5120 x 13824 at 65 / 700 / 4096 tokens 11.9 / 12.0, 19.0 / 18.3, 64 / 55; 4096 x 11008
    // r 32 at 2047 29.1 / 30.8; 4096 x 4096 at 300 / 4096 11.5 / 12.2, 25.3 / 29.9)
    if (cols >= 128 * 128 && M > 256) rg::launch<8>(j, (int)M, (int)r, (int)rp, alpha, s);
    else rg::launch<4>(j, (int)M, (int)r, (int)rp, alpha, s);
    prof_end(slot, s);
    return hipGetLastError();
}

}  // namespace fhpc
