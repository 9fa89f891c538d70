// Weight-streaming forward of the quantised finetuning layer for one to a few tokens, without partial-sum slabs:
//   Y = base_scale * X * deq(Wq, scales) + scaling * (X * A) * B.
//
// A workgroup owns 16 output channels and their whole reduction; its four waves take every fourth 128-byte piece of the
// channels' rows and their sums meet in LDS.  Nothing of the big product crosses workgroups: no slabs, no tickets, no last
// arriver that gathers through a chain of round trips.  The stream runs at 4.0 TB/s (what each further 1000 channels of
// 5120 int4 codes add) against 2.8 of the sliced kernel; the fixed part is 9 microseconds, 3.5 of them H's launch.
// What it costs is the token rows, which every workgroup takes into its LDS, so it is for a few tokens.
//
// Only H = X A, a few hundred numbers, crosses workgroups: a small launch ahead forms its 1024-deep chunks, and every
// streaming workgroup adds them up.  (In the same launch, with an arrival counter that the streaming workgroups look at, it
// costs more: the looks and the departures of all workgroups meet on one line of memory, 35 .. 40 nanoseconds apart, 40
// microseconds for the 1728 workgroups of a wide pair of weights.)  Bound by the HBM stream, then by that fixed part; code
// is kept short (two units ahead, not four: 31.1 -> 28.6 microseconds), since a launch starts with a cold instruction cache.
//
// Codes become matrix operands as in qskinny.hip (exact small integers, the offset taken out on the matrix unit, the fp16
// scale applied to fp32 sums).  The weight is the column operand here: a lane's accumulators are four tokens of the one
// channel whose row it loads, so a scale is one load and one factor per lane.
#include "qskinny.h"
#include "qskinny_codes.h"
#include "gemm_ring.h"
#include "profile.h"

#include <hip/hip_fp16.h>

namespace fhpc {
namespace skinny {

struct RowJobs {
    const void* Wq[QSKINNY_MAX_JOBS];
    const void* scales[QSKINNY_MAX_JOBS];
    const void* A[QSKINNY_MAX_JOBS];
    const void* B[QSKINNY_MAX_JOBS];
    void* Y[QSKINNY_MAX_JOBS];
    void* H_out[QSKINNY_MAX_JOBS];
    int N[QSKINNY_MAX_JOBS];
    int wg0[QSKINNY_MAX_JOBS + 1];            // first streaming workgroup of each weight
    float base_scale[QSKINNY_MAX_JOBS];
    float scaling[QSKINNY_MAX_JOBS];
    int count;
};

template <typename T>
__device__ __forceinline__ T pick_job(const T (&a)[QSKINNY_MAX_JOBS], int j)
{
    T v = a[0];
#pragma unroll
    for (int i = 1; i < QSKINNY_MAX_JOBS; i++) v = (j == i) ? a[i] : v;
    return v;
}

constexpr int RH_CHUNK = 1024;                // reduction depth of one chunk of H = X A
constexpr int RH_MAX = 64;                    // ranks

// hpart[job][c][m][j] = sum over the 1024 k of chunk c of X[m][k] A[k][j].  A workgroup per chunk and weight; every wave takes
// its share of the chunk on the matrix unit, all operands requested before the first wait, and the waves' sums are
// added in wave order.
// NB: blocks of 16 ranks.  PACKED (r a multiple of 4, at most 32): a wave's share of A lies together in memory; it is copied to LDS
// as it lies, 16 bytes a lane, and transposed as it is read (beyond the ranks: the next k's, columns that are not stored).  Loaded
// by two bytes, each lane its eight k of a rank, the requests alone keep the unit's address path
// busy for 1.7 microseconds.  A 13B decoder layer, one token, r 16: 80.7 -> 78.6 microseconds (two of these launches); four tokens of a
// 7B layer at r 32 99 -> 91.
constexpr int RH_NW = 8;
template <int NB, bool PACKED>
__global__ __launch_bounds__(64 * RH_NW) void qrows_h_kernel(RowJobs jb, const uint16_t* __restrict__ X, int M, int K, int r,
                                                             float* __restrict__ hpart, int chunks)
{
    constexpr int STEPS = RH_CHUNK / 32 / RH_NW;
    constexpr int SHARE = PACKED ? STEPS * 32 * NB * 32 + 64 : 16;      // (64: what the last reads reach beyond)
    __shared__ float red[RH_NW * 16 * RH_MAX];
    __shared__ __attribute__((aligned(16))) unsigned char share[RH_NW * SHARE];
    const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int job = (int)blockIdx.x / chunks, c = (int)blockIdx.x - job * chunks;
    const uint16_t* const A = static_cast<const uint16_t*>(pick_job(jb.A, job));
    const int m = lr < M ? lr : M - 1;         // (rows beyond M repeat the last; not used)
    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (PACKED) {
        const int k0 = c * RH_CHUNK + wave * (STEPS * 32), row_bytes = 2 * r;
        const ring::u32x4 ra = ring::make_rsrc(A, (uint32_t)K * (uint32_t)row_bytes);
        const __amdgpu_buffer_rsrc_t rx = rsrc(X, (int64_t)M * K * 2);
        unsigned char* const mine = share + wave * SHARE;
        const uint32_t base = ring::lds_addr(mine);
        // (k beyond K: A reads as zero, and X is not asked for)
        for (int q = 0; q < r / 4; q++) ring::dma_16B(ra, base + 1024u * q, (uint32_t)k0 * row_bytes + 1024u * q + 16u * lane);
        u32x4 xv[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; s++) xv[s] = __builtin_amdgcn_raw_buffer_load_b128(rx, k0 + 32 * s < K ? (uint32_t)(m * K + k0 + 32 * s + 8 * g) * 2u : OOB, 0, 0);
        FHPC_WAIT_VM(0);
        // the transposing read of 4 k x 16 ranks: lane i of 16 gives the address of k i / 4, ranks 4 (i % 4) .. + 3
        const unsigned char* const from = mine + (8 * g + (lr >> 2)) * row_bytes + 8 * (lr & 3);
#pragma unroll
        for (int s = 0; s < STEPS; s++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                union { ring::s16x4 p[2]; bf16x8 v; } a;
#pragma unroll
                for (int j = 0; j < 2; j++)
                    a.p[j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) ring::s16x4*)(const_cast<unsigned char*>(from + (s * 32 + 4 * j) * row_bytes + 32 * b)));
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xv[s]), a.v, acc[b], 0, 0, 0);
            }
    } else {
#pragma unroll
        for (int s = 0; s < STEPS; s++) {
            const int k = c * RH_CHUNK + (wave * STEPS + s) * 32 + 8 * g;
            if (k < K) {                       // (K is a multiple of 256: a 32-deep step is inside or outside as a whole)
                const u32x4 xv = *reinterpret_cast<const u32x4*>(X + (int64_t)m * K + k);
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    if (16 * b < r) {
                        const int j = (16 * b + lr < r) ? 16 * b + lr : r - 1;
                        uint32_t e[8];
#pragma unroll
                        for (int q = 0; q < 8; q++) e[q] = A[(int64_t)(k + q) * r + j];
                        const u32x4 av = {e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(xv), as_bf16x8(av), acc[b], 0, 0, 0);
                    }
                }
            }
        }
    }
    // a lane holds rank 16 b + lr of the tokens 4 g .. 4 g + 3
#pragma unroll
    for (int b = 0; b < NB; b++)
        if (16 * b < r)
#pragma unroll
            for (int v = 0; v < 4; v++) red[(wave * 16 + 4 * g + v) * RH_MAX + 16 * b + lr] = acc[b][v];
    __syncthreads();
    for (int i = threadIdx.x; i < M * r; i += 64 * RH_NW) {
        const int mm = i / r, j = i - mm * r;
        float s = red[mm * RH_MAX + j];
#pragma unroll
        for (int w = 1; w < RH_NW; w++) s += red[(w * 16 + mm) * RH_MAX + j];
        hpart[(int64_t)blockIdx.x * M * r + i] = s;
    }
}

constexpr int ROWS_CH = 16, ROWS_NW = 4;      // channels and waves of a workgroup
constexpr int ROWS_TOK = 16;                  // token rows of the matrix instructions: the most tokens of a call
constexpr int SUM_LD = 20;                    // floats between channels of a wave's sums (16 tokens)
constexpr int RX_PAD = 16;                    // bytes between token rows in LDS beyond their length
constexpr int RX_MOST = 20480;                // elements of X a workgroup holds
constexpr int RH_MOST = 8;                    // chunks of H a thread adds from registers

template <int SCHEME>
__global__ __launch_bounds__(64 * ROWS_NW) void qrows_fwd_kernel(RowJobs jb, const uint16_t* __restrict__ X, int M, int K, int r,
                                                            const float* __restrict__ hpart, int chunks)
{
    constexpr bool I4 = (SCHEME == 4);
    constexpr int CH = ROWS_CH, NW = ROWS_NW, NT = 64 * NW, AHEAD = 2;
    constexpr int UNIT = I4 ? 256 : 128;               // k of 128 bytes of a row
    constexpr int XC = UNIT / 32;                      // 16-byte pieces of a token row per lane and unit
    constexpr int XL = RX_MOST / 8 / NT;               // 16-byte pieces of X per thread
    constexpr int BL = (RH_MAX * CH + NT - 1) / NT;    // elements of B per thread
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];      // the token rows, then the waves' sums
    __shared__ float Hs[16 * RH_MAX];
    __shared__ uint16_t Bs[RH_MAX * CH];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = (int)blockIdx.x;
    int job = 0, first = 0;
#pragma unroll
    for (int i = 1; i < QSKINNY_MAX_JOBS; i++)
        if (i < jb.count && wg >= jb.wg0[i]) {
            job = i;
            first = jb.wg0[i];
        }
    const int N = pick_job(jb.N, job);
    const int n0 = (wg - first) * CH;
    const void* const scales = pick_job(jb.scales, job);
    const int64_t row_bytes = I4 ? K / 2 : K;
    const __amdgpu_buffer_rsrc_t rw = rsrc(pick_job(jb.Wq, job), (int64_t)N * row_bytes);
    const __amdgpu_buffer_rsrc_t rsc = rsrc(scales, I4 ? (int64_t)N * (K / 64) * 2 : (int64_t)N * 2);
    const __amdgpu_buffer_rsrc_t rx = rsrc(X, (int64_t)M * K * 2);
    const __amdgpu_buffer_rsrc_t rB = rsrc(pick_job(jb.B, job), (int64_t)r * N * 2);
    const __amdgpu_buffer_rsrc_t rh = rsrc(hpart, (int64_t)jb.count * chunks * M * r * 4);

    // Requested in the order in which they are waited for: the token rows, what the end needs (this workgroup's columns
    // of B, the chunks of H), the first weights.  Whatever lies beyond an operand reads as zero.
    u32x4 xr[XL];
#pragma unroll
    for (int i = 0; i < XL; i++) xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (uint32_t)(tid + NT * i) * 16u, 0, 0);
    uint16_t br[BL];
#pragma unroll
    for (int i = 0; i < BL; i++) {
        const int e = tid + NT * i, n = n0 + e % CH;
        br[i] = 0;
        if (NT * i < r * CH) br[i] = __builtin_amdgcn_raw_buffer_load_b16(rB, (n < N) ? (uint32_t)((e / CH) * N + n) * 2u : OOB, 0, 0);
    }
    float hr[RH_MOST];
#pragma unroll
    for (int c = 0; c < RH_MOST; c++) {
        hr[c] = 0.f;
        if (c < chunks) hr[c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rh, (tid < M * r) ? (uint32_t)((job * chunks + c) * M * r + tid) * 4u : OOB, 0, 0));
    }
    // this lane's row (rows beyond N read as zeros) and its 16 bytes of a 64-byte piece
    const uint32_t wlane = (n0 + lr < N) ? (uint32_t)((int64_t)(n0 + lr) * row_bytes) + 16u * (uint32_t)g : OOB;
    const uint32_t slane = (n0 + lr < N) ? (uint32_t)(I4 ? (n0 + lr) * (K / 64) * 2 : (n0 + lr) * 2) : OOB;
    const int units = K / UNIT;
    struct Unit {
        u32x4 w[2];
        uint32_t s[2];                                 // int4: four blocks' scales of the lane's channel
    };
    auto fetch = [&](Unit& q, int u) __attribute__((always_inline)) {
        // (units beyond the end repeat the last one: loaded, not used)
        const int at = (u < units) ? u : units - 1;
#pragma unroll
        for (int p = 0; p < 2; p++) q.w[p] = __builtin_amdgcn_raw_buffer_load_b128(rw, wlane + 64u * p, at * 128, 0);
        if constexpr (I4) {
            const auto h = __builtin_amdgcn_raw_buffer_load_b64(rsc, slane, at * 8, 0);
            q.s[0] = h[0];
            q.s[1] = h[1];
        }
    };
    Unit q[AHEAD];
#pragma unroll
    for (int a = 0; a < AHEAD; a++) fetch(q[a], wave + NW * a);

    const int ldx = K * 2 + RX_PAD;
#pragma unroll
    for (int i = 0; i < XL; i++) {
        const int e = (tid + NT * i) * 8;
        if (e < M * K) {
            const int m = e / K;
            *reinterpret_cast<u32x4*>(smem + m * ldx + (e - m * K) * 2) = I4 ? x_even_odd_order(xr[i]) : xr[i];
        }
    }
    __syncthreads();

    // Token row of this lane (rows beyond M repeat the last; their sums are not stored).  int4: after the exchange between
    // the halves of a wave, lane group g holds of each 64-block the 16 codes from 32 (g & 1) + 16 (g >> 1) on; int8: the
    // 16 codes from 16 g on of 64.
    const unsigned char* const xlane = smem + (lr < M ? lr : M - 1) * ldx + (I4 ? 32 * (g & 1) + 16 * (g >> 1) : 16 * g) * 2;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f}, ones_acc = {0.f, 0.f, 0.f, 0.f};
    const u32x4 ones_bits = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const u32x4 moff_bits = {0xc308c308u, 0xc308c308u, 0xc308c308u, 0xc308c308u};     // bf16(-136) x 8
    const bf16x8 ones = as_bf16x8(ones_bits), minus_offset = as_bf16x8(moff_bits);
    auto compute = [&](const Unit& q, int u) __attribute__((always_inline)) {
        // chunk (p, b, h) of int4: k = 128 p + 64 b + 8 h of the unit; (p, h) of int8: k = 64 p + 8 h
        bf16x8 xf[XC];
#pragma unroll
        for (int c = 0; c < XC; c++) xf[c] = as_bf16x8(*reinterpret_cast<const u32x4*>(xlane + u * (UNIT * 2) + (c / 2) * 128 + (c % 2) * 16));
        if constexpr (I4) {
            f32x4 off[4];                              // sum over each block of X (-136)
#pragma unroll
            for (int b = 0; b < 4; b++) off[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[2 * b], minus_offset, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 4; b++) off[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[2 * b + 1], minus_offset, off[b], 0, 0, 0);
            uint32_t c[2][4];
#pragma unroll
            for (int p = 0; p < 2; p++) {
                c[p][0] = q.w[p].x; c[p][1] = q.w[p].y; c[p][2] = q.w[p].z; c[p][3] = q.w[p].w;
                exchange_halves(c[p]);
            }
            f32x4 cw[4];                               // ... and of X (q + 136)
#pragma unroll
            for (int b = 0; b < 4; b++) cw[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[2 * b], int4_operand(c[b / 2][2 * (b % 2)]), off[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 4; b++) cw[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[2 * b + 1], int4_operand(c[b / 2][2 * (b % 2) + 1]), cw[b], 0, 0, 0);
#pragma unroll
            for (int b = 0; b < 4; b++) {
                const uint32_t word = q.s[b / 2];
                const float sc = __half2float(__ushort_as_half((unsigned short)((b % 2) ? (word >> 16) : (word & 0xffffu))));
#pragma unroll
                for (int v = 0; v < 4; v++) acc[v] += sc * cw[b][v];
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; c++) {
                const u32x4 w = q.w[c / 2];
                ones_acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[c], ones, ones_acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[c], (c % 2) ? int8_operand(w.z, w.w) : int8_operand(w.x, w.y), acc, 0, 0, 0);
            }
        }
    };
    // this wave's units: wave, wave + NW, ...; no branch between a request and its use but the loop's own end
    for (int u = wave; u < units;) {
#pragma unroll
        for (int a = 0; a < AHEAD; a++) {
            compute(q[a], u);
            fetch(q[a], u + NW * AHEAD);
            u += NW;
            if (u >= units) break;
        }
    }
    if constexpr (!I4) {
        // one fp16 scale per output channel, applied once
        const float sc = __half2float(__ushort_as_half((unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rsc, slane, 0, 0)));
#pragma unroll
        for (int v = 0; v < 4; v++) acc[v] = sc * (acc[v] - 128.f * ones_acc[v]);
    }
#pragma unroll
    for (int i = 0; i < BL; i++)
        if (tid + NT * i < r * CH) Bs[tid + NT * i] = br[i];
    {
        float h = hr[0];
#pragma unroll
        for (int c = 1; c < RH_MOST; c++)
            if (c < chunks) h += hr[c];
        if (tid < M * r) Hs[tid] = h;
    }
    __syncthreads();                                   // (the token rows have been read)
    float* const sums = reinterpret_cast<float*>(smem);
    // a lane holds channel lr, tokens 4 g .. 4 g + 3
    *reinterpret_cast<f32x4*>(sums + (wave * CH + lr) * SUM_LD + 4 * g) = acc;
    __syncthreads();
    const float base_scale = pick_job(jb.base_scale, job), scaling = pick_job(jb.scaling, job);
    uint16_t* const Y = static_cast<uint16_t*>(pick_job(jb.Y, job));
    for (int i = tid; i < CH * M; i += NT) {
        const int c = i % CH, m = i / CH, n = n0 + c;
        float s = sums[c * SUM_LD + m];
#pragma unroll
        for (int w = 1; w < NW; w++) s += sums[(w * CH + c) * SUM_LD + m];       // in wave order
        float l = 0.f;
        for (int j = 0; j < r; j++) l = fmaf(Hs[m * r + j], __uint_as_float((uint32_t)Bs[j * CH + c] << 16), l);
        if (n < N) {
            const __bf16 yb = (__bf16)(base_scale * s + scaling * l);
            Y[(int64_t)m * N + n] = __builtin_bit_cast(uint16_t, yb);
        }
    }
    if (wg == first) {
        uint16_t* const H_out = static_cast<uint16_t*>(pick_job(jb.H_out, job));
        if (H_out)
            for (int i = tid; i < M * r; i += NT) {
                const __bf16 hb = (__bf16)Hs[i];
                H_out[i] = __builtin_bit_cast(uint16_t, hb);
            }
    }
}

// What the kernels hold: one block of token rows, in LDS (four workgroups to a unit), a thread per number of H, its
// chunks in registers.
static bool rows_fit(int64_t M, int64_t K, int64_t r)
{
    return M >= 1 && M <= ROWS_TOK && r >= 1 && r <= RH_MAX && (K % 256) == 0 && M * K <= RX_MOST && M * r <= 64 * ROWS_NW && K <= RH_MOST * RH_CHUNK;
}

}  // namespace skinny

// Where it is taken (microseconds a call, twelve calls on four weights replayed from a graph, one token, sliced kernel / this one):
//   many channels, which are what the slabs cost: 5120 -> 15360 int4 19.7 / 15.2, 5120 -> 27648 41.9 / 25.5, 4096 -> 12288 int8
//   20.9 / 16.3;
//   more than 16 ranks, where the sliced kernel's chunks of H are what it waits for: 4096 -> 4096 r = 32 17.2 / 9.9,
//   r = 64 22.7 / 15.0;
//   a short reduction, few chunks of H to form: 2048 -> 4096 10.9 / 6.7.
// Over 240 calls it takes (1 .. 16 tokens, K 512 .. 8192, r 4 .. 64, both storages, ten calls a replay) it is 1.08 .. 2 times faster, 1.56 on
// average.  The line at 12288 channels dates from an H launch of 4.6 instead of 3.5 microseconds and lies high: with fewer channels a
// call alone in its graph takes as long either way (5120 -> 10240 19.4 / 19.4, 5120 -> 5120 16.7 / 17.0; 5120 -> 11776 24.6 / 19.5), calls one
// after another are faster here too (14.7 / 12.8, 12.1 / 10.7, 19.9 / 12.9).
// The rest are its limits.
bool qskinny_rows_pay(int64_t M, int64_t K, int64_t r, int64_t N_all, int num_cu)
{
    using namespace skinny;
    if (!rows_fit(M, K, r)) return false;
    return N_all >= (int64_t)3 * num_cu * ROWS_CH || r > 16 || K <= 2560;
}

hipError_t launch_qskinny_rows(const void* X, const QskinnyJob* jobs, int count, int scheme, int64_t M, int64_t K, int64_t r,
                               float* hpart, hipStream_t st)
{
    using namespace skinny;
    if (count < 1 || count > QSKINNY_MAX_JOBS || !rows_fit(M, K, r)) return hipErrorInvalidValue;
    RowJobs jb = {};
    jb.count = count;
    int wg = 0;
    for (int j = 0; j < QSKINNY_MAX_JOBS; j++) {
        const QskinnyJob& q = jobs[j < count ? j : 0];
        jb.Wq[j] = q.Wq; jb.scales[j] = q.scales; jb.A[j] = q.A; jb.B[j] = q.B; jb.Y[j] = q.Y; jb.H_out[j] = q.H_out;
        jb.N[j] = (int)q.N; jb.base_scale[j] = q.base_scale; jb.scaling[j] = q.scaling;
        jb.wg0[j] = wg;
        if (j < count) wg += (int)((q.N + ROWS_CH - 1) / ROWS_CH);
    }
    for (int j = count; j <= QSKINNY_MAX_JOBS; j++) jb.wg0[j] = wg;
    const int chunks = (int)((K + RH_CHUNK - 1) / RH_CHUNK);
    const uint16_t* const x = static_cast<const uint16_t*>(X);
    const dim3 hgrid((unsigned)(count * chunks)), hblock(64 * RH_NW);
    if (r % 4 == 0 && r <= 16) hipLaunchKernelGGL((qrows_h_kernel<1, true>), hgrid, hblock, 0, st, jb, x, (int)M, (int)K, (int)r, hpart, chunks);
    else if (r % 4 == 0 && r <= 32) hipLaunchKernelGGL((qrows_h_kernel<2, true>), hgrid, hblock, 0, st, jb, x, (int)M, (int)K, (int)r, hpart, chunks);
    else hipLaunchKernelGGL((qrows_h_kernel<RH_MAX / 16, false>), hgrid, hblock, 0, st, jb, x, (int)M, (int)K, (int)r, hpart, chunks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t xbytes = (size_t)M * (K * 2 + RX_PAD), sums = sizeof(float) * ROWS_NW * ROWS_CH * SUM_LD;
    const size_t lds = xbytes > sums ? xbytes : sums;
    if (scheme == 4) hipLaunchKernelGGL(qrows_fwd_kernel<4>, dim3((unsigned)wg), dim3(64 * ROWS_NW), lds, st, jb, x, (int)M, (int)K, (int)r, hpart, chunks);
    else hipLaunchKernelGGL(qrows_fwd_kernel<8>, dim3((unsigned)wg), dim3(64 * ROWS_NW), lds, st, jb, x, (int)M, (int)K, (int)r, hpart, chunks);
    return hipGetLastError();
}

}  // namespace fhpc
