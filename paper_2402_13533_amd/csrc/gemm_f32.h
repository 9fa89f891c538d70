// The fp32 products of the factorised layer, on the fp32 matrix instructions or, large ones, on the bf16 ones with operands in three parts.
// Internal; not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fhpc {

// How an operand element (row, k) is stored: ptr[row * ld + k] (F32_KC) or ptr[k * ld + row] (F32_XC).
enum F32Layout { F32_KC = 0, F32_XC = 1 };

// Output tiles: squares, on the fp32 matrix instructions (gemm_f32.hip) or with operands in three parts on the bf16 ones (gemm_f32x3.hip).
enum F32TileKind { F32_64, F32_32, F32_X3_128, F32_X3_64, F32_TILE_KINDS };
constexpr int F32_TILE[F32_TILE_KINDS] = {64, 32, 128, 64};          // edge

struct GemmF32Plan {
    F32TileKind tile;
    int splits;      // slices of the reduction; more than one: each stores a slab per tile; the last to arrive adds them (F32_X3: a second launch)
    int k_chunk;     // reduction length of a slice, a multiple of 32
};
constexpr int64_t F32_TICKETS = 4096;                        // tiles of a launch whose reductions may be cut: words of the workspace header
constexpr int64_t F32_LD_MAX = (int64_t)1 << 20;

// C[M][N] (row stride ldc) = sum_k a(m, k) b(n, k)
struct GemmF32Job {
    const float* a;
    const float* b;
    float* c;
    int64_t lda, ldb, ldc;
    int M, N, K;
    int splits, k_chunk;
    // (set by launch_gemm_f32)
    int tiles_n, items;
    float* part;
    uint32_t* tickets;
};

// Up to two products of the same operand layouts share a launch; `jobs` products of these sizes are planned together, without
// `three_parts` on the tiles of the fp32 instructions alone.
// part: scratch of gemm_f32_part_bytes of every job; tickets: F32_TICKETS zero words, left zero.
GemmF32Plan plan_gemm_f32(int jobs, const int64_t* M, const int64_t* N, const int64_t* K, int units, GemmF32Plan* each, bool three_parts = true);
int64_t gemm_f32_part_bytes(const GemmF32Plan& p, int64_t M, int64_t N);
hipError_t launch_gemm_f32(F32Layout al, F32Layout bl, const GemmF32Job* jobs, int count, F32TileKind tile, float* part, uint32_t* tickets, hipStream_t s);

// Which operands take 16-byte loads: bit 0 and 1 a and b of job 0, bit 2 and 3 of job 1.  An operand can where its rows start 16-byte
// aligned and its contiguous extent is a multiple of four, so with other ranks X, dY and B still do.  768 -> 191 -> 3072 at 8192 tokens,
// forward / backward in microseconds: every load by four bytes 193 / 300, this choice 157 / 246 (rank 192: 129 / 225).
constexpr unsigned F32_VEC_A = 5, F32_VEC_B = 10;
// launch_gemm_f32's second half for F32_X3 tiles: two jobs, complete (with count == 1 the second is not looked at)
hipError_t launch_gemm_f32x3(F32Layout al, F32Layout bl, const GemmF32Job* jobs, int count, unsigned blocks, F32TileKind tile, unsigned vec, hipStream_t s);

// out[i] = sum of the slabs' elements i, i < n.  With cols > 0 the output is bf16 [n / cols][cols] with row stride ldo
// (cols a multiple of 4, rows 8-byte aligned).
struct SumF32Job {
    const float* slabs;
    void* out;
    int64_t n, slab;
    int nslab, blocks;
    int cols;
    int64_t ldo;
};
constexpr int SUM_F32_MAX = 9;                    // jobs of a launch
hipError_t launch_sum_f32(const SumF32Job* jobs, int count, hipStream_t s);

// Two chained products with the rank-r intermediate kept in LDS (r <= 64), see gemm_f32.hip:
// P = L R (M x r, also stored to P_out when given), Out = P S (M x C; C = 0: P alone, with the same bits).
bool lowrank_chain_f32_pays(int64_t M, int64_t T, int64_t r);
hipError_t launch_lowrank_chain_f32(const float* L, int64_t ldl, const float* R, int64_t ldr, F32Layout rl,
                                    const float* S, int64_t lds, F32Layout sl, float* Out, int64_t ldo, float* P_out,
                                    int M, int T, int r, int C, int units, hipStream_t s);

// The r x r products of the rank-r factorisation, C = A' B with A' = A or A^T (all r x r, row-major, r a multiple of 8),
// with the polynomial step that follows in the same launch when `poly` is set:
//   C = post * (diag I + pre add_scale Add + scale A' B),   pre = *inv_trace and post = sqrt(pre) when inv_trace is given,
// 1 otherwise; Add may be NULL.  C may not alias an input.  With bf16_out the result goes there, rounded, and C is not touched.
struct SquareEpilogue {
    bool poly = false;
    float scale = 1.f, diag = 0.f, add_scale = 0.f;
    const float* add = nullptr;
    const float* inv_trace = nullptr;
};
hipError_t launch_square_f32(const float* A, bool transpose_a, const float* B, float* C, int64_t r, const SquareEpilogue& e, hipStream_t s, void* bf16_out = nullptr);

}  // namespace fhpc
