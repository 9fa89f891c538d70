// The factorised layer with at most 64 tokens (see few_lowrank.hip).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fhpc {

constexpr int FEW_MMAX = 64, FEW_RMAX = 1024;

// How a long reduction into the rank (H = X A, dH = dY B^T) is cut: workgroups of 16 row_frags rows x 32 ranks x `chunk` of it.
struct FewPlan {
    int row_frags, tiles, row_blocks, splits, chunk;
    int64_t part_bytes;         // slabs of the slices (0 with one slice)
};
FewPlan plan_few(int64_t M, int64_t Kred, int64_t r, int units);

// T[M][r] = left right, left bf16 [M][Kred], right bf16 [Kred][r] or [r][Kred] (`right_kc`).  part: scratch of the plan's size;
// tickets: the workspace header (zero words, left zero).
hipError_t launch_few_in(const void* left, const void* right, bool right_kc, void* T, int64_t M, int64_t Kred, int64_t r, const FewPlan& p,
                         float* part, uint32_t* tickets, hipStream_t s);

// In one launch, each part optional (NULL output):
//   out[M][n] = T right (bf16), T bf16 [M][r], right bf16 [r][n] or [n][r] (`right_kc`);
//   dA[K][r] = X^T dH,  dB[r][N] = H^T dY (fp32), X [M][K], dH and H [M][r], dY [M][N] bf16.
struct FewGrads {
    const void *X, *dH, *H, *dY;
    float *dA, *dB;
    int64_t K, N;
};
hipError_t launch_few_out(const void* T, const void* right, bool right_kc, void* out, int64_t M, int64_t r, int64_t n, const FewGrads* grads, int units, hipStream_t s);

}  // namespace fhpc
