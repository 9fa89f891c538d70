// Weight gradients of a rank of at most 32, both in one launch (see rank_grads.hip).  Not part of the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fhpc {

bool rank_grads_pay(int64_t M, int64_t rp);
// dA[k][j] = alpha sum_m X[m][k] dH[m][j]  (fp32 [K][r]),   dB[j][n] = alpha sum_m H[m][j] dY[m][n]  (fp32 [r][N]); either may be NULL.
// X [M][K], dY [M][N], dH and H [M][rp] are bf16, 16-byte aligned; K, N and rp multiples of 8, r <= rp <= 32.
hipError_t launch_rank_grads(const void* X, const void* dH, float* dA, const void* H, const void* dY, float* dB, int64_t M, int64_t K,
                             int64_t r, int64_t rp, int64_t N, float alpha, hipStream_t s);

}  // namespace fhpc
