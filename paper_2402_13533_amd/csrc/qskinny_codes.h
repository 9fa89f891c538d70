// Device helpers that the weight-streaming forward kernels share: codes as matrix operands, buffer descriptors, and
// data that crosses workgroups within a launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fhpc {
namespace skinny {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr uint32_t OOB = 0x80000000u;      // a byte offset beyond any operand

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Exchange between the two halves of a wave: lanes 0..31 keep w[0], w[1] and get the upper
// partner's (lane + 32) w[0], w[1] in w[2], w[3]; lanes 32..63 keep w[2], w[3] and get the lower
// partner's w[2], w[3] in w[0], w[1].
__device__ __forceinline__ void exchange_halves(uint32_t (&w)[4])
{
    // v_permlane32_swap a, b: lanes 32..63 of a <-> lanes 0..31 of b
    auto s0 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    auto s1 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    w[0] = s0[0]; w[2] = s0[1];
    w[1] = s1[0]; w[3] = s1[1];
}

// eight int4 codes (one 32-bit word, element 2j in the low nibble of byte j) -> eight bf16
// values 128 + (q + 8).  The even and the odd nibbles are isolated as bytes (u = n ^ 8), and one
// byte permute per result word interleaves two of them with the constant byte 0x43, so the
// operand's k order is 0 2 4 6 1 3 5 7; the token tile is stored in the same order
// (x_even_odd_order).
__device__ __forceinline__ bf16x8 int4_operand(uint32_t w)
{
    const uint32_t lo = (w & 0x0f0f0f0fu) ^ 0x08080808u;            // u of elements 0 2 4 6
    const uint32_t hi = ((w >> 4) & 0x0f0f0f0fu) ^ 0x08080808u;     // u of elements 1 3 5 7
    const uint32_t c43 = 0x43434343u;
    u32x4 r;
    r.x = __builtin_amdgcn_perm(c43, lo, 0x04010400u);
    r.y = __builtin_amdgcn_perm(c43, lo, 0x04030402u);
    r.z = __builtin_amdgcn_perm(c43, hi, 0x04010400u);
    r.w = __builtin_amdgcn_perm(c43, hi, 0x04030402u);
    return as_bf16x8(r);
}

// eight consecutive bf16 (four words) -> the order 0 2 4 6 1 3 5 7
__device__ __forceinline__ u32x4 x_even_odd_order(u32x4 v)
{
    u32x4 r;
    r.x = __builtin_amdgcn_perm(v.y, v.x, 0x05040100u);
    r.y = __builtin_amdgcn_perm(v.w, v.z, 0x05040100u);
    r.z = __builtin_amdgcn_perm(v.y, v.x, 0x07060302u);
    r.w = __builtin_amdgcn_perm(v.w, v.z, 0x07060302u);
    return r;
}

// eight int8 codes (two words) -> eight bf16 values q + 128
__device__ __forceinline__ bf16x8 int8_operand(uint32_t w0, uint32_t w1)
{
    const uint32_t a = w0 ^ 0x80808080u, b = w1 ^ 0x80808080u;
    const float f0 = (float)(a & 0xffu), f1 = (float)((a >> 8) & 0xffu), f2 = (float)((a >> 16) & 0xffu), f3 = (float)(a >> 24);
    const float f4 = (float)(b & 0xffu), f5 = (float)((b >> 8) & 0xffu), f6 = (float)((b >> 16) & 0xffu), f7 = (float)(b >> 24);
    // the values are integers below 256: the upper 16 bits of the fp32 pattern are the exact bf16
    u32x4 r;
    r.x = __builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u);
    r.y = __builtin_amdgcn_perm(__float_as_uint(f3), __float_as_uint(f2), 0x07060302u);
    r.z = __builtin_amdgcn_perm(__float_as_uint(f5), __float_as_uint(f4), 0x07060302u);
    r.w = __builtin_amdgcn_perm(__float_as_uint(f7), __float_as_uint(f6), 0x07060302u);
    return as_bf16x8(r);
}

// Data that one workgroup writes and another reads within the launch (slabs, chunk sums of H, H) moves with
// device-scope accesses: a store goes through to the level all compute units share and a load comes from there,
// instruction by instruction.  (Ordinary accesses would need a device-scope fence on either side, which writes
// back and invalidates a whole L2 on this chip: measured, that made a launch 8 to 50 times slower.)
__device__ __forceinline__ void shared_store(float* p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float shared_load(const float* p)
{
    return __hip_atomic_load(const_cast<float*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace skinny
}  // namespace fhpc
