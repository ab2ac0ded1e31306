// Device-side building blocks shared by the SSD kernels (gfx950 / CDNA4).
//
// Matrix-core convention used throughout.  A 16x16 output tile is produced by
// contraction steps in which lane l holds row (A operand) or column (B operand)
// r = l & 15 and, by its lane group g = l >> 4, some of the contraction indices:
//   * bf16: v_mfma_f32_16x16x32_bf16, eight indices per lane (32 a step);
//   * f32 : v_mfma_f32_16x16x4_f32, one index per lane (4 a step).
// Any assignment of indices to (group, slot) gives the same sum, as long as
// both operands use the same one.  The accumulator (4 floats per lane) holds
// D[4 g + v][r], v = 0..3.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssd {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;

// Activation element access: float, or bfloat16 stored as its 16 bits.
template <typename T>
struct Act;

// The block path's dt: softplus(v) = max(v, 0) + log(1 + e^-|v|) (no overflow
// on either side), after the head's bias, then the clamp.
__device__ __forceinline__ float softplus_f(float v) { return fmaxf(v, 0.f) + log1pf(expf(-fabsf(v))); }

template <>
struct Act<float> {
    static __device__ __forceinline__ float load(const float* p, int64_t i) { return p[i]; }
    static __device__ __forceinline__ void store(float* p, int64_t i, float v) { p[i] = v; }
};

template <>
struct Act<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t* p, int64_t i)
    {
        return __uint_as_float(static_cast<uint32_t>(p[i]) << 16);
    }
    // round to nearest even (inputs are finite)
    static __device__ __forceinline__ void store(uint16_t* p, int64_t i, float v)
    {
        uint32_t u = __float_as_uint(v);
        u += 0x7FFFu + ((u >> 16) & 1u);
        p[i] = static_cast<uint16_t>(u >> 16);
    }
};

__device__ __forceinline__ f32x4_t zero4()
{
    f32x4_t z = {0.f, 0.f, 0.f, 0.f};
    return z;
}

// Four consecutive activations as floats.  Rows are multiples of 16 elements,
// but the caller's pointers need only be aligned to their own type, so the
// vectors say so (the hardware reads and writes them at any alignment).
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t h4u_t __attribute__((ext_vector_type(4), aligned(2)));

__device__ __forceinline__ f32x4_t load4(const float* p)
{
    const f4u_t v = *reinterpret_cast<const f4u_t*>(p);
    return f32x4_t{v.x, v.y, v.z, v.w};
}

__device__ __forceinline__ f32x4_t load4(const uint16_t* p)
{
    const h4u_t v = *reinterpret_cast<const h4u_t*>(p);
    f32x4_t f;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = __uint_as_float(static_cast<uint32_t>(v[e]) << 16);
    return f;
}

__device__ __forceinline__ void store4(float* p, f32x4_t v) { *reinterpret_cast<f4u_t*>(p) = f4u_t{v[0], v[1], v[2], v[3]}; }

__device__ __forceinline__ void store4(uint16_t* p, f32x4_t v)
{
    h4u_t h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint16_t u;
        Act<uint16_t>::store(&u, 0, v[e]);   // round to nearest even
        h[e] = u;
    }
    *reinterpret_cast<h4u_t*>(p) = h;
}

// One float32 matrix instruction: D[4 g + v][r] += sum over the lane groups
// g' = 0..3 of A (row r of the lane) x B (column r of the lane).
__device__ __forceinline__ f32x4_t mma4(float a, float b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sixteen wait states between matrix instructions of a loop with a run-time
// trip count and the first read of their results after it (the compiler has
// been seen to leave too few on one path out of such a loop).
__device__ __forceinline__ void settle(f32x4_t& a) { asm volatile("s_nop 15" : "+v"(a)); }

// Cross-lane sums in registers (DPP and the permlane swaps; no trip through
// shared memory).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}

// Sum over the 16 lanes of each row (row_ror by 8, 4, 2, 1): every lane of the row gets it.
__device__ __forceinline__ float row_sum16(float v)
{
    v += dpp<0x128, 0xF>(v);
    v += dpp<0x124, 0xF>(v);
    v += dpp<0x122, 0xF>(v);
    v += dpp<0x121, 0xF>(v);
    return v;
}

// Sum over the four rows at each position (lanes r, r + 16, r + 32, r + 48):
// swapping odd rows with even ones, then the halves, and adding.
__device__ __forceinline__ float col_sum4(float v)
{
    uint32_t u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    u = __float_as_uint(v);
    const auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Sum over the 64 lanes of a wavefront (every lane gets it).
__device__ __forceinline__ float wave_sum(float v) { return col_sum4(row_sum16(v)); }

// Inclusive prefix sum over the 64 lanes: shifts by 1, 2, 4, 8 within each
// row, then the row totals carried up by broadcasts of lanes 15 (into rows 1
// and 3) and 31 (into rows 2 and 3).  Lanes with no source add zero.
__device__ __forceinline__ float wave_scan(float v)
{
    v += dpp<0x111, 0xF>(v);
    v += dpp<0x112, 0xF>(v);
    v += dpp<0x114, 0xF>(v);
    v += dpp<0x118, 0xF>(v);
    v += dpp<0x142, 0xA>(v);
    v += dpp<0x143, 0xC>(v);
    return v;
}

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Inclusive prefix sum over the first `nthreads` (a multiple of 64, <= 1024)
// threads of the block; `scratch` holds nthreads/64 floats of shared memory.
__device__ __forceinline__ float block_inclusive_scan(float v, float* scratch)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        float o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    if (lane == 63) scratch[wave] = v;
    __syncthreads();
    float off = 0.f;
    for (int w = 0; w < wave; ++w) off += scratch[w];
    __syncthreads();
    return v + off;
}

}  // namespace ssd
