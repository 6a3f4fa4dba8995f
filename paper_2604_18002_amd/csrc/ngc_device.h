// Shared device helpers for the gfx950 kernels: wave64 primitives, block
// scans and reductions.  Everything assumes 64-wide wavefronts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define NGC_WAVE 64

#define NGC_HIP_CHECK(expr)                         \
    do {                                            \
        hipError_t _e = (expr);                     \
        if (_e != hipSuccess) return NGC_EHIP;      \
    } while (0)

namespace ngc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// 2^x by the hardware instruction (-inf -> 0); for exponents <= 0 or small.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (NGC_WAVE - 1); }
__device__ __forceinline__ int wave_id() { return threadIdx.x >> 6; }

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ int popc_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// Reductions over the four lanes {l, l ^ 16, l ^ 32, l ^ 48} (the lane groups that share lane % 16 in the
// attention kernels), result in all four.  gfx950's lane-swap instructions exchange the halves / the odd and even
// rows of two registers inside the vector ALU: with both operands holding x, one comes back as [lo, lo] and the
// other as [hi, hi] (rows [r0, r0, r2, r2] and [r1, r1, r3, r3]), so combining the pair is the xor-32 (xor-16)
// step of a butterfly -- without the trip through LDS that a shuffle takes.
// max of two numbers that are known not to be NaN: the median of (a, b, +inf), one instruction, where fmaxf()
// first spends one more on each operand whose origin the compiler cannot see (a matrix-core result, a lane swap)
// to quiet a signalling NaN.
__device__ __forceinline__ float max_no_nan(float a, float b)
{
    return __builtin_amdgcn_fmed3f(a, b, __builtin_inff());
}
__device__ __forceinline__ float quad_rows_max(float v)
{
    uint32_t u = __float_as_uint(v);
    auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = __float_as_uint(max_no_nan(__uint_as_float(a[0]), __uint_as_float(a[1])));
    auto b = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return max_no_nan(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_rows_sum(float v)
{
    uint32_t u = __float_as_uint(v);
    auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// The same over the two lanes {l, l ^ 32} (the lane halves that share lane % 32 in 32-wide matrix tiles).
__device__ __forceinline__ float half_rows_max(float v)
{
    const uint32_t u = __float_as_uint(v);
    auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return max_no_nan(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float half_rows_sum(float v)
{
    const uint32_t u = __float_as_uint(v);
    auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// 16 bytes per lane from memory straight into LDS, lane l to lds + 16 l (lds wave-uniform).  Counts as a vector memory
// load; lds_loads_done() stands between it and the first use by any wave.
__device__ __forceinline__ void load_to_lds16(const void *src, void *lds)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) uint32_t *)(uintptr_t)src,
                                     (__attribute__((address_space(3))) uint32_t *)lds, 16, 0, 0);
}

__device__ __forceinline__ void lds_loads_done()
{
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's; the barrier makes it every wave's
    __syncthreads();
}

// Four 16-bit values per lane from LDS, transposed within each 16 lanes: lane x gets value x % 4 of the lanes x / 4,
// 4 + x / 4, 8 + x / 4, 12 + x / 4 (each lane's own address names four consecutive values).
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 read_transposed16(const void *lds)
{
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)lds));
}

// Whole-wave reductions and scans inside the vector ALU: lanes exchange within their row of 16 by data-parallel
// primitives (a shuffle through LDS costs ~60 cycles a step, these ~8), across rows by gfx950's lane-swap instructions.
namespace dpp {
constexpr int QUAD_XOR1 = 0xB1, QUAD_XOR2 = 0x4E, HALF_MIRROR = 0x141, MIRROR = 0x140;   // together: xor 1, 2, 4, 8
constexpr int ROW_SHR = 0x110;                                                           // + n: from n lanes below
constexpr int BCAST15 = 0x142, BCAST31 = 0x143;                                          // a row's last lane to the next row(s)
// lane's partner value; lanes without one (or outside ROWS) get `none`
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t from(uint32_t v, uint32_t none)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xF, false);
}
}  // namespace dpp

// op(a, b) over all 64 lanes, result in every lane.  T is a 32-bit type.
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op)
{
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    auto step = [&](uint32_t w) { u = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(T, u), __builtin_bit_cast(T, w))); };
    step(dpp::from<dpp::QUAD_XOR1>(u, u));
    step(dpp::from<dpp::QUAD_XOR2>(u, u));
    step(dpp::from<dpp::HALF_MIRROR>(u, u));
    step(dpp::from<dpp::MIRROR>(u, u));
    auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = a[0];
    step(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = b[0];
    step(b[1]);
    return __builtin_bit_cast(T, u);
}
// op over this lane and those below it (`none`: the neutral element)
template <class T, class Op>
__device__ __forceinline__ T wave_incl_scan(T v, T none, Op op)
{
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    const uint32_t z = __builtin_bit_cast(uint32_t, none);
    auto step = [&](uint32_t w) { u = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(T, w), __builtin_bit_cast(T, u))); };
    step(dpp::from<dpp::ROW_SHR + 1>(u, z));
    step(dpp::from<dpp::ROW_SHR + 2>(u, z));
    step(dpp::from<dpp::ROW_SHR + 4>(u, z));
    step(dpp::from<dpp::ROW_SHR + 8>(u, z));
    step(dpp::from<dpp::BCAST15, 0xA>(u, z));     // rows 1 and 3 take the row below's total
    step(dpp::from<dpp::BCAST31, 0xC>(u, z));     // rows 2 and 3 that of the lower half
    return __builtin_bit_cast(T, u);
}
struct OpAdd {
    template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; }
};
struct OpMaxF {
    __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
struct OpMaxU {
    __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};
__device__ __forceinline__ float wave_sum_f(float v) { return wave_reduce(v, OpAdd{}); }
__device__ __forceinline__ float wave_max_f(float v) { return wave_reduce(v, OpMaxF{}); }
__device__ __forceinline__ int wave_incl_scan_i(int v) { return wave_incl_scan(v, 0, OpAdd{}); }
__device__ __forceinline__ float wave_incl_scan_f(float v) { return wave_incl_scan(v, 0.f, OpAdd{}); }

// Block-wide exclusive scan of one int per thread.  `tmp` holds one int per
// wave (+1).  Returns the exclusive prefix; *total receives the block sum.
// Contains two barriers; every thread of the block must call it.
template <int THREADS>
__device__ __forceinline__ int block_excl_scan_i(int v, int *tmp, int *total)
{
    constexpr int NW = THREADS / NGC_WAVE;
    const int incl = wave_incl_scan_i(v);
    if (lane_id() == NGC_WAVE - 1) tmp[wave_id()] = incl;
    __syncthreads();
    int base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        int t = tmp[w];
        if (w < wave_id()) base += t;
        all += t;
    }
    __syncthreads();
    *total = all;
    return base + incl - v;
}

template <int THREADS>
__device__ __forceinline__ float block_excl_scan_f(float v, float *tmp, float *total)
{
    constexpr int NW = THREADS / NGC_WAVE;
    const float incl = wave_incl_scan_f(v);
    if (lane_id() == NGC_WAVE - 1) tmp[wave_id()] = incl;
    __syncthreads();
    float base = 0.f, all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        float t = tmp[w];
        if (w < wave_id()) base += t;
        all += t;
    }
    __syncthreads();
    *total = all;
    float prev = __shfl_up(incl, 1, NGC_WAVE);   // sum of the lanes below, no subtraction
    if (lane_id() == 0) prev = 0.f;
    return base + prev;
}

// Sum of the values of the threads ABOVE this one, and of all (an exclusive scan from the last thread down).
template <int THREADS>
__device__ __forceinline__ float block_above_scan_f(float v, float *tmp, float *total)
{
    constexpr int NW = THREADS / NGC_WAVE;
    float incl = v;   // this lane and those above it
#pragma unroll
    for (int o = 1; o < NGC_WAVE; o <<= 1) {
        const float t = __shfl_down(incl, o, NGC_WAVE);
        if (lane_id() + o < NGC_WAVE) incl += t;
    }
    if (lane_id() == 0) tmp[wave_id()] = incl;
    __syncthreads();
    float base = 0.f, all = 0.f;
#pragma unroll
    for (int w = NW - 1; w >= 0; --w) {
        const float t = tmp[w];
        if (w > wave_id()) base += t;
        all += t;
    }
    __syncthreads();
    *total = all;
    float prev = __shfl_down(incl, 1, NGC_WAVE);
    if (lane_id() == NGC_WAVE - 1) prev = 0.f;
    return base + prev;
}

template <int THREADS>
__device__ __forceinline__ float block_sum_f(float v, float *tmp)
{
    constexpr int NW = THREADS / NGC_WAVE;
    v = wave_sum_f(v);
    if (lane_id() == 0) tmp[wave_id()] = v;
    __syncthreads();
    float all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) all += tmp[w];
    __syncthreads();
    return all;
}

// Two maxima in one pass (same barriers as one).  `tmp` holds two floats per wave.
template <int THREADS>
__device__ __forceinline__ void block_max2_f(float &a, float &b, float *tmp)
{
    constexpr int NW = THREADS / NGC_WAVE;
    a = wave_max_f(a);
    b = wave_max_f(b);
    if (lane_id() == 0) { tmp[2 * wave_id()] = a; tmp[2 * wave_id() + 1] = b; }
    __syncthreads();
    a = tmp[0];
    b = tmp[1];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        a = fmaxf(a, tmp[2 * w]);
        b = fmaxf(b, tmp[2 * w + 1]);
    }
    __syncthreads();
}

template <int THREADS>
__device__ __forceinline__ uint32_t block_max_u(uint32_t v, uint32_t *tmp)
{
    constexpr int NW = THREADS / NGC_WAVE;
    v = wave_reduce(v, OpMaxU{});
    if (lane_id() == 0) tmp[wave_id()] = v;
    __syncthreads();
    uint32_t all = tmp[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) all = tmp[w] > all ? tmp[w] : all;
    __syncthreads();
    return all;
}

}  // namespace ngc
