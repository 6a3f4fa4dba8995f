// Shared device helpers for the gfx950 kernels: wave64 primitives, block
// scans and reductions.  Everything assumes 64-wide wavefronts.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ngc.h"

#define NGC_WAVE 64

#define NGC_HIP_CHECK(expr)                         \
    do {                                            \
        hipError_t _e = (expr);                     \
        if (_e != hipSuccess) return NGC_EHIP;      \
    } while (0)

namespace ngc {

// A launch of a kernel whose argument is one struct, by a single call of the runtime.  (The <<<>>> form makes three and another
// one asks for the error: 0.1-0.3 us of the 4.4-5 us that the smallest calls cost the host.)
template <class Args>
inline int launch(const void *kernel, dim3 grid, dim3 block, size_t lds, hipStream_t stream, Args &args)
{
    void *kargs[] = {&args};
    if (hipLaunchKernel(kernel, grid, block, kargs, lds, stream) == hipSuccess) return NGC_OK;
    (void)hipGetLastError();                 // not left for the next call to find
    return NGC_EHIP;
}

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
// IEEE maximum and minimum: NaN if an operand is one; two of them on the way to a third value are one instruction.
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float min_or_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }
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
constexpr int ROW_SHR = 0x110, ROW_SHL = 0x100;                                          // + n: from n lanes below, above
constexpr int WAVE_SHR1 = 0x138, WAVE_SHL1 = 0x130;                                      // from the lane below, above
constexpr int BCAST15 = 0x142, BCAST31 = 0x143;                                          // a row's last lane to the next row(s)
// the partner's value, for exchanges in which every lane has one (the compiler folds them into the operation that follows)
template <int CTRL>
__device__ __forceinline__ uint32_t swapped(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
// the value of the lane that CTRL names, 0 where there is none (likewise)
template <int CTRL>
__device__ __forceinline__ uint32_t shifted(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
// the same for lanes of the rows in ROWS; the others get 0
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t broadcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
}  // namespace dpp

// op(a, b) over all 64 lanes, result in every lane.  T is a 32-bit type.
template <class T, class Op>
__device__ __forceinline__ T wave_reduce(T v, Op op)
{
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    auto step = [&](uint32_t w) { u = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(T, u), __builtin_bit_cast(T, w))); };
    step(dpp::swapped<dpp::QUAD_XOR1>(u));
    step(dpp::swapped<dpp::QUAD_XOR2>(u));
    step(dpp::swapped<dpp::HALF_MIRROR>(u));
    step(dpp::swapped<dpp::MIRROR>(u));
    auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = a[0];
    step(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = b[0];
    step(b[1]);
    return __builtin_bit_cast(T, u);
}
// Sum over this lane and those below it.
template <class T>
__device__ __forceinline__ T wave_incl_scan(T v)
{
    auto bits = [](T x) { return __builtin_bit_cast(uint32_t, x); };
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 1>(bits(v)));
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 2>(bits(v)));
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 4>(bits(v)));
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 8>(bits(v)));
    v += __builtin_bit_cast(T, dpp::broadcast<dpp::BCAST15, 0xA>(bits(v)));   // rows 1 and 3 take the row below's total
    v += __builtin_bit_cast(T, dpp::broadcast<dpp::BCAST31, 0xC>(bits(v)));   // rows 2 and 3 that of the lower half
    return v;
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
__device__ __forceinline__ int wave_incl_scan_i(int v) { return wave_incl_scan(v); }
__device__ __forceinline__ float wave_incl_scan_f(float v) { return wave_incl_scan(v); }
// The same sum in 64 bits (both words travel).
__device__ __forceinline__ double wave_sum_d(double v)
{
    auto pair = [](uint32_t lo, uint32_t hi) { return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo); };
    uint32_t lo, hi;
    auto halves = [&] {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        lo = (uint32_t)b;
        hi = (uint32_t)(b >> 32);
    };
    halves(); v += pair(dpp::swapped<dpp::QUAD_XOR1>(lo), dpp::swapped<dpp::QUAD_XOR1>(hi));
    halves(); v += pair(dpp::swapped<dpp::QUAD_XOR2>(lo), dpp::swapped<dpp::QUAD_XOR2>(hi));
    halves(); v += pair(dpp::swapped<dpp::HALF_MIRROR>(lo), dpp::swapped<dpp::HALF_MIRROR>(hi));
    halves(); v += pair(dpp::swapped<dpp::MIRROR>(lo), dpp::swapped<dpp::MIRROR>(hi));
    halves();
    auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = pair(a[0], b[0]) + pair(a[1], b[1]);
    halves();
    a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return pair(a[0], b[0]) + pair(a[1], b[1]);
}
// The value of the lane below (above); 0 for the first (last).
__device__ __forceinline__ float lane_below_f(float v)
{
    return __uint_as_float(dpp::shifted<dpp::WAVE_SHR1>(__float_as_uint(v)));
}
__device__ __forceinline__ float lane_above_f(float v)
{
    return __uint_as_float(dpp::shifted<dpp::WAVE_SHL1>(__float_as_uint(v)));
}
// Sum over this lane and those above it.
__device__ __forceinline__ float wave_above_scan_f(float v)
{
    v += __uint_as_float(dpp::shifted<dpp::ROW_SHL + 1>(__float_as_uint(v)));
    v += __uint_as_float(dpp::shifted<dpp::ROW_SHL + 2>(__float_as_uint(v)));
    v += __uint_as_float(dpp::shifted<dpp::ROW_SHL + 4>(__float_as_uint(v)));
    v += __uint_as_float(dpp::shifted<dpp::ROW_SHL + 8>(__float_as_uint(v)));
    // the rows above: their sums stand in their first lanes
    auto first_of = [&](int lane) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane(__float_as_uint(v), lane)); };
    const float r3 = first_of(48), r2 = first_of(32) + r3, r1 = first_of(16) + r2;
    const int row = lane_id() >> 4;
    return v + (row == 0 ? r1 : row == 1 ? r2 : row == 2 ? r3 : 0.f);
}

// What the NW <= 16 waves of a workgroup have left in tmp[0], tmp[STRIDE], ... combined by every wave: a lane takes one
// of the values, data-parallel steps within the row of 16 do the rest (2 to 4 of them; a loop over the values costs
// every wave two or three instructions for each).
template <int NW, class T, class Op>
__device__ __forceinline__ T lanes_reduce(T v, Op op)      // of lanes that hold the NW values again and again
{
    static_assert(NW == 4 || NW == 8 || NW == 16, "whole rows of lanes");
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    auto step = [&](uint32_t w) { u = __builtin_bit_cast(uint32_t, op(__builtin_bit_cast(T, u), __builtin_bit_cast(T, w))); };
    step(dpp::swapped<dpp::QUAD_XOR1>(u));
    step(dpp::swapped<dpp::QUAD_XOR2>(u));
    if constexpr (NW > 4) step(dpp::swapped<dpp::HALF_MIRROR>(u));
    if constexpr (NW > 8) step(dpp::swapped<dpp::MIRROR>(u));
    return __builtin_bit_cast(T, u);
}
template <int NW, int STRIDE, class T, class Op>
__device__ __forceinline__ T across_waves(const T *tmp, Op op)
{
    return lanes_reduce<NW>(tmp[(lane_id() & (NW - 1)) * STRIDE], op);
}
// The sum of the values of the waves below this one, *total: of all.  ABOVE: of the waves above this one.
template <int NW, int STRIDE, bool ABOVE = false, class T>
__device__ __forceinline__ T below_waves(const T *tmp, T *total)
{
    static_assert(NW == 4 || NW == 8 || NW == 16, "whole rows of lanes");
    const int lane = lane_id() & (NW - 1);
    const int wv = __builtin_amdgcn_readfirstlane(wave_id());
    T v = tmp[(ABOVE ? NW - 1 - lane : lane) * STRIDE];
    auto bits = [](T x) { return __builtin_bit_cast(uint32_t, x); };
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 1>(bits(v)));
    v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 2>(bits(v)));
    if constexpr (NW > 4) v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 4>(bits(v)));
    if constexpr (NW > 8) v += __builtin_bit_cast(T, dpp::shifted<dpp::ROW_SHR + 8>(bits(v)));
    const uint32_t before = dpp::shifted<dpp::ROW_SHR + 1>(bits(v));
    *total = __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane((int)bits(v), NW - 1));
    return __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane((int)before, ABOVE ? NW - 1 - wv : wv));
}

// Block-wide exclusive scan of one int per thread.  `tmp` holds one int per
// wave (+1).  Returns the exclusive prefix; *total receives the block sum.
// Contains two barriers; every thread of the block must call it.
template <int THREADS>
__device__ __forceinline__ int block_excl_scan_i(int v, int *tmp, int *total)
{
    const int incl = wave_incl_scan_i(v);
    if (lane_id() == NGC_WAVE - 1) tmp[wave_id()] = incl;
    __syncthreads();
    const int base = below_waves<THREADS / NGC_WAVE, 1>(tmp, total);
    __syncthreads();
    return base + incl - v;
}

template <int THREADS>
__device__ __forceinline__ float block_excl_scan_f(float v, float *tmp, float *total)
{
    const float incl = wave_incl_scan_f(v);
    if (lane_id() == NGC_WAVE - 1) tmp[wave_id()] = incl;
    __syncthreads();
    const float base = below_waves<THREADS / NGC_WAVE, 1>(tmp, total);
    __syncthreads();
    return base + lane_below_f(incl);            // sum of the lanes below, no subtraction
}

// Sum of the values of the threads ABOVE this one, and of all (an exclusive scan from the last thread down).
template <int THREADS>
__device__ __forceinline__ float block_above_scan_f(float v, float *tmp, float *total)
{
    const float incl = wave_above_scan_f(v);     // this lane and those above it
    if (lane_id() == 0) tmp[wave_id()] = incl;
    __syncthreads();
    const float base = below_waves<THREADS / NGC_WAVE, 1, true>(tmp, total);
    __syncthreads();
    return base + lane_above_f(incl);
}

template <int THREADS>
__device__ __forceinline__ float block_sum_f(float v, float *tmp)
{
    v = wave_sum_f(v);
    if (lane_id() == 0) tmp[wave_id()] = v;
    __syncthreads();
    const float all = across_waves<THREADS / NGC_WAVE, 1>(tmp, OpAdd{});
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
    a = across_waves<NW, 2>(tmp, OpMaxF{});
    b = across_waves<NW, 2>(tmp + 1, OpMaxF{});
    __syncthreads();
}

// Largest of the first and smallest of the second over all threads, NaN if one of them is.  `tmp` as above.
template <int THREADS>
__device__ __forceinline__ void block_max_min(float &a, float &b, float *tmp)
{
    constexpr int NW = THREADS / NGC_WAVE;
    const auto larger = [](float x, float y) { return max_or_nan(x, y); };
    const auto smaller = [](float x, float y) { return min_or_nan(x, y); };
    a = wave_reduce(a, larger);
    b = wave_reduce(b, smaller);
    if (lane_id() == 0) { tmp[2 * wave_id()] = a; tmp[2 * wave_id() + 1] = b; }
    __syncthreads();
    a = across_waves<NW, 2>(tmp, larger);
    b = across_waves<NW, 2>(tmp + 1, smaller);
    __syncthreads();
}

template <int THREADS>
__device__ __forceinline__ uint32_t block_max_u(uint32_t v, uint32_t *tmp)
{
    v = wave_reduce(v, OpMaxU{});
    if (lane_id() == 0) tmp[wave_id()] = v;
    __syncthreads();
    const uint32_t all = across_waves<THREADS / NGC_WAVE, 1>(tmp, OpMaxU{});
    __syncthreads();
    return all;
}

}  // namespace ngc
