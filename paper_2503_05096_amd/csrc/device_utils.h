// Small device helpers shared by the gfx950 kernels: storage-type conversion,
// 64-lane wavefront reductions and scans.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace adaspec {

constexpr int kWave = 64;

// ---- storage types -------------------------------------------------------
struct F32 { using storage = float;    static constexpr int id = 0; };
struct F16 { using storage = uint16_t; static constexpr int id = 1; };
struct BF16 { using storage = uint16_t; static constexpr int id = 2; };

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ float f16_bits_to_float(uint16_t b)
{
    _Float16 h;
    __builtin_memcpy(&h, &b, 2);
    return (float)h;
}

// round-to-nearest-even from fp32
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x0040u);  // NaN stays NaN
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ uint16_t float_to_f16_bits(float f)
{
    _Float16 h = (_Float16)f;   // v_cvt_f16_f32, RNE
    uint16_t b;
    __builtin_memcpy(&b, &h, 2);
    return b;
}

template <class T> __device__ __forceinline__ float load_as_float(const void *base, int64_t idx);
template <> __device__ __forceinline__ float load_as_float<F32>(const void *base, int64_t idx)
{ return ((const float *)base)[idx]; }
template <> __device__ __forceinline__ float load_as_float<F16>(const void *base, int64_t idx)
{ return f16_bits_to_float(((const uint16_t *)base)[idx]); }
template <> __device__ __forceinline__ float load_as_float<BF16>(const void *base, int64_t idx)
{ return bf16_bits_to_float(((const uint16_t *)base)[idx]); }

// store one accumulator value in the requested output type
__device__ __forceinline__ void store_out(void *base, int64_t idx, float v, int out_dtype)
{
    if (out_dtype == 0)      ((float *)base)[idx] = v;
    else if (out_dtype == 1) ((uint16_t *)base)[idx] = float_to_f16_bits(v);
    else                     ((uint16_t *)base)[idx] = float_to_bf16_bits(v);
}

// ---- wavefront collectives ---------------------------------------------
// All of them use data-parallel-primitive moves inside the vector ALU: four shifts scan each row of 16 lanes, two row
// broadcasts carry the totals across, and lane 63 ends up with the reduction of all 64.  An exchange through LDS
// permutes costs a round trip of ~100 cycles per step (twice that for 8 bytes), and these reductions sit on the
// latency chains of the small kernels (MI355X: second acceptance pass of 64 requests 15.5 -> 14.6 us, fp32 rows 26.5 ->
// 25.1 us; draft sampling of 128 rows 26.2 -> 25.4 us).  All 64 lanes must be active.
// A lane without a source (first lanes of a row, rows a broadcast does not address) combines with `none`.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_move(uint32_t none, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows, class T>
__device__ __forceinline__ T dpp_shift(T none, T v)
{
    if constexpr (sizeof(T) == 8) {
        const unsigned long long n = __builtin_bit_cast(unsigned long long, none), x = __builtin_bit_cast(unsigned long long, v);
        const uint32_t lo = dpp_move<kCtrl, kRows>((uint32_t)n, (uint32_t)x);
        const uint32_t hi = dpp_move<kCtrl, kRows>((uint32_t)(n >> 32), (uint32_t)(x >> 32));
        return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(T, dpp_move<kCtrl, kRows>(__builtin_bit_cast(uint32_t, none), __builtin_bit_cast(uint32_t, v)));
    }
}
// inclusive scan over the 64 lanes with the operation f, whose neutral element is `none`
template <class T, class F>
__device__ __forceinline__ T wave_scan(T v, T none, F f)
{
    v = f(v, dpp_shift<0x111, 0xf>(none, v));   // row_shr:1
    v = f(v, dpp_shift<0x112, 0xf>(none, v));   // row_shr:2
    v = f(v, dpp_shift<0x114, 0xf>(none, v));   // row_shr:4
    v = f(v, dpp_shift<0x118, 0xf>(none, v));   // row_shr:8 -> scan inside each row of 16
    v = f(v, dpp_shift<0x142, 0xa>(none, v));   // row_bcast:15 into rows 1 and 3
    v = f(v, dpp_shift<0x143, 0xc>(none, v));   // row_bcast:31 into rows 2 and 3
    return v;
}
template <class T>
__device__ __forceinline__ T last_lane(T v)
{
    if constexpr (sizeof(T) == 8) {
        const unsigned long long x = __builtin_bit_cast(unsigned long long, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), 63);
        return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane((int)__builtin_bit_cast(uint32_t, v), 63));
    }
}
__device__ __forceinline__ float wave_max(float v)
{
    return last_lane(wave_scan(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); }));
}
__device__ __forceinline__ int wave_max(int v)
{
    return last_lane(wave_scan(v, (int)0x80000000, [](int a, int b) { return max(a, b); }));
}
__device__ __forceinline__ float wave_sum(float v)
{
    return last_lane(wave_scan(v, 0.f, [](float a, float b) { return a + b; }));
}
__device__ __forceinline__ double wave_sum(double v)
{
    return last_lane(wave_scan(v, 0.0, [](double a, double b) { return a + b; }));
}
__device__ __forceinline__ int wave_sum(int v)
{
    return last_lane(wave_scan(v, 0, [](int a, int b) { return a + b; }));
}
// inclusive scans over the 64 lanes
__device__ __forceinline__ double wave_scan_incl(double v, int)
{
    return wave_scan(v, 0.0, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ int wave_scan_incl(int v, int)
{
    return wave_scan(v, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_scan_incl_dpp(int v) { return wave_scan_incl(v, 0); }

// (value, index) max with the LOWEST index winning ties
struct ArgMax { float v; int i; };
__device__ __forceinline__ ArgMax argmax_merge(ArgMax a, ArgMax b)
{
    return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
__device__ __forceinline__ ArgMax wave_argmax(ArgMax a)
{
    a = wave_scan(a, ArgMax{-INFINITY, 0x7fffffff}, [](ArgMax x, ArgMax y) { return argmax_merge(x, y); });
    return last_lane(a);
}

// Lowest / highest thread number with a flag, over the workgroup (*word preset by the caller, read behind a barrier): one
// LDS atomic per wavefront.  An atomic by every flagged thread is a loop over the lanes (about 1 us per wavefront).
__device__ __forceinline__ void note_first(int *word, bool flag, int tid)
{
    const unsigned long long b = __ballot(flag);
    if (b && (tid & 63) == 0) atomicMin(word, (tid & ~63) + (int)__builtin_ctzll(b));
}
__device__ __forceinline__ void note_last(int *word, bool flag, int tid)
{
    const unsigned long long b = __ballot(flag);
    if (b && (tid & 63) == 0) atomicMax(word, (tid & ~63) + 63 - (int)__builtin_clzll(b));
}

// Workgroup barrier for data exchanged through LDS only.  __syncthreads() also drains the
// vector-memory counter (its fences cover global memory), which would stall on every global load
// that was deliberately left in flight across the barrier; this one waits for LDS traffic alone.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__host__ __device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ __forceinline__ size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

}  // namespace adaspec
