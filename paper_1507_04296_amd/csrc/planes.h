// fp32 products on v_mfma_f32_16x16x32_bf16: an operand is a sum of bf16
// planes (three hold an fp32 value: hi + mid + lo, each the rounded remainder
// of the previous, 8 + 8 + 8 significant bits; bf16 values are one plane), and
// of the nine plane products of two fp32 operands the three below 2^-24 of the
// value (mid*lo, lo*mid, lo*lo) are left out.  Each plane product is exact in
// fp32, so only the accumulation rounds.  An operand loses low bits below about
// 2^-110, and one that rounds to bf16's infinity (finite, from 0x1.ffp127 =
// 3.396e38 on) is infinite; infinite and NaN operands give the infinities and
// NaNs of the fp32 instruction (plane_sum).
//
// Operand layout: lane l holds row (A) or column (B) l % 16 and the reduction
// indices 8 (l / 16) .. +7; accumulator element e of lane l is row 4 (l / 16)
// + e, column l % 16.
#pragma once
#include "common.h"

namespace gorila {

// Four values as NP bf16 planes (two values per rounding; the remainders are exact).
template <int NP>
__device__ __forceinline__ void split4(f32x4 v, bf16x4 (&o)[NP]) {
    f32x2 a{v[0], v[1]}, b{v[2], v[3]};
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
        const bf16x2 ha = __builtin_convertvector(a, bf16x2), hb = __builtin_convertvector(b, bf16x2);
        o[pl] = __builtin_shufflevector(ha, hb, 0, 1, 2, 3);
        if (pl + 1 < NP) {
            const uint32_t ba = __builtin_bit_cast(uint32_t, ha), bb = __builtin_bit_cast(uint32_t, hb);
            a = f32x2{a[0] - __uint_as_float(ba << 16), a[1] - __uint_as_float(ba & 0xffff0000u)};
            b = f32x2{b[0] - __uint_as_float(bb << 16), b[1] - __uint_as_float(bb & 0xffff0000u)};
        }
    }
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The sum of the leading products' accumulator and the others' (of P planes an
// operand at most).  An infinite operand is (inf, NaN, NaN) in planes, so its
// leading products are infinite, or NaN against a zero, as the fp32
// instruction's are, but the others are NaN or infinite: they are held within
// the finite numbers (a NaN becomes the lowest), so that the leading sum decides
// (a ReLU would turn the NaN into zero).
template <int P>
__device__ __forceinline__ float plane_sum(float hi, float lo) {
    return hi + (P > 1 ? __builtin_amdgcn_fmed3f(lo, -0x1.fffffep127f, 0x1.fffffep127f) : lo);
}
template <int P>
__device__ __forceinline__ f32x4 plane_sum(f32x4 hi, f32x4 lo) {
    return f32x4{plane_sum<P>(hi[0], lo[0]), plane_sum<P>(hi[1], lo[1]), plane_sum<P>(hi[2], lo[2]),
                 plane_sum<P>(hi[3], lo[3])};
}

// A copy of a value that the compiler cannot see through: what derives from
// it is computed where it is used, per sample, instead of being kept in
// registers over the whole row loop.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Quads of fp32 values or of bf16 bit patterns (widened exactly; stored rounded).
__device__ inline f32x4 ldq(const float* p) { return ld4(p); }
__device__ inline f32x4 ldq(const uint16_t* p) {
    const uint2 v = *(const uint2*)p;
    return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                 __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
}
__device__ inline void stq(float* p, f32x4 v) { *(f32x4*)p = v; }
__device__ inline void stq(uint16_t* p, f32x4 v) {
    bf16x4 o[1];
    split4<1>(v, o);
    *(bf16x4*)p = o[0];
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

__device__ inline float ldv(const float* p) { return *p; }
__device__ inline float ldv(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }
__device__ inline void stv(float* p, float v) { *p = v; }
__device__ inline void stv(uint16_t* p, float v) { *p = __builtin_bit_cast(uint16_t, (__bf16)v); }
// The same quads at any element's address.
__device__ inline f32x4 ldqa(const float* p) { return *(const f32x4a*)p; }
__device__ inline f32x4 ldqa(const uint16_t* p) {
    const u16x4a v = *(const u16x4a*)p;
    return f32x4{__uint_as_float((uint32_t)v[0] << 16), __uint_as_float((uint32_t)v[1] << 16),
                 __uint_as_float((uint32_t)v[2] << 16), __uint_as_float((uint32_t)v[3] << 16)};
}

// One reduction step of 32: products of R row tiles with the column tiles J0 ..
// J0 + C - 1, the leading ones into hi, the others into lo.  Each plane pair is a
// round of R C independent instructions; the scheduling barriers (APART) keep the
// rounds apart, where the compiler would run one accumulator's chain back to back,
// each waiting for the one before, and let everything but matrix instructions pass.
template <int J0, bool APART = true, int PA, int PX, int R, int C, int N>
__device__ __forceinline__ void plane_products(const bf16x8 (&a)[R][PA], const bf16x8 (&x)[C][PX],
                                               f32x4 (&hi)[R][N], f32x4 (&lo)[R][N]) {
    auto round = [&](auto pc, auto qc, f32x4 (&acc)[R][N]) {
        constexpr int pa = decltype(pc)::value, px = decltype(qc)::value;
        if constexpr (pa < PA && px < PX) {
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < C; ++j) acc[i][J0 + j] = mfma16(a[i][pa], x[j][px], acc[i][J0 + j]);
            if constexpr (APART) __builtin_amdgcn_sched_barrier(0x7f6);
        }
    };
    constexpr std::integral_constant<int, 0> I0{};
    constexpr std::integral_constant<int, 1> I1{};
    constexpr std::integral_constant<int, 2> I2{};
    round(I0, I0, hi);
    round(I0, I1, lo);
    round(I1, I0, lo);
    round(I0, I2, lo);
    round(I1, I1, lo);
    round(I2, I0, lo);
}

}  // namespace gorila
