// f2.hpp -- arithmetic in F_{p^2} = F_p[i] / (i^2 + 1), p = 2^61 - 1, for the
// device kernels of fp2.hip and fs.hip: canonical helpers, and loose ones for
// the hot loops (parts are folded residues below 2^61 + 8, m61.hpp).
#pragma once
#include "common.hpp"
#include "m61.hpp"

namespace ra {

struct f2 {
    uint64_t re, im;
};

// ---- canonical parts ----
__device__ __forceinline__ f2 f2of(uint64_t a) { return f2{a, 0}; }
__device__ __forceinline__ f2 f2add(f2 a, f2 b) { return f2{m61::add(a.re, b.re), m61::add(a.im, b.im)}; }
__device__ __forceinline__ f2 f2sub(f2 a, f2 b) { return f2{m61::sub(a.re, b.re), m61::sub(a.im, b.im)}; }
// (a0 + a1 i)(b0 + b1 i) = (a0 b0 - a1 b1) + ((a0 + a1)(b0 + b1) - a0 b0 - a1 b1) i:
// three products of F_p instead of four
__device__ __forceinline__ f2 f2mul(f2 a, f2 b)
{
    const uint64_t p0 = m61::mul(a.re, b.re), p1 = m61::mul(a.im, b.im);
    const uint64_t p2 = m61::mul(m61::add(a.re, a.im), m61::add(b.re, b.im));
    return f2{m61::sub(p0, p1), m61::sub(m61::sub(p2, p0), p1)};
}
// a c for a small integer c (|c| < 2^31)
__device__ __forceinline__ f2 f2small(f2 a, int32_t c) { return f2{m61::mul_small(a.re, c), m61::mul_small(a.im, c)}; }
// a c for an F_p element c
__device__ __forceinline__ f2 f2scale(f2 a, uint64_t c) { return f2{m61::mul(a.re, c), m61::mul(a.im, c)}; }
__device__ __forceinline__ f2 ldp(const uint64_t *p) { return f2{p[0], p[1]}; }  // a challenge (re, im)
__device__ __forceinline__ void stp(uint64_t *p, f2 v)
{
    p[0] = v.re;
    p[1] = v.im;
}
__device__ __forceinline__ f2 ldt(const F2Tab &t, uint64_t i) { return f2{t.re[i], t.im[i]}; }
__device__ __forceinline__ void stt(const F2Tab &t, uint64_t i, f2 v)
{
    t.re[i] = v.re;
    t.im[i] = v.im;
}
// eq(z, b) for one variable and a bit b
__device__ __forceinline__ f2 eq1b(f2 z, int b) { return b ? z : f2sub(f2of(1), z); }
// eq(z, X) = (1 - X) + z (2 X - 1) for a small integer X
__device__ __forceinline__ f2 eq1x(f2 z, int X) { return f2add(f2of(m61::from_i64(1 - X)), f2small(z, 2 * X - 1)); }
// eq(a, b) for one variable, both points in F_{p^2}: a b + (1 - a)(1 - b) = 1 - a - b + 2 a b
__device__ __forceinline__ f2 eq1z(f2 a, f2 b)
{
    const f2 ab = f2mul(a, b);
    return f2add(f2sub(f2sub(f2of(1), a), b), f2add(ab, ab));
}

// ---- loose parts: operands and results folded (below 2^61 + 8) ----
__device__ __forceinline__ f2 l2add(f2 a, f2 b) { return f2{m61::fold(a.re + b.re), m61::fold(a.im + b.im)}; }
__device__ __forceinline__ f2 l2sub(f2 a, f2 b) { return f2{m61::lsub(a.re, b.re), m61::lsub(a.im, b.im)}; }
// the products of a Karatsuba product (folded), combined: p0 - p1 and
// p2 - p0 - p1; p0 + p1 < 4p and p2 + 4p < 2^64
__device__ __forceinline__ f2 l2comb(uint64_t p0, uint64_t p1, uint64_t p2)
{
    return f2{m61::fold(p0 + (4 * m61::P - p1)), m61::fold(p2 + (4 * m61::P - p0 - p1))};
}
__device__ __forceinline__ f2 l2mul(f2 a, f2 b)
{
    return l2comb(m61::lmul(a.re, b.re), m61::lmul(a.im, b.im), m61::lmul(a.re + a.im, b.re + b.im));
}
// lo + r (hi - lo)
__device__ __forceinline__ f2 l2fold(f2 lo, f2 hi, f2 r) { return l2add(lo, l2mul(r, l2sub(hi, lo))); }
__device__ __forceinline__ f2 l2canon(f2 a) { return f2{m61::canon(a.re), m61::canon(a.im)}; }

}  // namespace ra
