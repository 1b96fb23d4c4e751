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
// a c for 0 <= c <= 7
__device__ __forceinline__ f2 l2small(f2 a, uint32_t c) { return f2{m61::fold(a.re * c), m61::fold(a.im * c)}; }
// eq(z, X) for X >= 0
__device__ __forceinline__ f2 l2eq1x(f2 z, int X)
{
    const f2 one_x = f2{X ? m61::P + 1 - X : 1, 0};  // 1 - X
    return X ? l2add(one_x, l2small(z, 2 * X - 1)) : l2sub(one_x, z);
}
__device__ __forceinline__ f2 l2canon(f2 a) { return f2{m61::canon(a.re), m61::canon(a.im)}; }

// A sum of products with its three Karatsuba parts summed apart, combined once.
struct K3 {
    uint64_t p0 = 0, p1 = 0, p2 = 0;
    __device__ __forceinline__ void add(f2 a, f2 b)
    {
        p0 = m61::lmacc(p0, a.re, b.re);
        p1 = m61::lmacc(p1, a.im, b.im);
        p2 = m61::lmacc(p2, a.re + a.im, b.re + b.im);
    }
    __device__ __forceinline__ void add(f2 a, uint64_t b)  // b in F_p
    {
        p0 = m61::lmacc(p0, a.re, b);
        p2 = m61::lmacc(p2, a.re + a.im, b);
    }
    __device__ __forceinline__ f2 value() const { return l2comb(p0, p1, p2); }
};

// ---------------------------------------------------------------------------
// Sum-check rounds with a factored eq (Sec. II-D).  With x bound to z_{<j},
// EQ(x) = eq(r, x) is K_j eq(r_j, X) w_i, w_i = eq(r_{>j}, i), so a round's
// polynomial is K_j eq(r_j, X) s(X) with s quadratic, and no EQ table is read
// or folded.  Over the pairs (i, i + h), lo at X = 0 and hi at X = 1:
//   range   EQ B (c_eq (B - 1) + c_w):  P0 = sum w b0, P1 = sum w b1, Q0 = sum w b0^2,
//           M = sum w b0 b1, Q1 = sum w b1^2;
//           s = c_eq ((1-X)^2 Q0 + 2 X (1-X) M + X^2 Q1) + (c_w - c_eq) ((1-X) P0 + X P1)
//   ReLU    EQ D S (D = R - Y, S = R + Y):  T0 = sum w d0 s0, T1 = sum w d1 s1,
//           U = sum w (d0 + d1)(s0 + s1);  s = (1-X)^2 T0 + X (1-X) (U - T0 - T1) + X^2 T1
//   matrix  a b: as ReLU without weights, and g = s.
// A pair costs 5 (range: 15 products of F_p) or 5 (ReLU) products of F_{p^2},
// where evaluating the summand at X = 0..3 from tables of EQ took 12 and a
// fold more.
// ---------------------------------------------------------------------------
constexpr int f2_sum_words(int kind) { return kind == F2_RANGE ? 10 : 6; }

template <int KIND> struct F2Sums {  // ReLU, matrix
    K3 t0, t1, u;
    // d weighted (or, matrix, as it is)
    __device__ __forceinline__ void add(f2 d0, f2 d1, f2 s0, f2 s1)
    {
        t0.add(d0, s0);
        t1.add(d1, s1);
        u.add(l2add(d0, d1), l2add(s0, s1));
    }
    // weight w, the pair's products in F_p (integer tables)
    __device__ __forceinline__ void add_int(f2 w, uint64_t d0, uint64_t d1, uint64_t s0, uint64_t s1)
    {
        t0.add(w, m61::lmul(d0, s0));
        t1.add(w, m61::lmul(d1, s1));
        u.add(w, m61::lmul(m61::fold(d0 + d1), m61::fold(s0 + s1)));
    }
    __device__ __forceinline__ void words(uint64_t (&v)[6], bool scaled, f2 w) const
    {
        f2 x[3] = {t0.value(), t1.value(), u.value()};
#pragma unroll
        for (int q = 0; q < 3; q++) {
            if (scaled) x[q] = l2mul(x[q], w);
            v[2 * q] = x[q].re;
            v[2 * q + 1] = x[q].im;
        }
    }
};
template <> struct F2Sums<F2_RANGE> {
    f2 P0{0, 0}, P1{0, 0};
    K3 q0, m, q1;
    // u = w b
    __device__ __forceinline__ void add(f2 u0, f2 u1, f2 b0, f2 b1)
    {
        P0 = l2add(P0, u0);
        P1 = l2add(P1, u1);
        q0.add(u0, b0);
        m.add(u0, b1);
        q1.add(u1, b1);
    }
    __device__ __forceinline__ void words(uint64_t (&v)[10], bool scaled, f2 w) const
    {
        f2 x[5] = {P0, P1, q0.value(), m.value(), q1.value()};
#pragma unroll
        for (int q = 0; q < 5; q++) {
            if (scaled) x[q] = l2mul(x[q], w);
            v[2 * q] = x[q].re;
            v[2 * q + 1] = x[q].im;
        }
    }
};

// The round's value at X from the sums (canonical, the words of F2Sums), K =
// K_j, r = r_j, cst = (c_eq, c_w).
__device__ __forceinline__ f2 f2_round_value(int kind, const uint64_t *t, int X, f2 K, f2 r, const uint64_t *cst)
{
    const int u = 1 - X;
    auto at = [&](int q) { return f2{t[2 * q], t[2 * q + 1]}; };
    f2 s;
    if (kind == F2_RANGE) {
        const f2 lin = f2add(f2small(at(0), u), f2small(at(1), X));
        const f2 quad = f2add(f2add(f2small(at(2), u * u), f2small(at(3), 2 * X * u)), f2small(at(4), X * X));
        const f2 ceq = ldp(cst), cw = ldp(cst + 2);
        s = f2add(f2mul(ceq, quad), f2mul(f2sub(cw, ceq), lin));
    } else {
        const f2 cross = f2sub(f2sub(at(2), at(0)), at(1));
        s = f2add(f2add(f2small(at(0), u * u), f2small(cross, X * u)), f2small(at(1), X * X));
        if (kind == F2_MATMUL) return s;
    }
    return f2mul(f2mul(K, eq1x(r, X)), s);
}

// Sums over adjacent lanes (all of them active), in each of the lanes; in and
// out folded.  The partner values come by DPP moves in the adds' own registers
// (lane ^ 1, ^ 2, then the other quad and the other half by mirrors): a
// cross-lane read through LDS takes 100 cycles and more per step.
template <int CTRL> __device__ __forceinline__ uint64_t dpp_plus(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xF, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xF, 0xF, false);
    return v + ((uint64_t)hi << 32 | lo);  // two such adds of folded values stay below 2^64
}
__device__ __forceinline__ uint64_t sum8(uint64_t v)
{
    return m61::fold(dpp_plus<0x141>(m61::fold(dpp_plus<0x4E>(dpp_plus<0xB1>(v)))));
}
__device__ __forceinline__ uint64_t sum16(uint64_t v)
{
    return m61::fold(dpp_plus<0x140>(dpp_plus<0x141>(m61::fold(dpp_plus<0x4E>(dpp_plus<0xB1>(v))))));
}

// Totals of NW words per thread over the block's first nt threads (nt a
// multiple of 64, the others' words are zero): canonical, in tot (LDS) for
// every thread.  red: NW nt words.  Barriers on both sides.
template <int NW>
__device__ __forceinline__ void f2_totals(const uint64_t (&v)[NW], uint64_t *red, uint64_t *tot, int nt)
{
    const int tid = threadIdx.x, seg = nt >> 4;
    __syncthreads();
    if (tid < nt)
#pragma unroll
        for (int q = 0; q < NW; q++) red[q * nt + tid] = v[q];
    __syncthreads();
    for (int task = tid; task < NW * 16; task += blockDim.x) {  // 16 adjacent lanes per word
        const uint64_t *src = red + (task >> 4) * nt + (task & 15);
        uint64_t a0 = 0, a1 = 0;
        for (int e = 0; e < seg; e += 4) {
            a0 = m61::fold(a0 + src[16 * e] + src[16 * e + 32]);
            a1 = m61::fold(a1 + src[16 * e + 16] + src[16 * e + 48]);
        }
        const uint64_t x = sum16(m61::fold(a0 + a1));
        if ((task & 15) == 0) tot[task >> 4] = m61::canon(x);
    }
    __syncthreads();
}

// D = R - Y and S = R + Y of entry i as elements of F_p
__device__ __forceinline__ void relu_ints(const int32_t *R, const int32_t *Y, uint64_t i, uint64_t &d, uint64_t &s)
{
    const int64_t r = R[i], y = Y[i];
    d = m61::from_i64(r - y);
    s = m61::from_i64(r + y);
}

// lo + r (hi - lo) for lo, hi in F_p
__device__ __forceinline__ f2 fold_real(uint64_t lo, uint64_t hi, f2 r)
{
    const uint64_t d = m61::lsub(hi, lo);
    return f2{m61::lmacc(lo, r.re, d), m61::lmul(r.im, d)};
}

// The sums of eq(sigma_p, q) over the set bits q of a byte, for each byte of a
// bit word: tab[t][e], byte t (256 threads; tabs bytes, sig: 64 entries in
// LDS).  A word's plane-bound value is then one lookup and add per byte.
__device__ __forceinline__ void f2_byte_tables(const f2 *sig, int tabs, f2 (*tab)[256])
{
    for (int e = threadIdx.x; e < 256; e += blockDim.x)
        for (int t = 0; t < tabs; t++) {
            f2 s = f2of(0);
#pragma unroll
            for (int b = 0; b < 8; b++)
                if ((e >> b) & 1) s = f2{s.re + sig[8 * t + b].re, s.im + sig[8 * t + b].im};  // at most 8 2^61
            tab[t][e] = l2canon(s);
        }
}
__device__ __forceinline__ f2 f2_plane_bound(uint64_t w, int tabs, const f2 (*tab)[256])
{
    f2 s = f2of(0);
    for (int t = 0; t < tabs; t++) {
        const f2 x = tab[t][(w >> (8 * t)) & 255];
        s = f2{s.re + x.re, s.im + x.im};  // at most 8 canonical terms
    }
    return l2canon(s);
}

}  // namespace ra
