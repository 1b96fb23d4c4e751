// secp29.hpp -- secp256k1 on the device for the multi-scalar product: field
// elements of F_q, q = 2^256 - 2^32 - 977, as nine signed limbs of 29 bits, and
// points in XYZZ coordinates (x = X / ZZ, y = Y / ZZZ, ZZ^3 = ZZZ^2; the
// identity has ZZ = 0 in every limb).
//
// Why this form: a product is 81 v_mad_i64_i32 into 64-bit column sums with no
// carries between them (nine products of 29-bit limbs stay below 2^62), and
// sums and differences are nine plain additions, so the carries are paid once
// per product (about 160 instructions in all).  Eight canonical 32-bit limbs
// took about 400: a carry after every partial product, half of it moves to
// build 64-bit addends, and a comparison with q after every sum.
//
// A fresh value (a product's result) has limbs in (-2^21, 2^29 + 2^20) and any
// residue's representative below 2^261 or so in size; "magnitude" m below is a
// bound of m 2^29 on the limbs' size.  A product's operands need m1 m2 < 3.5
// (9 m1 m2 2^58 < 2^63), a difference of two products m1 m2 + m3 m4 < 3.5.
//
// The point formulas are those of the Explicit-Formulas Database (Bernstein,
// Lange) for y^2 = x^3 + b: in XYZZ coordinates madd-2008-s, add-2008-s and
// dbl-2008-s-1 (Sutherland), and the plain Jacobian doubling for a = 0.
#pragma once
#include "secp256k1.hpp"

namespace secp29 {

struct F {
    int32_t v[9];
};
constexpr int32_t kM = (1 << 29) - 1;
// 2^261 = 2^5 (2^32 + 977) = 2^8 2^29 + 31264 (mod q)
constexpr int32_t kR0 = 31264, kR1 = 256;

#define FE __device__ __forceinline__

FE F zero()
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) r.v[i] = 0;
    return r;
}
FE F one()
{
    F r = zero();
    r.v[0] = 1;
    return r;
}
FE F add(const F &a, const F &b)
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) r.v[i] = a.v[i] + b.v[i];
    return r;
}
FE F sub(const F &a, const F &b)
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) r.v[i] = a.v[i] - b.v[i];
    return r;
}
FE F neg(const F &a)
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) r.v[i] = -a.v[i];
    return r;
}
FE F times(const F &a, int32_t c)
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) r.v[i] = a.v[i] * c;
    return r;
}
FE F from_limbs32(const uint32_t *p)  // canonical 8 x 32 bits
{
    F r;
#pragma unroll
    for (int i = 0; i < 9; i++) {
        const int b = 29 * i, w = b >> 5, s = b & 31;
        uint32_t x = p[w] >> s;
        if (s > 3 && w < 7) x |= p[w + 1] << (32 - s);
        r.v[i] = (int32_t)(x & (uint32_t)kM);
    }
    return r;
}

// Column sums to a fresh value: lo[k] of weight 2^(29 k), hi[k] of 2^(29 (9 + k)).
FE F reduce(const int64_t (&lo)[9], const int64_t (&hi)[8])
{
    int32_t h[9];
    int64_t t = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        t += hi[k];
        h[k] = (int32_t)t & kM;
        t >>= 29;
    }
    h[8] = (int32_t)t;  // below 2^31 in size for m1 m2 < 3.5
    F r;
    t = 0;
#pragma unroll
    for (int k = 0; k < 9; k++) {
        t += lo[k] + (int64_t)h[k] * kR0;
        if (k) t += (int64_t)h[k - 1] * kR1;
        r.v[k] = (int32_t)t & kM;
        t >>= 29;
    }
    t += (int64_t)h[8] * kR1;  // what lies at 2^261: below 2^40 in size
    const int32_t v0 = (int32_t)t & kM, v1 = (int32_t)(t >> 29);
    int64_t u = (int64_t)v0 * kR0 + r.v[0];
    r.v[0] = (int32_t)u & kM;
    u = (u >> 29) + r.v[1] + (int64_t)v0 * kR1 + (int64_t)v1 * kR0;
    r.v[1] = (int32_t)u & kM;
    r.v[2] += (int32_t)(u >> 29) + v1 * kR1;
    return r;
}

FE void columns(const F &a, const F &b, int64_t (&lo)[9], int64_t (&hi)[8])
{
#pragma unroll
    for (int k = 0; k < 17; k++) {
        int64_t s = 0;
#pragma unroll
        for (int i = 0; i < 9; i++)
            if (k - i >= 0 && k - i < 9) s += (int64_t)a.v[i] * b.v[k - i];
        if (k < 9) lo[k] = s;
        else hi[k - 9] = s;
    }
}
FE void columns_sqr(const F &a, int64_t (&lo)[9], int64_t (&hi)[8])
{
    const F d = add(a, a);
#pragma unroll
    for (int k = 0; k < 17; k++) {
        int64_t s = 0;
#pragma unroll
        for (int i = 0; i < 9; i++)
            if (k - i > i && k - i < 9) s += (int64_t)d.v[i] * a.v[k - i];
        if (!(k & 1)) s += (int64_t)a.v[k / 2] * a.v[k / 2];
        if (k < 9) lo[k] = s;
        else hi[k - 9] = s;
    }
}
FE F mul(const F &a, const F &b)
{
    int64_t lo[9], hi[8];
    columns(a, b, lo, hi);
    return reduce(lo, hi);
}
FE F sqr(const F &a)
{
    int64_t lo[9], hi[8];
    columns_sqr(a, lo, hi);
    return reduce(lo, hi);
}
// a^2 - c s
FE F sqr_sub(const F &a, int32_t c, const F &s)
{
    int64_t lo[9], hi[8];
    columns_sqr(a, lo, hi);
#pragma unroll
    for (int k = 0; k < 9; k++) lo[k] -= (int64_t)c * s.v[k];
    return reduce(lo, hi);
}
// a b - c s
FE F mul_sub(const F &a, const F &b, int32_t c, const F &s)
{
    int64_t lo[9], hi[8];
    columns(a, b, lo, hi);
#pragma unroll
    for (int k = 0; k < 9; k++) lo[k] -= (int64_t)c * s.v[k];
    return reduce(lo, hi);
}
// a b - c d with one reduction
FE F mul_sub_mul(const F &a, const F &b, const F &c, const F &d)
{
    int64_t lo[9], hi[8];
    columns(a, b, lo, hi);
    const F n = neg(c);
#pragma unroll
    for (int k = 0; k < 17; k++)
#pragma unroll
        for (int i = 0; i < 9; i++)
            if (k - i >= 0 && k - i < 9) {
                if (k < 9) lo[k] += (int64_t)n.v[i] * d.v[k - i];
                else hi[k - 9] += (int64_t)n.v[i] * d.v[k - i];
            }
    return reduce(lo, hi);
}
// c a - b as a fresh value
FE F lin(int32_t c, const F &a, const F &b)
{
    int64_t lo[9], hi[8];
#pragma unroll
    for (int k = 0; k < 9; k++) lo[k] = (int64_t)c * a.v[k] - b.v[k];
#pragma unroll
    for (int k = 0; k < 8; k++) hi[k] = 0;
    return reduce(lo, hi);
}

// The canonical residue, eight 32-bit limbs.  Out of line: only ends of chains
// and the rare exact zero test need it.
static __device__ __noinline__ secp::Fe canon(F a)
{
    a = lin(1, a, zero());
    // q 2^6 added (the value is above -2^262), digits carried to [0, 2^29)
    // with whatever is left in the top one; bits from 2^256 on folded twice
    int64_t t = 0;
    int32_t d[10];
    for (int k = 0; k < 9; k++) {
        const int b = 29 * k - 6;  // digit k of q 2^6
        uint32_t w = 0;
        for (int i = 0; i < 29; i++) {
            const int p = b + i;
            if (p >= 0 && p < 256 && ((secp::kQ[p >> 5] >> (p & 31)) & 1)) w |= 1u << i;
        }
        t += (int64_t)a.v[k] + w;
        d[k] = (int32_t)t & kM;
        t >>= 29;
    }
    d[9] = (int32_t)t;  // q 2^6 has one bit at 2^261
    d[9] += 1;
    secp::Fe r;
    uint64_t top = 0;
    for (int pass = 0; pass < 2; pass++) {
        // bits from 2^256: limb 8 from its bit 24, limb 9
        top = ((uint64_t)(uint32_t)d[8] >> 24) | ((uint64_t)(uint32_t)d[9] << 5);
        d[8] &= (1 << 24) - 1;
        d[9] = 0;
        // top (2^32 + 977)
        int64_t c = (int64_t)(top * 977) + d[0];
        d[0] = (int32_t)c & kM;
        c = (c >> 29) + d[1] + (int64_t)(top << 3);
        d[1] = (int32_t)c & kM;
        c >>= 29;
        for (int k = 2; k < 9; k++) {
            c += d[k];
            d[k] = (int32_t)c & kM;
            c >>= 29;
        }
    }
    for (int w = 0; w < 8; w++) {
        const int b = 32 * w, k = b / 29, s = b % 29;
        uint64_t x = (uint64_t)(uint32_t)d[k] >> s;
        x |= (uint64_t)(uint32_t)d[k + 1] << (29 - s);
        if (58 - s < 32 && k + 2 < 9) x |= (uint64_t)(uint32_t)d[k + 2] << (58 - s);
        r.v[w] = (uint32_t)x;
    }
    return secp::fe_canon(r, (uint32_t)d[8] >> 24);
}

// a = 0 mod q: a representative k q, |k| < 128, has low limb -977 k mod 2^29,
// so k follows from it (977 inverted mod 2^29); one value in 2^21 passes and is
// settled exactly.  a of magnitude at most 2.
constexpr uint32_t inv977()
{
    uint32_t x = 977;
    for (int i = 0; i < 5; i++) x *= 2 - 977 * x;
    return x;
}
FE bool is_zero(const F &a)
{
    const uint32_t k = (0u - (uint32_t)a.v[0] * inv977() + 128u) & (uint32_t)kM;
    if (k >= 256u) return false;
    return secp::fe_is_zero(canon(a));
}

struct Pt {
    F X, Y, ZZ, ZZZ;
};
constexpr int kPtWords = 36;

FE Pt identity()
{
    Pt r;
    r.X = one();
    r.Y = one();
    r.ZZ = zero();
    r.ZZZ = zero();
    return r;
}
FE bool is_identity(const Pt &p)
{
    int32_t o = 0;
#pragma unroll
    for (int i = 0; i < 9; i++) o |= p.ZZ.v[i];
    return o == 0;
}
FE void store(uint32_t *p, const Pt &a)
{
#pragma unroll
    for (int i = 0; i < 9; i++) {
        p[i] = (uint32_t)a.X.v[i];
        p[9 + i] = (uint32_t)a.Y.v[i];
        p[18 + i] = (uint32_t)a.ZZ.v[i];
        p[27 + i] = (uint32_t)a.ZZZ.v[i];
    }
}
FE Pt load(const uint32_t *p)
{
    Pt a;
#pragma unroll
    for (int i = 0; i < 9; i++) {
        a.X.v[i] = (int32_t)p[i];
        a.Y.v[i] = (int32_t)p[9 + i];
        a.ZZ.v[i] = (int32_t)p[18 + i];
        a.ZZZ.v[i] = (int32_t)p[27 + i];
    }
    return a;
}

// 2 p (a = 0): U = 2Y, V = U^2, W = U V, S = X V, M = 3 X^2.  Out of line
// (equal points only).
static __device__ __noinline__ void dbl_slow(Pt &p)
{
    const F U = lin(2, p.Y, zero()), V = sqr(U), W = mul(U, V), S = mul(p.X, V), M = mul(p.X, times(p.X, 3));
    const F X = sqr_sub(M, 2, S);
    const F Y = mul_sub_mul(M, sub(S, X), W, p.Y);
    p.ZZ = mul(V, p.ZZ);
    p.ZZZ = mul(W, p.ZZZ);
    p.X = X;
    p.Y = Y;  // a point of order 2 does not exist on this curve
}

// The common end of an addition: P, R the differences, U1, S1 the first
// point's coordinates on the common denominators; false: the points have the
// same x (P = 0).
FE bool add_end(const F &U1, const F &S1, const F &P, const F &R, Pt &o, F &PP, F &PPP)
{
    if (is_zero(P)) return false;
    PP = sqr(P);
    PPP = mul(P, PP);
    const F Q = mul(U1, PP);
    o.X = sqr_sub(R, 1, add(PPP, add(Q, Q)));
    o.Y = mul_sub_mul(R, sub(Q, o.X), S1, PPP);
    return true;
}

// p + (x, y), x and y fresh or negated by limbs; so may p.Y be (a run's first
// point), where a plain difference for R would have magnitude 2, and R^2 twice
// the bound: p.Y goes into the product's reduction.  (Making a negated y fresh
// instead costs a reduction in nearly every step of a wave.)
FE void add_affine(Pt &p, const F &x, const F &y)
{
    const F P = sub(mul(x, p.ZZ), p.X), R = mul_sub(y, p.ZZZ, 1, p.Y);
    Pt o;
    F PP, PPP;
    if (!add_end(p.X, p.Y, P, R, o, PP, PPP)) {  // equal or opposite
        if (is_zero(R)) dbl_slow(p);
        else p = identity();
        return;
    }
    o.ZZ = mul(p.ZZ, PP);
    o.ZZZ = mul(p.ZZZ, PPP);
    p = o;
}

// p + q, either may be the identity
FE Pt add(const Pt &p, const Pt &q)
{
    if (is_identity(p)) return q;
    if (is_identity(q)) return p;
    const F U1 = mul(p.X, q.ZZ), S1 = mul(p.Y, q.ZZZ);
    const F P = sub(mul(q.X, p.ZZ), U1), R = sub(mul(q.Y, p.ZZZ), S1);
    Pt o;
    F PP, PPP;
    if (!add_end(U1, S1, P, R, o, PP, PPP)) {
        if (!is_zero(R)) return identity();
        o = p;
        dbl_slow(o);
        return o;
    }
    o.ZZ = mul(mul(p.ZZ, q.ZZ), PP);
    o.ZZZ = mul(mul(p.ZZZ, q.ZZZ), PPP);
    return o;
}

// Jacobian coordinates (x = X / Z^2, y = Y / Z^3) for runs of doublings: four
// products and three squares.  From XYZZ with Z = ZZ.
struct Jac {
    F X, Y, Z;
};
FE Jac to_jac(const Pt &p) { return Jac{mul(p.X, p.ZZ), mul(p.Y, p.ZZZ), p.ZZ}; }
FE Pt from_jac(const Jac &p)
{
    const F ZZ = sqr(p.Z);
    return Pt{p.X, p.Y, ZZ, mul(ZZ, p.Z)};
}
FE Jac dbl(const Jac &p)  // the identity (Z = 0) stays one
{
    const F E = mul(p.X, times(p.X, 3)), B = sqr(p.Y), D = mul(p.X, B), C = sqr(B);
    Jac r;
    r.X = sqr_sub(E, 8, D);
    r.Y = mul_sub(E, lin(4, D, r.X), 8, C);
    r.Z = mul(times(p.Y, 2), p.Z);
    return r;
}

// a^(q - 2), q - 2 = (2^223 - 1) 2^33 + (2^22 - 1) 2^10 + 45: runs of 223 and 22
// ones, then 45 = 5 8 + 5 in ten bits.  With ones(n) = a^(2^n - 1), ones(i + j) =
// ones(i)^(2^j) ones(j); the long run is reached through the short one, 223 =
// 10 22 + 3, and 22 = 2 (2 5 + 1).
static __device__ __noinline__ F inverse(F a)
{
    auto shift = [](F x, int n, const F &low) {  // x^(2^n) low
        for (int i = 0; i < n; i++) x = sqr(x);
        return mul(x, low);
    };
    const F ones2 = shift(a, 1, a);
    const F ones5 = shift(shift(ones2, 2, ones2), 1, a);
    const F ones11 = shift(shift(ones5, 5, ones5), 1, a);
    const F ones22 = shift(ones11, 11, ones11);
    const F ones44 = shift(ones22, 22, ones22);
    const F ones110 = shift(shift(ones44, 44, ones44), 22, ones22);
    const F ones223 = shift(shift(ones110, 110, ones110), 3, shift(ones2, 1, a));
    const F a5 = shift(a, 2, a);
    return shift(shift(shift(ones223, 23, ones22), 7, a5), 3, a5);
}

#undef FE

}  // namespace secp29
