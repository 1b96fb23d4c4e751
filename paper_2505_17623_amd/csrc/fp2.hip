// fp2.hip -- the layer protocol with the verifier's challenges in the
// quadratic extension F_{p^2} = F_p[i] / (i^2 + 1) (p = 2^61 - 1 is 3 mod 4,
// so x^2 + 1 is irreducible).  Sec. II-F asks for a field of more than 128
// bits; a sum-check round over F_{p^2} lets a cheating prover pass with
// probability about d / p^2 instead of d / p (Sec. II-D).
//
// The witness (C, R, Rm, Y, Z, the bit table) is integer-valued and is made
// by the F_p kernels.  Everything that depends on a challenge is an element
// of F_{p^2}, held as two F_p tables (real and imaginary parts, "SoA"):
//   - the eq tables E1 = eq(r1, .), E2 = eq(r2, .) and EQ(x) = E1 E2;
//   - the bound sides of the product (an integer table bound at a point of
//     F_{p^2} is the pair of its F_p bindings with the eq table's two parts,
//     so the F_p binding kernels serve);
//   - the plane rounds' Gram matrix G = sum_x EQ(x) bit bit^T, whose two
//     parts the F_p Gram pass computes from EQ's two parts;
//   - every folded table of the rounds.
// Rounds run one launch per round (a pass over the pairs that evaluates the
// round polynomial and folds the tables in place) while the tables are
// large, and the last rounds of an instance in one workgroup over LDS; this
// is slower than the F_p path's fused passes.
#include "common.hpp"
#include "f2.hpp"
#include "gram_reduce.hpp"
#include "fs_device.hpp"
#include "sha256.hpp"

namespace ra {

// Block sum of the eight words of four F_{p^2} values; thread 0 writes them.
__device__ __forceinline__ void f2_block_out(const f2 (&acc)[4], uint64_t *red, uint64_t *out)
{
    uint64_t v[8];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        v[2 * q] = acc[q].re;
        v[2 * q + 1] = acc[q].im;
    }
    m61::block_sum<8>(v, red);
    if (threadIdx.x == 0)
#pragma unroll
        for (int q = 0; q < 8; q++) out[q] = v[q];
}

// ---------------------------------------------------------------------------
// eq tables (Eq. (1)) of points of F_{p^2}: the point is v challenges stored
// as pairs (re, im); the table goes to two F_p arrays.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_f2_eq(const uint64_t *__restrict__ z, int v, F2Tab out)
{
    __shared__ f2 zl[64];
    if ((int)threadIdx.x < v) zl[threadIdx.x] = ldp(z + 2 * threadIdx.x);
    __syncthreads();
    const uint64_t n = 1ull << v;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        f2 acc = f2of(1);
        for (int j = 0; j < v; j++) acc = f2mul(acc, eq1b(zl[j], (int)((i >> (v - 1 - j)) & 1)));
        stt(out, i, acc);
    }
}

void launch_f2_eq(const uint64_t *z, int v, F2Tab out, hipStream_t st)
{
    const uint64_t n = 1ull << v;
    const int nb = (int)((n + kThreads - 1) / kThreads < 1024 ? (n + kThreads - 1) / kThreads : 1024);
    hipLaunchKernelGGL(k_f2_eq, dim3(nb), dim3(kThreads), 0, st, z, v, out);
}

// The eq tables of a layer in one launch: segments E1, E2 (SoA), LS, HS
// (f2.hpp; heaps, entry 2^k + y), each entry the product of its variables'
// factors.
__global__ __launch_bounds__(256) void k_f2_eqs(const uint64_t *__restrict__ r, int ln, int lk, F2Tab E1, F2Tab E2,
                                                f2 *__restrict__ HS, f2 *__restrict__ LS)
{
    __shared__ f2 z[64];
    const int lN = ln + lk, low = lN < kF2Low ? lN : kF2Low, hs = lN - low;
    if ((int)threadIdx.x < lN) z[threadIdx.x] = ldp(r + 2 * threadIdx.x);
    __syncthreads();
    const uint64_t n = 1ull << ln, k = 1ull << lk, ls = 2ull << low, nh = 2ull << hs;
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const f2 *v;  // the entry: eq over v[0 .. m) at y
    int m;
    uint64_t y;
    if (i < n + k) {
        const bool one = i < n;
        y = one ? i : i - n;
        v = one ? z : z + ln;
        m = one ? ln : lk;
    } else if (i < n + k + ls + nh) {
        const bool lo = i < n + k + ls;
        y = lo ? i - n - k : i - n - k - ls;
        if (!y) return;
        m = 63 - __builtin_clzll(y);
        y -= 1ull << m;
        v = lo ? z + lN - m : z + hs - m;
    } else {
        return;
    }
    f2 e = f2of(1);
    for (int j = 0; j < m; j++) e = l2mul(e, eq1b(v[j], (int)((y >> (m - 1 - j)) & 1)));
    e = l2canon(e);
    if (i < n) stt(E1, i, e);
    else if (i < n + k) stt(E2, y, e);
    else if (i < n + k + ls) LS[i - n - k] = e;
    else HS[i - n - k - ls] = e;
}

void launch_f2_eqs(const uint64_t *r, int ln, int lk, F2Tab E1, F2Tab E2, f2 *HS, f2 *LS, hipStream_t st)
{
    const int lN = ln + lk, low = lN < kF2Low ? lN : kF2Low;
    const uint64_t tot = (1ull << ln) + (1ull << lk) + (2ull << low) + (2ull << (lN - low));
    hipLaunchKernelGGL(k_f2_eqs, dim3((unsigned)((tot + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, r, ln, lk, E1,
                       E2, HS, LS);
}

// EQ(x) = E1[x >> lk] E2[x mod 2^lk] for x < N (the eq table of (r1, r2)).
__global__ __launch_bounds__(256) void k_f2_outer(F2Tab E1, F2Tab E2, int lk, uint64_t N, F2Tab out)
{
    const uint64_t mask = (1ull << lk) - 1;
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < N; x += (uint64_t)gridDim.x * blockDim.x)
        stt(out, x, f2mul(ldt(E1, x >> lk), ldt(E2, x & mask)));
}

void launch_f2_outer(F2Tab E1, F2Tab E2, int lk, uint64_t N, F2Tab out, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_outer, dim3(f2_blocks(N)), dim3(kThreads), 0, st, E1, E2, lk, N, out);
}

// The claims R~, Rm~, Y~, Z~ at (r1, r2): sum_x EQ(x) v(x), per-block
// partials (eight words per block).
__global__ __launch_bounds__(256) void k_f2_claims(F2Tab EQ, const int32_t *__restrict__ R,
                                                   const uint16_t *__restrict__ Rm, const int32_t *__restrict__ Y,
                                                   const int32_t *__restrict__ Z, uint64_t N, uint64_t *part)
{
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    f2 acc[4] = {f2of(0), f2of(0), f2of(0), f2of(0)};
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < N; x += (uint64_t)gridDim.x * blockDim.x) {
        const f2 e = ldt(EQ, x);
        acc[0] = f2add(acc[0], f2small(e, R[x]));
        acc[1] = f2add(acc[1], f2small(e, (int32_t)Rm[x]));
        acc[2] = f2add(acc[2], f2small(e, Y[x]));
        acc[3] = f2add(acc[3], f2small(e, Z[x]));
    }
    f2_block_out(acc, red, part + 8 * (size_t)blockIdx.x);
}

void launch_f2_claims(F2Tab EQ, const int32_t *R, const uint16_t *Rm, const int32_t *Y, const int32_t *Z, uint64_t N,
                      uint64_t *part, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_claims, dim3(f2_blocks(N)), dim3(kThreads), 0, st, EQ, R, Rm, Y, Z, N, part);
}

// Sum of nb rows of eight partial words -> out[0..7].
__global__ __launch_bounds__(256) void k_f2_sum8(const uint64_t *__restrict__ part, int nb, uint64_t *out)
{
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = m61::add(v[q], part[8 * (size_t)b + q]);
    m61::block_sum<8>(v, red);
    if (threadIdx.x == 0)
#pragma unroll
        for (int q = 0; q < 8; q++) out[q] = v[q];
}

void launch_f2_sum8(const uint64_t *part, int nb, uint64_t *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_sum8, dim3(1), dim3(kThreads), 0, st, part, nb, out);
}

// ---------------------------------------------------------------------------
// One round of a sum-check instance over tables of 2h entries (Sec. II-D):
// for every pair (i, i + h) the summand at X = 0..3 (each table is lo +
// X (hi - lo) there), summed per block, and the fold T[i] <- lo + rho
// (hi - lo) into the destination tables.  Summands:
//   F2_MATMUL  a b                                  (tables a, b; degree 2)
//   F2_RANGE   EQ B (c_eq (B - 1) + c_w)            (tables EQ, B; degree 3),
//              the range summand once the plane variables are bound:
//              c_eq = eq(tau_p, sigma_p), c_w = mu W~(sigma_p)
//   F2_RELU    EQ D S, D = R - Y, S = R + Y         (Eq. (6); degree 3)
// The first round of the ReLU instance reads R, Y (int32) for D, S.
// ---------------------------------------------------------------------------
// The summand of one pair at X = 0..3 added into acc, and the folded values
// lo + rho (hi - lo) into lo.
template <int KIND>
__device__ __forceinline__ void f2_pair(f2 (&lo)[3], const f2 (&hi)[3], f2 rho, f2 ceq, f2 cw, f2 (&acc)[4])
{
    constexpr int NT = KIND == F2_RELU ? 3 : 2;
    f2 v[3], d[3];
#pragma unroll
    for (int q = 0; q < NT; q++) {
        v[q] = lo[q];
        d[q] = f2sub(hi[q], lo[q]);
    }
#pragma unroll
    for (int X = 0; X < 4; X++) {
        if (X > 0)
#pragma unroll
            for (int q = 0; q < NT; q++) v[q] = f2add(v[q], d[q]);  // the tables at X
        f2 f;
        if (KIND == F2_MATMUL) {
            if (X == 3) break;
            f = f2mul(v[0], v[1]);
        } else if (KIND == F2_RANGE) {
            f = f2mul(f2mul(v[0], v[1]), f2add(f2mul(ceq, f2sub(v[1], f2of(1))), cw));
        } else {
            f = f2mul(f2mul(v[0], v[1]), v[2]);
        }
        acc[X] = f2add(acc[X], f);
    }
#pragma unroll
    for (int q = 0; q < NT; q++) lo[q] = f2add(lo[q], f2mul(rho, d[q]));
}

// The ReLU instance's first round reads D = R - Y and S = R + Y from the
// integer tables.
__device__ __forceinline__ void f2_relu_ints(const int32_t *R, const int32_t *Y, uint64_t i, f2 &d, f2 &s)
{
    const int64_t r = R[i], y = Y[i];
    d = f2of(m61::from_i64(r - y));
    s = f2of(m61::from_i64(r + y));
}

template <int KIND>
__global__ __launch_bounds__(256) void k_f2_round(F2RoundArgs a)
{
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    constexpr int NT = KIND == F2_RELU ? 3 : 2;
    const f2 rho = ldp(a.rho);
    f2 ceq = f2of(0), cw = f2of(0);
    if (KIND == F2_RANGE) {
        ceq = ldp(a.cst);
        cw = ldp(a.cst + 2);
    }
    f2 acc[4] = {f2of(0), f2of(0), f2of(0), f2of(0)};
    const uint64_t h = a.h;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < h; i += (uint64_t)gridDim.x * blockDim.x) {
        f2 lo[3], hi[3];
        lo[0] = ldt(a.src[0], i);
        hi[0] = ldt(a.src[0], i + h);
        if (KIND == F2_RELU && a.first) {
            f2_relu_ints(a.R, a.Y, i, lo[1], lo[2]);
            f2_relu_ints(a.R, a.Y, i + h, hi[1], hi[2]);
        } else {
#pragma unroll
            for (int q = 1; q < NT; q++) {
                lo[q] = ldt(a.src[q], i);
                hi[q] = ldt(a.src[q], i + h);
            }
        }
        f2_pair<KIND>(lo, hi, rho, ceq, cw, acc);
#pragma unroll
        for (int q = 0; q < NT; q++) stt(a.dst[q], i, lo[q]);
    }
    f2_block_out(acc, red, a.part + 8 * (size_t)blockIdx.x);
}

// ---------------------------------------------------------------------------
// The last v <= kF2TailLog rounds of an instance in one workgroup: the tables
// (2^v entries) are staged in LDS and folded there, round after round; each
// round's sums go to its first partial slot (the round's other slots are
// zeroed, so the finish kernel reads the same layout as after k_f2_round),
// and the final values to index 0 of the destination tables.
// ---------------------------------------------------------------------------
template <int KIND>
__global__ __launch_bounds__(256) void k_f2_tail(F2TailArgs a)
{
    constexpr int NT = KIND == F2_RELU ? 3 : 2, S = 1 << kF2TailLog;
    __shared__ uint64_t T[NT][2][S];  // (re, im) of each table
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    __shared__ uint64_t rz[2 * kF2TailLog];
    const int tid = threadIdx.x, n0 = 1 << a.v;
    f2 ceq = f2of(0), cw = f2of(0);
    if (KIND == F2_RANGE) {
        ceq = ldp(a.cst);
        cw = ldp(a.cst + 2);
    }
    if (tid < 2 * a.v) rz[tid] = a.rho[tid];
    for (int i = tid; i < n0; i += blockDim.x) {
        f2 t[3];
        t[0] = ldt(a.src[0], i);
        if (KIND == F2_RELU && a.first) {
            f2_relu_ints(a.R, a.Y, i, t[1], t[2]);
        } else {
#pragma unroll
            for (int q = 1; q < NT; q++) t[q] = ldt(a.src[q], i);
        }
#pragma unroll
        for (int q = 0; q < NT; q++) {
            T[q][0][i] = t[q].re;
            T[q][1][i] = t[q].im;
        }
    }
    __syncthreads();
    for (int c = 0; c < a.v; c++) {
        const int h = n0 >> (c + 1);
        const f2 rho{rz[2 * c], rz[2 * c + 1]};
        f2 acc[4] = {f2of(0), f2of(0), f2of(0), f2of(0)};
        // a pair's entries are read and its fold written by one thread only
        for (int i = tid; i < h; i += blockDim.x) {
            f2 lo[3], hi[3];
#pragma unroll
            for (int q = 0; q < NT; q++) {
                lo[q] = f2{T[q][0][i], T[q][1][i]};
                hi[q] = f2{T[q][0][i + h], T[q][1][i + h]};
            }
            f2_pair<KIND>(lo, hi, rho, ceq, cw, acc);
#pragma unroll
            for (int q = 0; q < NT; q++) {
                T[q][0][i] = lo[q].re;
                T[q][1][i] = lo[q].im;
            }
        }
        uint64_t *part = a.part + (size_t)c * kF2MaxBlocks * 8;
        const int nb = f2_blocks((uint64_t)h);
        if (tid >= 1 && tid < nb)
#pragma unroll
            for (int q = 0; q < 8; q++) part[8 * tid + q] = 0;
        f2_block_out(acc, red, part);  // its barriers also order this round's folds before the next reads
        __syncthreads();
    }
    if (tid == 0)
#pragma unroll
        for (int q = 0; q < NT; q++) stt(a.dst[q], 0, f2{T[q][0][0], T[q][1][0]});
}

void launch_f2_tail(const F2TailArgs &a, hipStream_t st)
{
    switch (a.kind) {
    case F2_MATMUL: hipLaunchKernelGGL(k_f2_tail<F2_MATMUL>, dim3(1), dim3(kThreads), 0, st, a); break;
    case F2_RANGE: hipLaunchKernelGGL(k_f2_tail<F2_RANGE>, dim3(1), dim3(kThreads), 0, st, a); break;
    default: hipLaunchKernelGGL(k_f2_tail<F2_RELU>, dim3(1), dim3(kThreads), 0, st, a); break;
    }
}

void launch_f2_round(const F2RoundArgs &a, hipStream_t st)
{
    const dim3 grid(f2_blocks(a.h));
    switch (a.kind) {
    case F2_MATMUL: hipLaunchKernelGGL(k_f2_round<F2_MATMUL>, grid, dim3(kThreads), 0, st, a); break;
    case F2_RANGE: hipLaunchKernelGGL(k_f2_round<F2_RANGE>, grid, dim3(kThreads), 0, st, a); break;
    default: hipLaunchKernelGGL(k_f2_round<F2_RELU>, grid, dim3(kThreads), 0, st, a); break;
    }
}

// ---------------------------------------------------------------------------
// The rounds' evaluations from the blocks' partials (one workgroup per
// round: round j of an instance over 2^v entries had f2_blocks(2^(v-1-j))
// blocks), written as pairs, D + 1 per round; workgroup 0 also writes the
// instance's final words:
//   F2_MATMUL  c0 = g_1(0) + g_1(1) (a b with no rounds), a*, b*
//   F2_RANGE   b~(sigma)
//   F2_RELU    R~(rho') = (D + S) / 2, Y~(rho') = (S - D) / 2
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_f2_finish(F2FinishArgs a)
{
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    const int j = blockIdx.x, D = a.kind == F2_MATMUL ? 2 : 3;
    uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (j < a.v) {
        const int nb = f2_blocks(1ull << (a.v - 1 - j));
        const uint64_t *p = a.part + (size_t)j * kF2MaxBlocks * 8;
        for (int b = threadIdx.x; b < nb; b += blockDim.x)
#pragma unroll
            for (int q = 0; q < 8; q++) v[q] = m61::add(v[q], p[8 * (size_t)b + q]);
        m61::block_sum<8>(v, red);
        if (threadIdx.x == 0)
            for (int q = 0; q < 2 * (D + 1); q++) a.ev[2 * (D + 1) * j + q] = v[q];
    }
    if (j != 0 || threadIdx.x != 0) return;
    if (a.kind == F2_MATMUL) {
        const f2 t0 = ldt(a.t[0], 0), t1 = ldt(a.t[1], 0);
        const f2 c0 = a.v > 0 ? f2add(f2{v[0], v[1]}, f2{v[2], v[3]}) : f2mul(t0, t1);
        stp(a.fin, c0);
        stp(a.fin + 2, t0);
        stp(a.fin + 4, t1);
    } else if (a.kind == F2_RANGE) {
        stp(a.fin, ldt(a.t[1], 0));
    } else {
        f2 Dv, Sv;
        if (a.v > 0) {
            Dv = ldt(a.t[1], 0);
            Sv = ldt(a.t[2], 0);
        } else {
            Dv = f2of(m61::from_i64((int64_t)a.R[0] - a.Y[0]));
            Sv = f2of(m61::from_i64((int64_t)a.R[0] + a.Y[0]));
        }
        constexpr uint64_t inv2 = 1ull << 60;  // 2 2^60 = 2^61 = 1 mod p
        stp(a.fin, f2scale(f2add(Dv, Sv), inv2));
        stp(a.fin + 2, f2scale(f2sub(Sv, Dv), inv2));
    }
}

void launch_f2_finish(const F2FinishArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_finish, dim3(a.v > 0 ? a.v : 1), dim3(kThreads), 0, st, a);
}

// ---------------------------------------------------------------------------
// The plane rounds of the range instance from the Gram matrix G[p][p'] =
// sum_x EQ(x) bit_p(x) bit_p'(x) (one workgroup).  A bit squared is itself, so
// with the diagonal g = diag(G) and the plane weights W the summand's sums
// over x are
//   g_j(X) = K_j eq(tau_j, X) sum_q es(q) (Q - L) + mu sum_q w L
// where q runs over the planes after the free one, es = eq(tau_{>j}, .), and
// Q, L, w are G, g and W bound at (sigma_<j, X): Q quadratic in X from G's
// entries (q, q), (q, q + h), (q + h, q + h), L and w linear from entries q
// and q + h.  So a round needs eight sums over at most 32 planes (five with
// es, three of W with g), one per group of 32 lanes; then g and W are folded at
// sigma_j, and G on both sides (its upper triangle, h (h + 1) / 2 entries).
// Keeping G unfolded and forming c^T G c anew each round took 106 us (118 us
// with the challenges hashed, MI355X, 64 planes); this takes 37 and 61.
//
// Also writes the x rounds' constants c_eq = eq(tau_p, sigma_p), c_w =
// mu W~(sigma_p), the claimed sum mu (l1 Rm~ + l2 (R~ + 2^(t+1)) + l3 Y~) and,
// where wanted, the table eq(sigma_p, .).
// ---------------------------------------------------------------------------
__device__ __forceinline__ f2 group32_sum(f2 v)
{
#pragma unroll
    for (int off = 1; off < 32; off <<= 1)
        v = f2{m61::fold(v.re + __shfl_xor(v.re, off, 64)), m61::fold(v.im + __shfl_xor(v.im, off, 64))};
    return v;
}

// eq(z, .) of k variables at index i (first variable most significant)
__device__ __forceinline__ f2 eq_entry(const f2 *z, int k, int i)
{
    f2 e = f2of(1);
    for (int j = 0; j < k; j++) e = l2mul(e, eq1b(z[j], (i >> (k - 1 - j)) & 1));
    return e;
}

__global__ __launch_bounds__(256) void k_f2_planes(F2PlaneArgs a)
{
    constexpr int GS = 65;  // row stride of the staged Gram matrix (odd, so rows start in different banks)
    __shared__ uint64_t g_re[64 * GS], g_im[64 * GS];
    __shared__ f2 W[64], dv[64], es[64], tau[8], sig[8], lam[4], pre[8], tot[8], gsh[4];
    __shared__ f2 ev[4 * kMaxPlaneLog];  // the rounds' values: stores to memory would be waited for at each barrier
    __shared__ FsLds fsl;  // the transcript (Fiat-Shamir mode)
    const int tid = threadIdx.x, lP = a.lP, P = a.P;
    for (int e = tid; e < P * P; e += blockDim.x) {
        const int p = e >> lP, q = e & (P - 1);
        g_re[p * GS + q] = a.G_re[p * 64 + q];
        g_im[p * GS + q] = a.G_im[p * 64 + q];
    }
    if (tid < lP) {
        tau[tid] = ldp(a.tau + 2 * tid);
        if (!a.fs) sig[tid] = ldp(a.sig + 2 * tid);  // else drawn after each round
    }
    if (tid < 4) lam[tid] = ldp(a.lam + 2 * tid);
    if (a.fs) fs_pull(fsl, a.fs);
    __syncthreads();
    const f2 mu = lam[3];
    if (tid < 64) {
        f2 w = f2of(0);
        const int s = a.s, t = a.t;
        if (tid < s) w = f2scale(lam[0], 1ull << tid);
        else if (tid < s + t + 2) w = f2scale(lam[1], 1ull << (tid - s));
        else if (a.relu && tid < s + 2 * t + 4) w = f2scale(lam[2], 1ull << (tid - s - t - 2));
        W[tid] = tid < P ? w : f2of(0);
        if (tid < P) dv[tid] = f2{g_re[tid * GS + tid], g_im[tid * GS + tid]};
    } else if (tid < 128) {  // the suffix eq tables as a heap: 2^k entries from index 2^k, over the last k variables
        const int i = tid - 64;
        if (i >= 1 && i < P) {
            const int k = 31 - __builtin_clz(i);
            es[i] = eq_entry(tau + lP - k, k, i - (1 << k));
        }
    } else if (tid == 128) {
        pre[0] = f2of(1);  // pre[i] = prod over i' < i of eq(tau_i', sigma_i'), after round i - 1
    }
    __syncthreads();
    for (int jj = 0; jj < lP; jj++) {
        const int h = P >> (jj + 1);
        {   // the round's eight sums
            const int T = tid >> 5, q = tid & 31;
            f2 v = f2of(0);
            if (q < h) {
                const int e00 = q * GS + q, e01 = e00 + h, e11 = e00 + h * GS + h;
                f2 x, y;
                if (T < 5) {
                    x = es[h + q];
                    if (T == 0) y = f2{g_re[e00], g_im[e00]};
                    else if (T == 1) y = f2{g_re[e01], g_im[e01]};
                    else if (T == 2) y = f2{g_re[e11], g_im[e11]};
                    else y = dv[T == 3 ? q : q + h];
                } else if (T == 5) {
                    x = W[q];
                    y = dv[q];
                } else if (T == 6) {
                    x = W[q + h];
                    y = dv[q + h];
                } else {
                    x = l2add(W[q], W[q + h]);
                    y = l2add(dv[q], dv[q + h]);
                }
                v = l2mul(x, y);
            }
            v = group32_sum(v);
            if (q == 0) tot[T] = l2canon(v);
        }
        __syncthreads();
        if (tid < 4) {
            const int X = tid, u = 1 - X;
            const f2 cross = f2sub(f2sub(tot[7], tot[5]), tot[6]);
            f2 A = f2add(f2add(f2small(tot[0], u * u), f2small(tot[1], 2 * X * u)), f2small(tot[2], X * X));
            A = f2sub(f2sub(A, f2small(tot[3], u)), f2small(tot[4], X));
            const f2 B = f2add(f2add(f2small(tot[5], u * u), f2small(cross, X * u)), f2small(tot[6], X * X));
            const f2 g = f2add(f2mul(f2mul(pre[jj], eq1x(tau[jj], X)), A), f2mul(mu, B));
            ev[4 * jj + tid] = g;
            gsh[tid] = g;
        }
        __syncthreads();
        if (a.fs) {  // the round's values absorbed, sigma_jj drawn
            if (!fs_absorb(fsl, (const uint32_t *)gsh, 16) && tid == 0) *a.err = 1;
            fs_draw(fsl);
            if (tid == 0) sig[jj] = f2{fsl.out[0], fsl.out[1]};
            __syncthreads();
        }
        const f2 sg = sig[jj];
        if (tid == 255) pre[jj + 1] = f2mul(pre[jj], eq1z(tau[jj], sg));
        // the folds; an entry's four sources are read by its own thread only
        if (tid < h) dv[tid] = l2fold(dv[tid], dv[tid + h], sg);
        else if (tid >= 64 && tid < 64 + h) W[tid - 64] = l2fold(W[tid - 64], W[tid - 64 + h], sg);
        if (h > 1)
            for (int e = tid; e < (h / 2) * (h + 1); e += blockDim.x) {
                // the upper triangle, rows r and h - 1 - r side by side (h + 1 entries)
                const int r = e / (h + 1), c = e - r * (h + 1), first = h - r;
                const int i = c < first ? r : h - 1 - r, k = c < first ? r + c : i + c - first;
                // (i, k), (i, k + h), (i + h, k) = (k, i + h) by symmetry, (i + h, k + h)
                const int e00 = i * GS + k, e01 = e00 + h, e10 = k * GS + i + h, e11 = e00 + h * GS + h;
                const f2 lo = l2fold(f2{g_re[e00], g_im[e00]}, f2{g_re[e10], g_im[e10]}, sg);
                const f2 hi = l2fold(f2{g_re[e01], g_im[e01]}, f2{g_re[e11], g_im[e11]}, sg);
                const f2 o = l2fold(lo, hi, sg);
                g_re[e00] = o.re;
                g_im[e00] = o.im;
            }
        __syncthreads();
    }
    if (a.fs) fs_push(a.fs, fsl);
    if (tid >= 192 && tid - 192 < 4 * lP) stp(a.ev + 2 * (tid - 192), ev[tid - 192]);
    if (tid < 64 && a.sig_tab.re) stt(a.sig_tab, tid, tid < P ? l2canon(eq_entry(sig, lP, tid)) : f2of(0));
    if (tid == 64) {  // x rounds' constants
        stp(a.cst, pre[lP]);
        stp(a.cst + 2, f2mul(mu, l2canon(W[0])));
    } else if (tid == 128) {  // the claimed sum
        const f2 r = ldp(a.claims), rm = ldp(a.claims + 2), y = ldp(a.claims + 4);
        f2 H = f2add(f2mul(lam[0], rm), f2mul(lam[1], f2add(r, f2of(1ull << (a.t + 1)))));
        if (a.relu) H = f2add(H, f2mul(lam[2], y));
        stp(a.range_sum, f2mul(mu, H));
    }
}

void launch_f2_planes(const F2PlaneArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_planes, dim3(1), dim3(kThreads), 0, st, a);
}

// The Gram matrix's two parts from the partial tiles of their passes.
__global__ __launch_bounds__(256) void k_f2_gram_sum(const uint64_t *__restrict__ gp_re,
                                                     const uint64_t *__restrict__ gp_im, int nblk, int tiles,
                                                     uint64_t *__restrict__ G_re, uint64_t *__restrict__ G_im)
{
    __shared__ uint64_t red[kGramReduceLdsWords];
    gram_reduce_block(blockIdx.y ? gp_im : gp_re, nblk, tiles, blockIdx.y ? G_im : G_re, blockIdx.x, red);
}

void launch_f2_gram_sum(const uint64_t *gp_re, const uint64_t *gp_im, int nblk, int tiles, uint64_t *G_re,
                        uint64_t *G_im, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_gram_sum, dim3(gram_reduce_groups(tiles), 2), dim3(kThreads), 0, st, gp_re, gp_im, nblk,
                       tiles, G_re, G_im);
}

}  // namespace ra
