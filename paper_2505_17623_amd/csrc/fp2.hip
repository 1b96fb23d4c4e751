// fp2.hip -- the layer protocol with the verifier's challenges in the
// quadratic extension F_{p^2} = F_p[i] / (i^2 + 1) (p = 2^61 - 1 is 3 mod 4,
// so x^2 + 1 is irreducible).  Sec. II-F asks for a field of more than 128
// bits; a sum-check round over F_{p^2} lets a cheating prover pass with
// probability about d / p^2 instead of d / p (Sec. II-D).
//
// The witness (C, R, Rm, Y, Z, the bit table) is integer-valued and is made
// by the F_p kernels.  Everything that depends on a challenge is an element
// of F_{p^2}, held as two F_p tables (real and imaginary parts, "SoA"):
//   - the eq tables E1 = eq(r1, .), E2 = eq(r2, .) and, for the claims and the
//     Gram pass, EQ(x) = E1 E2;
//   - the bound sides of the product (an integer table bound at a point of
//     F_{p^2} is the pair of its F_p bindings with the eq table's two parts,
//     formed in one pass);
//   - the plane rounds' Gram matrix G = sum_x EQ(x) bit bit^T, whose two
//     parts the F_p Gram pass computes from EQ's two parts;
//   - every folded table of the rounds.
#include <algorithm>

#include "common.hpp"
#include "f2.hpp"
#include "gram_reduce.hpp"
#include "limbs.hpp"
#include "ra.h"
#include "fs_device.hpp"
#include "sha256.hpp"

namespace ra {

// The eq tables of a layer in one launch, each entry the product of its
// variables' factors: E1, E2 (SoA) and the suffix eq tables of the point r = (r1,
// r2), which the rounds take their weights from.  LS: the last kF2Low variables,
// a heap: entry 2^k + y is eq over the last k variables at y.  HS: the variables
// before them, in the same form.
__global__ __launch_bounds__(256) void k_f2_eqs(const uint64_t *__restrict__ r, int ln, int lk, F2Tab E1, F2Tab E2,
                                                f2 *__restrict__ HS, f2 *__restrict__ LS,
                                                const uint64_t *__restrict__ sig, int lP, F2Tab SIG)
{
    __shared__ f2 z[64];
    const int lN = ln + lk, low = lN < kF2Low ? lN : kF2Low, hs = lN - low;
    if (sig && blockIdx.x == gridDim.x - 1) {  // eq(sig, .)
        if ((int)threadIdx.x < lP) z[threadIdx.x] = ldp(sig + 2 * threadIdx.x);
        __syncthreads();
        if (threadIdx.x < 64) {
            f2 e = f2of((int)threadIdx.x < (1 << lP) ? 1 : 0);
            for (int j = 0; j < lP; j++) e = l2mul(e, eq1b(z[j], (int)((threadIdx.x >> (lP - 1 - j)) & 1)));
            stt(SIG, threadIdx.x, l2canon(e));
        }
        return;
    }
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

void launch_f2_eqs(const uint64_t *r, int ln, int lk, F2Tab E1, F2Tab E2, f2 *HS, f2 *LS, hipStream_t st,
                   const uint64_t *sig, int lP, F2Tab SIG)
{
    const int lN = ln + lk, low = lN < kF2Low ? lN : kF2Low;
    const uint64_t tot = (1ull << ln) + (1ull << lk) + (2ull << low) + (2ull << (lN - low));
    hipLaunchKernelGGL(k_f2_eqs, dim3((unsigned)((tot + kThreads - 1) / kThreads) + (sig ? 1 : 0)), dim3(kThreads), 0, st,
                       r, ln, lk, E1, E2, HS, LS, sig, lP, SIG);
}

// ---------------------------------------------------------------------------
// The bound sides of the product.  Binding an integer table at a point of
// F_{p^2} is linear in the eq table, so one pass over the table sums both
// parts, by limbs of the eq values (limbs.hpp).  Two F_p
// bindings per side read each table twice and took six launches.
// ---------------------------------------------------------------------------
// part[chunk][2 cols]: the sums over a chunk's rows, real parts then imaginary
template <typename T>
__device__ __forceinline__ void f2_bind_rows(const T *__restrict__ A, uint32_t rows, uint32_t cols, F2Tab E,
                                             uint32_t per_chunk, uint64_t *__restrict__ part, uint32_t group,
                                             uint32_t chunk, uint64_t (*red)[2][64])
{
    using L = BindLimbs<T>;
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t c = group * 64 + lane;
    const uint32_t r0 = chunk * per_chunk;
    const uint32_t r1 = r0 + per_chunk < rows ? r0 + per_chunk : rows;
    uint64_t re = 0, im = 0;
    for (uint32_t b = r0 + wid; b < r1; b += 4 * L::kRun) {  // a wave's run: rows b, b + 4, ..
        const uint64_t e1 = (uint64_t)b + 4ull * L::kRun;
        const uint32_t e = e1 < r1 ? (uint32_t)e1 : r1;
        int64_t sr[L::kCount] = {}, si[L::kCount] = {};
#pragma unroll 4
        for (uint32_t r = b; r < e; r += 4) {
            const int32_t z = c < cols ? (int32_t)A[(size_t)r * cols + c] : 0;
            const uint64_t x = E.re[r], y = E.im[r];
#pragma unroll
            for (int i = 0; i < L::kCount; i++) {
                sr[i] += (int64_t)(int32_t)((x >> (L::kBits * i)) & ((1u << L::kBits) - 1)) * z;
                si[i] += (int64_t)(int32_t)((y >> (L::kBits * i)) & ((1u << L::kBits) - 1)) * z;
            }
        }
        re = m61::add(re, limbs_value<L::kBits>(sr));
        im = m61::add(im, limbs_value<L::kBits>(si));
    }
    red[wid][0][lane] = re;
    red[wid][1][lane] = im;
    __syncthreads();
    if (wid < 2 && c < cols)
        part[((size_t)chunk * 2 + wid) * cols + c] =
            m61::add(m61::add(red[0][wid][lane], red[1][wid][lane]), m61::add(red[2][wid][lane], red[3][wid][lane]));
}

// B's columns, a wave per four rows: lanes take eight consecutive columns (one
// 16-byte load per row) and read each eq value once for the four rows.
__device__ __forceinline__ void f2_bind_cols(const int16_t *__restrict__ B, uint32_t rows, uint32_t cols, F2Tab E,
                                             F2Tab out, uint32_t block)
{
    using L = BindLimbs<int16_t>;
    constexpr int RW = 4;
    const uint32_t r0 = ((block * blockDim.x + threadIdx.x) >> 6) * RW;  // wave-uniform
    const int lane = threadIdx.x & 63;
    if (r0 >= rows) return;
    typedef int v4i __attribute__((ext_vector_type(4)));
    f2 acc[RW];
#pragma unroll
    for (int rr = 0; rr < RW; rr++) acc[rr] = f2of(0);
    for (uint64_t b = 8 * lane; b < cols; b += (uint64_t)512 * (L::kRun / 8)) {  // at most kRun entries per lane
        int64_t sr[RW][2] = {}, si[RW][2] = {};
        const uint64_t e = b + (uint64_t)512 * (L::kRun / 8) < cols ? b + (uint64_t)512 * (L::kRun / 8) : cols;
        for (uint64_t c0 = b; c0 < e; c0 += 512) {
            int32_t x[8][4];
#pragma unroll
            for (int t = 0; t < 8; t++) {
                const uint64_t re = E.re[c0 + t], im = E.im[c0 + t];
                x[t][0] = (int32_t)(re & 0x7FFFFFFFull);
                x[t][1] = (int32_t)(re >> 31);
                x[t][2] = (int32_t)(im & 0x7FFFFFFFull);
                x[t][3] = (int32_t)(im >> 31);
            }
#pragma unroll
            for (int rr = 0; rr < RW; rr++) {
                if (r0 + rr >= rows) break;
                const v4i z4 = *(const v4i *)&B[(size_t)(r0 + rr) * cols + c0];
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    const int32_t z = (int32_t)(int16_t)(z4[t >> 1] >> (16 * (t & 1)));
                    sr[rr][0] += (int64_t)x[t][0] * z;
                    sr[rr][1] += (int64_t)x[t][1] * z;
                    si[rr][0] += (int64_t)x[t][2] * z;
                    si[rr][1] += (int64_t)x[t][3] * z;
                }
            }
        }
#pragma unroll
        for (int rr = 0; rr < RW; rr++)
            acc[rr] = f2add(acc[rr], f2{limbs_value<31>(sr[rr]), limbs_value<31>(si[rr])});
    }
#pragma unroll
    for (int rr = 0; rr < RW; rr++) {
        f2 v = acc[rr];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) v = l2add(v, f2{__shfl_xor(v.re, off, 64), __shfl_xor(v.im, off, 64)});
        if (lane == 0 && r0 + rr < rows) stt(out, r0 + rr, l2canon(v));
    }
}

// EQ(x) = E1[x >> lk] E2[x mod 2^lk] for x < N (the eq table of (r1, r2),
// folded parts) and, on the way, the claims R~, Rm~, Y~ and Z~ = (R~ + Y~) / 2
// (ReLU, else R~) at (r1, r2): sum_x EQ(x) v(x) in 21-bit limbs of EQ, exact in
// int64 over runs of 1024 entries.  Per-block partials, eight words per block.
__device__ __forceinline__ void f2_claims(F2Tab E1, F2Tab E2, int lk, F2Tab EQ, const int32_t *__restrict__ R,
                                          const uint16_t *__restrict__ Rm, const int32_t *__restrict__ Y, int relu,
                                          uint64_t N, uint64_t *part, uint32_t block, uint32_t blocks, uint64_t *red,
                                          uint64_t *tot)
{
    const uint64_t mask = (1ull << lk) - 1, stride = (uint64_t)blocks * blockDim.x;
    uint64_t acc[6] = {0, 0, 0, 0, 0, 0};
    for (uint64_t b = (uint64_t)block * blockDim.x + threadIdx.x; b < N; b += 1024 * stride) {
        int64_t s[6][3] = {};
        const uint64_t e1 = b + 1024 * stride, end = e1 < N ? e1 : N;
        for (uint64_t x = b; x < end; x += stride) {
            const int32_t r = R[x], rm = Rm[x], y = Y[x];
            const f2 e = l2mul(ldt(E1, x >> lk), ldt(E2, x & mask));
            stt(EQ, x, e);
#pragma unroll
            for (int i = 0; i < 3; i++) {
                const int32_t a = (int32_t)((e.re >> (21 * i)) & 0x1FFFFF), c = (int32_t)((e.im >> (21 * i)) & 0x1FFFFF);
                s[0][i] += (int64_t)a * r;
                s[1][i] += (int64_t)c * r;
                s[2][i] += (int64_t)a * rm;
                s[3][i] += (int64_t)c * rm;
                s[4][i] += (int64_t)a * y;
                s[5][i] += (int64_t)c * y;
            }
        }
#pragma unroll
        for (int q = 0; q < 6; q++) acc[q] = m61::add(acc[q], limbs_value<21>(s[q]));
    }
    f2_totals<6>(acc, red, tot, blockDim.x);
    if (threadIdx.x < 8) {
        const int p = threadIdx.x & 1;
        uint64_t v = threadIdx.x < 6 ? tot[threadIdx.x] : tot[p];
        if (threadIdx.x >= 6 && relu) v = m61::rotl(m61::add(v, tot[4 + p]), 60);  // 1 / 2 = 2^60
        part[8 * (size_t)block + threadIdx.x] = v;
    }
}

// The column binding, the claims and the row binding in one launch, longest
// first: each alone leaves the chip waiting on loads (one or two waves per
// SIMD), and none needs another's results.  Three launches one after the other
// took 53 us for a 512 x 4096 by 4096 x 4096 layer, this and the launch that
// sums the row chunks 36 to 40 (MI355X).
template <typename T>
__global__ __launch_bounds__(256) void k_f2_sides(F2Sides a, const T *__restrict__ A)
{
    __shared__ union {
        uint64_t red[6 * 256];
        uint64_t rows[4][2][64];
    } u;
    __shared__ uint64_t tot[6];
    uint32_t b = blockIdx.x;
    if (b < a.ncols) {
        f2_bind_cols(a.B, a.m, a.k, a.E2, a.Tb, b);
        return;
    }
    b -= a.ncols;
    if (b < a.nclaims) {
        f2_claims(a.E1, a.E2, a.lk, a.EQ, a.R, a.Rm, a.Y, a.relu, a.N, a.cpart, b, a.nclaims, u.red, tot);
        return;
    }
    b -= a.nclaims;
    f2_bind_rows<T>(A, a.n, a.m, a.E1, a.per, a.chunks, b % a.groups, b / a.groups, u.rows);
}

// out = the chunk rows of part (cols words each) added up
__global__ __launch_bounds__(256) void k_f2_sum_chunks(const uint64_t *__restrict__ part, int nch, uint32_t cols,
                                                       uint64_t *__restrict__ out)
{
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    if (c >= cols) return;
    uint64_t v = 0;
#pragma unroll 8
    for (int q = 0; q < nch; q++) v = m61::fold(v + part[(size_t)q * cols + c]);
    out[c] = m61::canon(v);
}

void launch_f2_sides(F2Sides a, const void *A, int a_dtype, uint64_t *scr, F2Tab Ta, hipStream_t st)
{
    const int nch = bind_rows_chunks(a.n, a.m);
    a.per = (a.n + nch - 1) / nch;
    a.groups = (a.m + 63) / 64;
    a.chunks = nch > 1 ? scr : Ta.re;  // one chunk: its sums are canonical and Ta's parts lie one after the other
    // 16-byte loads of eight columns where B's rows allow them, else the two parts one after the other
    const bool vec = a.k >= 8 && ((uintptr_t)a.B & 15) == 0;
    a.ncols = vec ? ((a.m + 3) / 4 + 3) / 4 : 0;
    a.nclaims = f2_blocks(a.N);
    const dim3 grid(a.ncols + a.nclaims + a.groups * nch);
    if (a_dtype == RA_I16)
        hipLaunchKernelGGL(k_f2_sides<int16_t>, grid, dim3(256), 0, st, a, (const int16_t *)A);
    else
        hipLaunchKernelGGL(k_f2_sides<int32_t>, grid, dim3(256), 0, st, a, (const int32_t *)A);
    if (nch > 1)
        hipLaunchKernelGGL(k_f2_sum_chunks, dim3((2 * a.m + 255) / 256), dim3(256), 0, st, (const uint64_t *)scr, nch,
                           2 * a.m, Ta.re);
    if (!vec) {
        launch_bind_cols(a.B, RA_I16, a.m, a.k, a.E2.re, a.Tb.re, st);
        launch_bind_cols(a.B, RA_I16, a.m, a.k, a.E2.im, a.Tb.im, st);
    }
}

// ---------------------------------------------------------------------------
// The rounds over tables with given challenges (Sec. II-D; eq factored, see
// F2Sums): the matrix instance, the range instance once its plane variables
// are bound, and the ReLU zero-check.
//
// While a table holds more than 2^kF2TailLog entries a pass takes two rounds
// per launch in registers: a thread reads the four entries of a quad, sums
// both rounds and writes the one entry left, so a table crosses memory 1.25
// times per two rounds, and the range and the ReLU instance share the launch.
// Bound by the field products (19 of F_{p^2} per range quad, about 1100 VALU
// instructions).  One round per launch over tables that carried EQ took 430 us
// for the two instances of 2^21 and the one of 2^21 without ReLU; this takes
// 160 (MI355X).
// ---------------------------------------------------------------------------
template <int KIND, bool INTS>
__device__ __forceinline__ void f2_pass(const F2PassArgs &a, uint64_t *red, uint64_t *tot)
{
    constexpr int NW = f2_sum_words(KIND), NT = KIND == F2_RANGE ? 1 : 2;
    const f2 rho0 = ldp(a.rho), rho1 = ldp(a.rho + 2);
    f2 r1 = f2of(0);
    if (KIND != F2_MATMUL) r1 = ldp(a.r + 2);  // the second round's variable
    const f2 nr1 = f2sub(f2of(1), r1);
    F2Sums<KIND> s0, s1;
    const uint64_t n = a.n, first = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (uint64_t i = first; i < n; i += (uint64_t)f2_blocks(n) * blockDim.x) {
        // weights: the high variables here (the same for the whole workgroup), the low ones at the end;
        // the first round's pairs (x0, x2), (x1, x3) carry the second variable's factors
        f2 w = f2of(1), w0 = f2of(1), w1 = f2of(1);
        if (KIND != F2_MATMUL) {
            w = a.HS[(n >> kF2Low ? n >> kF2Low : 1) + (i >> kF2Low)];
            w0 = l2mul(w, nr1);
            w1 = l2sub(w, w0);
        }
        f2 y[2][2];
        if (INTS) {
            uint64_t d[4], s[4];
#pragma unroll
            for (int t = 0; t < 4; t++) relu_ints(a.R, a.Y, i + t * n, d[t], s[t]);
            if constexpr (KIND == F2_RELU) {
                s0.add_int(w0, d[0], d[2], s[0], s[2]);
                s0.add_int(w1, d[1], d[3], s[1], s[3]);
            }
            y[0][0] = fold_real(d[0], d[2], rho0);
            y[0][1] = fold_real(d[1], d[3], rho0);
            y[1][0] = fold_real(s[0], s[2], rho0);
            y[1][1] = fold_real(s[1], s[3], rho0);
        } else {
            f2 x[NT][4];
#pragma unroll
            for (int q = 0; q < NT; q++)
#pragma unroll
                for (int t = 0; t < 4; t++) x[q][t] = ldt(a.src[q], i + t * n);
            if constexpr (KIND == F2_MATMUL) {
                s0.add(x[0][0], x[0][2], x[NT - 1][0], x[NT - 1][2]);
                s0.add(x[0][1], x[0][3], x[NT - 1][1], x[NT - 1][3]);
            } else {
                s0.add(l2mul(w0, x[0][0]), l2mul(w0, x[0][2]), x[NT - 1][0], x[NT - 1][2]);
                s0.add(l2mul(w1, x[0][1]), l2mul(w1, x[0][3]), x[NT - 1][1], x[NT - 1][3]);
            }
#pragma unroll
            for (int q = 0; q < NT; q++)
#pragma unroll
                for (int t = 0; t < 2; t++) y[q][t] = l2fold(x[q][t], x[q][t + 2], rho0);
        }
        if constexpr (KIND == F2_MATMUL) s1.add(y[0][0], y[0][1], y[NT - 1][0], y[NT - 1][1]);
        else s1.add(l2mul(w, y[0][0]), l2mul(w, y[0][1]), y[NT - 1][0], y[NT - 1][1]);
#pragma unroll
        for (int q = 0; q < NT; q++) stt(a.dst[q], i, l2fold(y[q][0], y[q][1], rho1));
    }
    f2 w = f2of(1);
    if (KIND != F2_MATMUL) {
        const uint32_t low = n < (1u << kF2Low) ? (uint32_t)n : 1u << kF2Low;
        w = a.LS[low + (uint32_t)(first & (low - 1))];
    }
    uint64_t v[NW];
    s0.words(v, KIND != F2_MATMUL, w);
    f2_totals<NW>(v, red, tot, blockDim.x);
    if (threadIdx.x < NW) a.part[(size_t)threadIdx.x * kF2MaxBlocks + blockIdx.x] = tot[threadIdx.x];
    s1.words(v, KIND != F2_MATMUL, w);
    f2_totals<NW>(v, red, tot, blockDim.x);
    if (threadIdx.x < NW) a.part[(size_t)(10 + threadIdx.x) * kF2MaxBlocks + blockIdx.x] = tot[threadIdx.x];
}

template <int KIND> __global__ __launch_bounds__(256) void k_f2_pass(F2PassArgs a)
{
    __shared__ uint64_t red[10 * 256], tot[10];
    f2_pass<KIND, false>(a, red, tot);
}

// The range and the ReLU instance side by side.
template <bool INTS> __global__ __launch_bounds__(256) void k_f2_pass_both(F2PassArgs range, F2PassArgs relu)
{
    __shared__ uint64_t red[10 * 256], tot[10];
    if (blockIdx.y == 0) f2_pass<F2_RANGE, false>(range, red, tot);
    else f2_pass<F2_RELU, INTS>(relu, red, tot);
}

void launch_f2_pass(const F2PassArgs &a, const F2PassArgs *relu, hipStream_t st)
{
    const dim3 grid(f2_blocks(a.n), relu ? 2 : 1), blk(kThreads);
    if (relu && relu->R) hipLaunchKernelGGL(k_f2_pass_both<true>, grid, blk, 0, st, a, *relu);
    else if (relu) hipLaunchKernelGGL(k_f2_pass_both<false>, grid, blk, 0, st, a, *relu);
    else if (a.kind == F2_RANGE) hipLaunchKernelGGL(k_f2_pass<F2_RANGE>, grid, blk, 0, st, a);
    else hipLaunchKernelGGL(k_f2_pass<F2_MATMUL>, grid, blk, 0, st, a);
}

// ---------------------------------------------------------------------------
// The last v <= kF2TailLog rounds of every instance, all rounds' values and
// the final values, in one launch.  The challenges are known, so the rounds
// need not wait for each other: workgroup c folds the table c times in LDS
// (each half the work of the one before) and sums round c alone; the rounds
// of the passes have a workgroup each too, which sums their partials.  (All
// rounds of an instance in one workgroup took 53 us.)
// ---------------------------------------------------------------------------
struct F2TailLds {
    f2 T[2][1 << kF2TailLog], g[4], K;
    uint64_t red[10 * kF2TailThreads], tot[10];
};

template <int KIND> __device__ __forceinline__ void f2_tail(const F2TailArgs &a, F2TailLds &s)
{
    constexpr int NW = f2_sum_words(KIND), NT = KIND == F2_RANGE ? 1 : 2, D1 = KIND == F2_MATMUL ? 3 : 4;
    const int tid = threadIdx.x, rounds = a.j0 + a.v, j = blockIdx.x;  // this workgroup's round; j = rounds: the final values
    if (j > rounds) return;
    if (tid < 64) {  // K_j
        f2 k = f2of(1);
        if (KIND != F2_MATMUL && tid < j && j < rounds) k = eq1z(ldp(a.r + 2 * tid), ldp(a.rho + 2 * tid));
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) k = l2mul(k, f2{__shfl_xor(k.re, off, 64), __shfl_xor(k.im, off, 64)});
        if (tid == 0) s.K = l2canon(k);
    }
    if (j < a.j0) {  // a pass's round
        const uint64_t *part = a.part + (size_t)(j >> 1) * kF2PassPart + (size_t)(j & 1) * 10 * kF2MaxBlocks;
        const int nb = f2_blocks(a.n0 >> (j & ~1)), lane = tid & 63;
        for (int q = tid >> 6; q < NW; q += blockDim.x >> 6) {
            uint64_t v = 0;
            for (int b = lane; b < nb; b += 64) v = m61::fold(v + part[(size_t)q * kF2MaxBlocks + b]);
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) v = m61::fold(v + __shfl_xor(v, off, 64));
            if (lane == 0) s.tot[q] = m61::canon(v);
        }
        __syncthreads();
    } else {
        const int c = j - a.j0;
        int n = 1 << a.v;  // entries
        for (int i = tid; i < n; i += blockDim.x)
#pragma unroll
            for (int q = 0; q < NT; q++) {
                f2 x;
                if (KIND == F2_RELU && a.R) {
                    const int64_t r = a.R[i], y = a.Y[i];
                    x = f2of(m61::from_i64(q == 0 ? r - y : r + y));
                } else {
                    x = ldt(a.src[q], i);
                }
                s.T[q][i] = x;
            }
        __syncthreads();
        for (int b = 0; b < c; b++) {  // an entry's two sources are read by its own thread only
            const f2 rho = ldp(a.rho + 2 * (a.j0 + b));
            n >>= 1;
            for (int i = tid; i < n; i += blockDim.x)
#pragma unroll
                for (int q = 0; q < NT; q++) s.T[q][i] = l2fold(s.T[q][i], s.T[q][i + n], rho);
            __syncthreads();
        }
        if (j == rounds) {
            constexpr uint64_t inv2 = 1ull << 60;  // 2 2^60 = 2^61 = 1 mod p
            if (tid != 0) return;
            const f2 x = l2canon(s.T[0][0]), y = l2canon(s.T[NT - 1][0]);
            if (KIND == F2_MATMUL) {  // a*, b*, and with no rounds c0 = a b
                if (rounds == 0) stp(a.out, f2mul(x, y));
                stp(a.out + 2, x);
                stp(a.out + 4, y);
            } else if (KIND == F2_RANGE) {
                stp(a.out, x);
            } else {  // R~ = (D + S) / 2, Y~ = (S - D) / 2
                stp(a.out, f2scale(f2add(x, y), inv2));
                stp(a.out + 2, f2scale(f2sub(y, x), inv2));
            }
            return;
        }
        const int h = n >> 1;
        F2Sums<KIND> acc;
        for (int i = tid; i < h; i += blockDim.x) {
            if constexpr (KIND == F2_MATMUL) {
                acc.add(s.T[0][i], s.T[0][i + h], s.T[NT - 1][i], s.T[NT - 1][i + h]);
            } else {
                const f2 w = a.LS[h + i];
                acc.add(l2mul(w, s.T[0][i]), l2mul(w, s.T[0][i + h]), s.T[NT - 1][i], s.T[NT - 1][i + h]);
            }
        }
        uint64_t v[NW];
        acc.words(v, false, f2of(1));
        f2_totals<NW>(v, s.red, s.tot, h < 64 ? 64 : (h < kF2TailThreads ? h : kF2TailThreads));
    }
    if (tid < D1) {
        const f2 r = KIND == F2_MATMUL ? f2of(0) : ldp(a.r + 2 * j);
        const f2 g = f2_round_value(KIND, s.tot, tid, s.K, r, a.cst);
        stp(a.ev + 2 * (D1 * j + tid), g);
        s.g[tid] = g;
    }
    __syncthreads();
    if (KIND == F2_MATMUL && j == 0 && tid == 0) stp(a.out, f2add(s.g[0], s.g[1]));  // c0 = g_1(0) + g_1(1)
}

__global__ __launch_bounds__(kF2TailThreads) void k_f2_tails(F2TailArgs mm, F2TailArgs rs, F2TailArgs zc)
{
    __shared__ F2TailLds s;
    if (blockIdx.y == 0) f2_tail<F2_MATMUL>(mm, s);
    else if (blockIdx.y == 1) f2_tail<F2_RANGE>(rs, s);
    else f2_tail<F2_RELU>(zc, s);
}

void launch_f2_tails(const F2TailArgs &mm, const F2TailArgs &rs, const F2TailArgs *zc, hipStream_t st)
{
    const int x = 1 + std::max(mm.j0 + mm.v, rs.j0 + rs.v);
    hipLaunchKernelGGL(k_f2_tails, dim3(x, zc ? 3 : 2), dim3(kF2TailThreads), 0, st, mm, rs, zc ? *zc : F2TailArgs{});
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
// with the challenges hashed, MI355X, 64 planes); the evaluation on four
// threads in canonical arithmetic and sums through LDS lane reads 37 and 61; this
// takes 28 and 44.
//
// Also writes the x rounds' constants c_eq = eq(tau_p, sigma_p), c_w =
// mu W~(sigma_p), the claimed sum mu (l1 Rm~ + l2 (R~ + 2^(t+1)) + l3 Y~) and,
// where wanted, the table eq(sigma_p, .).
// ---------------------------------------------------------------------------
__device__ __forceinline__ f2 group32_sum(f2 v)
{
    v = f2{sum16(v.re), sum16(v.im)};
    return f2{m61::fold(v.re + __shfl_xor(v.re, 16, 64)), m61::fold(v.im + __shfl_xor(v.im, 16, 64))};
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
    __shared__ f2 ke[2][4];  // K_j eq(tau_j, X), by j's parity
    __shared__ f2 ev[4 * kMaxPlaneLog];  // the rounds' values: stores to memory would be waited for at each barrier
    __shared__ FsLds fsl;  // the transcript (Fiat-Shamir mode)
    const int tid = threadIdx.x, lP = a.lP, P = a.P;
#pragma unroll 8
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
    } else if (tid >= 192 && tid < 196 && lP) {
        ke[0][tid - 192] = l2eq1x(tau[0], tid - 192);
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
        if (tid < 64) {
            // lanes 0 .. 3: K_j eq(tau_j, X) A(X); 4 .. 7: mu B(X); each from
            // its values at 0 and 1 and its leading coefficient
            const int X = tid & 3;
            const bool second = tid & 4;
            const f2 t0 = tot[second ? 5 : 0], t1 = tot[second ? 6 : 2], tm = tot[second ? 7 : 1], t = l2add(t0, t1);
            const f2 lo = second ? t0 : l2sub(t0, tot[3]), hi = second ? t1 : l2sub(t1, tot[4]);
            const f2 inf = second ? l2sub(l2add(t, t), tm) : l2sub(t, l2add(tm, tm));
            f2 g = l2add(l2add(lo, l2small(l2sub(hi, lo), X)), l2small(inf, X * (X - 1)));
            g = l2mul(second ? mu : ke[jj & 1][X], g);
            g = l2canon(l2add(g, f2{__shfl_xor(g.re, 4, 64), __shfl_xor(g.im, 4, 64)}));
            if (tid < 4) ev[4 * jj + tid] = g;
            if (a.fs) {
                if (tid < 4) gsh[tid] = g;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const uint32_t ql = fsl.m[8];
                const bool ok = fs_append(fsl, ql, gsh, 16, tid, 64);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (tid == 0) {
                    if (ok) fsl.m[8] = ql + 64;
                    else *a.err = 1;
                }
            }
        }
        if (a.fs) {  // the round's values absorbed, sigma_jj drawn
            fs_draw(fsl);
            if (tid == 0) sig[jj] = f2{fsl.out[0], fsl.out[1]};
        }
        const f2 sg = a.fs ? f2{fsl.out[0], fsl.out[1]} : sig[jj];
        if (tid >= 192 && tid < 196) {  // K_{j+1} and the factors of the next round's values
            const f2 ab = l2mul(tau[jj], sg);
            const f2 K = l2mul(pre[jj], l2add(l2sub(l2sub(f2of(1), tau[jj]), sg), l2add(ab, ab)));
            if (tid == 192) pre[jj + 1] = l2canon(K);
            if (jj + 1 < lP) ke[(jj + 1) & 1][tid - 192] = l2mul(K, l2eq1x(tau[jj + 1], tid - 192));
        }
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

// The Gram matrix's two parts from the partial tiles of their passes; the last
// workgroup in x (part 0) sums the claims' partials.
__global__ __launch_bounds__(256) void k_f2_gram_sum(const uint64_t *__restrict__ gp_re,
                                                     const uint64_t *__restrict__ gp_im, int nblk, int tiles,
                                                     uint64_t *__restrict__ G_re, uint64_t *__restrict__ G_im,
                                                     int groups, const uint64_t *__restrict__ cpart, int cblocks,
                                                     uint64_t *__restrict__ claims)
{
    __shared__ uint64_t red[kGramReduceLdsWords > 8 * 256 ? kGramReduceLdsWords : 8 * 256], tot[8];
    if ((int)blockIdx.x == groups) {
        if (blockIdx.y) return;
        uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int b = threadIdx.x; b < cblocks; b += blockDim.x)
#pragma unroll
            for (int q = 0; q < 8; q++) v[q] = m61::add(v[q], cpart[8 * (size_t)b + q]);
        f2_totals<8>(v, red, tot, blockDim.x);
        if (threadIdx.x < 8) claims[threadIdx.x] = tot[threadIdx.x];
        return;
    }
    gram_reduce_block(blockIdx.y ? gp_im : gp_re, nblk, tiles, blockIdx.y ? G_im : G_re, blockIdx.x, red);
}

void launch_f2_gram_sum(const uint64_t *gp_re, const uint64_t *gp_im, int nblk, int tiles, uint64_t *G_re,
                        uint64_t *G_im, const uint64_t *cpart, int cblocks, uint64_t *claims, hipStream_t st)
{
    const int groups = gram_reduce_groups(tiles);
    hipLaunchKernelGGL(k_f2_gram_sum, dim3(groups + (cpart ? 1 : 0), 2), dim3(kThreads), 0, st, gp_re, gp_im, nblk,
                       tiles, G_re, G_im, groups, cpart, cblocks, claims);
}

// The transcript and the statuses to mapped host memory (one launch instead
// of two to four copies).
__global__ __launch_bounds__(256) void k_f2_publish(F2Publish a)
{
    for (int i = threadIdx.x; i < a.nw; i += blockDim.x) a.dst[i] = a.tr[i];
    uint64_t *d = a.dst + a.nw;
    int any = 0;
    if (a.wit.known)
        for (int b = threadIdx.x; b < a.wit.nblk; b += blockDim.x) any |= a.wit.flags[b] != 0;
    any = __syncthreads_or(any);
    if (threadIdx.x == 0) {
        WitParams p = a.wit.known ? a.wit.hp : *a.wit.prm;
        if (any) p.status = RA_E_RANGE;
        *(WitParams *)d = p;
        d[8] = a.err ? *a.err : 0;
    }
    if (a.root && threadIdx.x >= 64 && threadIdx.x < 72) ((uint32_t *)(d + 9))[threadIdx.x - 64] = a.root[threadIdx.x - 64];
}

void launch_f2_publish(const F2Publish &a, hipStream_t st)
{
    hipLaunchKernelGGL(k_f2_publish, dim3(1), dim3(kThreads), 0, st, a);
}

}  // namespace ra
