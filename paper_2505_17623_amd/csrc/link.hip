// link.hip -- the gather link between layers.  Sec. III-C chains layers
// through their outputs; a convolution's input is a gather of the previous
// output (im2col: each input entry read by up to kh kw patch positions,
// zero padding; flattening: a permutation).  With A[a] = Z[src[a]] (0 where
// src[a] = -1), the next layer's claim A~(z) at the point z = (r1, rho) of its
// matrix sum-check is
//     A~(z) = sum_y Z[y] W_z[y],   W_z[y] = sum over the a with src[a] = y of eq(z, a),
// a degree-2 sum-check (Sec. II-D) over the entries of Z.  It ends in Z~(y*)
// (a claim on the previous output) and W~_z(y*) (computable from the public
// gather map).
//
// Kernels: the eq tables of the point and a cleared W, the weight table W (one
// pass over src, modular atomic adds since several entries read one y), the
// first rounds three per pass over the tables, and one launch in which every
// round has a workgroup of its own: it sums the passes' partials, or folds the
// small table up to its round and takes that round's sums.  The round
// challenges are fixed in advance, so no round waits for another's value.
#include <algorithm>

#include "common.hpp"
#include "m61.hpp"

namespace ra {

constexpr int kWeightRun = 4 * kThreads;  // entries per block and step of the weight pass

// eq(z, a) = E1[a >> lm] E2[a mod 2^lm] (row variables first), added to
// W[src[a]].  A source index outside [-1, nz) is not followed: it sets *bad.
// W[y] holds its sum mod p in any representative below 2^64: a word that wraps
// has lost 2^64 = 8, which is added back, so one atomic add serves an entry
// (reading, adding mod p and exchanging took two round trips and repeats under
// contention).  Four entries per thread keep four adds in flight.
__global__ __launch_bounds__(256) void k_link_weights(const int32_t *__restrict__ src, uint64_t na, int lm,
                                                      const uint64_t *__restrict__ E1, const uint64_t *__restrict__ E2,
                                                      uint64_t nz, unsigned long long *__restrict__ W,
                                                      uint32_t *__restrict__ bad)
{
    const uint64_t cmask = (1ull << lm) - 1, step = (uint64_t)gridDim.x * kWeightRun;
    for (uint64_t a0 = (uint64_t)blockIdx.x * kWeightRun + threadIdx.x; a0 < na; a0 += step) {
        int32_t y[4];
        unsigned long long v[4], old[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint64_t a = a0 + 256 * u;
            y[u] = a < na ? src[a] : -1;
            if (y[u] < -1 || (y[u] >= 0 && (uint64_t)y[u] >= nz)) {
                atomicOr(bad, 1u);
                y[u] = -1;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint64_t a = a0 + 256 * u;
            v[u] = y[u] >= 0 ? m61::lmul(E1[a >> lm], E2[a & cmask]) : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; u++) old[u] = y[u] >= 0 ? atomicAdd(W + y[u], v[u]) : 0;
#pragma unroll
        for (int u = 0; u < 4; u++)
            for (unsigned long long o = old[u], d = v[u]; o + d < o; d = 8) o = atomicAdd(W + y[u], 8ull);
    }
}

// R rounds over tables of 2^R q entries in one pass.  A round's polynomial is
// g(X) = sum_i T0(X) T1(X), T(X) = lo + X (hi - lo), then T <- lo + rho (hi -
// lo); a thread holds the 2^R entries that end in its entry of the folded
// tables.  Each round's block sums are those of lo lo, hi hi and (hi - lo)
// (hi - lo), the values at 0 and 1 and the leading coefficient.  The first pass
// reads T0 from the int32 table Z and W as the weights left it (any word).
template <int R, bool FIRST>
__global__ __launch_bounds__(256) void k_link_pass(const int32_t *__restrict__ Z, uint64_t *T0, uint64_t *T1, uint64_t q,
                                                   const uint64_t *__restrict__ rho_p, uint64_t *__restrict__ part)
{
    __shared__ uint64_t red[m61::block_sum_words(3 * R, 256)];
    uint64_t rho[R], g[3 * R] = {};
#pragma unroll
    for (int j = 0; j < R; j++) rho[j] = rho_p[j];
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < q; i += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t a[1 << R], b[1 << R];
#pragma unroll
        for (int k = 0; k < 1 << R; k++) {
            a[k] = FIRST ? m61::from_i32(Z[i + k * q]) : T0[i + k * q];
            b[k] = T1[i + k * q];
        }
        if (FIRST)
#pragma unroll
            for (int k = 0; k < 1 << R; k++) b[k] = m61::fold(b[k]);
#pragma unroll
        for (int j = 0; j < R; j++) {
            const int h = 1 << (R - 1 - j);
#pragma unroll
            for (int k = 0; k < h; k++) {
                const uint64_t da = m61::lsub(a[k + h], a[k]), db = m61::lsub(b[k + h], b[k]);
                g[3 * j] = m61::lmacc(g[3 * j], a[k], b[k]);
                g[3 * j + 1] = m61::lmacc(g[3 * j + 1], a[k + h], b[k + h]);
                g[3 * j + 2] = m61::lmacc(g[3 * j + 2], da, db);
                a[k] = m61::lmacc(a[k], rho[j], da);
                b[k] = m61::lmacc(b[k], rho[j], db);
            }
        }
        T0[i] = a[0];
        T1[i] = b[0];
    }
    const uint64_t *t = m61::block_sum_lds<3 * R>(g, red);
    if (threadIdx.x < 3 * R) part[(size_t)threadIdx.x * kLinkMaxBlocks + blockIdx.x] = t[threadIdx.x];
}

// One workgroup per round and one for the end, blockIdx.x = vz.  A round j <
// j0 sums its pass's partials; a later one folds the tables the passes left (Z
// itself when j0 = 0; at most 2^kLinkTailLog entries) in LDS up to its round and
// takes its sums.  Writes g_j(0), g_j(1), g_j(2) to tr[3 j ..], the claim
// g_1(0) + g_1(1) to fin[0] and, folded to the end, fin[1..3] = Z~(y*), W~(y*) and
// the map's status.  (All of the last rounds in one workgroup, one after the
// other, took 19.7 us and a launch for the others' partials 3.1.)
__global__ __launch_bounds__(kLinkTailThreads) void k_link_tails(const int32_t *__restrict__ Z,
                                                                 const uint64_t *__restrict__ T0g,
                                                                 const uint64_t *__restrict__ Wg, int vz, int j0,
                                                                 const uint64_t *__restrict__ rho,
                                                                 const uint64_t *__restrict__ part,
                                                                 uint64_t *__restrict__ tr, uint64_t *__restrict__ fin,
                                                                 const uint32_t *__restrict__ bad)
{
    __shared__ uint64_t t0[1 << kLinkTailLog], t1[1 << kLinkTailLog];
    __shared__ uint64_t red[m61::block_sum_words(3, kLinkTailThreads)];
    const int j = blockIdx.x, tid = threadIdx.x;
    uint64_t g[3] = {0, 0, 0};
    if (j < j0) {
        const int s = j - j % kLinkPass, r = link_pass_rounds(j0 - s), nb = link_blocks(1ull << (vz - s - r));
        const uint64_t *p = part + 3 * (size_t)j * kLinkMaxBlocks;
        for (int b = tid; b < nb; b += blockDim.x)
            for (int q = 0; q < 3; q++) g[q] = m61::fold(g[q] + p[(size_t)q * kLinkMaxBlocks + b]);
    } else {
        int n = 1 << (vz - j0);
        for (int i = tid; i < n; i += blockDim.x) {
            t0[i] = j0 == 0 ? m61::from_i32(Z[i]) : T0g[i];
            t1[i] = m61::fold(Wg[i]);
        }
        __syncthreads();
        for (int b = j0; b < j; b++) {  // an entry's two sources are read by its own thread only
            const uint64_t r = rho[b];
            n >>= 1;
            for (int i = tid; i < n; i += blockDim.x) {
                t0[i] = m61::lmacc(t0[i], r, m61::lsub(t0[i + n], t0[i]));
                t1[i] = m61::lmacc(t1[i], r, m61::lsub(t1[i + n], t1[i]));
            }
            __syncthreads();
        }
        if (j == vz) {
            if (tid != 0) return;
            const uint64_t z = m61::canon(t0[0]), w = m61::canon(t1[0]);
            if (vz == 0) fin[0] = m61::mul(z, w);
            fin[1] = z;
            fin[2] = w;
            fin[3] = *bad;
            return;
        }
        const int h = n >> 1;
        for (int i = tid; i < h; i += blockDim.x) {
            g[0] = m61::lmacc(g[0], t0[i], t1[i]);
            g[1] = m61::lmacc(g[1], t0[i + h], t1[i + h]);
            g[2] = m61::lmacc(g[2], m61::lsub(t0[i + h], t0[i]), m61::lsub(t1[i + h], t1[i]));
        }
    }
    m61::block_sum<3>(g, red);
    if (tid != 0) return;
    tr[3 * (size_t)j] = g[0];
    tr[3 * (size_t)j + 1] = g[1];
    tr[3 * (size_t)j + 2] = m61::sub(m61::add(m61::add(g[1], g[1]), m61::add(g[2], g[2])), g[0]);
    if (j == 0) fin[0] = m61::add(g[0], g[1]);
}

// The gathered input itself: A[a] = Z[src[a]], 0 where src[a] = -1.  An
// index outside [-1, nz) is not followed (A[a] = 0); ra_link_prove refuses
// the same map.
__global__ __launch_bounds__(256) void k_link_gather(const int32_t *__restrict__ Z, uint64_t nz,
                                                     const int32_t *__restrict__ src, uint64_t na,
                                                     int32_t *__restrict__ A)
{
    for (uint64_t a = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; a < na; a += (uint64_t)gridDim.x * blockDim.x) {
        const int32_t y = src[a];
        A[a] = (y >= 0 && (uint64_t)y < nz) ? Z[y] : 0;
    }
}

void launch_link_gather(const int32_t *Z, uint64_t nz, const int32_t *src, uint64_t na, int32_t *A, hipStream_t st)
{
    const int nb = (int)std::min<uint64_t>((na + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(k_link_gather, dim3(nb > 0 ? nb : 1), dim3(kThreads), 0, st, Z, nz, src, na, A);
}

template <int R> static void link_pass(const LinkArgs &a, int j, hipStream_t st)
{
    const uint64_t q = 1ull << (a.vz - j - R);
    const dim3 grid(link_blocks(q)), blk(kThreads);
    uint64_t *part = a.part + 3 * (size_t)j * kLinkMaxBlocks;
    if (j == 0) hipLaunchKernelGGL((k_link_pass<R, true>), grid, blk, 0, st, a.Z, a.T0, a.W, q, a.rho, part);
    else hipLaunchKernelGGL((k_link_pass<R, false>), grid, blk, 0, st, a.Z, a.T0, a.W, q, a.rho + j, part);
}

void launch_link(const LinkArgs &a, hipStream_t st)
{
    const int wb = (int)std::min<uint64_t>((a.na + kWeightRun - 1) / kWeightRun, 2048);
    hipLaunchKernelGGL(k_link_weights, dim3(wb > 0 ? wb : 1), dim3(kThreads), 0, st, a.src, a.na, a.lm, a.E1,
                       a.E2, 1ull << a.vz, (unsigned long long *)a.W, a.bad);
    const int j0 = a.vz > kLinkTailLog ? a.vz - kLinkTailLog : 0;  // rounds over the global tables
    for (int j = 0; j < j0; j += kLinkPass) {
        const int r = link_pass_rounds(j0 - j);
        if (r == 3) link_pass<3>(a, j, st);
        else if (r == 2) link_pass<2>(a, j, st);
        else link_pass<1>(a, j, st);
    }
    hipLaunchKernelGGL(k_link_tails, dim3(a.vz + 1), dim3(kLinkTailThreads), 0, st, a.Z, a.T0, a.W, a.vz, j0, a.rho,
                       a.part, a.tr, a.fin, a.bad);
}

}  // namespace ra
