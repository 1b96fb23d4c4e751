// fs.hip -- the non-interactive layer proof (Fiat-Shamir over F_{p^2}) on
// the device: the Merkle root of the witness tables, the transcript (absorb
// and draw, one workgroup: the hash chain is sequential), and the sum-check
// rounds reordered for challenges that exist only after a round's values are
// hashed.
#include <algorithm>

#include "common.hpp"
#include "f2.hpp"
#include "fs_device.hpp"
#include "sha256.hpp"

namespace ra {

// ---------------------------------------------------------------------------
// Merkle root: 1 KiB chunks, leaf H(0x00 || chunk), nodes H(0x01 || 4
// digests), root H(0x02 || LE64(leaves) || top).  A 4-ary node is 129 bytes
// (three compressions), which keeps the sequential levels short.
//
// Even the largest tables leave the chip less than one wave of leaves per
// SIMD, so the 17 compressions of a leaf and the three of every level are
// chains of latency.  A leaf's schedule is expanded by a second wave one block
// ahead of the rounds; a workgroup goes on from its 64 leaves to the node
// above them (three levels), and one workgroup takes the rest of the tree and
// the root, with the schedules of a level's blocks all at once and eight nodes
// per wave (ShaLanes).  One thread per hash and a launch per level: 113 us for
// 352 leaves, 155 us for 45056; so 65 and 131 (MI355X).
// ---------------------------------------------------------------------------
constexpr int kLeafThreads = 128, kLeafGroup = 64, kLeafLevels = 3;
constexpr int kTopThreads = 128, kTopNodes = 64;  // digests the last workgroup starts from, at most: its levels take two waves
constexpr int kNodeRow = 3 * 16 + 1;  // a node's three schedules, rows one bank group apart

// Message word from stored words (digests and data as their bytes in order):
// the last byte of `prev`, then the first three of `cur`, big-endian.
__device__ __forceinline__ uint32_t shifted_word(uint32_t prev, uint32_t cur)
{
    return (prev & 0xFF000000u) | ((cur & 0xFFu) << 16) | (cur & 0xFF00u) | ((cur >> 16) & 0xFFu);
}

// The schedule of block b of a node over `kids` digests (8 words each) at d.
__device__ __forceinline__ void node_schedule(const uint32_t *d, int kids, int b, uint4 *kw)
{
    uint32_t w[16];
    const int n = 8 * kids, g0 = 16 * b;
    uint32_t prev = b ? (g0 - 1 < n ? d[g0 - 1] : 0u) : 0x01000000u;
    if (b < 2) {
#pragma unroll
        for (int t = 0; t < 16; t++) {
            const uint32_t cur = g0 + t < n ? d[g0 + t] : 0u;
            w[t] = shifted_word(prev, cur);
            prev = cur;
        }
    } else {  // the last byte, the 0x80 marker, the length
        w[0] = (prev & 0xFF000000u) | 0x00800000u;
#pragma unroll
        for (int t = 1; t < 15; t++) w[t] = 0;
        w[15] = 129u * 8u;
    }
    sha_schedule(w, kw);
}

// A level of nodes in place: digests dig[0 .. count) to dig[0 .. (count + 3) /
// 4), at most 8 per wave at a time, whose schedules kw holds.  A chunk's nodes
// are written below every digest that a later chunk reads.  Barriers on both
// sides; the block.
__device__ __forceinline__ void node_level(uint32_t *dig, int count, uint4 *kw)
{
    const int tid = threadIdx.x, lane = tid & 63, per = (blockDim.x >> 6) * 8, nodes = (count + 3) / 4;
    for (int first = 0; first < nodes; first += per) {
        __syncthreads();
        for (int i = tid; i < 3 * per; i += blockDim.x) {
            const int j = i / 3, g = first + j;
            if (g < nodes) node_schedule(dig + 32 * g, count - 4 * g < 4 ? count - 4 * g : 4, i % 3, kw + kNodeRow * j + 16 * (i % 3));
        }
        __syncthreads();
        const int j0 = (tid >> 6) * 8;  // this wave's nodes
        if (first + j0 < nodes) {
            const int j = j0 + (lane >> 3);
            uint32_t st[4];
            sha_lanes_hash(kw + kNodeRow * (first + j < nodes ? j : j0), 3, st);
            if ((lane & 3) == 0 && first + j < nodes)
#pragma unroll
                for (int i = 0; i < 4; i++) dig[8 * (first + j) + (lane & 4) + i] = __builtin_bswap32(st[i]);
        }
    }
    __syncthreads();
}

// Sixteen rounds of one hash per lane, kw read at a stride of 64 vectors.
__device__ __forceinline__ void sha_rounds16(uint32_t (&v)[8], const uint4 *kw)
{
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint4 x = kw[64 * q];
        const uint32_t k4[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const uint32_t e = v[4], a = v[0];
            const uint32_t S1 = sha::xor3(sha::rotr(e, 6), sha::rotr(e, 11), sha::rotr(e, 25));
            const uint32_t T1 = (v[7] + k4[u]) + S1 + sha::choose(e, v[5], v[6]);
            const uint32_t S0 = sha::xor3(sha::rotr(a, 2), sha::rotr(a, 13), sha::rotr(a, 22));
            const uint32_t T2 = S0 + sha::majority(a, v[1], v[2]);
            v[7] = v[6];
            v[6] = v[5];
            v[5] = e;
            v[4] = v[3] + T1;
            v[3] = v[2];
            v[2] = v[1];
            v[1] = a;
            v[0] = T1 + T2;
        }
    }
}

// 64 leaves (src: from their tables; else 64 digests of `in`) and the levels
// above them, at most `levels`, to out[blockIdx.x].  count: leaves, or digests.
template <bool LEAVES>
__global__ __launch_bounds__(kLeafThreads) void k_merkle_group(MerkleArgs a, const uint32_t *__restrict__ in,
                                                               uint64_t count, int levels, uint32_t *__restrict__ out)
{
    __shared__ uint4 buf[2][16][64];   // the schedules of a block of 64 leaves, twice
    __shared__ uint32_t dig[kLeafGroup * 8];
    static_assert(sizeof(buf) >= sizeof(uint4) * 16 * kNodeRow, "the first level's 16 nodes");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t first = (uint64_t)blockIdx.x * kLeafGroup;
    const int here = (int)(count - first < kLeafGroup ? count - first : kLeafGroup);
    if (!LEAVES) {
        for (int i = tid; i < 8 * here; i += kLeafThreads) dig[i] = in[8 * first + i];
    } else {
        const uint64_t leaf = first + (lane < here ? lane : 0);
        int sg = 0;
        while (sg < 4 && leaf >= a.seg[sg + 1].first_leaf) sg++;
        const uint64_t off = (leaf - a.seg[sg].first_leaf) * 1024, left = a.seg[sg].bytes - off;
        const uint8_t *src = a.seg[sg].p + off;  // 16-byte aligned
        const uint32_t avail = left < 1024 ? (uint32_t)left : 1024u;
        // the 16 words of data block blk, zero past avail
        auto data = [&](int blk, uint32_t (&c)[16]) {
            if (64u * blk + 64u <= avail) {
                const uint4 *q = (const uint4 *)(src + 64 * blk);
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const uint4 x = q[v];
                    c[4 * v] = x.x;
                    c[4 * v + 1] = x.y;
                    c[4 * v + 2] = x.z;
                    c[4 * v + 3] = x.w;
                }
            } else {
#pragma unroll
                for (int t = 0; t < 16; t++) {
                    uint32_t v = 0;
                    for (uint32_t at = 64u * blk + 4u * t, b = 0; b < 4 && at + b < avail; b++)
                        v |= (uint32_t)src[at + b] << (8 * b);
                    c[t] = v;
                }
            }
        };
        uint32_t v[8], st[8], c[16], prev = 0;  // prefix 0x00
#pragma unroll
        for (int i = 0; i < 8; i++) st[i] = sha::kConsts.h[i];
        if (wave == 1) data(0, c);
#pragma unroll 1
        for (int it = 0; it <= 17; it++) {  // wave 1: block it; wave 0: block it - 1
            if (wave == 1 && it < 17) {
                uint32_t w[16];
                if (it < 16) {
#pragma unroll
                    for (int t = 0; t < 16; t++) {
                        w[t] = shifted_word(prev, c[t]);
                        prev = c[t];
                    }
                    if (it < 15) data(it + 1, c);  // the next block's loads beside this one's schedule
                } else {  // the last data byte, the 0x80 marker, the length
                    w[0] = (prev & 0xFF000000u) | 0x00800000u;
#pragma unroll
                    for (int t = 1; t < 15; t++) w[t] = 0;
                    w[15] = 1025u * 8u;
                }
                uint4(*kw)[64] = buf[it & 1];
                uint4 row[16];
                sha_schedule(w, row);
#pragma unroll
                for (int q = 0; q < 16; q++) kw[q][lane] = row[q];
            } else if (wave == 0 && it > 0) {
                const uint4 *kw = &buf[(it - 1) & 1][0][lane];
#pragma unroll
                for (int i = 0; i < 8; i++) v[i] = st[i];
#pragma unroll 1
                for (int p = 0; p < 4; p++) sha_rounds16(v, kw + 256 * p);
#pragma unroll
                for (int i = 0; i < 8; i++) st[i] += v[i];
            }
            __syncthreads();
        }
        if (wave == 0 && lane < here)
#pragma unroll
            for (int i = 0; i < 8; i++) dig[8 * lane + i] = __builtin_bswap32(st[i]);
    }
    int n = here;
    for (int l = 0; l < levels; l++) {
        node_level(dig, n, &buf[0][0][0]);
        n = (n + 3) / 4;
    }
    __syncthreads();
    if (tid < 8) out[8 * (size_t)blockIdx.x + tid] = dig[tid];
}

// The levels above `count` digests (at most kTopNodes) and the root.
__global__ __launch_bounds__(kTopThreads) void k_merkle_top(const uint32_t *__restrict__ in, int count, uint64_t leaves,
                                                            uint32_t *__restrict__ root)
{
    __shared__ uint32_t dig[8 * kTopNodes];
    __shared__ uint4 kw[kTopThreads / 64 * 8 * kNodeRow];
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < 8 * count; i += kTopThreads) dig[i] = in[i];
    __syncthreads();
    for (; count > 1; count = (count + 3) / 4) node_level(dig, count, kw);
    if (tid == 0) {  // 0x02, the leaves, the digest: 41 bytes
        uint32_t w[16], prev = (uint32_t)(leaves >> 32);
        w[0] = 0x02000000u | __builtin_bswap32((uint32_t)leaves) >> 8;
        w[1] = (uint32_t)(leaves >> 24 & 0xFF) << 24 | __builtin_bswap32(prev) >> 8;
#pragma unroll
        for (int t = 0; t < 8; t++) {
            w[2 + t] = shifted_word(prev, dig[t]);
            prev = dig[t];
        }
        w[10] = (prev & 0xFF000000u) | 0x00800000u;
#pragma unroll
        for (int t = 11; t < 15; t++) w[t] = 0;
        w[15] = 41u * 8u;
        sha_schedule(w, kw);
    }
    __syncthreads();
    if (tid < 64) {
        uint32_t st[4];
        sha_lanes_hash(kw, 1, st);
        if (lane < 8 && (lane & 3) == 0)
#pragma unroll
            for (int i = 0; i < 4; i++) root[lane + i] = __builtin_bswap32(st[i]);
    }
}

uint64_t merkle_leaves(const MerkleArgs &a)
{
    uint64_t n = 0;
    for (int s = 0; s < 5; s++) n += (a.seg[s].bytes + 1023) / 1024;
    return n;
}

// digests: two areas, of merkle_leaves() and a quarter as many of 8 words
void launch_merkle_root(MerkleArgs a, uint32_t *dig0, uint32_t *dig1, uint8_t *root, hipStream_t st)
{
    uint64_t first = 0;
    for (int s = 0; s < 5; s++) {
        a.seg[s].first_leaf = first;
        first += (a.seg[s].bytes + 1023) / 1024;
    }
    a.leaves = first;
    // a group's levels: those of the tree where it is one group, which ends at the top
    auto levels = [](uint64_t n) {
        int l = 0;
        for (; l < kLeafLevels && n > 1; l++) n = (n + 3) / 4;
        return l;
    };
    uint64_t count = (first + kLeafGroup - 1) / kLeafGroup;
    hipLaunchKernelGGL((k_merkle_group<true>), dim3((unsigned)count), dim3(kLeafThreads), 0, st, a, nullptr, first,
                       levels(first), dig0);
    uint32_t *in = dig0, *out = dig1;
    while (count > kTopNodes) {
        const uint64_t next = (count + kLeafGroup - 1) / kLeafGroup;
        hipLaunchKernelGGL((k_merkle_group<false>), dim3((unsigned)next), dim3(kLeafThreads), 0, st, a, in, count,
                           kLeafLevels, out);
        std::swap(in, out);
        count = next;
    }
    hipLaunchKernelGGL(k_merkle_top, dim3(1), dim3(kTopThreads), 0, st, in, (int)count, first, (uint32_t *)root);
}

// ---------------------------------------------------------------------------
// Transcript kernels (fs_device.hpp): one workgroup; a failed absorb sets *err.
// ---------------------------------------------------------------------------
constexpr int kFsThreads = 128;  // one wave runs the rounds, one the message schedules

// ndraw challenges (at most kFsDraws) in a row to out, the first with what is
// pending.
constexpr int kFsDraws = 64;
__device__ __forceinline__ void fs_draws(FsLds &f, uint64_t *out, int ndraw)
{
    __shared__ uint32_t raw[4 * kFsDraws];
    if (ndraw == 0) return;
    fs_draw(f);
    fs_hash_more(f, ndraw - 1, raw);
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * ndraw; i += blockDim.x)
        out[i] = i < 2 ? f.out[i] : fs_challenge_word(raw + 2 * (i - 2));
}

__global__ __launch_bounds__(kFsThreads) void k_fs_header(sha::Transcript *fs, FsHeader h,
                                                          const uint8_t *__restrict__ root, uint64_t *out, int ndraw,
                                                          uint32_t *err)
{
    __shared__ FsLds f;
    __shared__ uint32_t msg[24];  // the header, then the root
    const int tid = threadIdx.x;
    fs_pull(f, fs);
    if (tid < 16) msg[tid] = h.words[tid];
    else if (tid < 24) msg[tid] = ((const uint32_t *)root)[tid - 16];
    const bool ok = fs_absorb(f, msg, 24);
    if (tid == 0) *err = ok ? 0 : 1;  // the layer's first transcript kernel
    fs_draws(f, out, ndraw);
    __syncthreads();
    fs_push(fs, f);
}

void launch_fs_header(sha::Transcript *fs, const FsHeader &h, const uint8_t *root, uint64_t *out, int ndraw,
                      uint32_t *err, hipStream_t st)
{
    hipLaunchKernelGGL(k_fs_header, dim3(1), dim3(kFsThreads), 0, st, fs, h, root, out, ndraw, err);
}

// The claims R~, Rm~, Y~, Z~ from their partials (eight words per block),
// written to `out` and absorbed; ndraw challenges drawn.
__global__ __launch_bounds__(256) void k_fs_claims(const uint64_t *__restrict__ part, int nb, uint64_t *out8,
                                                   sha::Transcript *fs, uint64_t *out, int ndraw, uint32_t *err)
{
    __shared__ uint64_t red[m61::block_sum_words(8, 256)];
    __shared__ FsLds f;
    const int tid = threadIdx.x;
    fs_pull(f, fs);
    uint64_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = tid; b < nb; b += blockDim.x)
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = m61::add(v[q], part[8 * (size_t)b + q]);
    const uint64_t *tot = m61::block_sum_lds<8>(v, red);
    if (tid < 8) out8[tid] = tot[tid];
    if (!fs_absorb(f, tot, 16) && tid == 0) *err = 1;
    fs_draws(f, out, ndraw);
    __syncthreads();
    fs_push(fs, f);
}

void launch_fs_claims(const uint64_t *part, int nb, uint64_t *out8, sha::Transcript *fs, uint64_t *out, int ndraw,
                      uint32_t *err, hipStream_t st)
{
    hipLaunchKernelGGL(k_fs_claims, dim3(1), dim3(kThreads), 0, st, part, nb, out8, fs, out, ndraw, err);
}

// ---------------------------------------------------------------------------
// Rounds whose challenges exist only after their values are hashed.  Pass j
// (one launch per round while the tables hold more than 2^kFsTailLog
// entries) first finishes round j - 1: every workgroup sums that round's
// partials, forms its values, absorbs them and draws rho_{j-1}, so no launch
// of one workgroup sits between two passes (it took 7.6 us and the gaps of
// two launches per round); workgroup 0 writes the values and the transcript,
// to the other of two copies, since the rest still read the first.  Then it
// folds with rho_{j-1} (4h entries to 2h) and sums round j (f2.hpp).
// The last rounds run in one workgroup over LDS, hashing as they go.
// ---------------------------------------------------------------------------
// Round j - 1 finished in every workgroup: its challenge; f holds the
// transcript after it.  K: K_j in LDS.
struct FsFinLds {
    FsLds f;
    f2 g[4], K, k[2];
    f2 co[4][2];  // by X: the factors of the round's quadratic and linear sums in its value
    uint64_t tot[10];
};

// The transcript pulled; round j - 1's sums added up from the blocks'
// partials, its values formed and absorbed, its challenge drawn, K_j-1 (K_in;
// null: 1) advanced.  What does not depend on the sums (the factors K eq(r, X)
// of the values, K's next value as a line in rho) is formed beside them by
// the last wave, and nothing is stored to memory before the last barrier (it
// would be waited for there).
template <int KIND>
__device__ __forceinline__ f2 fs_finish_prev(FsFinLds &l, const FsFinArgs &a, bool writer)
{
    constexpr int NW = f2_sum_words(KIND), D1 = KIND == F2_MATMUL ? 3 : 4;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, nw = blockDim.x >> 6;
    fs_pull(l.f, a.fs_in);
    uint64_t v[3] = {0, 0, 0};  // at least four waves: at most three words each
#pragma unroll 4
    for (int b = lane; b < a.nb; b += 64)
#pragma unroll
        for (int u = 0; u < 3; u++)
            if (wave + u * nw < NW) v[u] = m61::fold(v[u] + a.part[(size_t)(wave + u * nw) * kF2MaxBlocks + b]);
    if (KIND != F2_MATMUL && wave == nw - 1) {
        const f2 K = a.K_in ? ldp(a.K_in) : f2of(1), r = ldp(a.r);
        f2 w = l2mul(K, l2eq1x(r, lane & 3));
        if (KIND == F2_RANGE) {
            const f2 ceq = ldp(a.cst), cd = f2sub(ldp(a.cst + 2), ceq);
            w = l2mul(w, lane & 4 ? cd : ceq);
        }
        if (lane < 8) l.co[lane & 3][lane >> 2] = w;
        const f2 k = l2mul(K, lane & 1 ? f2sub(f2add(r, r), f2of(1)) : f2sub(f2of(1), r));
        if (lane < 2) l.k[lane] = k;
    }
#pragma unroll
    for (int u = 0; u < 3; u++) v[u] = sum16(v[u]);
#pragma unroll
    for (int off = 16; off < 64; off <<= 1)
#pragma unroll
        for (int u = 0; u < 3; u++) v[u] = m61::fold(v[u] + __shfl_xor(v[u], off, 64));
#pragma unroll
    for (int u = 0; u < 3; u++)
        if (lane == 0 && wave + u * nw < NW) l.tot[wave + u * nw] = m61::canon(v[u]);
    __syncthreads();
    if (wave == 0) {
        const int X = lane & 3, j = (lane >> 2) & 1;
        auto at = [&](int q) { return f2{l.tot[2 * q], l.tot[2 * q + 1]}; };
        f2 lo, hi, inf;  // the sum (linear: j = 1) at 0 and 1, its leading coefficient
        if (KIND == F2_RANGE) {
            lo = at(j ? 0 : 2);
            hi = at(j ? 1 : 4);
            const f2 m = at(3);
            inf = j ? f2of(0) : l2sub(l2add(lo, hi), l2add(m, m));
        } else {
            lo = at(0);
            hi = at(1);
            const f2 t = l2add(lo, hi);
            inf = l2sub(l2add(t, t), at(2));
        }
        f2 g = l2add(l2add(lo, l2small(l2sub(hi, lo), X)), l2small(inf, X * (X - 1)));
        if (KIND != F2_MATMUL) g = l2mul(l.co[X][j], g);
        if (KIND == F2_RANGE) g = l2add(g, f2{__shfl_xor(g.re, 4, 64), __shfl_xor(g.im, 4, 64)});
        g = l2canon(g);
        if (lane < D1) l.g[lane] = g;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t q = l.f.m[8];
        const bool ok = fs_append(l.f, q, l.g, 4 * D1, lane, 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane == 0) {
            if (ok) l.f.m[8] = q + 16 * D1;
            else if (writer) *a.err = 1;
        }
    }
    fs_draw(l.f);
    const f2 rho{l.f.out[0], l.f.out[1]};
    if (writer && tid < D1) stp(a.ev + 2 * tid, l.g[tid]);
    if (KIND != F2_MATMUL && writer && tid == 64) {  // K (1 - r) + rho K (2 r - 1)
        const f2 K = l2canon(l2add(l.k[0], l2mul(rho, l.k[1])));
        l.K = K;
        if (a.K_out) stp(a.K_out, K);
    }
    return rho;
}

// Sources of a pass: field tables, the integer tables R, Y (ReLU), the bit
// words (range: Bx formed from them and written).
enum { FS_FIELD = 0, FS_INTS = 1, FS_BITS = 2 };

template <int KIND, int SRC, bool FOLD>
__global__ __launch_bounds__(256) void k_fs_pass(FsPassArgs a)
{
    constexpr int NW = f2_sum_words(KIND), NT = KIND == F2_RANGE ? 1 : 2;
    __shared__ FsFinLds l;
    __shared__ uint64_t red[NW * 256];
    __shared__ f2 tab[SRC == FS_BITS ? 8 : 1][256], sig[SRC == FS_BITS ? 64 : 1];
    const int tid = threadIdx.x;
    f2 rho{0, 0};
    if (FOLD) {
        rho = fs_finish_prev<KIND>(l, a.fin, blockIdx.x == 0);
        if (blockIdx.x == 0) fs_push(a.fin.fs_out, l.f);
    }
    if (SRC == FS_BITS) {
        if (tid < 64) sig[tid] = ldt(a.sig, tid);
        __syncthreads();
        f2_byte_tables(sig, a.tabs, tab);
        __syncthreads();
    }
    F2Sums<KIND> acc;
    const uint64_t h = a.h, first = (uint64_t)blockIdx.x * blockDim.x + tid;
    for (uint64_t i = first; i < h; i += (uint64_t)gridDim.x * blockDim.x) {
        f2 lo[2], hi[2];
        // weights: the high variables here (the same for the whole workgroup), the low ones at the end
        f2 w = f2of(1);
        if (KIND != F2_MATMUL) w = a.HS[(h >> kF2Low) + (i >> kF2Low)];
        if (SRC == FS_INTS) {
            uint64_t d[4], s[4];
#pragma unroll
            for (int q = 0; q < (FOLD ? 4 : 2); q++) relu_ints(a.R, a.Y, i + q * h, d[q], s[q]);
            if (!FOLD) {
                if constexpr (KIND == F2_RELU) acc.add_int(w, d[0], d[1], s[0], s[1]);
                continue;
            }
            lo[0] = fold_real(d[0], d[2], rho);
            hi[0] = fold_real(d[1], d[3], rho);
            lo[1] = fold_real(s[0], s[2], rho);
            hi[1] = fold_real(s[1], s[3], rho);
        } else if (SRC == FS_BITS) {
            lo[0] = f2_plane_bound(a.bits[i], a.tabs, tab);
            hi[0] = f2_plane_bound(a.bits[i + h], a.tabs, tab);
        } else {
#pragma unroll
            for (int q = 0; q < NT; q++) {
                lo[q] = ldt(a.src[q], i);
                hi[q] = ldt(a.src[q], i + h);
                if (FOLD) {
                    lo[q] = l2fold(lo[q], ldt(a.src[q], i + 2 * h), rho);
                    hi[q] = l2fold(hi[q], ldt(a.src[q], i + 3 * h), rho);
                }
            }
        }
        if (FOLD || SRC == FS_BITS)
#pragma unroll
            for (int q = 0; q < NT; q++) {
                stt(a.dst[q], i, lo[q]);
                stt(a.dst[q], i + h, hi[q]);
            }
        if constexpr (KIND == F2_MATMUL) acc.add(lo[0], hi[0], lo[1], hi[1]);
        else if constexpr (KIND == F2_RANGE) acc.add(l2mul(w, lo[0]), l2mul(w, hi[0]), lo[0], hi[0]);
        else acc.add(l2mul(w, lo[0]), l2mul(w, hi[0]), lo[1], hi[1]);
    }
    uint64_t v[NW];
    acc.words(v, KIND != F2_MATMUL,
              KIND != F2_MATMUL ? a.LS[(1u << kF2Low) + (uint32_t)(first & ((1u << kF2Low) - 1))] : f2of(1));
    f2_totals<NW>(v, red, l.tot, blockDim.x);
    if (tid < NW) a.part[(size_t)tid * kF2MaxBlocks + blockIdx.x] = l.tot[tid];
}

void launch_fs_pass(const FsPassArgs &a, hipStream_t st)
{
    const dim3 grid(f2_blocks(a.h)), blk(kThreads);
    const bool fold = a.fin.nb > 0;
    if (a.kind == F2_MATMUL) {
        if (fold) hipLaunchKernelGGL((k_fs_pass<F2_MATMUL, FS_FIELD, true>), grid, blk, 0, st, a);
        else hipLaunchKernelGGL((k_fs_pass<F2_MATMUL, FS_FIELD, false>), grid, blk, 0, st, a);
    } else if (a.kind == F2_RANGE) {
        if (fold) hipLaunchKernelGGL((k_fs_pass<F2_RANGE, FS_FIELD, true>), grid, blk, 0, st, a);
        else hipLaunchKernelGGL((k_fs_pass<F2_RANGE, FS_BITS, false>), grid, blk, 0, st, a);
    } else if (!a.R) {
        hipLaunchKernelGGL((k_fs_pass<F2_RELU, FS_FIELD, true>), grid, blk, 0, st, a);
    } else if (fold) {
        hipLaunchKernelGGL((k_fs_pass<F2_RELU, FS_INTS, true>), grid, blk, 0, st, a);
    } else {
        hipLaunchKernelGGL((k_fs_pass<F2_RELU, FS_INTS, false>), grid, blk, 0, st, a);
    }
}

// ---------------------------------------------------------------------------
// The last v rounds (tables of 2^v <= 2^kFsTailLog entries once the previous
// pass's round is finished and folded), the instance's final values, and
// their absorption, in one workgroup.
//
// A round's hash takes 3.5 us on two waves, so all the rest of a round runs
// beside it on the others: with T_c the tables bound at rho_{<c}, the sums of
// round c + 1 are quadratic in rho_c, its pairs being lo = x0 + rho (x2 - x0),
// hi = x1 + rho (x3 - x1) over T_c's quads, and are taken at rho = 0 (x0, x1),
// 1 (x2, x3) and infinity (the differences) while rho_c is being hashed; the
// last of the waves turns them into the values g_{c+1}(X), X = 0 .. 3, as
// cubics in rho_c (their eq factor is linear in it).  Once rho_c is there,
// wave 0 evaluates these and goes on hashing, and the other waves fold.
// Per round, sums over the block, values, hash and fold one after the other
// took 10 us; with the sums beside the hash 7.5; with the cubics 4.2 to 4.6 from
// 64 quads down (11 range rounds 86 -> 70 us with their start, MI355X).
// ---------------------------------------------------------------------------
constexpr int kTailWorkers = kFsTailThreads / 64 - 2;  // waves 2 ..
constexpr int kTailSplit = 512;                        // short rounds: the other place of a table
static_assert(kFsTailThreads == 512, "six waves beside the chain's two");

// Sums over pairs weighted by w: ll = lo lo', hh = hi hi', and lo hi' (range)
// or (lo + hi)(lo' + hi') (else).
struct PairSums {
    K3 ll, lh, hh;
    template <int KIND> __device__ __forceinline__ void add(f2 a0, f2 a1, f2 b0, f2 b1)
    {
        ll.add(a0, b0);
        if (KIND == F2_RANGE) lh.add(a0, b1);
        else lh.add(l2add(a0, a1), l2add(b0, b1));
        hh.add(a1, b1);
    }
};
// values (3 e + q) for e = 0, 1, infinity and q = ll, lh, hh; range: 9 + 2 e + b the sums of lo (b = 0), hi at e = 0, 1
constexpr int tail_values(int kind) { return kind == F2_RANGE ? 13 : 9; }

struct FsTailLds {
    uint64_t part[kTailWorkers][2 * 13];  // a wave's sums, canonical
    uint64_t tr[kTailWorkers][8 * 64];    // its transposes
    f2 co[4][4];                          // by X: the factors of tail_cubics
    f2 val[16];                           // the waves' sums added up
};

// Sums of NV values per lane of the wave, to out (2 NV words); tr: 512 words.
template <int NV>
__device__ __forceinline__ void wave_totals(const f2 (&x)[NV], uint64_t *tr, uint64_t *out)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q0 = 0; q0 < NV; q0 += 4) {  // eight words at a time: 8 lanes per word, 8 entries each
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const f2 v = q0 + q < NV ? x[q0 + q < NV ? q0 + q : 0] : f2of(0);
            tr[(2 * q) * 64 + lane] = v.re;
            tr[(2 * q + 1) * 64 + lane] = v.im;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint64_t *src = tr + (lane >> 3) * 64 + (lane & 7);
        uint64_t v = 0;
#pragma unroll
        for (int e = 0; e < 8; e += 2) v = m61::fold(v + src[8 * e] + src[8 * e + 8]);
        v = sum8(v);
        const int w = 2 * q0 + (lane >> 3);
        if ((lane & 7) == 0 && w < 2 * NV) out[w] = m61::canon(v);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

__device__ __forceinline__ f2 lane_of(f2 v, int i) { return f2{__shfl(v.re, i, 64), __shfl(v.im, i, 64)}; }

// Lanes 0 .. 15 (X = lane & 3, j = lane >> 2): the factors of the values of a
// round at X, with K = k0 + rho k1, r the round's coordinate: of the quadratic
// and the linear sums (c_eq, c_d = c_w - c_eq; ReLU: 1, none) times rho^0, rho^1.
template <int KIND>
__device__ __forceinline__ void tail_factors(FsTailLds &t, f2 k0, f2 k1, f2 r, f2 ceq, f2 cd)
{
    const int lane = threadIdx.x & 63, X = lane & 3, j = (lane >> 2) & 3;
    f2 v = l2mul(j < 2 ? k0 : k1, l2eq1x(r, X));
    if (KIND == F2_RANGE) v = l2mul(v, j & 1 ? cd : ceq);
    else if (j & 1) v = f2of(0);
    if (lane < 16) t.co[X][j] = v;
}

// One wave: the values of round c + 1 at X = 0 .. 3 as cubics in rho_c from
// nw waves' sums (split: from three waves' sums, those of wave e at rho = 0, 1,
// infinity): cub[X][d], the coefficient of rho_c^d.  Lane (j, d, X) forms the
// product with factor j, the four products of a (d, X) are added over lanes.
template <int KIND>
__device__ __forceinline__ void tail_cubics(FsTailLds &t, int nw, bool split, f2 (*cub)[4])
{
    constexpr int NV = tail_values(KIND);
    const int lane = threadIdx.x & 63, X = lane & 3, d = (lane >> 2) & 3, j = lane >> 4;
    if (lane < NV) {
        f2 v = f2of(0);
        if (split) {
            const int e = lane < 9 ? lane / 3 : (lane - 9) >> 1, q = lane < 9 ? lane % 3 : 3 + ((lane - 9) & 1);
            v = f2{t.part[e][2 * q], t.part[e][2 * q + 1]};
        } else {
            for (int w = 0; w < nw; w++) v = l2add(v, f2{t.part[w][2 * lane], t.part[w][2 * lane + 1]});
        }
        t.val[lane] = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int at = KIND == F2_MATMUL || j < 2 ? d : d - 1;  // of rho in the sum
    auto coef = [&](int q) {  // of rho^at in the sum q, from its values at 0, 1 and infinity
        const f2 p0 = t.val[q], pi = t.val[6 + q];
        const f2 b = l2sub(l2sub(t.val[3 + q], p0), pi);
        return at == 0 ? p0 : (at == 1 ? b : (at == 2 ? pi : f2of(0)));
    };
    f2 lo = coef(0), hi = coef(2), inf = coef(1);
    const f2 t2 = l2add(lo, hi);
    inf = KIND == F2_RANGE ? l2sub(t2, l2add(inf, inf)) : l2sub(l2add(t2, t2), inf);
    if (KIND == F2_RANGE && (j & 1)) {  // the linear sums
        lo = t.val[9];
        hi = t.val[10];
        if (at == 1) {
            lo = l2sub(t.val[11], lo);
            hi = l2sub(t.val[12], hi);
        } else if (at != 0) {
            lo = hi = f2of(0);
        }
        inf = f2of(0);
    }
    f2 s = l2add(l2add(lo, l2small(l2sub(hi, lo), X)), l2small(inf, X * (X - 1)));
    if (KIND != F2_MATMUL) {
        s = l2mul(t.co[X][j], s);
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) s = l2add(s, f2{__shfl_xor(s.re, off, 64), __shfl_xor(s.im, off, 64)});
    }
    if (lane < 16) cub[X][d] = s;
}

template <int KIND>
__global__ __launch_bounds__(kFsTailThreads) void k_fs_tail(FsTailArgs a)
{
    constexpr int NW = f2_sum_words(KIND), NT = KIND == F2_RANGE ? 1 : 2, S = 1 << kFsTailLog, NV = tail_values(KIND);
    constexpr int D1 = KIND == F2_MATMUL ? 3 : 4;
    // red: also the byte tables while Bx is formed
    constexpr int RED = NW * kFsTailThreads > 8 * 512 ? NW * kFsTailThreads : 8 * 512;
    __shared__ f2 T[NT][S], LS[KIND == F2_MATMUL ? 1 : S];
    __shared__ union {
        uint64_t red[RED];
        FsTailLds t;
    } u;
    __shared__ FsFinLds l;
    __shared__ f2 sig[KIND == F2_RANGE ? 64 : 1], fin[3];
    __shared__ f2 cub[2][4][4];  // the values of round c as cubics in rho_{c-1}, by c's parity
    __shared__ uint32_t arrived;
    __shared__ uint64_t drawn[2][2];  // rho_c, by c's parity: rho_{c-1} may still be read while rho_c is drawn
    __shared__ f2 ev[D1 * kFsTailLog], rs[kFsTailLog];  // the rounds' values, written out at the end; r_j0 ..
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, n0 = 1 << a.v;
    f2 rho{0, 0};
    if (KIND != F2_MATMUL)
        for (int i = tid; i < n0; i += blockDim.x) LS[i] = a.LS[i];  // entries 2^k + y, k < v
    if (KIND != F2_MATMUL && tid < a.v) rs[tid] = ldp(a.r + 2 * (a.j0 + tid));
    const bool prev = a.fin.nb > 0;
    if (prev) {
        rho = fs_finish_prev<KIND>(l, a.fin, true);
    } else {
        fs_pull(l.f, a.fin.fs_in);
        if (tid == 0) l.K = f2of(1);
    }
    if (KIND == F2_RANGE && !prev) {
        f2(*tab)[256] = (f2(*)[256])u.red;
        if (tid < 64) sig[tid] = ldt(a.sig, tid);
        __syncthreads();
        f2_byte_tables(sig, a.tabs, tab);
        __syncthreads();
        for (int i = tid; i < n0; i += blockDim.x) T[0][i] = f2_plane_bound(a.bits[i], a.tabs, tab);
    } else if (KIND == F2_RELU && a.R) {
        for (int i = tid; i < n0; i += blockDim.x) {
            uint64_t d0, s0, d1, s1;
            relu_ints(a.R, a.Y, i, d0, s0);
            if (prev) {
                relu_ints(a.R, a.Y, i + n0, d1, s1);
                T[0][i] = fold_real(d0, d1, rho);
                T[NT - 1][i] = fold_real(s0, s1, rho);
            } else {
                T[0][i] = f2of(d0);
                T[NT - 1][i] = f2of(s0);
            }
        }
    } else {
        for (int i = tid; i < n0; i += blockDim.x)
#pragma unroll
            for (int q = 0; q < NT; q++) {
                const f2 x = ldt(a.src[q], i);
                T[q][i] = prev ? l2fold(x, ldt(a.src[q], i + n0), rho) : x;
            }
    }
    __syncthreads();
    f2 ceq = f2of(0), cd = f2of(0);
    if (KIND == F2_RANGE) {
        ceq = ldp(a.cst);
        cd = f2sub(ldp(a.cst + 2), ceq);
    }
    if (a.v > 0) {  // the first round's sums, by every thread
        const int h = n0 >> 1;
        F2Sums<KIND> acc;
        for (int i = tid; i < h; i += blockDim.x) {
            f2 lo[2], hi[2];
#pragma unroll
            for (int q = 0; q < NT; q++) {
                lo[q] = T[q][i];
                hi[q] = T[q][i + h];
            }
            if constexpr (KIND == F2_MATMUL) {
                acc.add(lo[0], hi[0], lo[1], hi[1]);
            } else {
                const f2 w = LS[h + i], u0 = l2mul(w, lo[0]), u1 = l2mul(w, hi[0]);
                if constexpr (KIND == F2_RANGE) acc.add(u0, u1, lo[0], hi[0]);
                else acc.add(u0, u1, lo[1], hi[1]);
            }
        }
        uint64_t v[NW];
        acc.words(v, false, f2of(1));
        f2_totals<NW>(v, u.red, l.tot, h < 64 ? 64 : (h < kFsTailThreads ? h : kFsTailThreads));
        // the first round's values as cubics (no rho before it: constants)
        if (wave == 0) {
            if (KIND != F2_MATMUL) tail_factors<KIND>(u.t, l.K, f2of(0), rs[0], ceq, cd);
            constexpr int omap[3] = {0, 2, 1};  // of F2Sums' words: ll, lh, hh
            if (lane < 13) {
                int at = KIND == F2_RANGE ? (lane >= 9 ? (lane - 9) & 1 : 2 + lane % 3) : omap[lane % 3];
                const bool inf = lane >= 6 && lane < 9;
                u.t.part[0][2 * lane] = inf ? 0 : l.tot[2 * at];
                u.t.part[0][2 * lane + 1] = inf ? 0 : l.tot[2 * at + 1];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            tail_cubics<KIND>(u.t, 1, false, cub[0]);
            if (lane == 0) {
                l.f.go = 0;
                arrived = 0;
            }
        }
        __syncthreads();
    }
    // the other waves in the order they take a long round's work: those that
    // share a SIMD with the chain's two (waves w and w + 4) last
    const int w = wave < 4 ? wave - 2 : (wave < 6 ? wave : wave - 4), wt = 64 * w + lane;
    f2 kk0 = l.K, kk1 = f2of(0);  // wave 7's: K_c, linear in rho_{c-1}
    int base = 0;                    // T_{c-1}'s place
    if (wave < 2) __builtin_amdgcn_s_setprio(3);  // the chain's waves before the one they share a SIMD with
    for (int c = 0; c < a.v; c++) {
        const int lg = a.v - c;                         // T_c holds 2^lg entries
        const int n = lg >= 2 ? 1 << (lg - 2) : 0;      // its quads
        const f2 z = c ? f2{drawn[(c - 1) & 1][0], drawn[(c - 1) & 1][1]} : f2of(0);  // rho_{c-1}
        if (wave == 0) {
            // the round's values: lanes 0 .. 3 form z^2, 4 .. 7 z D1, 8 .. 11 z D3
            const int X = lane & 3;
            const f2(*D)[4] = cub[c & 1];
            const f2 pr = l2mul(z, lane < 4 ? z : D[X][lane < 8 ? 1 : 3]);
            const f2 hi = l2add(D[X][2], lane_of(pr, 8 + X)), lo = l2add(D[X][0], lane_of(pr, 4 + X));
            const f2 g = l2canon(l2add(lo, l2mul(lane_of(pr, X), hi)));
            // to the transcript, behind what is pending
            const uint32_t qlen = l.f.m[8];
            if (lane < D1) {
                ev[D1 * c + lane] = g;
                l.g[lane] = g;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const bool ok = fs_append(l.f, qlen, l.g, 4 * D1, lane, 64);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane == 0) {
                if (ok) l.f.m[8] = qlen + 16 * D1;
                else *a.err = 1;
                __hip_atomic_store(&l.f.go, (uint32_t)(c + 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            fs_hash_rounds(l.f, drawn[c & 1]);
        } else if (wave == 1) {
            while (__hip_atomic_load(&l.f.go, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < (uint32_t)(c + 1)) {
            }
            fs_hash_schedules(l.f);
        } else {
            const int hs = 1 << lg;
            const bool split = n <= 64;
            int of = 0, nw = 3;  // the waves whose results the round's cubics take
            if (KIND != F2_MATMUL && n && wave == 7) {
                // K_{c+1} = K_c eq(r_c, rho_c) = K_c (1 - r_c) + rho_c K_c (2 r_c - 1)
                const f2 K = l2add(kk0, l2mul(z, kk1)), r = rs[c];
                kk0 = l2mul(K, f2sub(f2of(1), r));
                kk1 = l2mul(K, f2sub(f2add(r, r), f2of(1)));
                tail_factors<KIND>(u.t, kk0, kk1, rs[c + 1], ceq, cd);
            }
            if (split) {
                // short rounds: waves 2, 3, 6 take the sums at rho = 0, 1,
                // infinity (folding what they need themselves), waves 5 and 7 fold
                const int e = wave == 6 ? 2 : wave - 2;
                if (n && (wave < 4 || wave == 6)) {
                    const int i = lane & (n - 1);
                    f2 x[2], y[2];
#pragma unroll
                    for (int q = 0; q < NT; q++)
#pragma unroll
                        for (int b = 0; b < 2; b++) {
                            const f2 *src = &T[q][base + i + b * n];
                            f2 v = src[e ? 2 * n : 0], o = c ? src[(e ? 2 * n : 0) + hs] : f2of(0);
                            if (e == 2) {
                                v = l2sub(v, src[0]);
                                if (c) o = l2sub(o, src[hs]);
                            }
                            if (c) v = l2fold(v, o, z);
                            (q == NT - 1 ? y : x)[b] = v;
                            if (NT == 1) x[b] = v;
                        }
                    if (KIND != F2_MATMUL) {
                        const f2 wt1 = LS[n + i];
                        x[0] = l2mul(wt1, x[0]);
                        x[1] = l2mul(wt1, x[1]);
                    }
                    PairSums at;
                    at.template add<KIND>(x[0], x[1], y[0], y[1]);
                    f2 val[KIND == F2_RANGE ? 5 : 3] = {at.ll.value(), at.lh.value(), at.hh.value()};
                    if constexpr (KIND == F2_RANGE) {
                        val[3] = x[0];
                        val[4] = x[1];
                    }
                    if (lane >= n)
#pragma unroll
                        for (auto &v : val) v = f2of(0);
                    wave_totals<KIND == F2_RANGE ? 5 : 3>(val, u.t.tr[w], u.t.part[e]);
                }
                if ((wave == 5 || wave == 7) && c > 0) {
                    const int db = base ^ kTailSplit;
                    for (int i = 32 * (wave - 5) + lane; i < NT << lg; i += 128) {
                        const int q = i >> lg, p = i & (hs - 1);
                        T[q][db + p] = l2fold(T[q][base + p], T[q][base + p + hs], z);
                    }
                }
                if (n && (wave < 4 || wave == 6 || wave == 7)) of = 4;
            } else {
                nw = n < 64 * kTailWorkers ? (n + 63) >> 6 : kTailWorkers;
                if (c > 0)  // T_c from T_{c-1}: an entry's two sources are read by its own thread only
                    for (int i = wt; i < n; i += 64 * kTailWorkers)
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            const int p = i + e * n;
#pragma unroll
                            for (int q = 0; q < NT; q++) T[q][p] = l2fold(T[q][p], T[q][p + hs], z);
                        }
                if (w < nw) {
                    PairSums at[3];
                    f2 lin[2][2] = {{f2of(0), f2of(0)}, {f2of(0), f2of(0)}};
                    for (int i = wt; i < n; i += 64 * kTailWorkers) {
                        f2 x[4], y[4];
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            y[e] = T[NT - 1][i + e * n];
                            x[e] = T[0][i + e * n];
                            if (KIND != F2_MATMUL) x[e] = l2mul(LS[n + i], x[e]);
                        }
                        at[0].template add<KIND>(x[0], x[1], y[0], y[1]);
                        at[1].template add<KIND>(x[2], x[3], y[2], y[3]);
                        at[2].template add<KIND>(l2sub(x[2], x[0]), l2sub(x[3], x[1]), l2sub(y[2], y[0]), l2sub(y[3], y[1]));
                        if (KIND == F2_RANGE)
#pragma unroll
                            for (int e = 0; e < 4; e++) lin[e >> 1][e & 1] = l2add(lin[e >> 1][e & 1], x[e]);
                    }
                    f2 val[NV];
#pragma unroll
                    for (int e = 0; e < 3; e++) {
                        val[3 * e] = at[e].ll.value();
                        val[3 * e + 1] = at[e].lh.value();
                        val[3 * e + 2] = at[e].hh.value();
                    }
                    if constexpr (KIND == F2_RANGE)
#pragma unroll
                        for (int e = 0; e < 4; e++) val[9 + e] = lin[e >> 1][e & 1];
                    wave_totals<NV>(val, u.t.tr[w], u.t.part[w]);
                }
                if (w < nw || wave == 7) of = nw + (nw <= 3 ? 1 : 0);  // wave 7 is the fourth to take work
            }
            if (of) {  // the last of these waves to arrive has all of their results
                uint32_t before = 0;
                if (lane == 0) before = __hip_atomic_fetch_add(&arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (__builtin_amdgcn_readfirstlane((int)before) == of - 1) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    tail_cubics<KIND>(u.t, nw, split, cub[(c + 1) & 1]);
                    if (lane == 0) arrived = 0;
                }
            }
        }
        if (c > 0 && n <= 64) base ^= kTailSplit;
        __syncthreads();
    }
    if (a.v > 0) {
        if (tid < NT) T[tid][0] = l2fold(T[tid][base], T[tid][base + 1], f2{drawn[(a.v - 1) & 1][0], drawn[(a.v - 1) & 1][1]});
        if (tid >= 64 && tid - 64 < D1 * a.v) stp(a.ev + 2 * (D1 * a.j0 + tid - 64), ev[tid - 64]);
        __syncthreads();
    }
    constexpr uint64_t inv2 = 1ull << 60;  // 2 2^60 = 2^61 = 1 mod p
    constexpr int nfin = KIND == F2_MATMUL ? 2 : (KIND == F2_RANGE ? 1 : 2);
    if (tid == 0) {  // a*, b*; b~(sigma); R~ = (D + S) / 2, Y~ = (S - D) / 2
        const f2 x = l2canon(T[0][0]), y = l2canon(T[NT - 1][0]);
        fin[0] = KIND == F2_RELU ? f2scale(f2add(x, y), inv2) : x;
        fin[1] = KIND == F2_RELU ? f2scale(f2sub(y, x), inv2) : y;
        if (KIND == F2_MATMUL) {  // c0 = g_1(0) + g_1(1), or a b with no rounds
            const bool any = a.j0 + a.v > 0;
            stp(a.out, any ? (a.j0 ? f2add(ldp(a.ev), ldp(a.ev + 2)) : f2add(ev[0], ev[1])) : f2mul(x, y));
        }
        for (int q = 0; q < nfin; q++) stp(a.out + (KIND == F2_MATMUL ? 2 : 0) + 2 * q, fin[q]);
    }
    if (!fs_absorb(l.f, fin, 4 * nfin) && tid == 0) *a.err = 1;
    fs_push(a.fs_out, l.f);
}

void launch_fs_tail(const FsTailArgs &a, hipStream_t st)
{
    const dim3 blk(kFsTailThreads);
    if (a.kind == F2_MATMUL) hipLaunchKernelGGL(k_fs_tail<F2_MATMUL>, dim3(1), blk, 0, st, a);
    else if (a.kind == F2_RANGE) hipLaunchKernelGGL(k_fs_tail<F2_RANGE>, dim3(1), blk, 0, st, a);
    else hipLaunchKernelGGL(k_fs_tail<F2_RELU>, dim3(1), blk, 0, st, a);
}

__global__ __launch_bounds__(256) void k_fill0(uint64_t *__restrict__ p, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

void launch_fill0(uint64_t *p, uint64_t n, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill0, dim3(f2_blocks(n)), dim3(kThreads), 0, st, p, n);
}

}  // namespace ra
