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
// ---------------------------------------------------------------------------
// SHA-256 of prefix || NB bytes at src (NB a multiple of 64; bytes at or
// beyond `avail` read as zero), src 16-byte aligned; digest stored as its 32
// bytes in order.
template <int NB>
__device__ void hash_chunk(uint8_t prefix, const uint8_t *__restrict__ src, uint32_t avail, uint32_t *__restrict__ out)
{
    static_assert(NB % 64 == 0, "whole blocks of data");
    uint32_t st[8];
#pragma unroll
    for (int i = 0; i < 8; i++) st[i] = sha::kConsts.h[i];
    const uint32_t *s32 = (const uint32_t *)src;
    auto word = [&](int i) -> uint32_t {  // little-endian word i of the chunk, zero past avail
        if (4u * i + 4u <= avail) return s32[i];
        uint32_t v = 0;
        for (int b = 0; b < 4; b++)
            if (4u * i + b < avail) v |= (uint32_t)src[4 * i + b] << (8 * b);
        return v;
    };
    uint32_t prev = (uint32_t)prefix << 24;  // the byte before chunk word 0 sits in the top byte
    for (int blk = 0; blk <= NB / 64; blk++) {
        uint32_t w[16];
        if (blk < NB / 64) {
            uint32_t c[16];
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
                for (int t = 0; t < 16; t++) c[t] = word(16 * blk + t);
            }
            // message word g = 16 blk + t holds bytes chunk[4g - 1], chunk[4g .. 4g + 2]
#pragma unroll
            for (int t = 0; t < 16; t++) {
                const uint32_t cw = c[t];
                w[t] = (prev & 0xFF000000u) | ((cw & 0xFFu) << 16) | (cw & 0xFF00u) | ((cw >> 16) & 0xFFu);
                prev = cw;
            }
        } else {
            // the last data byte, the 0x80 marker, zeros, the length (1 + NB) * 8 bits
            w[0] = (prev & 0xFF000000u) | 0x00800000u;
#pragma unroll
            for (int t = 1; t < 15; t++) w[t] = 0;
            w[15] = (1u + NB) * 8u;
        }
        sha::compress(st, w);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) out[i] = __builtin_bswap32(st[i]);
}

__global__ __launch_bounds__(256) void k_merkle_leaves(MerkleArgs a, uint32_t *__restrict__ dig)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.leaves) return;
    int sg = 0;
    while (sg < 4 && i >= a.seg[sg + 1].first_leaf) sg++;
    const uint64_t off = (i - a.seg[sg].first_leaf) * 1024;
    const uint64_t left = a.seg[sg].bytes - off;
    hash_chunk<1024>(0x00, a.seg[sg].p + off, (uint32_t)(left < 1024 ? left : 1024), dig + 8 * i);
}

__global__ __launch_bounds__(256) void k_merkle_nodes(const uint32_t *__restrict__ in, uint64_t count,
                                                      uint32_t *__restrict__ out)
{
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (count + 3) / 4) return;
    const uint64_t kids = std::min<uint64_t>(4, count - 4 * g);
    hash_chunk<128>(0x01, (const uint8_t *)(in + 8 * 4 * g), (uint32_t)(32 * kids), out + 8 * g);
}

__global__ void k_merkle_root(const uint32_t *__restrict__ top, uint64_t leaves, uint8_t *__restrict__ root)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    sha::Hasher h;
    h.init();
    h.byte(0x02);
    h.le(leaves, 8);
    h.update((const uint8_t *)top, 32);
    h.final(root);
}

uint64_t merkle_leaves(const MerkleArgs &a)
{
    uint64_t n = 0;
    for (int s = 0; s < 5; s++) n += (a.seg[s].bytes + 1023) / 1024;
    return n;
}

// digests: two areas of merkle_leaves() x 8 words each
void launch_merkle_root(MerkleArgs a, uint32_t *dig0, uint32_t *dig1, uint8_t *root, hipStream_t st)
{
    uint64_t first = 0;
    for (int s = 0; s < 5; s++) {
        a.seg[s].first_leaf = first;
        first += (a.seg[s].bytes + 1023) / 1024;
    }
    a.leaves = first;
    hipLaunchKernelGGL(k_merkle_leaves, dim3((unsigned)((first + 255) / 256)), dim3(256), 0, st, a, dig0);
    uint64_t count = first;
    uint32_t *in = dig0, *out = dig1;
    while (count > 1) {
        const uint64_t next = (count + 3) / 4;
        hipLaunchKernelGGL(k_merkle_nodes, dim3((unsigned)((next + 255) / 256)), dim3(256), 0, st, in, count, out);
        std::swap(in, out);
        count = next;
    }
    hipLaunchKernelGGL(k_merkle_root, dim3(1), dim3(64), 0, st, in, first, root);
}

// ---------------------------------------------------------------------------
// Transcript kernels (fs_device.hpp): one workgroup; a failed absorb sets *err.
// ---------------------------------------------------------------------------
constexpr int kFsThreads = 128;  // one wave runs the rounds, one the message schedules

// ndraw challenges (at most kFsDraws) in a row to out.  They are kept in LDS
// until the last: a store to memory before a barrier is waited for there.
constexpr int kFsDraws = 64;
__device__ __forceinline__ void fs_draws(FsLds &f, uint64_t *out, int ndraw)
{
    __shared__ uint64_t drawn[2 * kFsDraws];
    for (int i = 0; i < ndraw; i++) {
        fs_draw(f);
        if (threadIdx.x < 2) drawn[2 * i + threadIdx.x] = f.out[threadIdx.x];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * ndraw; i += blockDim.x) out[i] = drawn[i];
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
    if (!fs_absorb(f, (const uint32_t *)tot, 16) && tid == 0) *err = 1;
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
    f2 g[4], K;
    uint64_t tot[10];
};

// The values of a round from its sums in l.tot (after a barrier): to l.g, and
// by the writer to ev; absorbed, the challenge drawn; K advanced.
template <int KIND>
__device__ __forceinline__ f2 fs_finish_round(FsFinLds &l, f2 r, const uint64_t *cst, uint64_t *ev, bool writer,
                                              uint32_t *err)
{
    constexpr int D1 = KIND == F2_MATMUL ? 3 : 4;
    const int tid = threadIdx.x;
    if (tid < D1) {
        const f2 g = f2_round_value(KIND, l.tot, tid, l.K, r, cst);
        l.g[tid] = g;
        if (writer) stp(ev + 2 * tid, g);
    }
    if (!fs_absorb(l.f, (const uint32_t *)l.g, 4 * D1) && tid == 0 && writer) *err = 1;
    fs_draw(l.f);
    return f2{l.f.out[0], l.f.out[1]};
}

// As above, with the sums taken from the blocks' partials first and the
// transcript pulled; K_j-1 read from K_in (null: 1).
template <int KIND>
__device__ __forceinline__ f2 fs_finish_prev(FsFinLds &l, const FsFinArgs &a, bool writer)
{
    constexpr int NW = f2_sum_words(KIND);
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    fs_pull(l.f, a.fs_in);
    for (int q = tid >> 6; q < NW; q += nw) {
        uint64_t v = 0;
        for (int b = lane; b < a.nb; b += 64) v = m61::fold(v + a.part[(size_t)q * kF2MaxBlocks + b]);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) v = m61::fold(v + __shfl_xor(v, off, 64));
        if (lane == 0) l.tot[q] = m61::canon(v);
    }
    const f2 r = KIND == F2_MATMUL ? f2of(0) : ldp(a.r);
    if (tid == 0) l.K = KIND != F2_MATMUL && a.K_in ? ldp(a.K_in) : f2of(1);
    __syncthreads();
    const f2 rho = fs_finish_round<KIND>(l, r, a.cst, a.ev, writer, a.err);
    if (KIND != F2_MATMUL) {
        if (tid == 64) {
            const f2 K = f2mul(l.K, eq1z(r, rho));
            l.K = K;
            if (writer && a.K_out) stp(a.K_out, K);
        }
        __syncthreads();
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
// A round's hash takes 3.5 us on two waves, so the rest of a round runs
// beside it on the others: with T_c the tables bound at rho_{<c}, the sums of
// round c + 1 are quadratic in rho_c, its pairs being lo = x0 + rho (x2 - x0),
// hi = x1 + rho (x3 - x1) over T_c's quads, and are taken at rho = 0 (x0, x1),
// 1 (x2, x3) and infinity (the differences) while rho_c is being hashed.  Once
// it is there, wave 0 alone interpolates them, forms the round's values and
// goes on hashing while the other waves fold.  Eleven rounds in sequence (sums
// over the block, values, hash, fold) took 111 us; so they take 88 (range).
// ---------------------------------------------------------------------------
constexpr int kTailWorkers = kFsTailThreads / 64 - 2;  // waves 2 ..

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
    f2 co[5][2];                          // K_{c+1} eq(r_{c+1}, Y), Y = 0 .. 3, and K_{c+1}, linear in rho_c
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
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) v = m61::fold(v + __shfl_xor(v, off, 64));
        const int w = 2 * q0 + (lane >> 3);
        if ((lane & 7) == 0 && w < 2 * NV) out[w] = m61::canon(v);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

__device__ __forceinline__ f2 lane_of(f2 v, int i) { return f2{__shfl(v.re, i, 64), __shfl(v.im, i, 64)}; }

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
        // the factors of the first round's values (no rho before it)
        if (KIND != F2_MATMUL && tid < 5)
            u.t.co[tid][0] = tid < 4 ? f2mul(l.K, eq1x(rs[0], tid)) : l.K;
        if (tid < 5) u.t.co[tid][1] = f2of(0);
        __syncthreads();
    }
    for (int c = 0; c < a.v; c++) {
        const int lg = a.v - c;                         // T_c holds 2^lg entries
        const int n = lg >= 2 ? 1 << (lg - 2) : 0;      // its quads
        const f2 z = c ? f2{l.f.out[0], l.f.out[1]} : f2of(0);  // rho_{c-1}
        if (wave == 0) {
            // the round's sums at rho_{c-1}, in lanes 0 .. 4: ll, lh, hh, l, h; in lanes 5 .. 9 the factors
            f2 p0 = f2of(0), p1 = f2of(0), pi = f2of(0);
            const int q = lane < 3 ? lane : (KIND == F2_RANGE && lane < 5 ? lane : 0);
            if (c == 0) {
                constexpr int rmap[5] = {2, 3, 4, 0, 1}, omap[3] = {0, 2, 1};  // of F2Sums' words
                const int at = KIND == F2_RANGE ? (q == 0 ? rmap[0] : q == 1 ? rmap[1] : q == 2 ? rmap[2] : q == 3 ? rmap[3] : rmap[4])
                                                : (q == 0 ? omap[0] : q == 1 ? omap[1] : omap[2]);
                p0 = p1 = f2{l.tot[2 * at], l.tot[2 * at + 1]};
            } else {
                const int nq = 1 << (lg - 1), nw = nq < 64 * kTailWorkers ? (nq + 63) >> 6 : kTailWorkers;  // of T_{c-1}
                const int i0 = q < 3 ? q : 6 + q, i1 = q < 3 ? 3 + q : 8 + q, ii = q < 3 ? 6 + q : i0;
                for (int w = 0; w < nw; w++) {
                    const uint64_t *t = u.t.part[w];
                    p0 = l2add(p0, f2{t[2 * i0], t[2 * i0 + 1]});
                    p1 = l2add(p1, f2{t[2 * i1], t[2 * i1 + 1]});
                    if (q < 3) pi = l2add(pi, f2{t[2 * ii], t[2 * ii + 1]});
                }
            }
            f2 b = l2sub(p1, p0);
            if (KIND != F2_MATMUL && lane >= 5 && lane < 10) {
                p0 = u.t.co[lane - 5][0];
                b = u.t.co[lane - 5][1];
                pi = f2of(0);
            }
            const f2 v = l2add(p0, l2mul(z, l2add(b, l2mul(l2sub(z, f2of(1)), pi))));
            // s(0), s(1), s(infinity) (the leading coefficient) in lanes 0, 1, 2
            const f2 ll = lane_of(v, 0), lh = lane_of(v, 1), hh = lane_of(v, 2), t2 = l2add(ll, hh);
            f2 sv;
            if (KIND == F2_RANGE) {
                const f2 inf = l2sub(t2, l2add(lh, lh)), l0 = lane_of(v, 3), h0 = lane_of(v, 4);
                const f2 lin = l2mul(cd, lane == 0 ? l0 : h0), qd = l2mul(ceq, lane == 0 ? ll : (lane == 1 ? hh : inf));
                sv = lane == 2 ? qd : l2add(qd, lin);
            } else {
                sv = lane == 0 ? ll : (lane == 1 ? hh : l2sub(l2add(t2, t2), lh));
            }
            const f2 s0 = lane_of(sv, 0), s1 = lane_of(sv, 1), si = lane_of(sv, 2);
            const int X = lane & 3;
            f2 g = l2add(l2add(s0, l2small(l2sub(s1, s0), X)), l2small(si, X * (X - 1)));
            if (KIND != F2_MATMUL) {
                const f2 ke = lane_of(v, 5 + X);
                g = l2mul(ke, g);
                if (lane == 9) l.K = v;  // K_c
            }
            g = l2canon(g);
            // the values: to the transcript, behind what is pending
            const uint32_t qlen = l.f.m[8];
            if (lane < D1) {
                ev[D1 * c + lane] = g;
                l.g[lane] = g;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const bool ok = fs_append(l.f, qlen, (const uint32_t *)l.g, 4 * D1, lane, 64);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane == 0) {
                if (ok) l.f.m[8] = qlen + 16 * D1;
                else *a.err = 1;
            }
        } else if (wave >= 2 && c > 0) {  // T_c from T_{c-1}: an entry's two sources are read by its own thread only
            for (int i = tid - 128; i < (n ? n : 1); i += 64 * kTailWorkers)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int p = n ? i + e * n : e, hs = 1 << lg;
                    if (p < hs)
#pragma unroll
                        for (int q = 0; q < NT; q++) T[q][p] = l2fold(T[q][p], T[q][p + hs], z);
                }
        }
        __syncthreads();
        if (wave < 2) {
            fs_hash(l.f);
        } else if (n) {
            if (tid - 128 < (n > 64 ? n : 64) || wave == 2) {
                PairSums at[3];
                f2 lin[2][2] = {{f2of(0), f2of(0)}, {f2of(0), f2of(0)}};
                for (int i = tid - 128; i < n; i += 64 * kTailWorkers) {
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
                wave_totals<NV>(val, u.t.tr[wave - 2], u.t.part[wave - 2]);
            }
            if (KIND != F2_MATMUL && wave == kTailWorkers + 1 && lane < 5) {
                // K_{c+1} = K_c eq(r_c, rho_c) = K_c (1 - r_c) + rho_c K_c (2 r_c - 1), with its factors for round c + 1
                const f2 K = l.K, r = rs[c];
                const f2 k0 = l2mul(K, f2sub(f2of(1), r)), k1 = l2mul(K, f2sub(f2add(r, r), f2of(1)));
                f2 e = f2of(1);
                if (lane < 4) e = l2eq1x(rs[c + 1], lane);
                u.t.co[lane][0] = l2mul(k0, e);
                u.t.co[lane][1] = l2mul(k1, e);
            }
        }
        __syncthreads();
    }
    if (a.v > 0) {
        if (tid < NT) T[tid][0] = l2fold(T[tid][0], T[tid][1], f2{l.f.out[0], l.f.out[1]});
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
    if (!fs_absorb(l.f, (const uint32_t *)fin, 4 * nfin) && tid == 0) *a.err = 1;
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
