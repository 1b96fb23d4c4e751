// commit.hip -- Pedersen vector commitments P = sum_i v_i G_i on secp256k1
// (Sec. II-C commits a vector a as g^a; Sec. IV names the curve), for the
// integer tables of a layer.
//
// The multi-scalar product is the bucket (Pippenger) method with 9-bit
// windows of signed digits (two windows for 16-bit values, four for 32-bit,
// eight for 64-bit words), the signs applied to the point:
//   P = sum_w 2^(9w) sum_{b=1}^{256} b S_{w,b},  S_{w,b} = sum of +-G_i
//   over the i whose window-w digit is +-b.
// A workgroup takes a chunk of values and one window: it sorts the chunk by
// digit in LDS (a counting sort), then every thread adds an equal run of the
// sorted list with mixed additions, so a heavy bucket is spread over many
// threads; the runs' partial sums, in bucket order, are added per bucket.
// The chunks' bucket sums are then added per bucket, and sum_b b S_{w,b} is
// formed as sum_k 2^k (sum over the b with bit k set).  Every table of a
// batch is in each of the four launches.
#include <algorithm>

#include "commit.hpp"
#include "secp29.hpp"
#include "sha256.hpp"

namespace ra {

using secp::Fe;

// ---------------------------------------------------------------------------
// Generators by try-and-increment: x = SHA-256(tag || domain || LE64(i) ||
// LE32(c)) big-endian mod q for c = 0, 1, ...; the first x with x^3 + 7 a
// square gives (x, y), y the even root.
// ---------------------------------------------------------------------------
struct GenArgs {
    uint8_t domain[32];
    uint64_t first, count;
    uint32_t *gens, *err;
};

__global__ __launch_bounds__(256) void k_commit_generators(GenArgs a)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.count) return;
    const uint64_t idx = a.first + i;
    const char tag[] = "range-arithmetic generators v1";
    for (uint32_t c = 0; c < 256; c++) {
        sha::Hasher h;
        h.init();
        h.update((const uint8_t *)tag, sizeof(tag) - 1);
        h.update(a.domain, 32);
        h.le(idx, 8);
        h.le(c, 4);
        uint8_t d[32];
        h.final(d);
        Fe x;
        for (int l = 0; l < 8; l++)
            x.v[l] = ((uint32_t)d[31 - 4 * l - 3] << 24) | ((uint32_t)d[31 - 4 * l - 2] << 16) |
                     ((uint32_t)d[31 - 4 * l - 1] << 8) | d[31 - 4 * l];
        x = secp::fe_canon(x, 0);
        const Fe rhs = secp::fe_add(secp::fe_mul(secp::fe_sqr(x), x), secp::fe_small(7));
        Fe y = secp::fe_sqrt(rhs);
        if (!secp::fe_eq(secp::fe_sqr(y), rhs)) continue;
        if (y.v[0] & 1) y = secp::fe_neg(y);
        uint32_t *o = a.gens + 16 * i;
        for (int l = 0; l < 8; l++) {
            o[l] = x.v[l];
            o[8 + l] = y.v[l];
        }
        return;
    }
    atomicOr(a.err, 1u);
}

void launch_commit_generators(const uint8_t *domain, uint64_t first, uint64_t count, uint32_t *gens, uint32_t *err,
                              hipStream_t st)
{
    GenArgs a{};
    for (int i = 0; i < 32; i++) a.domain[i] = domain[i];
    a.first = first;
    a.count = count;
    a.gens = gens;
    a.err = err;
    hipLaunchKernelGGL(k_commit_generators, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, a);
}

// ---------------------------------------------------------------------------
// The bucket method
// ---------------------------------------------------------------------------
using secp29::F;
using secp29::Pt;
constexpr int kPipThreads = 512;
constexpr int kPipSub = 16384;             // values a workgroup sorts at a time, at most (LDS)
constexpr int kPipBits = 9;                // window width; digits -256 .. 255, buckets 1 .. 256
constexpr int kPipBuckets = 256;
constexpr int kPipParts = kPipThreads + kPipBuckets - 1;  // run partials of one sort, at most
constexpr int kPipChunks = 128;            // chunks of a table, at most
constexpr int kPtWords = secp29::kPtWords;
constexpr int kBitSums = kPipBits;         // bits of a bucket's number

int msm_windows(int kind) { return kind == 3 ? 8 : (kind == 2 ? 4 : 2); }

// Room per window: kPipChunks + 1 rows of 256 points and kBitSums more (what
// the kernels use), within what earlier forms of the workspace held: a
// caller's workspace of that size stays large enough, and the check of its
// size what it was.
size_t msm_workspace_bytes(int kind)
{
    constexpr size_t per_window = (size_t)256 * 257 * 96 + 8 * 96;
    static_assert(((size_t)(kPipChunks + 1) * kPipBuckets + kBitSums) * kPtWords * 4 <= per_window, "workspace");
    return (size_t)msm_windows(kind) * per_window + 256;
}

// |v| and its sign for value i
__device__ __forceinline__ void scalar(const void *vals, int kind, uint64_t i, uint64_t &mag, int &neg)
{
    int64_t s;
    switch (kind) {
    case 0: s = ((const int16_t *)vals)[i]; break;
    case 1: mag = ((const uint16_t *)vals)[i]; neg = 0; return;
    case 2: s = ((const int32_t *)vals)[i]; break;
    default: mag = ((const uint64_t *)vals)[i]; neg = 0; return;
    }
    neg = s < 0;
    mag = (uint64_t)(s < 0 ? -s : s);
}

// Digit w of W of mag, in -256 .. 255 below the top one: with 256 added to
// each of the lower digits, digit w is the 9-bit field less 256; the top
// digit is what is left (at most 2^7 + 1 for every value type, the carry out of 64
// bits included).
__device__ __forceinline__ int signed_digit(uint64_t mag, int w, int W)
{
    uint64_t bias = 0;
    for (int i = 0; i < W - 1; i++) bias |= 256ull << (kPipBits * i);
    const uint64_t t = mag + bias;
    if (w < W - 1) return (int)((t >> (kPipBits * w)) & 511) - 256;
    const uint64_t carry = t < mag ? 1 : 0;  // 2^64; W = 8: the top digit starts at bit 63
    return (int)((t >> (kPipBits * w)) | (carry << (64 - kPipBits * w)));
}

// Exclusive prefix sums of one value per thread (kPipThreads threads); the
// total to *total.  sc: a word per wave.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *sc, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t inc = v;
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) sc[wv] = inc;
    __syncthreads();
    uint32_t before = 0;
    for (int q = 0; q < wv; q++) before += sc[q];
    if (total && threadIdx.x == kPipThreads - 1) *total = before + inc;
    const uint32_t ex = before + inc - v;
    __syncthreads();
    return ex;
}

// The tables of one batch: windows of table t are the global windows
// wpre[t] .. wpre[t + 1] - 1; its workspace starts off[t] bytes into ws:
// the chunks' bucket sums (W C 256 points, window-major), the bucket sums S
// (W 256), their bit sums U (W kBitSums).
struct MsmBatch {
    int count;
    uint32_t wpre[kCommitBatchMax + 1];
    uint32_t C[kCommitBatchMax];     // chunks
    uint8_t kind[kCommitBatchMax];
    uint64_t off[kCommitBatchMax];
    uint64_t n[kCommitBatchMax];
    const void *vals[kCommitBatchMax];
    uint64_t per;                    // values per chunk, the same for every table
    uint32_t sort;                   // values per sort
};
__device__ __forceinline__ int batch_table(const MsmBatch &b, uint32_t gw)
{
    int t = 0;
    while (t + 1 < b.count && gw >= b.wpre[t + 1]) t++;
    return t;
}
__device__ __forceinline__ uint32_t *batch_chunks(char *ws, const MsmBatch &b, int t)
{
    return (uint32_t *)(ws + b.off[t]);
}
__device__ __forceinline__ uint32_t *batch_S(char *ws, const MsmBatch &b, int t)
{
    const uint32_t W = b.wpre[t + 1] - b.wpre[t];
    return batch_chunks(ws, b, t) + (size_t)W * kPipChunks * kPipBuckets * kPtWords;
}
__device__ __forceinline__ uint32_t *batch_U(char *ws, const MsmBatch &b, int t)
{
    const uint32_t W = b.wpre[t + 1] - b.wpre[t];
    return batch_S(ws, b, t) + (size_t)W * kPipBuckets * kPtWords;
}

// Workgroup (window, chunk): the window's bucket sums over the chunk's values,
// in sorts of bt.sort values.  A table with fewer chunks has no work for the
// rest.
//
// Bound by the field products of the additions (VALU issue): about 1700
// instructions per addition, one per nonzero digit, 1.7 of the pass's
// 2.6 ms for the five witness tables of 2^21 outputs.  512 threads over
// 148 KB of LDS are one workgroup, two waves per SIMD.  A sort's partials
// cost full additions (1.1 ms with sorts of 8192 values), so a sort takes
// 16384 values where there are enough; the digits are formed twice rather
// than kept, and the sorted list holds position and sign in 16 bits.  Nine-bit
// signed digits fill 256 buckets (8-bit unsigned ones 255) with fewer digits:
// 2 instead of 3 for 18-bit values, 7 instead of 8 for 60-bit words.  The
// windows of one chunk are adjacent workgroups on one XCD (workgroups go to
// the XCDs in turn), so its generators are fetched into one L2.
__global__ __launch_bounds__(kPipThreads) void k_pip_buckets(char *ws, MsmBatch bt, const uint32_t *__restrict__ gens)
{
    __shared__ uint16_t perm[kPipSub];  // position, sign in the top bit; sorted by |digit|
    __shared__ uint16_t pd[kPipParts];
    __shared__ uint32_t cnt[kPipBuckets + 1], end[kPipBuckets + 1], first[kPipBuckets + 1];
    __shared__ uint32_t sc[kPipThreads / 64], tot[2];
    __shared__ uint32_t pp[kPipParts][kPtWords];
    static_assert(kPipSub <= 1 << 14, "a position and a sign in 16 bits; counts in 16");
    const int tid = threadIdx.x;
    const uint32_t nw = bt.wpre[bt.count], x = blockIdx.x >> 3;
    const uint32_t gw = x % nw, c = x / nw * 8 + (blockIdx.x & 7);
    const int t = batch_table(bt, gw);
    const int W = (int)(bt.wpre[t + 1] - bt.wpre[t]), w = (int)(gw - bt.wpre[t]), kind = bt.kind[t];
    if (c >= bt.C[t]) return;
    const void *vals = bt.vals[t];
    const uint64_t lo = (uint64_t)c * bt.per, hi = lo + bt.per < bt.n[t] ? lo + bt.per : bt.n[t];
    // thread b - 1's bucket b, kept in memory between the sorts
    uint32_t *bucket =
        batch_chunks(ws, bt, t) + (((size_t)w * bt.C[t] + c) * kPipBuckets + (tid & (kPipBuckets - 1))) * kPtWords;
    bool empty = true;
    for (uint64_t base = lo; base < hi; base += bt.sort) {
        const int len = (int)(hi - base < (uint64_t)bt.sort ? hi - base : (uint64_t)bt.sort);
        // f(i, digit of value i), every i once; eight loads in flight per thread
        auto each_digit = [&](auto f) {
            constexpr int U = 8;
            for (int i0 = tid; i0 < len; i0 += U * kPipThreads) {
                uint64_t mag[U];
                int neg[U];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int i = i0 + u * kPipThreads;
                    scalar(vals, kind, base + (i < len ? i : i0), mag[u], neg[u]);
                }
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int i = i0 + u * kPipThreads, d = signed_digit(mag[u], w, W);
                    if (i < len) f(i, neg[u] ? -d : d);
                }
            }
        };
        if (tid <= kPipBuckets) {
            cnt[tid] = 0;
            first[tid] = 0xFFFFFFFFu;
        }
        __syncthreads();
        each_digit([&](int, int d) { atomicAdd(&cnt[abs(d)], 1u); });
        __syncthreads();
        // counting sort by |digit|; end[d] is the start of digit d, and after the scatter its end
        const uint32_t st = block_scan(tid <= kPipBuckets ? cnt[tid] : 0, sc, nullptr);
        if (tid <= kPipBuckets) end[tid] = st;
        const int skip = (int)cnt[0];  // zero digits
        __syncthreads();
        if (skip == len) continue;  // no digit in this window
        each_digit([&](int i, int d) {
            if (d) perm[atomicAdd(&end[abs(d)], 1u)] = (uint16_t)(i | (d < 0 ? 1 << 15 : 0));
        });
        __syncthreads();
        // runs of the sorted list past the zero digits: thread t takes [r0, r1)
        const int run = (len - skip + kPipThreads - 1) / kPipThreads;
        const int r0 = skip + tid * run < len ? skip + tid * run : len;
        const int r1 = r0 + run < len ? r0 + run : len;
        int d0 = 0;       // the digit at r0: the first whose end is past it
        uint32_t np = 0;  // partials of this run: its distinct digits
        if (r0 < r1) {
            int a = 1, b = kPipBuckets;
            while (a < b) {
                const int m = (a + b) >> 1;
                if ((int)end[m] > r0) b = m;
                else a = m + 1;
            }
            d0 = a;
            np = 1;
            for (int d = a; (int)end[d] < r1; d++) np += cnt[d + 1] != 0;
        }
        const uint32_t off = block_scan(np, sc, &tot[1]);
        if (r0 < r1) {
            Pt acc = secp29::identity();
            uint32_t k = off;
            uint32_t nx[16];
            auto fetch = [&](int i) {  // the next generator, while this one is added
                const uint4 *gp = (const uint4 *)(gens + 16 * (base + i));
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const uint4 y = gp[v];
                    nx[4 * v] = y.x;
                    nx[4 * v + 1] = y.y;
                    nx[4 * v + 2] = y.z;
                    nx[4 * v + 3] = y.w;
                }
            };
            int i = perm[r0], de = (int)end[d0];
            fetch(i & 0x7FFF);
            bool fresh = true;
#pragma unroll 1
            for (int q = r0; q < r1; q++) {
                const F x = secp29::from_limbs32(nx);
                F y = secp29::from_limbs32(nx + 8);
                if (i >> 15) y = secp29::neg(y);
                if (q + 1 < r1) {
                    i = perm[q + 1];
                    fetch(i & 0x7FFF);
                }
                if (q == de) {  // a new bucket starts with this point
                    secp29::store(pp[k], acc);
                    pd[k++] = (uint16_t)d0;
                    do de = (int)end[++d0];
                    while (de == q);
                    fresh = true;
                }
                if (fresh) acc = Pt{x, y, secp29::one(), secp29::one()};
                else secp29::add_affine(acc, x, y);
                fresh = secp29::is_identity(acc);  // a point and its opposite
            }
            secp29::store(pp[k], acc);
            pd[k] = (uint16_t)d0;
        }
        __syncthreads();
        // The partials are in digit order.  A digit spread over many runs (a
        // heavy bucket) has many partials: they are summed by a segmented tree
        // (round s: partial p of a segment, p a multiple of 2s, adds the one
        // s after it) until every segment's first partial holds its sum.
        const uint32_t nparts = tot[1];
        if (tid == 0) tot[0] = 1;  // the longest segment
        for (uint32_t k = tid; k < nparts; k += kPipThreads) {
            if (k == 0 || pd[k] != pd[k - 1]) first[pd[k]] = k;
            atomicAdd(&cnt[pd[k]], 1u << 16);  // the partials of digit d, above its count
        }
        __syncthreads();
        if (tid < kPipBuckets) atomicMax(&tot[0], cnt[tid + 1] >> 16);
        __syncthreads();
        const uint32_t longest = tot[0];
        for (uint32_t sd = 1; sd < longest; sd <<= 1) {
            // the round's additions, listed (at most nparts / 2, less than the threads) where perm was
            if (tid == 0) tot[1] = 0;
            __syncthreads();
            for (uint32_t k = tid; k + sd < nparts; k += kPipThreads)
                if (((k - first[pd[k]]) & (2 * sd - 1)) == 0 && pd[k + sd] == pd[k])
                    perm[atomicAdd(&tot[1], 1u)] = (uint16_t)k;
            __syncthreads();
            if ((uint32_t)tid < tot[1]) {
                const uint32_t k = perm[tid];
                secp29::store(pp[k], secp29::add(secp29::load(pp[k]), secp29::load(pp[k + sd])));
            }
            __syncthreads();
        }
        if (tid < kPipBuckets && first[tid + 1] != 0xFFFFFFFFu) {
            const Pt s = secp29::load(pp[first[tid + 1]]);
            secp29::store(bucket, empty ? s : secp29::add(secp29::load(bucket), s));
            empty = false;
        }
        __syncthreads();  // LDS reused by the next sort
    }
    if (tid < kPipBuckets && empty) secp29::store(bucket, secp29::identity());
}

// Sums of G points per group of G threads (each thread's point in p[tid]) by a
// tree in LDS; the group's first thread ends with the sum in p.
template <int G> __device__ __forceinline__ void group_tree(uint32_t (*p)[kPtWords])
{
    const int tid = threadIdx.x, j = tid & (G - 1);
#pragma unroll 1
    for (int st = G / 2; st >= 1; st >>= 1) {
        __syncthreads();
        if (j < st) secp29::store(p[tid], secp29::add(secp29::load(p[tid]), secp29::load(p[tid + st])));
    }
    __syncthreads();
}

// S[w][b] = sum over the C chunks of the chunks' bucket b of window w: 16
// threads per bucket, each a strided share, then a tree.  Sixteen buckets of
// one window per workgroup; the workgroups run over the batch's windows.
__global__ __launch_bounds__(256) void k_pip_bucket_sums(char *ws, MsmBatch bt)
{
    __shared__ uint32_t part[256][kPtWords];
    const int tid = threadIdx.x, j = tid & 15;
    const uint32_t wb = blockIdx.x * 16 + (tid >> 4), gw = wb / kPipBuckets, b = wb % kPipBuckets;
    const int t = batch_table(bt, gw);  // workgroup-uniform
    const uint32_t w = gw - bt.wpre[t], C = bt.C[t];
    const uint32_t *in = batch_chunks(ws, bt, t);
    Pt acc = secp29::identity();
#pragma unroll 1
    for (uint32_t c = j; c < C; c += 16)
        acc = secp29::add(acc, secp29::load(in + (((size_t)w * C + c) * kPipBuckets + b) * kPtWords));
    secp29::store(part[tid], acc);
    group_tree<16>(part);
    if (j == 0) secp29::store(batch_S(ws, bt, t) + ((size_t)w * kPipBuckets + b) * kPtWords, secp29::load(part[tid]));
}

// U[w][k] = sum over the buckets b with bit k of S[w][b]: 64 threads per (w,
// k), two buckets each (k < 8: 128 of them; k = 8: bucket 256 alone).
__global__ __launch_bounds__(64) void k_pip_bit_sums(char *ws, MsmBatch bt)
{
    __shared__ uint32_t part[64][kPtWords];
    const int tid = threadIdx.x;
    const uint32_t gw = blockIdx.x / kBitSums, k = blockIdx.x % kBitSums;
    const int t = batch_table(bt, gw);
    const uint32_t w = gw - bt.wpre[t];
    const uint32_t *S = batch_S(ws, bt, t) + (size_t)w * kPipBuckets * kPtWords;
    Pt acc = secp29::identity();
    if (k == 8) {
        if (tid == 0) acc = secp29::load(S + 255 * kPtWords);
    } else {
#pragma unroll 1
        for (uint32_t q = tid; q < 128; q += 64) {  // the q-th b below 256 with bit k set
            const uint32_t b = ((q >> k) << (k + 1)) | (1u << k) | (q & ((1u << k) - 1));
            acc = secp29::add(acc, secp29::load(S + (size_t)(b - 1) * kPtWords));
        }
    }
    secp29::store(part[tid], acc);
    group_tree<64>(part);
    if (tid == 0) secp29::store(batch_U(ws, bt, t) + ((size_t)w * kBitSums + k) * kPtWords, secp29::load(part[0]));
}

// P = sum over (w, k) of 2^(9w + k) U[w][k]: each pair's doublings by a thread
// of its own, side by side, then a tree and the affine bytes to out + 64 t.
// One workgroup per table.
__global__ __launch_bounds__(128) void k_pip_final(char *ws, MsmBatch bt, uint8_t *__restrict__ out)
{
    __shared__ uint32_t T[128][kPtWords];
    const int tid = threadIdx.x, t = blockIdx.x;
    const int W = (int)(bt.wpre[t + 1] - bt.wpre[t]);
    const uint32_t *U = batch_U(ws, bt, t);
    Pt p = secp29::identity();
    if (tid < W * kBitSums) {
        p = secp29::load(U + (size_t)tid * kPtWords);  // 9 w + k is the thread's number
        if (!secp29::is_identity(p)) {
            secp29::Jac q = secp29::to_jac(p);
#pragma unroll 1
            for (int i = 0; i < tid; i++) q = secp29::dbl(q);
            p = secp29::from_jac(q);
        }
    }
    secp29::store(T[tid], p);
    group_tree<128>(T);
    if (tid == 0) {
        p = secp29::load(T[0]);
        uint8_t bytes[64];
        for (int i = 0; i < 64; i++) bytes[i] = 0;
        if (!secp29::is_identity(p)) {  // x = X / ZZ, y = Y / ZZZ, 1 / ZZ = (ZZ / ZZZ)^2
            const F iz3 = secp29::inverse(p.ZZZ), iz = secp29::mul(iz3, p.ZZ);
            const secp::Fe x = secp29::canon(secp29::mul(p.X, secp29::sqr(iz)));
            const secp::Fe y = secp29::canon(secp29::mul(p.Y, iz3));
            for (int i = 0; i < 32; i++) {
                bytes[i] = (uint8_t)(x.v[7 - i / 4] >> (8 * (3 - i % 4)));
                bytes[32 + i] = (uint8_t)(y.v[7 - i / 4] >> (8 * (3 - i % 4)));
            }
        }
        for (int i = 0; i < 64; i++) out[64 * (size_t)t + i] = bytes[i];
    }
}

size_t msm_batch_offsets(const int *kinds, int count, size_t *offs)
{
    size_t o = 0;
    for (int t = 0; t < count; t++) {
        offs[t] = o;
        o += (msm_workspace_bytes(kinds[t]) + 255) & ~(size_t)255;
    }
    return o;
}

void launch_commit_batch(const void *const *vals, const int *kinds, const uint64_t *ns, int count,
                         const uint32_t *gens, void *ws, uint8_t *out, hipStream_t st)
{
    MsmBatch bt{};
    bt.count = count;
    size_t offs[kCommitBatchMax];
    msm_batch_offsets(kinds, count, offs);
    uint64_t nmax = 1;
    for (int t = 0; t < count; t++) nmax = std::max(nmax, ns[t]);
    for (int t = 0; t < count; t++) bt.wpre[t + 1] = bt.wpre[t] + (uint32_t)msm_windows(kinds[t]);
    // Sorts of kPipSub values (their partials' additions weigh least), less
    // while that leaves fewer than 1024 workgroups (four per CU), but at least
    // two values per thread.
    const uint64_t want = nmax * bt.wpre[count] / 1024;
    bt.sort = (uint32_t)(std::min<uint64_t>(std::max<uint64_t>(want, 1024), kPipSub) + 511) / 512 * 512;
    const uint64_t subs = (nmax + bt.sort - 1) / bt.sort, Cmax = std::min<uint64_t>(subs, kPipChunks);
    bt.per = (subs + Cmax - 1) / Cmax * bt.sort;  // whole sorts per chunk but the last
    uint32_t chunks = 1;
    for (int t = 0; t < count; t++) {
        bt.C[t] = (uint32_t)((ns[t] + bt.per - 1) / bt.per);
        chunks = std::max(chunks, bt.C[t]);
        bt.kind[t] = (uint8_t)kinds[t];
        bt.off[t] = offs[t];
        bt.n[t] = ns[t];
        bt.vals[t] = vals[t];
    }
    const uint32_t nw = bt.wpre[count];
    hipLaunchKernelGGL(k_pip_buckets, dim3((chunks + 7) / 8 * 8 * nw), dim3(kPipThreads), 0, st, (char *)ws, bt, gens);
    hipLaunchKernelGGL(k_pip_bucket_sums, dim3(nw * (kPipBuckets / 16)), dim3(256), 0, st, (char *)ws, bt);
    hipLaunchKernelGGL(k_pip_bit_sums, dim3(nw * kBitSums), dim3(64), 0, st, (char *)ws, bt);
    hipLaunchKernelGGL(k_pip_final, dim3(count), dim3(128), 0, st, (char *)ws, bt, out);
}

void launch_commit(const void *vals, int kind, uint64_t n, const uint32_t *gens, void *ws, uint8_t *out,
                   hipStream_t st)
{
    launch_commit_batch(&vals, &kind, &n, 1, gens, ws, out, st);
}

}  // namespace ra
