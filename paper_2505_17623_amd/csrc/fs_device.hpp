// fs_device.hpp -- the Fiat-Shamir transcript on the device, worked by one
// workgroup of at least 128 threads from LDS.  The transcript
// (sha::Transcript in device memory: S, the pending length, the pending
// bytes) is pulled into LDS laid out as the next draw's message, S ||
// LE32(|Q|) || Q, so that absorbing appends to it and drawing hashes it in
// place.  Everything absorbed is whole 32-bit words, so the message is worked
// by words throughout.
//
// A draw is a chain of SHA-256 compressions, each 64 dependent rounds, and
// one wave issues an instruction every four cycles (8-byte encodings: 4.6)
// whatever its lanes do, so the instructions of the chain are its time.  Wave
// 1 expands the message schedules (one block per lane, every block of the
// message at once) sixteen words ahead of wave 0, which only runs the rounds,
// both halves of the state side by side in its lanes (ShaLanes): 19 ns per
// round, 25 with all eight variables in one lane.  Nothing is loaded from
// memory inside a draw (the initial state and the constants wait in LDS), the
// padding is written with what is absorbed, and wave 0 starts on the message
// itself.  Against rounds of 14 instructions on one lane: a draw with nothing
// pending 2.5 -> 1.8 us, with a round's values 4.5 -> 3.5 us (MI355X).
#pragma once
#include "sha256.hpp"

namespace ra {

constexpr int kFsMsgWords = 9 + sha::kFsPending / 4;        // S, |Q|, Q
constexpr int kFsMaxBlocks = (4 * kFsMsgWords + 9 + 63) / 64;
struct FsLds {
    uint32_t m[kFsMaxBlocks * 16];    // the message, room for its padding
    uint4 kw[kFsMaxBlocks * 16];      // schedule plus round constants, 64 words per block
    uint64_t out[2];                  // the last challenge drawn
    uint32_t h0[8], k16[16];          // the initial state, the first sixteen round constants
    uint32_t go;                      // messages complete, where no barrier says so (0 before and after)
    uint32_t ready;                   // quarters of the schedules after the first that wave 1 has stored (0 between draws)
};

__device__ __forceinline__ uint32_t vgpr(uint32_t x)  // the value, kept in vector registers
{
    asm("" : "+v"(x));
    return x;
}

// Blocks of the padded message of `words` words.
__device__ __forceinline__ int fs_blocks(int words) { return (4 * words + 9 + 63) / 64; }

// Thread t of nt: the padding behind a message of `words` words (0x80, zeros,
// the length in bits, as bytes in order), which f.m holds whenever a draw may
// follow, so that a draw reads whole blocks.
__device__ __forceinline__ void fs_pad(FsLds &f, int words, int t, int nt)
{
    const int end = 16 * fs_blocks(words);
    for (int i = words + t; i < end; i += nt)
        f.m[i] = i == words ? 0x80u : (i == end - 1 ? __builtin_bswap32(32u * (uint32_t)words) : 0u);
}

// The block: the transcript into f (visible after the caller's next barrier).
__device__ inline void fs_pull(FsLds &f, const sha::Transcript *g)
{
    const uint32_t *s = (const uint32_t *)g;
    const int words = 9 + (int)(s[8] >> 2);
    for (int i = threadIdx.x; i < kFsMsgWords; i += blockDim.x) {  // all of it: the loads do not wait for the length
        const uint32_t x = s[i];
        if (i < words) f.m[i] = x;
    }
    fs_pad(f, words, threadIdx.x, blockDim.x);
    if (threadIdx.x < 16) f.k16[threadIdx.x] = sha::kConsts.k[threadIdx.x];
    if (threadIdx.x < 8) f.h0[threadIdx.x] = sha::kConsts.h[threadIdx.x];
    if (threadIdx.x == 0) f.ready = f.go = 0;
}

// The block: f back into the transcript (after a barrier).
__device__ inline void fs_push(sha::Transcript *g, const FsLds &f)
{
    uint32_t *d = (uint32_t *)g;
    const int words = 9 + (int)(f.m[8] >> 2);
    for (int i = threadIdx.x; i < words; i += blockDim.x) d[i] = f.m[i];
}

// Threads t of nt: the nw 32-bit words at w (of any type) behind the pending
// ones and the padding behind them, where they fit (false: more than
// sha::kFsPending bytes pending).  The length is the caller's to set, once
// f.m[8] has been read.
__device__ __forceinline__ bool fs_append(FsLds &f, uint32_t q, const void *w, int nw, int t, int nt)
{
    if (q + 4 * (uint32_t)nw > sha::kFsPending) return false;
    const int at = 9 + (int)(q >> 2);
    for (int i = t; i < nw; i += nt) {
        uint32_t x;
        __builtin_memcpy(&x, (const char *)w + 4 * i, 4);  // the words of 64-bit values: a copy, not a read as another type
        f.m[at + i] = x;
    }
    fs_pad(f, at + nw, t, nt);
    return true;
}

// The block: append the nw 32-bit words at w (of any type, readable by every
// thread).  Barriers on both sides; false: more than sha::kFsPending bytes pending.
__device__ inline bool fs_absorb(FsLds &f, const void *w, int nw)
{
    __syncthreads();
    const uint32_t q = f.m[8];
    const bool ok = fs_append(f, q, w, nw, threadIdx.x, blockDim.x);
    __syncthreads();
    if (ok && threadIdx.x == 0) f.m[8] = q + 4 * (uint32_t)nw;
    __syncthreads();
    return ok;
}

// The rounds of one hash over the lanes of a wave.  In each group of eight
// lanes the first four hold a, b, c, d and the others e, f, g, h, so that one
// instruction forms both big sigmas (the rotations differ by lane), and one
// pair of them both majority and choice: with x = a ^ b the majority is
// x ? c : b, with x = ~e the choice is x ? g : f.  The halves meet in adds
// whose operand is the other half's lane (DPP row_half_mirror: lane i reads
// 7 - i): 10 instructions per round where one lane alone needs 14.
struct ShaLanes {
    uint32_t v[4];         // a, b, c, d or e, f, g, h
    uint32_t q;            // h + schedule word + constant of the round to come (e's half), 0 (a's half)
    uint32_t s1, s2, s3;   // the rotations of the half's sigma
    uint32_t m;            // all ones in e's half
    __device__ __forceinline__ void init(int lane)
    {
        const bool e = lane & 4;
        s1 = vgpr(e ? 6 : 2);
        s2 = vgpr(e ? 11 : 13);
        s3 = vgpr(e ? 25 : 22);
        m = vgpr(e ? ~0u : 0u);
    }
    __device__ __forceinline__ void start(const uint32_t (&st)[4], uint32_t kw0)
    {
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = st[i];
        q = (v[3] + kw0) & m;
        // a DPP operand may not be written in the two instructions before it is read
        asm volatile("s_nop 1" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(q));
    }
    // four rounds; k: schedule words + constants of the second to the fourth
    // and of the round after them.  A round: sigma in s; x = m ? ~v0 : v0 ^ v1
    // and the choice by it; s = T1 in e's half, T2 in a's; e' = T1 + d, a' = T2
    // + T1 in the place of h and d.  Two instructions lie between the write of
    // s and its DPP read.  (In one block, since the compiler puts a wait
    // between two blocks that pass a register on.)
    __device__ __forceinline__ void rounds4(uint32_t k0, uint32_t k1, uint32_t k2, uint32_t k3)
    {
#define RA_SHA_ROUND(A, B, C, D, K)                                                   \
    "v_alignbit_b32 %[s], " A ", " A ", %[s1]\n\t"                                    \
    "v_alignbit_b32 %[x], " A ", " A ", %[s2]\n\t"                                    \
    "v_alignbit_b32 %[y], " A ", " A ", %[s3]\n\t"                                    \
    "v_bitop3_b32 %[s], %[s], %[x], %[y] bitop3:0x96\n\t"                             \
    "v_bitop3_b32 %[x], " A ", " B ", %[m] bitop3:0x1e\n\t"                           \
    "v_bitop3_b32 %[x], %[x], " C ", " B " bitop3:0xca\n\t"                           \
    "v_add3_u32 %[s], %[q], %[s], %[x]\n\t"                                           \
    "v_add_u32_dpp " D ", " D ", %[s] row_half_mirror row_mask:0xf bank_mask:0xf\n\t"  \
    "v_add_u32_dpp %[q], " C ", " K " quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xa\n\t" \
    "v_add_u32_dpp " D ", %[s], %[s] row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
        uint32_t s, x, y;
        asm(RA_SHA_ROUND("%[a]", "%[b]", "%[c]", "%[d]", "%[k0]")
            RA_SHA_ROUND("%[d]", "%[a]", "%[b]", "%[c]", "%[k1]")
            RA_SHA_ROUND("%[c]", "%[d]", "%[a]", "%[b]", "%[k2]")
            RA_SHA_ROUND("%[b]", "%[c]", "%[d]", "%[a]", "%[k3]")
            : [s] "=&v"(s), [x] "=&v"(x), [y] "=&v"(y), [q] "+&v"(q), [a] "+&v"(v[0]), [b] "+&v"(v[1]),
              [c] "+&v"(v[2]), [d] "+&v"(v[3])
            : [k0] "v"(k0), [k1] "v"(k1), [k2] "v"(k2), [k3] "v"(k3), [s1] "v"(s1), [s2] "v"(s2), [s3] "v"(s3),
              [m] "v"(m));
#undef RA_SHA_ROUND
    }
    // sixteen rounds; k: the words of the rounds, next: of the one after them
    __device__ __forceinline__ void rounds16(const uint4 (&k)[4], uint32_t next)
    {
#pragma unroll
        for (int i = 0; i < 4; i++) rounds4(k[i].y, k[i].z, k[i].w, i < 3 ? k[i < 3 ? i + 1 : 0].x : next);
    }
};

// Words 16 (p + 1) .. 16 (p + 1) + 15 of the schedule from the sixteen before
// them (w, replaced), stored with their round constants.
template <int P>
__device__ __forceinline__ void fs_schedule16(uint32_t (&w)[16], uint4 *kw)
{
    uint32_t o[16];
#pragma unroll
    for (int t = 0; t < 16; t++) {
        const uint32_t w15 = w[(t + 1) & 15], w2 = w[(t + 14) & 15];
        const uint32_t s0 = sha::xor3(sha::rotr(w15, 7), sha::rotr(w15, 18), w15 >> 3);
        const uint32_t s1 = sha::xor3(sha::rotr(w2, 17), sha::rotr(w2, 19), w2 >> 10);
        w[t] = w[t] + s0 + (w[(t + 9) & 15] + s1);
        o[t] = w[t] + sha::kConsts.k[16 * P + t];
    }
#pragma unroll
    for (int q = 0; q < 4; q++) kw[4 * P + q] = make_uint4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
}

// A block's schedule with its round constants, 64 words, from its message
// words (replaced).
__device__ __forceinline__ void sha_schedule(uint32_t (&w)[16], uint4 *kw)
{
#pragma unroll
    for (int q = 0; q < 4; q++)
        kw[q] = make_uint4(w[4 * q] + sha::kConsts.k[4 * q], w[4 * q + 1] + sha::kConsts.k[4 * q + 1],
                           w[4 * q + 2] + sha::kConsts.k[4 * q + 2], w[4 * q + 3] + sha::kConsts.k[4 * q + 3]);
    fs_schedule16<1>(w, kw);
    fs_schedule16<2>(w, kw);
    fs_schedule16<3>(w, kw);
}

// Eight hashes per wave, one per group of eight lanes: nblk blocks whose
// schedules lie at kw (16 vectors each).  Lane 8 g: words 0 .. 3 of hash g's
// state, lane 8 g + 4: words 4 .. 7.
__device__ __forceinline__ void sha_lanes_hash(const uint4 *kw, int nblk, uint32_t (&st)[4])
{
    ShaLanes l;
    l.init(threadIdx.x & 63);
#pragma unroll
    for (int i = 0; i < 4; i++)
        st[i] = vgpr(sha::kConsts.h[i]) ^ (l.m & vgpr(sha::kConsts.h[i] ^ sha::kConsts.h[4 + i]));
    uint4 x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; i++) x[i] = kw[i];
#pragma unroll 1
    for (int b = 0; b < nblk; b++) {
        l.start(st, x[0].x);
#pragma unroll
        for (int p = 0; p < 4; p++) {
            const int next = b + 1 < nblk || p < 3 ? 4 * (4 * b + p + 1) : 0;
#pragma unroll
            for (int i = 0; i < 4; i++) y[i] = kw[next + i];
            l.rounds16(x, y[0].x);
#pragma unroll
            for (int i = 0; i < 4; i++) x[i] = y[i];
        }
#pragma unroll
        for (int i = 0; i < 4; i++) st[i] += l.v[i];
    }
}

// Word q of the challenge from S's bytes in order: LE64(S[8q .. 8q + 8]) mod p.
__device__ __forceinline__ uint64_t fs_challenge_word(const uint32_t *s)
{
    constexpr uint64_t p = 0x1FFFFFFFFFFFFFFFull;
    const uint64_t x = (uint64_t)s[0] | ((uint64_t)s[1] << 32);
    const uint64_t r = (x & p) + (x >> 61);
    return r >= p ? r - p : r;
}

// The draw proper: S = H(S || LE32(|Q|) || Q), Q emptied, the challenge's two
// words to out; one wave for each part, both started once the message is
// complete.  The rounds wait in LDS for each later quarter of the first
// block's schedule; the schedules are stored without waiting for anything.
__device__ __forceinline__ void fs_hash_schedules(FsLds &f)
{
    const int lane = threadIdx.x & 63;
    if (lane >= fs_blocks(9 + (int)(f.m[8] >> 2))) return;  // lanes without a block would publish ahead of the others
    auto publish = [&](uint32_t p) {  // LDS operations of a wave stay in order
        __hip_atomic_store(&f.ready, p, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    uint32_t w[16];
    uint4 *kw = f.kw + 16 * lane;
#pragma unroll
    for (int t = 0; t < 16; t++) w[t] = __builtin_bswap32(f.m[16 * lane + t]);
    if (lane > 0)  // wave 0 forms the first block's
#pragma unroll
        for (int q = 0; q < 4; q++)
            kw[q] = make_uint4(w[4 * q] + sha::kConsts.k[4 * q], w[4 * q + 1] + sha::kConsts.k[4 * q + 1],
                               w[4 * q + 2] + sha::kConsts.k[4 * q + 2], w[4 * q + 3] + sha::kConsts.k[4 * q + 3]);
    fs_schedule16<1>(w, kw);
    publish(1);
    fs_schedule16<2>(w, kw);
    publish(2);
    fs_schedule16<3>(w, kw);
    publish(3);
}

__device__ __forceinline__ void fs_hash_rounds(FsLds &f, uint64_t *out)
{
    const int lane = threadIdx.x & 63, nblk = fs_blocks(9 + (int)(f.m[8] >> 2));
    ShaLanes l;
    l.init(lane);
    uint32_t st[4];
#pragma unroll
    for (int i = 0; i < 4; i++) st[i] = f.h0[(lane & 4) + i];
    if (lane < 16) ((uint32_t *)f.kw)[lane] = __builtin_bswap32(f.m[lane]) + f.k16[lane];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    auto load = [&](uint4 (&x)[4], int q) {
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = f.kw[4 * q + i];
    };
    auto add = [&]() {
#pragma unroll
        for (int i = 0; i < 4; i++) st[i] += l.v[i];
    };
    uint4 x[4];
    load(x, 0);
    l.start(st, x[0].x);
#pragma unroll 1
    for (int p = 1; p < 4; p++) {  // the first block: each quarter as it comes
        // the round before a quarter's first needs its first word: it is
        // run with 0 in its place, which is added once the quarter is there
        l.rounds16(x, 0);
        uint32_t got;
        do {  // a wave's LDS operations stay in order: the words are those of a quarter stored before `got`
            got = __hip_atomic_load(&f.ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("" ::: "memory");
            load(x, p);
            asm volatile("" ::: "memory");
        } while (got < (uint32_t)p);
        l.q += x[0].x & l.m;
    }
    l.rounds16(x, 0);
    add();
    if (nblk > 1) {
        load(x, 4);
#pragma unroll 1
        for (int b = 1; b < nblk; b++) {
            l.start(st, x[0].x);
#pragma unroll
            for (int p = 0; p < 4; p++) {
                uint4 y[4];
                load(y, b + 1 < nblk || p < 3 ? 4 * b + p + 1 : 0);
                l.rounds16(x, y[0].x);
#pragma unroll
                for (int i = 0; i < 4; i++) x[i] = y[i];
            }
            add();
        }
    }
    if ((lane & ~4) == 0) {  // lanes 0 and 4: S as its bytes in order
#pragma unroll
        for (int i = 0; i < 4; i++) f.m[lane + i] = st[i] = __builtin_bswap32(st[i]);
    }
    if (lane >= 8 && lane < 16)  // nothing pending: |Q| = 0 and the padding of nine words
        f.m[lane] = lane == 9 ? 0x80u : (lane == 15 ? __builtin_bswap32(32u * 9u) : 0u);
    if (lane == 0) {
        f.ready = 0;
        out[0] = fs_challenge_word(st);
        out[1] = fs_challenge_word(st + 2);
    }
}

// Waves 0 and 1, between two barriers of the block (the other waves may do
// other work).
__device__ __forceinline__ void fs_hash(FsLds &f)
{
    if (threadIdx.x < 64) fs_hash_rounds(f, f.out);
    else if (threadIdx.x < 128) fs_hash_schedules(f);
}

// n draws in a row with nothing pending (a draw came before), by waves 0 and
// 1 between two barriers: the first four words of each new S, as its bytes in
// order, to raw[4 i ..].  A message is then S and constants, so a draw hands
// the new state straight to the next one's schedule, with no barrier between.
__device__ __forceinline__ void fs_hash_more(FsLds &f, int n, uint32_t *raw)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (wave == 1 && lane == 0) {
        for (int i = 0; i < n; i++) {
            while (__hip_atomic_load(&f.go, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < (uint32_t)(i + 1)) {
            }
            auto publish = [&](uint32_t p) {
                __hip_atomic_store(&f.ready, 3 * (uint32_t)i + p, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            uint32_t w[16];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const uint4 x = f.kw[q];
                w[4 * q] = x.x - sha::kConsts.k[4 * q];
                w[4 * q + 1] = x.y - sha::kConsts.k[4 * q + 1];
                w[4 * q + 2] = x.z - sha::kConsts.k[4 * q + 2];
                w[4 * q + 3] = x.w - sha::kConsts.k[4 * q + 3];
            }
#pragma unroll
            for (int t = 8; t < 16; t++) w[t] = t == 9 ? 0x80000000u : (t == 15 ? 32u * 9u : 0u);
            fs_schedule16<1>(w, f.kw);
            publish(1);
            fs_schedule16<2>(w, f.kw);
            publish(2);
            fs_schedule16<3>(w, f.kw);
            publish(3);
        }
    } else if (wave == 0) {
        ShaLanes l;
        l.init(lane);
        uint32_t st[4], h[4], k[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            h[i] = f.h0[(lane & 4) + i];
            k[i] = f.k16[(lane & 4) + i];
            st[i] = __builtin_bswap32(f.m[(lane & 4) + i]);
        }
        if (lane >= 8 && lane < 16)
            ((uint32_t *)f.kw)[lane] = (lane == 9 ? 0x80000000u : (lane == 15 ? 32u * 9u : 0u)) + f.k16[lane];
#pragma unroll 1
        for (int i = 0; i < n; i++) {
            if ((lane & ~4) == 0) f.kw[lane >> 2] = make_uint4(st[0] + k[0], st[1] + k[1], st[2] + k[2], st[3] + k[3]);
            if (lane == 0) __hip_atomic_store(&f.go, (uint32_t)(i + 1), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            uint4 x[4];
#pragma unroll
            for (int q = 0; q < 4; q++) x[q] = f.kw[q];
            l.start(h, x[0].x);
#pragma unroll 1
            for (int p = 1; p < 4; p++) {
                l.rounds16(x, 0);
                uint32_t got;
                do {  // as in fs_hash_rounds
                    got = __hip_atomic_load(&f.ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int q = 0; q < 4; q++) x[q] = f.kw[4 * p + q];
                    asm volatile("" ::: "memory");
                } while (got < 3 * (uint32_t)i + (uint32_t)p);
                l.q += x[0].x & l.m;
            }
            l.rounds16(x, 0);
#pragma unroll
            for (int q = 0; q < 4; q++) st[q] = h[q] + l.v[q];
            if (lane == 0)
#pragma unroll
                for (int q = 0; q < 4; q++) raw[4 * i + q] = __builtin_bswap32(st[q]);
        }
        if (n > 0 && (lane & ~4) == 0)
#pragma unroll
            for (int q = 0; q < 4; q++) f.m[lane + q] = __builtin_bswap32(st[q]);
        if (lane == 0) f.ready = f.go = 0;
    }
}

// The block: a draw with its barriers.
__device__ inline void fs_draw(FsLds &f)
{
    __syncthreads();
    fs_hash(f);
    __syncthreads();
}

}  // namespace ra
