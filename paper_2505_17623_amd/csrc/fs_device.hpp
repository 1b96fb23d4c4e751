// fs_device.hpp -- the Fiat-Shamir transcript on the device, worked by one
// workgroup of at least 128 threads from LDS.  The transcript
// (sha::Transcript in device memory: S, the pending length, the pending
// bytes) is pulled into LDS laid out as the next draw's message, S ||
// LE32(|Q|) || Q, so that absorbing appends to it and drawing hashes it in
// place.  Everything absorbed is whole 32-bit words, so the message is worked
// by words throughout.
//
// A draw is a chain of SHA-256 compressions, each 64 dependent rounds, and
// one wave issues an instruction every four cycles whatever its lanes do, so
// the instructions of the chain are its time.  Wave 1 expands the message
// schedules (one block per lane, every block of the message at once) sixteen
// words ahead of wave 0, which only runs the rounds: 14 instructions each,
// the three-input logic on v_bitop3_b32.  All lanes of wave 0 carry the same
// values; the state is kept out of the scalar unit, which has no rotate.
// Against one thread working the message through a generic compression: a
// round's draw with its sums 14.1 -> 7.6 us, the header of a layer with 2^14
// outputs 88 -> 43 us (MI355X).
#pragma once
#include "sha256.hpp"

namespace ra {

constexpr int kFsMsgWords = 9 + sha::kFsPending / 4;        // S, |Q|, Q
constexpr int kFsMaxBlocks = (4 * kFsMsgWords + 9 + 63) / 64;
struct FsLds {
    uint32_t m[kFsMaxBlocks * 16];    // the message, room for its padding
    uint4 kw[kFsMaxBlocks * 16];      // schedule plus round constants, 64 words per block
    uint64_t out[2];                  // the last challenge drawn
    uint32_t ready;                   // quarters of the first schedules wave 1 has stored (0 between draws)
};

__device__ __forceinline__ uint32_t vgpr(uint32_t x)  // the value, kept in vector registers
{
    asm("" : "+v"(x));
    return x;
}

// The block: the transcript into f (visible after the caller's next barrier).
__device__ inline void fs_pull(FsLds &f, const sha::Transcript *g)
{
    const uint32_t *s = (const uint32_t *)g;
    for (int i = threadIdx.x; i < kFsMsgWords; i += blockDim.x) f.m[i] = s[i];
    if (threadIdx.x == 0) f.ready = 0;
}

// The block: f back into the transcript (after a barrier).
__device__ inline void fs_push(sha::Transcript *g, const FsLds &f)
{
    uint32_t *d = (uint32_t *)g;
    const int words = 9 + (int)(f.m[8] >> 2);
    for (int i = threadIdx.x; i < words; i += blockDim.x) d[i] = f.m[i];
}

// The block: append nw 32-bit words (readable by every thread).  Barriers on
// both sides; false: more than sha::kFsPending bytes pending.
__device__ inline bool fs_absorb(FsLds &f, const uint32_t *w, int nw)
{
    __syncthreads();
    const uint32_t q = f.m[8];
    const bool ok = q + 4 * (uint32_t)nw <= sha::kFsPending;
    if (ok)
        for (int i = threadIdx.x; i < nw; i += blockDim.x) f.m[9 + (q >> 2) + i] = w[i];
    __syncthreads();
    if (ok && threadIdx.x == 0) f.m[8] = q + 4 * (uint32_t)nw;
    __syncthreads();
    return ok;
}

// Sixteen rounds on the working variables, kw read as four vectors.
__device__ __forceinline__ void fs_rounds16(uint32_t (&v)[8], const uint4 *kw)
{
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint4 x = kw[q];
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

// The draw proper, by waves 0 and 1 between two barriers of the block (the
// message complete before the first; the other waves may do other work):
// S = H(S || LE32(|Q|) || Q), Q emptied, the challenge's two words to f.out.
// Wave 0 waits in LDS for each quarter of the first block's schedule; wave 1
// stores every quarter without waiting for anything.
__device__ inline void fs_hash(FsLds &f)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int words = 9 + (int)(f.m[8] >> 2), nblk = (4 * words + 9 + 63) / 64;
    auto publish = [&](uint32_t p) {  // LDS operations of a wave stay in order
        __hip_atomic_store(&f.ready, p, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto await = [&](uint32_t p) {
        while (__hip_atomic_load(&f.ready, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < p) {
        }
    };
    if (wave == 1 && lane < nblk) {  // the lanes without a block take no part: they would publish ahead of the others
        uint32_t w[16];
        uint4 *kw = f.kw + 16 * lane;
        // the padded message: 0x80 after its last word, its bit length at the end
#pragma unroll
        for (int t = 0; t < 16; t++) w[t] = f.m[16 * lane + t];  // m has room for the last block
#pragma unroll
        for (int t = 0; t < 16; t++) {
            const int g = 16 * lane + t;
            w[t] = g < words ? __builtin_bswap32(w[t]) : (g == words ? 0x80000000u : 0u);
        }
        if (lane == nblk - 1) w[15] = 32u * (uint32_t)words;
#pragma unroll
        for (int q = 0; q < 4; q++)
            kw[q] = make_uint4(w[4 * q] + sha::kConsts.k[4 * q], w[4 * q + 1] + sha::kConsts.k[4 * q + 1],
                               w[4 * q + 2] + sha::kConsts.k[4 * q + 2], w[4 * q + 3] + sha::kConsts.k[4 * q + 3]);
        publish(1);
        fs_schedule16<1>(w, kw);
        publish(2);
        fs_schedule16<2>(w, kw);
        publish(3);
        fs_schedule16<3>(w, kw);
        publish(4);
    } else if (wave == 0) {
        uint32_t v[8], st[8];
#pragma unroll
        for (int i = 0; i < 8; i++) st[i] = vgpr(sha::kConsts.h[i]);
#pragma unroll 1
        for (int b = 0; b < nblk; b++) {
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = st[i];
#pragma unroll 1
            for (int p = 0; p < 4; p++) {
                if (b == 0) await(p + 1);
                fs_rounds16(v, f.kw + 16 * b + 4 * p);
            }
#pragma unroll
            for (int i = 0; i < 8; i++) st[i] += v[i];
        }
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < 8; i++) f.m[i] = st[i] = __builtin_bswap32(st[i]);  // S as its bytes in order
            f.m[8] = 0;
            f.ready = 0;
            constexpr uint64_t p = 0x1FFFFFFFFFFFFFFFull;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const uint64_t x = (uint64_t)st[2 * q] | ((uint64_t)st[2 * q + 1] << 32);  // LE64 of S[8q .. 8q + 8]
                const uint64_t r = (x & p) + (x >> 61);                                     // x mod p (x < 2^64)
                f.out[q] = r >= p ? r - p : r;
            }
        }
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
