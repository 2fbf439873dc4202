// Device helpers and launch constants shared by the decode kernels (decode.hip, decode_rope.hip).
#pragma once
#include <type_traits>

#include "csr_internal.h"
#include "lane_ops.h"

namespace csr {
namespace dec {

using namespace lane;

// Threads of a workgroup of the position-free streaming kernel = tokens per round: 16 waves (enough loads in flight
// with one workgroup per CU) of 128 registers each.
constexpr int kStreamThreads = 1024;
constexpr int kMaxDevices = 64;      // devices a process may use this library on
// Rounds per chunk: a thread keeps the scores of its tokens (one per round and query head) in registers.  With four
// query heads per workgroup only 8 (32 of the 128 registers) ...
constexpr int max_rounds(int GB) { return GB == 4 ? 8 : 16; }
// ... which makes long contexts many short chunks, and every chunk costs a fixed 10 us (dispatch, table load, histogram
// clear and read-out, checks).  For those the four-head kernel has a second shape: 8 waves of 256 registers keep 32
// rounds - chunks of 16384 tokens, like the other variants' (measured at 8 sequences x 8 KV heads x 131072 tokens:
// 185 against 211 us per call).  Built for codes that are requested as a whole (NP > 0 below).
constexpr int kLongThreads4 = 512;
constexpr int kLongRounds4 = 32;
constexpr int kMaxChunks = 128;
// The rotary-key kernel (decode_rope.hip).  One query head at a time: 16 waves with 128 registers each; a query group
// keeps a rebuilt key and the group's scores in registers: 8 waves with 256 each.
constexpr int rope_threads(int GB) { return GB >= 2 ? 512 : 1024; }  // tokens per round
// rounds a chunk may have: one score per round and query head stays in registers
constexpr int rope_rounds(int GB) { return GB == 2 ? 16 : 8; }
// the rotary-key kernel keeps the key dictionary of its KV head in LDS when it fits (at most 512 atoms of 128 halves)
constexpr bool rope_dictionary_fits_lds(int N) { return (size_t)N * 256 <= 128 * 1024; }
// 32-bit words of a lane class's rotation constants: 5 x 16, and 4 that spread the 8 classes' 16-byte reads over the banks
constexpr int kRopeTurn = 84;
constexpr size_t kRopeTableBytes = 8 * kRopeTurn * 4 + 8 * 4 * 8 * 4 + 64 * 8;  // rotation constants, a group's query pairs, theta
// What of them counts against the LDS budget below: the largest dictionary that is taken does not depend on the tables' layout.
constexpr size_t kRopeTableCounted = 2560;
constexpr size_t kLdsBudget = 150 * 1024;
static_assert(kRopeTableBytes >= kRopeTableCounted && kLdsBudget + kRopeTableBytes - kRopeTableCounted <= 160 * 1024, "within a CU's LDS");
// Reduction scratch of the streaming kernels, in 4-byte words behind the table / histogram (WAVES <= 16, GB <= 4):
constexpr int kRedMax = 0;     // [WAVES][GB]  wave maxima of the scores
constexpr int kRedCm = 64;     // [WAVES]      wave maxima of the sampled |value coefficients|
constexpr int kRedL = 80;      // [WAVES][GB]  wave sums of p
constexpr int kRedChk = 144;   // [WAVES][12]  the scatter's self-check: see finish_chunk
constexpr int kRedWords = 144 + 16 * 12;
constexpr size_t kRedBytes = 2048;
static_assert(kRedWords * 4 <= kRedBytes, "reduction scratch");

__device__ __forceinline__ float h2f(__half v) { return __half2float(v); }

template <typename T> __device__ __forceinline__ void load8(const T *p, float (&o)[8]);
template <> __device__ __forceinline__ void load8<__half>(const __half *p, float (&o)[8])
{
    const uint4 raw = *reinterpret_cast<const uint4 *>(p);
    const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 f = __half22float2(h2[j]);
        o[2 * j] = f.x;
        o[2 * j + 1] = f.y;
    }
}
__device__ __forceinline__ void load8_raw(const uint4 &raw, float (&o)[8])   // 8 packed halves, already in registers
{
    const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 f = __half22float2(h2[j]);
        o[2 * j] = f.x;
        o[2 * j + 1] = f.y;
    }
}
template <> __device__ __forceinline__ void load8<float>(const float *p, float (&o)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    const float4 b = *reinterpret_cast<const float4 *>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
}

// ---------------------------------------------------------------------------------------------
// Code-stream loads: PV pairs of one token at a time, widened to int / float registers.
template <typename TI, int PV> struct IdxLoad;
template <> struct IdxLoad<uint16_t, 8> {
    static __device__ __forceinline__ void ld(const uint16_t *p, int (&o)[8]) {
        const uint4 r = *reinterpret_cast<const uint4 *>(p);
        o[0] = r.x & 0xffff; o[1] = r.x >> 16; o[2] = r.y & 0xffff; o[3] = r.y >> 16;
        o[4] = r.z & 0xffff; o[5] = r.z >> 16; o[6] = r.w & 0xffff; o[7] = r.w >> 16;
    }
};
template <> struct IdxLoad<uint16_t, 4> {
    static __device__ __forceinline__ void ld(const uint16_t *p, int (&o)[4]) {
        const uint2 r = *reinterpret_cast<const uint2 *>(p);
        o[0] = r.x & 0xffff; o[1] = r.x >> 16; o[2] = r.y & 0xffff; o[3] = r.y >> 16;
    }
};
template <> struct IdxLoad<uint16_t, 2> {
    static __device__ __forceinline__ void ld(const uint16_t *p, int (&o)[2]) {
        const uint32_t r = *reinterpret_cast<const uint32_t *>(p);
        o[0] = r & 0xffff; o[1] = r >> 16;
    }
};
template <> struct IdxLoad<uint16_t, 1> {
    static __device__ __forceinline__ void ld(const uint16_t *p, int (&o)[1]) { o[0] = p[0]; }
};
template <> struct IdxLoad<int32_t, 8> {
    static __device__ __forceinline__ void ld(const int32_t *p, int (&o)[8]) {
        const int4 a = *reinterpret_cast<const int4 *>(p);
        const int4 b = *reinterpret_cast<const int4 *>(p + 4);
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    }
};
template <> struct IdxLoad<int32_t, 4> {
    static __device__ __forceinline__ void ld(const int32_t *p, int (&o)[4]) {
        const int4 a = *reinterpret_cast<const int4 *>(p);
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    }
};
template <> struct IdxLoad<int32_t, 2> {
    static __device__ __forceinline__ void ld(const int32_t *p, int (&o)[2]) {
        const int2 a = *reinterpret_cast<const int2 *>(p);
        o[0] = a.x; o[1] = a.y;
    }
};
template <> struct IdxLoad<int32_t, 1> {
    static __device__ __forceinline__ void ld(const int32_t *p, int (&o)[1]) { o[0] = p[0]; }
};

template <typename TC, int PV> struct CoefLoad;
template <> struct CoefLoad<__half, 8> {
    static __device__ __forceinline__ void ld(const __half *p, float (&o)[8]) { load8<__half>(p, o); }
};
template <> struct CoefLoad<__half, 4> {
    static __device__ __forceinline__ void ld(const __half *p, float (&o)[4]) {
        const uint2 raw = *reinterpret_cast<const uint2 *>(p);
        const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
        const float2 f0 = __half22float2(h2[0]), f1 = __half22float2(h2[1]);
        o[0] = f0.x; o[1] = f0.y; o[2] = f1.x; o[3] = f1.y;
    }
};
template <> struct CoefLoad<__half, 2> {
    static __device__ __forceinline__ void ld(const __half *p, float (&o)[2]) {
        const float2 f = __half22float2(*reinterpret_cast<const __half2 *>(p));
        o[0] = f.x; o[1] = f.y;
    }
};
template <> struct CoefLoad<__half, 1> {
    static __device__ __forceinline__ void ld(const __half *p, float (&o)[1]) { o[0] = h2f(p[0]); }
};
template <> struct CoefLoad<float, 8> {
    static __device__ __forceinline__ void ld(const float *p, float (&o)[8]) { load8<float>(p, o); }
};
template <> struct CoefLoad<float, 4> {
    static __device__ __forceinline__ void ld(const float *p, float (&o)[4]) {
        const float4 a = *reinterpret_cast<const float4 *>(p);
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
    }
};
template <> struct CoefLoad<float, 2> {
    static __device__ __forceinline__ void ld(const float *p, float (&o)[2]) {
        const float2 a = *reinterpret_cast<const float2 *>(p);
        o[0] = a.x; o[1] = a.y;
    }
};
template <> struct CoefLoad<float, 1> {
    static __device__ __forceinline__ void ld(const float *p, float (&o)[1]) { o[0] = p[0]; }
};

// x as a 64-bit fixed-point number in units of 2^-32 (two's complement), rounded to the nearest unit; |x| must
// stay below 2^31 (the integer part is saturated there rather than wrapped).  fl = floor(x) and x - fl are exact in
// fp32, but x - fl can be exactly 1 (a tiny negative x), so the scaled fraction is kept below 2^32 before the
// conversion; adding one half only matters where the scaled fraction still has fraction bits (below 2^23).  The
// caller scales p * c by a power of two first (see stream_kernel), so that the unit follows the data and the
// result does not depend on the scale of the coefficients.
__device__ __forceinline__ unsigned long long to_fixed(float x)
{
    const float fl = floorf(fminf(fmaxf(x, -2147483648.0f), 2147483520.0f));
    const int hi = (int)fl;
    const unsigned lo = (unsigned)fminf((x - fl) * 4294967296.0f + 0.5f, 4294967040.0f);
    return ((unsigned long long)(unsigned)hi << 32) | lo;
}
__device__ __forceinline__ float from_fixed(unsigned long long v)
{
    return (float)(int)(unsigned)(v >> 32) + (float)(unsigned)(v & 0xffffffffull) * 2.3283064365386963e-10f;
}

// ---------------------------------------------------------------------------------------------
// The V side of a chunk, common to the streaming kernels (position-free and rotary keys): softmax weights of
// the chunk's tokens, the scatter of p * c of the value codes into the LDS histogram (D4), and the chunk's
// histogram (fp32), maximum and sum of weights to scratch.
//
// The histogram is fixed point, summed with integer LDS atomics: integer sums are exact, so the result does
// not depend on the order in which the hardware serves the adds, and the float atomic add of this LDS is
// serialised lane by lane.  Fast form: 32-bit adds (1.7 times the rate of 64-bit ones).  Every query head has
// bins [n][sign]: p >= 0, so the sign of an add is the sign of its coefficient, and with the magnitudes of the
// two signs kept apart every bin only grows - an overflow (a wrap, or a bin beyond 2^31) cannot cancel and is
// found exactly: the bins' total is compared with the total the threads add up themselves (in fp32, to 2^-17
// relative: a wrap is off by 2^32), and every bin is looked at when it is read out.  The unit is a power of two
// per query head chosen BEFORE the scatter from what is known then - the sum l of the weights and the largest
// |coefficient| among the chunk's first tokens: 2^-28 .. 2^-27 of c_est * max(1, l s / N) (the |p c| an average bin
// would collect if every coefficient were the largest sampled one), which leaves 8- to 16-fold headroom over that.
// After the scatter two things are checked:
//   * no overflow (above);
//   * resolution: the rounding of the n adds to the unit (each within half a unit, signs random) perturbs the
//     histogram by about unit * sqrt(n / 12) in the 2-norm; that must stay below 2^-15 of the histogram's own
//     2-norm (taken at the read-out): 3e-5, a thirtieth of the tolerance of the whole call.
// If either fails - coefficients far larger than the sampled ones, a hot atom hit by most tokens, weights and
// coefficients spanning more than the 32 bits can hold - the scatter is repeated ONCE in the wide form: 64-bit
// bins [n] in units of 2^-62 .. 2^-61 of the total |p c| just measured, which can neither overflow nor lose
// anything an fp32 product carries.  The decision depends on exact sums and on fp32 sums formed in a fixed
// order, so it is the same on every run, and so are the output bits.
//
// sc[i][g]: score of the token this thread owns in round i (token t0 + i * THREADS + owner_off), -inf if none.
// NP > 0: a token's value code has NP pairs in all its chunks together; its NP indices and NP coefficients are then
// requested as a whole, PF steps ahead of their use.  What bounds the scatter and the scores is how many bytes of codes are
// under way: loaded where they are used, 268 MB of codes took (8 sequences x 8 KV heads x 4 query heads, 4096 atoms)
// 151 us with 4 pairs, 177 with 6, 299 with 2 x 2 and 96 with 16; requested ahead 120, 121, 164 and 83.
template <typename TI, typename TC, int NP> struct CodeVec {
    static_assert(NP == 0 || (sizeof(TI) == sizeof(TC) && NP * sizeof(TI) % 4 == 0), "whole 32-bit words, as many of each");
    static constexpr int W = NP > 0 ? NP * (int)sizeof(TI) / 4 : 1;   // 32-bit words of the indices and of the coefficients
    // Held and requested as 16-byte vectors, indices and coefficients in turn (word by word, all indices first, the same
    // requests take 0.5 % longer: 4 x 32 heads x 32768 tokens, 16 pairs on 8192 atoms 135.7 against 135.2 us)
    static constexpr bool kQuads = W % 4 == 0 && sizeof(TI) == 2;
    typename std::conditional<kQuads, uint4, uint32_t>::type i[kQuads ? W / 4 : W], c[kQuads ? W / 4 : W];
};
// Steps whose codes are requested ahead, as far as the registers go without spilling: 8 words with one query head per
// workgroup (what bounds that kernel is the number of bytes in flight per CU), else 4, at least one step.
template <int GB, int TPT, int W> constexpr int prefetch_steps()
{
    constexpr int words = GB == 1 && TPT >= 4 ? 8 : 4;
    return words >= W ? words / W : 1;
}
// pairs worked on at a time
template <int NP> constexpr int pair_block() { return NP % 8 == 0 ? 8 : NP; }
// Pairs requested at a time: the whole code, or with four query heads per workgroup half of a code of 16 (the scores
// leave no registers for two whole ones).  With two heads whole ones cost 3 spilled registers and are worth it: 4 sequences x
// 16 KV heads x 2 query heads, 32768 tokens, 4096 atoms 72.5 us against 75.9 in halves.  A "step" is one such piece of one token.
template <int GB, int NP> constexpr int pair_piece() { return GB > 2 && NP > 8 ? 8 : NP; }

// The code streams of a thread's tokens, walked round by round: two workgroup-uniform base addresses (the codes of the
// chunk's first token) and one 32-bit offset per thread, in bytes or 16-byte vectors.  The offset passes
// through an empty asm statement at every step, so that the compiler cannot work out all rounds' addresses ahead of
// time (they would occupy registers from the start of the loop).
template <typename TI, typename TC, int NP, int PIECE, int THREADS> struct CodeWalk {
    static constexpr uint32_t kUnit = CodeVec<TI, TC, PIECE>::kQuads ? 16 : 1;   // bytes the offset counts in
    const unsigned char *ib, *cb;   // uniform
    uint32_t off;                   // the piece of this thread's token at which the walk stands
    __device__ __forceinline__ CodeWalk(const TI *idx, const TC *coef, int64_t first_token, int owner_off)
        : ib(reinterpret_cast<const unsigned char *>(idx + first_token * NP)),
          cb(reinterpret_cast<const unsigned char *>(coef + first_token * NP)), off((uint32_t)owner_off * (NP * (uint32_t)sizeof(TI) / kUnit)) {}
    // `step`: the step at which the walk stands
    __device__ __forceinline__ void next(int step)
    {
        constexpr int P = PIECE > 0 ? NP / PIECE : 1;
        off += (step % P == P - 1 ? THREADS * NP - (P - 1) * PIECE : PIECE) * (uint32_t)sizeof(TI) / kUnit;
        asm volatile("" : "+v"(off));
    }
};
typedef uint32_t word3 __attribute__((ext_vector_type(3), aligned(4)));   // 12 bytes at any word
template <int W> __device__ __forceinline__ void load_words(const unsigned char *p, uint32_t (&o)[W])
{
    if constexpr (W == 3) {
        const word3 r = *reinterpret_cast<const word3 *>(p);
        o[0] = r.x; o[1] = r.y; o[2] = r.z;
    } else if constexpr (W % 4 == 0) {
#pragma unroll
        for (int k = 0; k < W; k += 4) {
            const uint4 r = *reinterpret_cast<const uint4 *>(p + 4 * k);
            o[k] = r.x; o[k + 1] = r.y; o[k + 2] = r.z; o[k + 3] = r.w;
        }
    } else if constexpr (W % 2 == 0) {
#pragma unroll
        for (int k = 0; k < W; k += 2) {
            const uint2 r = *reinterpret_cast<const uint2 *>(p + 4 * k);
            o[k] = r.x; o[k + 1] = r.y;
        }
    } else {
#pragma unroll
        for (int k = 0; k < W; ++k) o[k] = reinterpret_cast<const uint32_t *>(p)[k];
    }
}
// Requests the piece of a code at which the walk stands.  Without such a token (`have` false: past the
// end of the chunk) the chunk's first token is requested instead and the caller ignores what arrives: a request
// under a branch would make the destination registers the meeting point of two paths, and the compiler then copies
// them - and waits for the request - right behind it.
// PAST: non-temporal (see launch_stream_t).
template <bool PAST, typename TI, typename TC, int NP, int PIECE, int THREADS>
__device__ __forceinline__ void fetch_codes(CodeVec<TI, TC, PIECE> &r, const CodeWalk<TI, TC, NP, PIECE, THREADS> &w, bool have)
{
    static_assert(!PAST || CodeVec<TI, TC, PIECE>::kQuads, "only 16-byte vectors are requested non-temporally");
    const uint32_t o = have ? w.off : 0u;
    if constexpr (CodeVec<TI, TC, PIECE>::kQuads) {
#pragma unroll
        for (int v = 0; v < CodeVec<TI, TC, PIECE>::W / 4; ++v) {
            if constexpr (PAST) {
                typedef uint32_t word4 __attribute__((ext_vector_type(4)));
                r.i[v] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const word4 *>(w.ib) + (o + v)));
                r.c[v] = __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const word4 *>(w.cb) + (o + v)));
            } else {
                r.i[v] = reinterpret_cast<const uint4 *>(w.ib)[o + v];
                r.c[v] = reinterpret_cast<const uint4 *>(w.cb)[o + v];
            }
        }
    } else {
        load_words(w.ib + o, r.i);
        load_words(w.cb + o, r.c);
    }
}
// The codes of the current step must have arrived BEFORE a later round's request is issued: the empty asm
// statements make the compiler place the wait for them here, where only older requests are outstanding, instead of
// behind the new request, where it would wait for both.
template <typename TI, typename TC, int NP>
__device__ __forceinline__ void await_codes(CodeVec<TI, TC, NP> &cur)
{
    constexpr int W = CodeVec<TI, TC, NP>::W;
    if constexpr (CodeVec<TI, TC, NP>::kQuads) {   // a request at a time
#pragma unroll
        for (int v = 0; v < W / 4; ++v) {
            asm volatile("" : "+v"(cur.i[v].x), "+v"(cur.i[v].y), "+v"(cur.i[v].z), "+v"(cur.i[v].w));
            asm volatile("" : "+v"(cur.c[v].x), "+v"(cur.c[v].y), "+v"(cur.c[v].z), "+v"(cur.c[v].w));
        }
    } else {
#pragma unroll
        for (int k = 0; k < W; ++k) asm volatile("" : "+v"(cur.i[k]), "+v"(cur.c[k]));
    }
}
// pairs B * j0 .. of a code, B = pair_block
template <typename TI, typename TC, int NP, int B>
__device__ __forceinline__ void unpack_codes(const CodeVec<TI, TC, NP> &r, int j0, int (&id)[B], float (&cf)[B])
{
    if constexpr (CodeVec<TI, TC, NP>::kQuads) {
        const uint4 &ri = r.i[j0 / 8], &rc = r.c[j0 / 8];
        id[0] = ri.x & 0xffff; id[1] = ri.x >> 16; id[2] = ri.y & 0xffff; id[3] = ri.y >> 16;
        id[4] = ri.z & 0xffff; id[5] = ri.z >> 16; id[6] = ri.w & 0xffff; id[7] = ri.w >> 16;
        load8_raw(rc, cf);
    } else if constexpr (sizeof(TI) == 2) {
#pragma unroll
        for (int j = 0; j < B; j += 2) {
            const uint32_t wi = r.i[(j0 + j) / 2], wc = r.c[(j0 + j) / 2];
            id[j] = wi & 0xffff; id[j + 1] = wi >> 16;
            const float2 f = __half22float2(*reinterpret_cast<const __half2 *>(&wc));
            cf[j] = f.x; cf[j + 1] = f.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < B; ++j) { id[j] = (int)r.i[j0 + j]; cf[j] = __uint_as_float(r.c[j0 + j]); }
    }
}
// The table (or histogram) entry at which the chunk of pair j of a token starts, s pairs and n entries per chunk.  Scalars.
template <bool CH, int NP> struct ChunkBase {
    int at[CH && NP > 0 ? NP : 1];
    __device__ __forceinline__ ChunkBase(int s, int n)
    {
        if constexpr (CH && NP > 0) {
            int base = 0, left = s;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                at[j] = base;
                if (--left == 0) { base += n; left = s; }
            }
        }
    }
    template <int B> __device__ __forceinline__ void shift(int j0, int (&id)[B]) const
    {
        if constexpr (CH && NP > 0) {
#pragma unroll
            for (int j = 0; j < B; ++j) id[j] += at[j0 + j];
        }
    }
};

// A thread keeps one value per round and query head in registers, sc[round][head]: the loops over the rounds are
// fully unrolled (registers cannot be indexed by a loop counter).  Left alone, the compiler then pulls the loads and
// address arithmetic of all rounds ahead until it spills; round_fence() between two rounds keeps memory accesses on
// their side of it, so that only the explicitly requested vectors (fetch_codes) are in flight.
__device__ __forceinline__ void round_fence() { asm volatile("" ::: "memory"); }

// Long chunks (this many tokens or more), several per sequence, are cut anew where lengths are given: see chunk_of.
constexpr int kCutFromStream = 12288, kCutFromRope = 4096;
inline bool cut_by_lengths(const int32_t *seq_lens, int nchunks, int B, int64_t chunk_tokens, int from)
{
    return seq_lens && nchunks > 1 && B <= 64 && chunk_tokens >= from;
}

template <int CTRL, int ROWS> __device__ __forceinline__ int scan_step(int v) { return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
// sum of v over the lanes up to this one
__device__ __forceinline__ int wave_scan(int v)
{
    v = scan_step<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: sums within the rows of 16 lanes
    v = scan_step<0x112, 0xf>(v);
    v = scan_step<0x114, 0xf>(v);
    v = scan_step<0x118, 0xf>(v);
    v = scan_step<0x142, 0xa>(v);   // row_bcast 15: rows 0 and 2 to rows 1 and 3
    return scan_step<0x143, 0xc>(v);   // row_bcast 31: the first half to the second
}

// A workgroup's part of the work: tokens [t0, t_end) of sequence b, its chunk c (of slots 0 .. nchunks - 1; one without tokens has
// t_end <= t0).  The grid is (heads, nchunks, B): KV heads x group slices first.
struct Chunk {
    int b, c;
    int64_t t0, t_end;
};
// The plan's chunks are cut for sequences that fill the buffer.  Where lengths are given, long chunks (CUT_FROM tokens or more,
// several of them per sequence) are cut anew, every sequence by its own length and evenly, and the workgroups are numbered
// so that those without tokens come last: one that ends at once in the middle of the numbers gives one shader engine a
// workgroup more than it has CUs, and another one less.  A workgroup costs about kFixedRounds rounds besides its own, so a
// sequence gets as few chunks as the plan's size allows, or more (at most the plan's number) where the whole launch then
// makes cheaper generations of 256 workgroups, one per CU.  All of it follows from the lengths alone - of all sequences: the low bits
// of one's output depend on the others' - and every wave works it out for itself, in about a microsecond: shorter chunks, one chunk per
// sequence and more than 64 sequences keep the plan's.  CUT_FROM = 0: all calls do, and the kernel is the one without any of this.
// 8 sequences of 73728 to 131072 tokens, 8 KV heads x 4 query heads 146 us with the plan's chunks, 134 longest first, 136 to 143 in other
// orders; 20 sequences of 15000 to 30000, 4 x 8 heads 134 and 113; 50 random batches of 2 to 64 sequences 0.83 of the time, the worst 1.03.
// The lines, by the time with the cut over the time without (9 random batches each): chunks of up to 4096 tokens 0.99, 8192 0.92, 12288
// 0.97, 16384 0.82; rotary keys of up to 1024 0.95, 2048 0.92, 3072 0.90.  So a lower line would pay, too, with more variants of
// the kernels.  0.92: with 1.0 the same (stream), 5 % either way (rotary keys).  Tried: longest first in every batch, and prices by
// the chunks as they come out; what every workgroup pays for that is more than it brings (64 sequences 91 -> 112 us).
template <int THREADS, int CUT_FROM>
__device__ __forceinline__ Chunk chunk_of(const int32_t *__restrict__ seq_lens, int64_t T, int nchunks, int64_t chunk_tokens)
{
    if constexpr (CUT_FROM == 0) {
        const int c = blockIdx.y, b = blockIdx.z;
        int64_t len = T;
        if (seq_lens) {
            const int32_t l = seq_lens[b];
            len = l < 0 ? 0 : (l > T ? T : l);
        }
        const int64_t t0 = (int64_t)c * chunk_tokens;
        return {b, c, t0, min(t0 + chunk_tokens, len)};
    }
    constexpr float kFixedRounds = 7.0f;
    const int B = gridDim.z, heads = gridDim.x, lane = threadIdx.x & 63;
    if (__builtin_expect(!seq_lens || nchunks == 1 || B > 64 || chunk_tokens < CUT_FROM, 1)) {
        int64_t len = T;
        if (seq_lens) {
            const int32_t l = seq_lens[blockIdx.z];
            len = l < 0 ? 0 : (l > T ? T : l);
        }
        const int64_t t0 = (int64_t)blockIdx.y * chunk_tokens;
        return {(int)blockIdx.z, (int)blockIdx.y, t0, min(t0 + chunk_tokens, len)};
    }
    const int most = (int)(chunk_tokens / THREADS);   // rounds per chunk of the plan
    // lane i: sequence i (T is at most 2^20)
    const int l = lane < B ? seq_lens[lane] : 0;
    const int len = l < 0 ? 0 : (l > (int)T ? (int)T : l), R = (len + THREADS - 1) / THREADS;
    // chunks of R rounds at r rounds a chunk: ceil(R / r); the quotient is at least 1 / (2 r) away from a whole number
    auto chunks = [&](float r) { return min(nchunks, (int)(((float)R + r - 0.5f) * (1.0f / r))); };
    const float sum = wave_sum((float)R) * (float)heads, g = ceilf(sum / (256.0f * (float)most));
    float r = (float)most, best = INFINITY;
#pragma unroll
    for (int k = 0; k < 3; ++k) {   // the plan's size; what fills g and g + 1 generations, half a chunk lost per sequence
        const float room = 256.0f * (g + (float)(k - 1)) - 0.5f * (float)(B * heads);
        const float rk = k == 0 || !(room > 0.0f) ? (float)most : fminf((float)most, fmaxf(1.0f, ceilf(sum / room)));
        const float groups = wave_sum((float)chunks(rk)) * (float)heads;
        const float cost = ceilf(groups * (1.0f / 256.0f)) * (rk + kFixedRounds);
        if (k == 0 || cost < 0.92f * best) { best = cost; r = rk; }
    }
    // workgroup j of a head: the j-th of all sequences' chunks, or, behind the last, the (j - all)-th empty slot
    const int n = lane < B ? chunks(r) : 0;
    int upto = n;
    if constexpr (CUT_FROM == kCutFromRope) {   // with the shorter form the rotary kernel's loop comes out 1 - 3 % slower (one head, 8 pairs)
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int o = __shfl_up(upto, m, 64);
            if (lane >= m) upto += o;
        }
    } else {
        upto = wave_scan(n);
    }
    const int j = (int)(blockIdx.y + nchunks * blockIdx.z), all = __builtin_amdgcn_readlane(upto, 63);
    const bool empty = j >= all;
    // empty slots up to a lane's sequence: nchunks per sequence less its chunks
    const int past_of = empty ? all + nchunks * (lane + 1) - upto : upto, mine = empty ? nchunks - n : n;
    const unsigned long long past = __ballot(lane < B && j < past_of);
    const int at = past ? __ffsll((long long)past) - 1 : 0;   // never none: chunks and empty slots are as many as the grid's workgroups
    const int before = __builtin_amdgcn_readlane(past_of - mine, at), n_at = __builtin_amdgcn_readlane(n, at);
    if (empty) return {at, n_at + j - before, 0, 0};
    const int own = (__builtin_amdgcn_readlane(R, at) + n_at - 1) / n_at * THREADS, t0 = (j - before) * own;
    return {at, j - before, t0, min(t0 + own, __builtin_amdgcn_readlane(len, at))};
}

template <int GB, typename TI, typename TC, int PV, bool CH, int TPT, int THREADS, int NP, bool PAST = false>
__device__ __forceinline__ void finish_chunk(unsigned char *smem_raw, float *red, float (&sc)[TPT][GB], const float (&mx)[GB],
                                             int n_mine, int64_t t0, int64_t t_end, int64_t code_row, int owner_off,
                                             const TI *__restrict__ idxV, const TC *__restrict__ coefV, int32_t N,
                                             int32_t sV, int32_t snV_arg, float *ml, float *part_hist, int64_t slot)
{
    constexpr int WAVES = THREADS / 64;
    static_assert(WAVES <= 16 && GB <= 4, "layout of the reduction scratch");
    static_assert(NP == 0 || PV == pair_block<NP>(), "pairs worked on at a time");
    const int snV = CH ? snV_arg : 1;
    // 32-bit form: |sum| of c > 0 and of c < 0 per (query head, atom).  [g][n][sign]; for an even number of heads
    // [g / 2][n][sign][g % 2]: the bins of two heads side by side, so that ONE 64-bit add serves both (a loop of 16
    // ds_add_u64 takes 8 % less LDS time than one of 32 ds_add_u32, and the second head needs no address).  A bin that
    // wraps then carries into its neighbour's - which the check of the totals finds like any other wrap (the sum of
    // all bins is off by 2^32 - 1).
    constexpr bool PAIRED = GB % 2 == 0;
    uint32_t *h32 = reinterpret_cast<uint32_t *>(smem_raw);
    unsigned long long *h64 = reinterpret_cast<unsigned long long *>(smem_raw);  // wide form: [GB][NV]
    uint32_t *redw = reinterpret_cast<uint32_t *>(red);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int NV = snV * N, sVt = snV * sV;
    const int bins = NV * GB;
    const int64_t tok0 = t0 + owner_off;  // this thread's token of round 0

    // ---- the chunk's maximum; a sample of the value coefficients (the first round's tokens) ---------------
    float cm = 0.0f;
    constexpr int PIECE = pair_piece<GB, NP>(), STEPS = NP > 0 ? NP / PIECE : 1;   // steps per round
    constexpr int PF = prefetch_steps<GB, TPT, CodeVec<TI, TC, PIECE>::W>();
    CodeVec<TI, TC, PIECE> ring[PF + 1];  // step i reads slot i % (PF + 1) while step i + PF is requested into the slot step i - 1 left
    auto prime = [&](CodeWalk<TI, TC, NP, PIECE, THREADS> &w) {   // requests steps 0 .. PF-1, leaves w at step PF
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            fetch_codes<PAST>(ring[k], w, k / STEPS < n_mine && tok0 + (int64_t)(k / STEPS) * THREADS < t_end);
            w.next(k);
        }
    };
    static_assert(STEPS <= 2 && (STEPS == 1 || PF == 1), "the sample below takes the coefficients of the steps that prime left out");
    uint32_t other[STEPS > 1 ? CodeVec<TI, TC, PIECE>::W : 1];   // the second half's coefficients of the first round's token
    if constexpr (NP > 0) {
        CodeWalk<TI, TC, NP, PIECE, THREADS> w0(idxV, coefV, code_row + t0, owner_off);
        prime(w0);
        if constexpr (STEPS > 1) load_words(w0.cb + (n_mine > 0 && tok0 < t_end ? w0.off * w0.kUnit : 0u), other);
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        const float wm = wave_max(mx[g]);
        if (lane == 0) red[kRedMax + wave * GB + g] = wm;
    }
    if constexpr (NP > 0) {
#pragma unroll
        for (int j0 = 0; j0 < PIECE; j0 += PV) {
            int id[PV];
            float cf[PV];
            unpack_codes(ring[0], j0, id, cf);
            if (n_mine > 0 && tok0 < t_end) {   // else the vectors are not this thread's
#pragma unroll
                for (int j = 0; j < PV; ++j) cm = fmaxf(cm, fabsf(cf[j]));
                if constexpr (STEPS > 1) {
#pragma unroll
                    for (int j = 0; j < PV; j += 2) {
                        const float2 f = __half22float2(*reinterpret_cast<const __half2 *>(&other[(j0 + j) / 2]));
                        cm = fmaxf(cm, fmaxf(fabsf(f.x), fabsf(f.y)));
                    }
                }
            }
        }
    } else {
        if (n_mine > 0 && tok0 < t_end) {
            const TC *vp = coefV + (code_row + tok0) * sVt;
            for (int j0 = 0; j0 < sVt; j0 += PV) {
                float cf[PV];
                CoefLoad<TC, PV>::ld(vp + j0, cf);
#pragma unroll
                for (int j = 0; j < PV; ++j) cm = fmaxf(cm, fabsf(cf[j]));
            }
        }
    }
    cm = wave_max(cm);
    if (lane == 0) red[kRedCm + wave] = cm;
    __syncthreads();  // every score is computed: the table (or the dictionary rows) is free
    // the waves' partial results meet: lane l takes wave l % WAVES's, a reduction inside rows of WAVES lanes follows
    const int wsel = lane & (WAVES - 1);
    float m_c[GB];
#pragma unroll
    for (int g = 0; g < GB; ++g) m_c[g] = row_reduce<WAVES>(red[kRedMax + wsel * GB + g], OpMax());
    const float c_est = row_reduce<WAVES>(red[kRedCm + wsel], OpMax());

    // ---- p = exp(score - max) in place of the scores, their sum; the histogram cleared -------------------
    float l_thr[GB];
#pragma unroll
    for (int g = 0; g < GB; ++g) l_thr[g] = 0.0f;
#pragma unroll
    for (int i = 0; i < TPT; ++i) {
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            const float p = (i < n_mine && sc[i][g] > -INFINITY) ? __expf(sc[i][g] - m_c[g]) : 0.0f;
            sc[i][g] = p;
            l_thr[g] += p;
        }
    }
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        const float ws = wave_sum(l_thr[g]);
        if (lane == 0) red[kRedL + wave * GB + g] = ws;
    }
    {
        uint4 *z = reinterpret_cast<uint4 *>(smem_raw);
        const int n16 = (bins * 8 + 15) / 16;  // the table region is a multiple of 16 bytes
        for (int e = tid; e < n16; e += THREADS) z[e] = make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    int k_exp[GB];   // p is scattered as p * 2^k_exp
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        const float l = row_reduce<WAVES>(red[kRedL + wsel * GB + g], OpAdd());
        if (tid == g) { ml[2 * g] = m_c[g]; ml[2 * g + 1] = l; }
        const float b_est = c_est * fmaxf(1.0f, l * (float)sVt / (float)NV);
        k_exp[g] = 20;  // nothing sampled (or nothing finite): any unit will do, the checks below decide
        if (b_est > 0.0f && b_est < INFINITY) {
            int e2;
            (void)frexpf(b_est, &e2);  // b_est in [2^(e2-1), 2^e2)
            k_exp[g] = 28 - e2;        // b_est * 2^k in [2^27, 2^28)
        }
    }

    // ---- scatter ----------------------------------------------------------------------------------------
    float *dst = part_hist + slot * (int64_t)bins;
    const ChunkBase<CH, NP> chunk_base(sV, N);
    const float n_adds = (float)(t_end - t0) * (float)sVt;
    bool wide = false;
#pragma unroll 1
    for (int attempt = 0; attempt < 2; ++attempt) {
        float scale[GB];
#pragma unroll
        for (int g = 0; g < GB; ++g) scale[g] = ldexpf(1.0f, k_exp[g]);
        float s_thr = 0.0f, m_thr = 0.0f;  // sum and maximum of p' * sum_j |c_j| over this thread's tokens and heads
        CodeWalk<TI, TC, NP, PIECE, THREADS> walk(idxV, coefV, code_row + t0, owner_off);  // walks PF steps ahead of the current one
        if constexpr (NP > 0) {
            if (attempt > 0) prime(walk);
            else {
#pragma unroll
                for (int k = 0; k < PF; ++k) walk.next(k);
            }
        }
        // (inlined by order: unrolled as a function of its own, its body would be too large for the compiler to inline, and the
        // scores it is handed would live in scratch memory)
        auto rounds = [&](auto wide_c) __attribute__((always_inline)) {
            constexpr bool WIDE = decltype(wide_c)::value;
#pragma unroll
            for (int i = 0; i < TPT; ++i) {
                if (i < n_mine) {
                    round_fence();
                    const int64_t t = tok0 + (int64_t)i * THREADS;
                    float pp[GB];
#pragma unroll
                    for (int g = 0; g < GB; ++g) pp[g] = sc[i][g] * scale[g];
                    float a_t = 0.0f;
                    auto pairs = [&](int base, const int (&id)[PV], const float (&cf)[PV]) {
#pragma unroll
                        for (int j = 0; j < PV; ++j) {
                            const float ac = fabsf(cf[j]);
                            a_t += ac;
                            if constexpr (WIDE) {
#pragma unroll
                                for (int g = 0; g < GB; ++g) atomicAdd(&h64[g * NV + base + id[j]], to_fixed(pp[g] * cf[j]));
                            } else {
                                const int cell = 2 * (base + id[j]) + (int)(__float_as_uint(cf[j]) >> 31);
                                if constexpr (PAIRED) {
#pragma unroll
                                    for (int g = 0; g < GB; g += 2) {
                                        const uint32_t a0 = __float2uint_rz(fmaf(pp[g], ac, 0.5f));
                                        const uint32_t a1 = __float2uint_rz(fmaf(pp[g + 1], ac, 0.5f));
                                        atomicAdd(h64 + cell + g * NV, ((unsigned long long)a1 << 32) | a0);
                                    }
                                } else {
#pragma unroll
                                    for (int g = 0; g < GB; ++g)
                                        atomicAdd(h32 + cell + 2 * g * NV, __float2uint_rz(fmaf(pp[g], ac, 0.5f)));
                                }
                            }
                            // one pair after the other (the next pair's products depend on this statement), so
                            // that the values of all 8 x GB adds are not computed ahead and held in registers
#pragma unroll
                            for (int g = 0; g < GB; ++g) asm volatile("" : "+v"(pp[g]));
                        }
                    };
                    auto totals = [&]() {
#pragma unroll
                        for (int g = 0; g < GB; ++g) {
                            const float pa = pp[g] * a_t;
                            s_thr += pa;
                            m_thr = fmaxf(m_thr, pa);
                        }
                    };
                    if constexpr (NP > 0) {
#pragma unroll
                        for (int st = i * STEPS; st < (i + 1) * STEPS; ++st) {
                            // the codes of this step are awaited; behind them step st + PF is requested
                            CodeVec<TI, TC, PIECE> &cur = ring[st % (PF + 1)];
                            await_codes(cur);
                            const int nx = st + PF;
                            if (nx < TPT * STEPS) {
                                fetch_codes<PAST>(ring[nx % (PF + 1)], walk, nx / STEPS < n_mine && tok0 + (int64_t)(nx / STEPS) * THREADS < t_end);
                                walk.next(nx);
                            }
                            if (t < t_end) {
#pragma unroll
                                for (int j0 = 0; j0 < PIECE; j0 += PV) {
                                    int id[PV];
                                    float cf[PV];
                                    unpack_codes(cur, j0, id, cf);
                                    chunk_base.shift((st % STEPS) * PIECE + j0, id);
                                    pairs(0, id, cf);
                                }
                                if (st == (i + 1) * STEPS - 1) totals();
                            }
                        }
                    } else if (t < t_end) {
                        const TI *ip = idxV + (code_row + t) * sVt;
                        const TC *cp = coefV + (code_row + t) * sVt;
                        int base = 0;
                        for (int ch = 0; ch < snV; ++ch, base += N, ip += sV, cp += sV) {
                            for (int j0 = 0; j0 < sV; j0 += PV) {  // PV divides sV: a vector load stays in its chunk
                                int id[PV];
                                float cf[PV];
                                IdxLoad<TI, PV>::ld(ip + j0, id);
                                CoefLoad<TC, PV>::ld(cp + j0, cf);
                                pairs(base, id, cf);
                            }
                        }
                        totals();
                    }
                }
            }
        };
        if (wide) rounds(std::true_type{});
        else rounds(std::false_type{});
        __syncthreads();  // all atomics landed

        // ---- read-out: histogram to scratch as fp32; the checks' sums on the way ------------------------
        if (wide) {
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                const float from_units = ldexpf(1.0f, -k_exp[g]);
                for (int e = tid; e < NV; e += THREADS) dst[g * NV + e] = from_fixed(h64[g * NV + e]) * from_units;
            }
            break;
        }
        unsigned long long tot = 0ull;  // this thread's bins added up
        uint32_t high = 0u;             // OR of this thread's bins
        float h2[GB];                   // squares of this thread's histogram entries, per query head
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            h2[g] = 0.0f;
            const float from_units = ldexpf(1.0f, -k_exp[g]);
            constexpr int U = 4;   // bins read together: the LDS round trips of a thread overlap
            for (int e0 = tid; e0 < NV; e0 += U * THREADS) {
                uint2 pn[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {   // past the end: bin 0, ignored below (no load under a branch)
                    const int e = e0 + u * THREADS;
                    const int ec = e < NV ? e : 0;
                    if constexpr (PAIRED) {
                        const uint32_t *c2 = h32 + 4 * ((g >> 1) * NV + ec) + (g & 1);
                        pn[u] = make_uint2(c2[0], c2[2]);
                    } else {
                        pn[u] = *reinterpret_cast<const uint2 *>(h32 + 2 * (g * NV + ec));
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = e0 + u * THREADS;
                    if (e < NV) {
                        tot += (unsigned long long)pn[u].x + pn[u].y;
                        high |= pn[u].x | pn[u].y;
                        const float v = (float)(int)(pn[u].x - pn[u].y);  // exact while both stay below 2^31
                        h2[g] = fmaf(v, v, h2[g]);
                        // Of several heads non-temporal: the next launch reads it on other XCDs, and what is dirty in an L2 at the end is
                        // written back before that starts (8 sequences x 8 KV heads x 4 query heads, 8192 tokens: a step 84.2 -> 82.7 us; one query
                        // head 0 to 1.7 % slower)
                        if constexpr (GB > 1) __builtin_nontemporal_store(v * from_units, dst + g * NV + e);
                        else dst[g * NV + e] = v * from_units;
                    }
                }
            }
        }
        // per wave: s - tot (as integers: the sums are exact from here on), max single add, high bits, |hist|^2
        unsigned long long dif = wave_reduce((unsigned long long)fminf(s_thr, 1.0e19f) - tot, OpAdd());
        high = wave_reduce(high, OpOr());
        m_thr = wave_max(m_thr);
        const float s_wave = wave_sum(fminf(s_thr, 1.0e19f));
#pragma unroll
        for (int g = 0; g < GB; ++g) h2[g] = wave_sum(h2[g]);
        if (lane == 0) {
            uint32_t *c = redw + kRedChk + wave * 12;
            c[0] = (uint32_t)dif; c[1] = (uint32_t)(dif >> 32);
            c[2] = __float_as_uint(s_wave);
            c[4] = __float_as_uint(m_thr); c[5] = high;
#pragma unroll
            for (int g = 0; g < GB; ++g) c[6 + g] = __float_as_uint(h2[g]);
        }
        __syncthreads();
        const uint32_t *c = redw + kRedChk + wsel * 12;
        const unsigned long long DIF = row_reduce<WAVES>(((unsigned long long)c[1] << 32) | c[0], OpAdd());
        const float M = row_reduce<WAVES>(__uint_as_float(c[4]), OpMax());
        const float S_f = row_reduce<WAVES>(__uint_as_float(c[2]), OpAdd());
        const uint32_t HIGH = row_reduce<WAVES>(c[5], OpOr());
        float H2[GB];
#pragma unroll
        for (int g = 0; g < GB; ++g) H2[g] = row_reduce<WAVES>(__uint_as_float(c[6 + g]), OpAdd());
        const long long diff = (long long)DIF;
        bool ok = HIGH < 0x80000000u && M < 2147483648.0f && diff < 2147483648ll && diff > -2147483648ll;
        // resolution: unit * sqrt(n / 12) against 2^-15 |hist|, both in units (an all-zero histogram passes)
#pragma unroll
        for (int g = 0; g < GB; ++g) ok = ok && (n_adds * (1.0f / 12.0f) * 1073741824.0f <= H2[g] || M == 0.0f);
        if (ok) break;
        // wide form: the integer part of an add counts 2^32 units; all adds of a head together stay below 2^30 of
        // them.  S is the total over the heads in units of 2^-k_exp (as a float it may have saturated: then the
        // maximum single add, which has not, gives the scale)
        wide = true;
        const float total = fmaxf(S_f, M) * 1.0001f;
        int e2 = 0;
        if (total > 0.0f && total < INFINITY) (void)frexpf(total, &e2);  // total < 2^e2
#pragma unroll
        for (int g = 0; g < GB; ++g) k_exp[g] += 30 - e2;
        {
            uint4 *z = reinterpret_cast<uint4 *>(smem_raw);
            const int n16 = (bins * 8 + 15) / 16;
            for (int e = tid; e < n16; e += THREADS) z[e] = make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
    }
}

}  // namespace dec
}  // namespace csr
