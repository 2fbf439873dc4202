// Decode attention on codes whose KEYS were sparsely represented before the rotary position embedding
// (Section "Position embedding makes nonstationary Keys": the key cache is processed ahead of the embedding,
// so attention has to rotate the rebuilt key K~_t = D_K r_t of Eq.12 to its position t).
//
// The rotation depends on the token, so the one score table q . d_n of the position-free path no longer
// exists: every (token, pair) costs a gathered atom row and d multiply-adds instead of one table entry.  That
// only pays while the atom rows come from LDS: the kernel keeps the whole key dictionary of its KV head there
// (N * d * 2 bytes <= 128 KB, the paper's own dictionary sizes) and is bound by the vector ALU (the count of its
// instructions), not by HBM.  Values carry no position: the V side is the same histogram scatter as in stream_kernel, and out_kernel /
// finalize_kernel run unchanged on its results.
//
// Two ways to spend the multiply-adds, chosen by the number of query heads that share the KV head:
//   one query head:  (Rot(t) K~_t) . q = K~_t . (Rot(-t) q) = sum_j c_j (d_{i_j} . q~_t): the query is turned back
//                    to the token's position and dotted with each gathered row (packed fp16 dot products);
//   a query group:   K~_t is rebuilt in fp32 from the gathered rows, turned to its position once and dotted with
//                    every query of the group.
//
// Mapping of pass 1.  A wave handles 64 consecutive tokens per round.  The 8 lanes of an eighth of the wave share the
// work of one token at a time: each holds 8 of the 64 frequency pairs and reads the matching two 16-byte pieces of
// every gathered row.  In step u eighth e works on token 8u + e: all its lanes read that token's codes straight from
// memory (the same 16 bytes; the eighths' tokens are neighbours, so the wave reads one 128-byte line per stream and
// step, requested one step ahead, across rounds too).  The rotating state stands at the middle of the round, and steps
// 3 - i and 4 + i turn it by the same angle in opposite directions: two products serve both (three operations per pair
// and step), the result of a single query is rounded to fp16 by the multiply-add that forms it (v_fma_mixlo / mixhi),
// and the fp32 recurrence takes one step per round.  The eight steps' partial scores are transposed and added in three
// exchanges: lane (e, u) ends up with the score of token 8u + e, whose value codes it handles in pass 2.  The starting
// angle of every lane is reduced in double precision, so positions in the hundreds of thousands stay accurate.
// Bound by the count of vector instructions (16.5 per token of one head with 8 pairs; the vector ALU is busy 80 % of the
// time) and, before them, by codes that were requested one step ahead and came late.  4 sequences x 32 heads x 32768 tokens,
// 256 atoms, 8 key pairs: 193 us a call; with one recurrence step and one reduction per step, and codes one step ahead,
// it was 219; with 4 key pairs on 512 atoms 137 against 183, 8 sequences x 8 KV heads x 4 query heads 192 against 202.  Two copies
// of a small dictionary, so that two eighths never meet on the same LDS banks, change nothing.
#include <atomic>
#include <cmath>

#include "csr_internal.h"
#include "decode_common.h"

namespace csr {
namespace {

using namespace dec;

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint4v LdsVec;   // 16 bytes of LDS, addressed by their offset in it

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2(*reinterpret_cast<const half2v *>(&a), *reinterpret_cast<const half2v *>(&b), c, false);
}

// (a, b) as an fp16 pair; where a and b are fused multiply-adds, they round to fp16 themselves
__device__ __forceinline__ uint32_t turned_half2(float a, float b)
{
    half2v h;
    h.x = (_Float16)a;
    h.y = (_Float16)b;
    return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ float lo_half(uint32_t w)
{
    const uint16_t v = (uint16_t)(w & 0xffffu);
    return h2f(*reinterpret_cast<const __half *>(&v));
}
__device__ __forceinline__ float hi_half(uint32_t w)
{
    const uint16_t v = (uint16_t)(w >> 16);
    return h2f(*reinterpret_cast<const __half *>(&v));
}

// v + (v of the lane whose number differs in bit 0 / 1 / all three): cross-lane adds inside a row of 16 lanes
template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false);
    return v + __int_as_float(o);
}
__device__ __forceinline__ float sum8(float v)
{
    v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);  // row_half_mirror: lane i of every 8 with lane 7 - i, which lies in the other quad
    return v;
}
// Sums over the 8 lanes of an eighth of eight values each, value u to lane u: three exchanges that each halve what a lane
// holds (a lane keeps the values whose number has its own bit and adds the partner's).  row_half_mirror pairs lane i with
// 7 - i, whose bits all differ: bit 2 goes first, then quad_perm [1,0,3,2] (bit 0) and [2,3,0,1] (bit 1).
template <int CTRL> __device__ __forceinline__ float keep_and_add(bool upper, float low, float high)
{
    const float send = upper ? low : high;
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(send), CTRL, 0xf, 0xf, false);
    return (upper ? high : low) + __int_as_float(o);
}
__device__ __forceinline__ float transpose_sum8(const float (&v)[8], int sub)
{
    const bool b0 = sub & 1, b1 = sub & 2, b2 = sub & 4;
    float w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = keep_and_add<0x141>(b2, v[u], v[u + 4]);
    const float x0 = keep_and_add<0xB1>(b0, w[0], w[1]), x1 = keep_and_add<0xB1>(b0, w[2], w[3]);
    return keep_and_add<0x4E>(b1, x0, x1);
}

// LDS: atom rows of D_K[h], 256 bytes each, the two members of every frequency pair side by side (pass 1), later the
// fixed-point histogram (pass 2, finish_chunk) | reduction scratch | rotation constants [8 lane classes][kRopeTurn] |
// the group's query pairs, packed fp16 [8 lane classes][4][8] (ROTK only) | theta_k as doubles [64]
// TPT: rounds of rope_threads(GB) tokens a chunk may have (a lane keeps one score per round and query head).
// NP, PV: pairs of a value code, see finish_chunk.
// ONEB: a key code is exactly one block of PVK pairs.
// GLOBAL: the key dictionary does not fit the LDS (more than 512 atoms): every gathered row piece then comes from
// device memory - the L2 for dictionaries of a few MB - instead, brought into the same pair-adjacent form in
// registers.  The arithmetic is the same; the call is then bound by those gathers (256 bytes per code pair).
template <int GB, bool ROTK, int PVK, bool ONEB, int PV, int NP, int TPT, bool GLOBAL>
__global__ __launch_bounds__(rope_threads(GB)) void stream_rope_kernel(
    const __half *__restrict__ q, const __half *__restrict__ DK, const uint16_t *__restrict__ idxK,
    const __half *__restrict__ coefK, const uint16_t *__restrict__ idxV, const __half *__restrict__ coefV,
    const int32_t *__restrict__ seq_lens, float *__restrict__ part_hist, float *__restrict__ part_ml, int32_t Hq,
    int32_t Hkv, int32_t G, int32_t ngs, int64_t T, int32_t N, int32_t sK, int32_t sV, int32_t snV, float scale,
    float rope_base, int32_t layout, int64_t pos0, int64_t chunk_tokens, int32_t nchunks, uint32_t tab_bytes)
{
    constexpr int THREADS = rope_threads(GB);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    float *red = reinterpret_cast<float *>(smem_raw + tab_bytes);
    float *ctab = red + kRedBytes / sizeof(float);  // [8][kRopeTurn]: 5 x (8 cos, 8 sin), of 4 + 8 i positions, i < 4, and of a round
    uint32_t *qtab = reinterpret_cast<uint32_t *>(ctab + 8 * kRopeTurn);  // [8][GB][8]

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int sub = lane & 7, eighth = lane >> 3;
    const int h = blockIdx.x / ngs, gs = blockIdx.x % ngs;
    const Chunk part = chunk_of<THREADS, kCutFromRope>(seq_lens, T, nchunks, chunk_tokens);
    const int c = part.c, b = part.b;
    const int64_t t0 = part.t0, t_end = part.t_end;
    const int64_t slot = (((int64_t)b * Hkv + h) * ngs + gs) * nchunks + c;
    float *ml = part_ml + slot * (2 * GB);
    if (t_end <= t0) {  // nothing cached in this chunk: weight zero, histogram never read
        if (tid < GB) { ml[2 * tid] = -INFINITY; ml[2 * tid + 1] = 0.0f; }
        return;
    }
    const int64_t code_row = ((int64_t)b * Hkv + h) * T;
    const int n_mine = (int)((t_end - t0 + THREADS - 1) / THREADS);  // rounds of THREADS tokens

    // ---- the key dictionary into LDS, frequency pairs made adjacent -----------------------------------------
    // frequency pairs of a lane: slot e < 4 lives in row piece `sub`, e >= 4 in piece 8 + sub (128 bytes further); piece p
    // holds pairs 4p .. 4p+3.  theta_k of all 64 pairs, in double, once per workgroup, while the first rows are under way
    double *theta = reinterpret_cast<double *>(qtab + 8 * 4 * 8);  // [64]
    auto theta_out = [&]() {
        if (tid < 64) theta[tid] = exp2(-(2.0 * tid / 128.0) * log2((double)rope_base));
    };
    if constexpr (!GLOBAL) {
        const __half *src = DK + (int64_t)h * N * 128;
        constexpr int U = 4;   // pieces of 16 bytes a thread requests together: 256 atoms in one round trip of 1024 threads
        for (int e0 = tid; e0 < N * 16; e0 += U * THREADS) {
            uint4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {   // past the end: the first piece again, not stored
                const int e = e0 + u * THREADS < N * 16 ? e0 + u * THREADS : tid;
                const int row = e >> 4, j = e & 15;
                if (layout == 0) {  // pair k = dimensions (k, k + 64): take 4 + 4
                    const uint2 lo = *reinterpret_cast<const uint2 *>(src + row * 128 + 4 * j);
                    const uint2 hi = *reinterpret_cast<const uint2 *>(src + row * 128 + 64 + 4 * j);
                    v[u] = make_uint4(lo.x, lo.y, hi.x, hi.y);
                } else {            // pair k = dimensions (2k, 2k + 1): already adjacent
                    v[u] = *reinterpret_cast<const uint4 *>(src + row * 128 + 8 * j);
                }
            }
            if (e0 == tid) theta_out();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * THREADS;
                if (e < N * 16) {
                    uint4 w = v[u];
                    if (layout == 0)   // and interleave
                        w = make_uint4((v[u].x & 0xffffu) | (v[u].z << 16), (v[u].x >> 16) | (v[u].z & 0xffff0000u),
                                       (v[u].y & 0xffffu) | (v[u].w << 16), (v[u].y >> 16) | (v[u].w & 0xffff0000u));
                    *reinterpret_cast<uint4 *>(smem_raw + (e >> 4) * 256 + (e & 15) * 16) = w;
                }
            }
        }
        if (N * 16 <= tid && tid < 64) theta_out();   // fewer than 64 pieces: the threads that had none
    } else {
        theta_out();
    }
    // What depends on `sub` only goes to LDS, computed once
    __syncthreads();
    auto pair_of = [](int sb, int e) { return 4 * (e < 4 ? sb : sb + 8) + (e & 3); };
    // cos and sin of positions * theta_k: the angle is reduced to [-1/2, 1/2] revolutions in double, then the
    // hardware sine and cosine (which take revolutions) are accurate to about 1e-6
    auto cos_sin = [&](int k, double positions, float &co, float &si) {
        const double r = positions * theta[k] * 0.15915494309189533577;
        const float f = (float)(r - rint(r));
        co = __builtin_amdgcn_cosf(f);
        si = __builtin_amdgcn_sinf(f);
    };
    // the turning angles' constants are applied over and over, so they get the library's accurate sine and cosine (one thread
    // per constant: 5 x 64 of them, once per workgroup); a lane's starting phase above is applied once
    static_assert(THREADS >= 320, "one thread per constant");
    if (tid < 320) {
        const int i = tid >> 6, sb = (tid >> 3) & 7, e = tid & 7;
        const double r = (i < 4 ? 4.0 + 8.0 * i : (double)THREADS) * theta[pair_of(sb, e)] * 0.15915494309189533577;
        double co, si;
        sincospi(2.0 * (r - rint(r)), &si, &co);
        float *at = ctab + sb * kRopeTurn + 16 * i + e;
        at[0] = (float)co;
        at[8] = (float)si;
    }
    if (tid < 64) {
        const int sb = tid >> 3, e = tid & 7, k = pair_of(sb, e);
        if constexpr (ROTK) {
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                const __half *qp = q + ((int64_t)b * Hq + (int64_t)h * G + gs * GB + g) * 128;
                const __half2 pk = __halves2half2(layout == 0 ? qp[k] : qp[2 * k], layout == 0 ? qp[k + 64] : qp[2 * k + 1]);
                qtab[(sb * GB + g) * 8 + e] = *reinterpret_cast<const uint32_t *>(&pk);
            }
        }
    }
    // GLOBAL: this lane's two 16-byte pieces (pairs 4 sub .. 4 sub + 3 and 32 + 4 sub .. + 3) of the atom row at byte
    // offset `off` of the head's dictionary, the members of every pair made adjacent
    const unsigned char *grow = reinterpret_cast<const unsigned char *>(DK + (int64_t)h * N * 128);
    auto global_pieces = [&](uint32_t off, uint4 &d0, uint4 &d1) {
        if (layout == 0) {  // pair k = dimensions (k, k + 64): 4 + 4 halves from both halves of the row, interleaved
            auto weave = [](const uint2 &lo, const uint2 &hi) {
                return make_uint4((lo.x & 0xffffu) | (hi.x << 16), (lo.x >> 16) | (hi.x & 0xffff0000u),
                                  (lo.y & 0xffffu) | (hi.y << 16), (lo.y >> 16) | (hi.y & 0xffff0000u));
            };
            const unsigned char *r = grow + off + sub * 8;
            const uint2 a0 = *reinterpret_cast<const uint2 *>(r), b0 = *reinterpret_cast<const uint2 *>(r + 128);
            const uint2 a1 = *reinterpret_cast<const uint2 *>(r + 64), b1 = *reinterpret_cast<const uint2 *>(r + 192);
            d0 = weave(a0, b0);
            d1 = weave(a1, b1);
        } else {            // pair k = dimensions (2k, 2k + 1): already adjacent
            d0 = *reinterpret_cast<const uint4 *>(grow + off + sub * 16);
            d1 = *reinterpret_cast<const uint4 *>(grow + off + 128 + sub * 16);
        }
    };
    const float *my_c = ctab + sub * kRopeTurn;
    const uint32_t *my_q = qtab + sub * GB * 8;
    // the rotating state, at the middle of the eight tokens this eighth handles in the first round
    // ROTK: (ra, rb) = (cos, sin) of position * theta; else: the query pair turned back by that angle, scaled
    constexpr int NR = ROTK ? 1 : GB;
    float ra[NR][8], rb[NR][8];
    {
        const int64_t pos_start = pos0 + t0 + wave * 64 + eighth + 28;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = pair_of(sub, e);
            float c0, s0;
            cos_sin(k, (double)pos_start, c0, s0);
            if constexpr (ROTK) {
                ra[0][e] = c0;
                rb[0][e] = s0;
            } else {
#pragma unroll
                for (int g = 0; g < GB; ++g) {  // Rot(-pos) (a, b)
                    const __half *qp = q + ((int64_t)b * Hq + (int64_t)h * G + gs * GB + g) * 128;
                    const float a = scale * h2f(layout == 0 ? qp[k] : qp[2 * k]);
                    const float bb = scale * h2f(layout == 0 ? qp[k + 64] : qp[2 * k + 1]);
                    ra[g][e] = a * c0 + bb * s0;
                    rb[g][e] = bb * c0 - a * s0;
                }
            }
        }
    }
    __syncthreads();

    // ---- pass 1 ---------------------------------------------------------------------------------------------
    const int nblk = ONEB ? 1 : sK / PVK;  // pair blocks per token (ONEB: known to be one)
    float sc[TPT][GB];
    float mx[GB];
#pragma unroll
    for (int g = 0; g < GB; ++g) {
        mx[g] = -INFINITY;
#pragma unroll
        for (int i = 0; i < TPT; ++i) sc[i][g] = -INFINITY;
    }
    // PVK pairs of a token, read by all 8 lanes of the eighth (one 16-byte piece, and the 8 eighths' tokens are neighbours:
    // a wave reads 128 contiguous bytes per stream and step); indices and coefficients as packed 16-bit words, at a 32-bit
    // byte offset from the chunk's first token.  Whole codes are requested three steps ahead of their use, blocks of
    // longer ones one block ahead.
    constexpr int AHEAD = ONEB ? 3 : 1, SLOTS = ONEB ? 4 : 1;
    uint32_t ni[SLOTS][PVK / 2], nc[SLOTS][PVK / 2];
    const unsigned char *ibase = reinterpret_cast<const unsigned char *>(idxK + (code_row + t0) * sK);
    const unsigned char *cbase = reinterpret_cast<const unsigned char *>(coefK + (code_row + t0) * sK);
    const uint32_t code_bytes = 2u * (uint32_t)(ONEB ? PVK : sK);
    const uint32_t last_code = (uint32_t)(t_end - t0 - 1) * code_bytes;
    auto fetch = [&](int slot, uint32_t code, int jb) {   // past the end: the last token again, score unused
        const uint32_t o = min(code, last_code) + (ONEB ? 0u : (uint32_t)jb * (2u * PVK));
        if constexpr (PVK == 8) {
            const uint4 a = *reinterpret_cast<const uint4 *>(ibase + o);
            const uint4 bq = *reinterpret_cast<const uint4 *>(cbase + o);
            ni[slot][0] = a.x; ni[slot][1] = a.y; ni[slot][2] = a.z; ni[slot][3] = a.w;
            nc[slot][0] = bq.x; nc[slot][1] = bq.y; nc[slot][2] = bq.z; nc[slot][3] = bq.w;
        } else {
            const uint2 a = *reinterpret_cast<const uint2 *>(ibase + o);
            const uint2 bq = *reinterpret_cast<const uint2 *>(cbase + o);
            ni[slot][0] = a.x; ni[slot][1] = a.y;
            nc[slot][0] = bq.x; nc[slot][1] = bq.y;
        }
    };
    // The order of a round's steps: 3, 4, 2, 5, 1, 6, 0, 7; the tokens of step `o` of this order, counted on into the next
    // round, stand 8 * step_at(o) tokens behind the eighth's first one
    auto step_at = [](int o) { return (o >> 3) * (THREADS / 8) + ((o & 1) ? 4 + ((o & 7) >> 1) : 3 - ((o & 7) >> 1)); };
    const int nwave = (int)min((int64_t)n_mine, (t_end - t0 - wave * 64 + THREADS - 1) / THREADS);  // rounds with tokens of this wave
    uint32_t code0 = (uint32_t)(wave * 64 + eighth) * code_bytes;   // the code of this eighth's token of step 0
    if (nwave > 0) {
#pragma unroll
        for (int o = 0; o < AHEAD; ++o) fetch(o % SLOTS, code0 + (uint32_t)step_at(o) * (8 * code_bytes), 0);
    }
    const uint32_t row_low = GLOBAL ? 0u : (uint32_t)sub * 16u;   // lowest byte of a row piece's address
#pragma unroll 1
    for (int i = 0; i < nwave; ++i) {
        // half `up` of pair w of the order: step up ? 4 + w : 3 - w; part: its partial scores
        auto step = [&](int w, auto up_c, float (&part)[GB]) {
            constexpr bool kUp = decltype(up_c)::value;
            // the state turned by 4 + 8 w positions, back for the steps below the middle
            float cc[8], ss[8];
            {
                const float *cs = my_c + w * 16;
#pragma unroll
                for (int e = 0; e < 8; e += 4) {
                    *reinterpret_cast<float4 *>(&cc[e]) = *reinterpret_cast<const float4 *>(cs + e);
                    *reinterpret_cast<float4 *>(&ss[e]) = *reinterpret_cast<const float4 *>(cs + 8 + e);
                }
            }
            float ka[ROTK ? 8 : 1], kb[ROTK ? 8 : 1];  // ROTK: K~ of this lane's 8 pairs, fp32
            uint32_t qp[ROTK ? 1 : GB][8];             // else: the turned-back queries as fp16 pairs
            constexpr float sgn = kUp ? 1.0f : -1.0f;
            if constexpr (ROTK) {
#pragma unroll
                for (int e = 0; e < 8; ++e) ka[e] = kb[e] = 0.0f;
            } else {
#pragma unroll
                for (int g = 0; g < GB; ++g) {
                    part[g] = 0.0f;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        qp[g][e] = turned_half2(fmaf(rb[g][e], sgn * ss[e], ra[g][e] * cc[e]), fmaf(-ra[g][e], sgn * ss[e], rb[g][e] * cc[e]));
                }
            }
#pragma unroll 1
            for (int jb = 0; jb < nblk; ++jb) {
                const int o = 2 * w + (kUp ? 1 : 0), slot = o % SLOTS;
                uint32_t to[PVK], tc[PVK / 2];
#pragma unroll
                for (int jj = 0; jj < PVK; ++jj)   // 256 * index + 16 * sub, by one byte permute
                    to[jj] = __builtin_amdgcn_perm(ni[slot][jj >> 1], row_low, (jj & 1) ? 0x0c070600u : 0x0c050400u);
#pragma unroll
                for (int k = 0; k < PVK / 2; ++k) tc[k] = nc[slot][k];
                if (jb + 1 < nblk) fetch(slot, code0 + (uint32_t)step_at(o) * (8 * code_bytes), jb + 1);
                else fetch((o + AHEAD) % SLOTS, code0 + (uint32_t)step_at(o + AHEAD) * (8 * code_bytes), 0);
                auto coef = [&](int jj) { return (jj & 1) ? hi_half(tc[jj >> 1]) : lo_half(tc[jj >> 1]); };
                auto read_row = [&](int jj, uint4 &d0, uint4 &d1) {
                    if constexpr (GLOBAL) {
                        global_pieces(to[jj], d0, d1);
                    } else {
                        // the dictionary starts the workgroup's LDS (launch_rope_t checks that nothing stands before it),
                        // so that the permuted bytes are the address
                        const LdsVec *row = reinterpret_cast<const LdsVec *>(to[jj]);
                        d0 = __builtin_bit_cast(uint4, row[0]);
                        d1 = __builtin_bit_cast(uint4, row[8]);
                    }
                };
                if constexpr (ROTK) {
#pragma unroll
                    for (int jj = 0; jj < PVK; ++jj) {
                        uint4 d0, d1;
                        read_row(jj, d0, d1);
                        const float cf = coef(jj);
                        const uint32_t dw[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            ka[e] = fmaf(cf, lo_half(dw[e]), ka[e]);
                            kb[e] = fmaf(cf, hi_half(dw[e]), kb[e]);
                        }
                    }
                } else {
                    // two rows at a time, so that two chains of dot products alternate, the next two rows requested before
                    // these are awaited
                    uint4 d[2][2][2];   // [pair of rows][row][piece]
                    auto request = [&](int jj) {
#pragma unroll
                        for (int r = 0; r < 2; ++r) read_row(jj + r, d[(jj >> 1) & 1][r][0], d[(jj >> 1) & 1][r][1]);
                        round_fence();
                    };
                    request(0);
#pragma unroll
                    for (int jj = 0; jj < PVK; jj += 2) {
                        if (jj + 2 < PVK) request(jj + 2);
                        auto &x = d[(jj >> 1) & 1];
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int k = 0; k < 2; ++k) asm volatile("" : "+v"(x[r][k].x), "+v"(x[r][k].y), "+v"(x[r][k].z), "+v"(x[r][k].w));
#pragma unroll
                        for (int g = 0; g < GB; ++g) {
                            float p0 = 0.0f, p1 = 0.0f;
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                p0 = dot2(qp[g][4 * k], x[0][k].x, p0);
                                p1 = dot2(qp[g][4 * k], x[1][k].x, p1);
                                p0 = dot2(qp[g][4 * k + 1], x[0][k].y, p0);
                                p1 = dot2(qp[g][4 * k + 1], x[1][k].y, p1);
                                p0 = dot2(qp[g][4 * k + 2], x[0][k].z, p0);
                                p1 = dot2(qp[g][4 * k + 2], x[1][k].z, p1);
                                p0 = dot2(qp[g][4 * k + 3], x[0][k].w, p0);
                                p1 = dot2(qp[g][4 * k + 3], x[1][k].w, p1);
                            }
                            part[g] = fmaf(coef(jj), p0, part[g]);
                            part[g] = fmaf(coef(jj + 1), p1, part[g]);
                        }
                    }
                }
            }
            if constexpr (ROTK) {
                // turned to the token's position, rounded to fp16 pairs, dotted with every query of the group
                uint32_t kp[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float co = fmaf(-rb[0][e], sgn * ss[e], ra[0][e] * cc[e]), si = fmaf(ra[0][e], sgn * ss[e], rb[0][e] * cc[e]);
                    kp[e] = turned_half2(fmaf(-kb[e], si, ka[e] * co), fmaf(ka[e], si, kb[e] * co));
                }
#pragma unroll
                for (int g = 0; g < GB; ++g) {
                    const uint4 q0 = *reinterpret_cast<const uint4 *>(my_q + g * 8);
                    const uint4 q1 = *reinterpret_cast<const uint4 *>(my_q + g * 8 + 4);
                    float p = dot2(q0.x, kp[0], 0.0f);
                    p = dot2(q0.y, kp[1], p);
                    p = dot2(q0.z, kp[2], p);
                    p = dot2(q0.w, kp[3], p);
                    p = dot2(q1.x, kp[4], p);
                    p = dot2(q1.y, kp[5], p);
                    p = dot2(q1.z, kp[6], p);
                    p = dot2(q1.w, kp[7], p);
                    part[g] = p;
                }
            }
            round_fence();   // requests and row reads of a step stay in it
        };
        float mine[GB];
        if constexpr (ONEB || !ROTK) {
            float part[8][GB];   // [step][head]
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                step(w, std::false_type{}, part[3 - w]);
                step(w, std::true_type{}, part[4 + w]);
            }
#pragma unroll
            for (int g = 0; g < GB; ++g) {
                const float v[8] = {part[0][g], part[1][g], part[2][g], part[3][g], part[4][g], part[5][g], part[6][g], part[7][g]};
                mine[g] = transpose_sum8(v, sub);
            }
        } else {   // a loop of blocks in every step: with the steps unrolled around it 330 registers spill
#pragma unroll
            for (int g = 0; g < GB; ++g) mine[g] = 0.0f;
#pragma unroll 1
            for (int w = 0; w < 4; ++w) {
                float lo[GB], hi[GB];
                step(w, std::false_type{}, lo);
                step(w, std::true_type{}, hi);
#pragma unroll
                for (int g = 0; g < GB; ++g) {
                    const float a = sum8(lo[g]), b2 = sum8(hi[g]);
                    mine[g] = sub == 3 - w ? a : sub == 4 + w ? b2 : mine[g];
                }
            }
        }
        {   // the state one round on
            float cc[8], ss[8];
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                *reinterpret_cast<float4 *>(&cc[e]) = *reinterpret_cast<const float4 *>(my_c + 64 + e);
                *reinterpret_cast<float4 *>(&ss[e]) = *reinterpret_cast<const float4 *>(my_c + 72 + e);
            }
#pragma unroll
            for (int g = 0; g < NR; ++g) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float a = ra[g][e], bb = rb[g][e];
                    if constexpr (ROTK) {  // (cos, sin) forward
                        ra[g][e] = fmaf(-bb, ss[e], a * cc[e]);
                        rb[g][e] = fmaf(a, ss[e], bb * cc[e]);
                    } else {               // the query further back
                        ra[g][e] = fmaf(bb, ss[e], a * cc[e]);
                        rb[g][e] = fmaf(-a, ss[e], bb * cc[e]);
                    }
                }
            }
        }
        code0 += THREADS * code_bytes;
        // the score of the token whose value codes this lane handles; registers take no index: kept by comparison
        const bool have = t0 + (int64_t)i * THREADS + wave * 64 + 8 * sub + eighth < t_end;
#pragma unroll
        for (int g = 0; g < GB; ++g) {
            const float v = have ? (ROTK ? mine[g] * scale : mine[g]) : -INFINITY;
            mx[g] = fmaxf(mx[g], v);
#pragma unroll
            for (int k = 0; k < TPT; ++k) sc[k][g] = i == k ? v : sc[k][g];
        }
    }
    finish_chunk<GB, uint16_t, __half, PV, true, TPT, THREADS, NP>(smem_raw, red, sc, mx, n_mine, t0, t_end, code_row,
                                                                  wave * 64 + 8 * sub + eighth, idxV, coefV, N, sV, snV, ml,
                                                                  part_hist, slot);
}

template <int GB, bool ROTK, int PVK, bool ONEB, int PV, int NP, bool GLOBAL>
hipError_t launch_rope_t(const DecodeArgs &a, const DecodePlan &p, float *hist, float *ml)
{
    auto kern = stream_rope_kernel<GB, ROTK, PVK, ONEB, PV, NP, rope_rounds(GB), GLOBAL>;
    static std::atomic<bool> attr_set[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
        hipFuncAttributes fa;
        e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(kern));
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidDeviceFunction;   // the kernel's row addresses start at LDS address 0
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)(kLdsBudget + kRopeTableBytes - kRopeTableCounted));
        if (e != hipSuccess) return e;
        attr_set[dev].store(true, std::memory_order_release);
    }
    // the plan's LDS size = dictionary / histogram | reductions | constant tables (see plan_decode)
    const uint32_t tab_bytes = (uint32_t)(p.lds_bytes - kRedBytes - kRopeTableBytes);
    const dim3 grid((unsigned)(a.Hkv * p.ngs), (unsigned)p.nchunks, (unsigned)a.B);
    hipLaunchKernelGGL(kern, grid, dim3(rope_threads(GB)), p.lds_bytes, a.stream, (const __half *)a.q,
                       (const __half *)a.DK, (const uint16_t *)a.idxK, (const __half *)a.coefK,
                       (const uint16_t *)a.idxV, (const __half *)a.coefV, a.seq_lens, hist, ml, a.Hq, a.Hkv, a.G, p.ngs,
                       a.T, a.N, a.sK, a.sV, a.snV, a.scale, a.rope_base, a.rope_layout, a.rope_pos0, p.chunk_tokens,
                       p.nchunks, tab_bytes);
    return hipGetLastError();
}

template <int GB, bool ROTK, int PVK, bool ONEB, bool GLOBAL>
hipError_t launch_rope_pv(const DecodeArgs &a, const DecodePlan &p, float *hist, float *ml)
{
    // Value codes read as a whole, requested ahead - except in the variant that has no registers for it (one query head, 8
    // key rows at a time from device memory: 240 spilled registers become 279, 32 heads x 4096 tokens on 4096 atoms take
    // 101.9 us instead of 92.9; with groups of 2 and 4 the requests are worth 1 - 2 %).
    if constexpr (!(GLOBAL && GB == 1 && PVK == 8)) {
        switch (a.snV * a.sV) {
            case 4: return launch_rope_t<GB, ROTK, PVK, ONEB, 4, 4, GLOBAL>(a, p, hist, ml);
            case 8: return launch_rope_t<GB, ROTK, PVK, ONEB, 8, 8, GLOBAL>(a, p, hist, ml);
            case 16: return launch_rope_t<GB, ROTK, PVK, ONEB, 8, 16, GLOBAL>(a, p, hist, ml);
        }
    }
    if (a.sV % 8 == 0) return launch_rope_t<GB, ROTK, PVK, ONEB, 8, 0, GLOBAL>(a, p, hist, ml);
    if (a.sV % 4 == 0) return launch_rope_t<GB, ROTK, PVK, ONEB, 4, 0, GLOBAL>(a, p, hist, ml);
    return launch_rope_t<GB, ROTK, PVK, ONEB, 1, 0, GLOBAL>(a, p, hist, ml);
}

template <int GB, bool ROTK>
hipError_t launch_rope_gb(const DecodeArgs &a, const DecodePlan &p, float *hist, float *ml)
{
    if (!rope_dictionary_fits_lds(a.N)) {  // rows gathered from device memory
        if (a.sK % 8 == 0) return launch_rope_pv<GB, ROTK, 8, false, true>(a, p, hist, ml);
        return launch_rope_pv<GB, ROTK, 4, false, true>(a, p, hist, ml);
    }
    if (a.sK == 8) return launch_rope_pv<GB, ROTK, 8, true, false>(a, p, hist, ml);  // the paper's key codes
    if (a.sK == 4) return launch_rope_pv<GB, ROTK, 4, true, false>(a, p, hist, ml);
    if (a.sK % 8 == 0) return launch_rope_pv<GB, ROTK, 8, false, false>(a, p, hist, ml);
    return launch_rope_pv<GB, ROTK, 4, false, false>(a, p, hist, ml);
}

}  // namespace

bool decode_rope_shape_supported(int32_t d, int32_t N, int32_t sK, int32_t snK)
{
    return d == 128 && snK == 1 && sK % 4 == 0 && N <= 65536;
}

hipError_t launch_stream_rope(const DecodeArgs &a, const DecodePlan &p, float *hist, float *ml)
{
    switch (p.GB) {
        case 4: return launch_rope_gb<4, true>(a, p, hist, ml);
        case 2: return launch_rope_gb<2, true>(a, p, hist, ml);
        case 1: return launch_rope_gb<1, false>(a, p, hist, ml);
    }
    return hipErrorInvalidValue;
}

}  // namespace csr
