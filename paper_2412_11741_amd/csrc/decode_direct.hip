// Decode attention for SHORT contexts: the cached tokens rebuilt from their codes on the fly.
//
// The code-domain form (decode.hip) reads both dictionaries once per KV head and pays a score table, a histogram and four
// launches, about 25 us whatever the context - right when thousands of tokens share them.  A short context touches fewer
// atoms than the dictionary has: here every cached token is rebuilt (Eq.12, K~_t = D_K r_t and V~_t = D_V r_t) from its
// s + s gathered atom rows, and ordinary softmax attention runs on it in registers - 256 bytes from L2 per pair instead of 4
// from the cache, and two launches.
//
//   direct_kernel   one workgroup per (token chunk, sequence, KV head).  16 lanes - a team - share a token, 8 dimensions
//                   each: an atom row is one 256-byte request of the team.  The team dots the rebuilt key with the KV
//                   head's query heads (held in registers), keeps a running maximum and sum per query head and adds the
//                   weighted rebuilt value to its partial output; the 16 teams of the workgroup meet at the end.
//   combine_kernel  the chunks' partial outputs of a (sequence, query head), weighted by their maxima and sums.
//
// Keys coded before the rotary position embedding (ROPE) are turned in registers: the lane's 8 dimensions are 4 frequency
// pairs, whose angle is reduced to a revolution in double precision.
//
// Bound: L2 gathers (11.6 TB/s, 0.022 us per 1000 rows) once a few hundred workgroups are in flight, before that the chain of one token - codes,
// rows, reduction, combine.  All sums run in a fixed order: the same inputs give the same bits.  When it is taken: see
// kMostGathers.
#include <cfloat>
#include <cmath>

#include "csr_internal.h"
#include "decode_common.h"

namespace csr {
namespace {

using namespace dec;

constexpr int kThreads = 256;
constexpr int kTeams = kThreads / 16;   // tokens a workgroup has in work at a time
// Atom rows of 256 bytes (pairs of all cached tokens; fp32 rows count twice) up to which a context is a short one.  The
// time here is about 9 us + 0.022 us per 1000 rows, the code-domain form's 23 to 26 us with few (sequence, query head) pairs
// per KV head (31 to 35 with many, or 8192 atoms).  Measured (us, this / the other): 8 KV heads x 4 query heads, N = 4096,
// s = 8: T = 64 8.4 / 22.7, 1024 11.8 / 24.1, 4096 (524000 rows) 19.8 / 25.7; 32 heads: 256 11.5 / 22.4, 1024 (524000 rows)
// 19.4 / 23.0, 2048 30.2 / 23.3; rotary keys, N = 256, 4 sequences: 1024 (524000 rows) 17.6 / 31.2.
constexpr int64_t kMostGathers = 512 * 1024;

// 8 elements of an atom row, raw and unpacked
template <typename TD> struct Piece;
template <> struct Piece<__half> {
    uint4 v;
    __device__ __forceinline__ void zero() { v = make_uint4(0u, 0u, 0u, 0u); }
    __device__ __forceinline__ void get(float (&f)[8]) const { load8_raw(v, f); }
};
template <> struct Piece<float> {
    float4 a, b;
    __device__ __forceinline__ void zero() { a = b = make_float4(0.0f, 0.0f, 0.0f, 0.0f); }
    __device__ __forceinline__ void get(float (&f)[8]) const
    {
        f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
};
// SPLIT: 4 + 4 elements, `far` elements apart (rotary layout 0: dimensions 4 sub .. and 64 + 4 sub ..)
template <bool SPLIT> __device__ __forceinline__ void fetch(Piece<__half> &p, const __half *row)
{
    if constexpr (SPLIT) {
        const uint2 x = *reinterpret_cast<const uint2 *>(row), y = *reinterpret_cast<const uint2 *>(row + 64);
        p.v = make_uint4(x.x, x.y, y.x, y.y);
    } else {
        p.v = *reinterpret_cast<const uint4 *>(row);
    }
}
template <bool SPLIT> __device__ __forceinline__ void fetch(Piece<float> &p, const float *row)
{
    p.a = *reinterpret_cast<const float4 *>(row);
    p.b = *reinterpret_cast<const float4 *>(row + (SPLIT ? 64 : 4));
}

// An index as it is used: one outside the dictionary counts as the last atom.  The rows are read from device memory, where an
// index that a program left stale would otherwise read outside the allocation (the score-table form's stays in the LDS).
__device__ __forceinline__ int inside(int id, uint32_t last) { return (int)min((uint32_t)id, last); }

// up to 8 pairs of a code: indices (at most `last`) and coefficients, zero past the end
template <typename TI, typename TC, int PV>
__device__ __forceinline__ void load_pairs(const TI *ip, const TC *cp, int n, uint32_t last, int (&id)[8], float (&cf)[8])
{
#pragma unroll
    for (int j0 = 0; j0 < 8; j0 += PV) {
        int i[PV];
        float c[PV];
#pragma unroll
        for (int j = 0; j < PV; ++j) { i[j] = 0; c[j] = 0.0f; }
        if (j0 < n) {   // (uniform; PV divides n)
            IdxLoad<TI, PV>::ld(ip + j0, i);
            CoefLoad<TC, PV>::ld(cp + j0, c);
        }
#pragma unroll
        for (int j = 0; j < PV; ++j) { id[j0 + j] = inside(i[j], last); cf[j0 + j] = c[j]; }
    }
}

struct DirectParams {
    const void *q, *DK, *DV, *idxK, *coefK, *idxV, *coefV;
    const int32_t *seq_lens;
    void *out;
    float *part;      // [B * Hq][nchunks][128]
    float2 *ml;       // [B * Hq][nchunks]: maximum, sum of weights
    int64_t T, rope_pos0;
    int32_t Hq, Hkv, G, N, sK, sV, snK, snV, chunk_tokens, nchunks, out16;
    float scale, rope_base;
};

__device__ __forceinline__ int64_t context_length(const DirectParams &p, int b)
{
    if (!p.seq_lens) return p.T;
    const int32_t l = p.seq_lens[b];
    return l < 0 ? 0 : (l > p.T ? p.T : l);
}
__device__ __forceinline__ void store8(const DirectParams &p, int64_t at, const float (&v)[8])
{
    if (p.out16) {
        uint4 raw;
        __half2 *h = reinterpret_cast<__half2 *>(&raw);
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = __floats2half2_rn(v[2 * j], v[2 * j + 1]);
        *reinterpret_cast<uint4 *>(reinterpret_cast<__half *>(p.out) + at) = raw;
    } else {
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.out) + at) = make_float4(v[0], v[1], v[2], v[3]);
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(p.out) + at + 4) = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// Waves per SIMD the register budget is set for: a workgroup is a chain of dependent requests, what hides it is the others.
template <int GM, typename TD> constexpr int waves_per_simd() { return sizeof(TD) == 2 ? (GM == 1 ? 4 : GM == 2 ? 3 : 2) : GM <= 4 ? 2 : 1; }

// v of this lane plus v of the lanes 32 (16) away, two values at a time: the lower half (even rows) of the wave ends up with
// the sums of `a`, the upper half (odd rows) with those of `b`
__device__ __forceinline__ float fold32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// GM: query heads per KV head, rounded up to 1, 2, 4 or 8 (the excess ones compute on zeros).  ROPE: 0 none, 1 pairs
// (k, k + 64), 2 pairs (2 k, 2 k + 1).
template <int GM, typename TD, typename TI, typename TC, int PV, int ROPE>
__global__ __launch_bounds__(kThreads, (waves_per_simd<GM, TD>())) void direct_kernel(const DirectParams p)
{
    __shared__ float acc_s[4][GM][128];
    __shared__ float2 ml_s[4][GM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = tid & 15, team = tid >> 4;
    // an XCD gets a contiguous run of the work, ordered by KV head first: its L2 then gathers from few dictionaries
    unsigned id = blockIdx.x;
    const unsigned per = gridDim.x >> 3;
    if (id < per * 8u) id = (id & 7u) * per + (id >> 3);
    const int c = (int)(id % (unsigned)p.nchunks);
    const int bh = (int)(id / (unsigned)p.nchunks);
    const int B = (int)(gridDim.x / (unsigned)(p.nchunks * p.Hkv));
    const int h = bh / B, b = bh - h * B;

    const int64_t len = context_length(p, b);
    const int64_t t0 = (int64_t)c * p.chunk_tokens, t_end = min(t0 + p.chunk_tokens, len);
    const int64_t oq = (int64_t)b * p.Hq + h * p.G;   // first query head
    if (t_end <= t0) {                                // no tokens: weight zero
        if (p.nchunks > 1) {
            if (tid < p.G) p.ml[(oq + tid) * p.nchunks + c] = make_float2(-INFINITY, 0.0f);
        } else {
            const float zero[8] = {};
            if (tid < 16 * p.G) store8(p, (oq + tid / 16) * 128 + sub * 8, zero);
        }
        return;
    }

    // this lane's 8 dimensions: of the values 8 sub .. 8 sub + 7, of keys and queries the same or, with pairs (k, k + 64),
    // 4 sub .. + 3 and 64 + 4 sub .. + 3
    const int kd = ROPE == 1 ? 4 * sub : 8 * sub;
    const int dcK = 128 / p.snK, dcV = 128 / p.snV;
    const int chK = kd / dcK, chV = 8 * sub / dcV;
    const TD *DKh = reinterpret_cast<const TD *>(p.DK) + ((int64_t)h * p.snK + chK) * p.N * dcK + (kd - chK * dcK);
    const TD *DVh = reinterpret_cast<const TD *>(p.DV) + ((int64_t)h * p.snV + chV) * p.N * dcV + (8 * sub - chV * dcV);
    const int64_t row0 = ((int64_t)b * p.Hkv + h) * p.T;
    const TI *iK = reinterpret_cast<const TI *>(p.idxK) + (row0 * p.snK + chK) * p.sK;
    const TC *cK = reinterpret_cast<const TC *>(p.coefK) + (row0 * p.snK + chK) * p.sK;
    const TI *iV = reinterpret_cast<const TI *>(p.idxV) + (row0 * p.snV + chV) * p.sV;
    const TC *cV = reinterpret_cast<const TC *>(p.coefV) + (row0 * p.snV + chV) * p.sV;

    float q[GM][8];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
        Piece<TD> raw;
        raw.zero();
        if (g < p.G) fetch<ROPE == 1>(raw, reinterpret_cast<const TD *>(p.q) + (oq + g) * 128 + kd);
        raw.get(q[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) q[g][e] *= p.scale;
    }
    double turns[4];   // revolutions per position of this lane's four frequency pairs
    if constexpr (ROPE != 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            turns[e] = exp2(-(2.0 * (4 * sub + e) / 128.0) * log2((double)p.rope_base)) * 0.15915494309189533577;
    }

    const uint32_t last = (uint32_t)p.N - 1u;
    float m[GM], l[GM], acc[GM][8];
#pragma unroll
    for (int g = 0; g < GM; ++g) {
        m[g] = -FLT_MAX;   // below every finite score, and a difference with a score of minus infinity is no NaN
        l[g] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.0f;
    }
    int ik[8], iv[8];
    float ck[8], cv[8];
    auto codes = [&](int64_t t) {   // the first 8 pairs of token t's codes
        load_pairs<TI, TC, PV>(iK + t * p.snK * p.sK, cK + t * p.snK * p.sK, p.sK, last, ik, ck);
        load_pairs<TI, TC, PV>(iV + t * p.snV * p.sV, cV + t * p.snV * p.sV, p.sV, last, iv, cv);
    };
    // The score as the code-domain form has it, sum_j c_j (q . d_j): an infinite coefficient is an infinite score there, while
    // the rebuilt key mixes infinities of both signs.  One pair at a time: codes of finite numbers never come here.
    auto score_by_pairs = [&](int64_t t, const float (&qg)[8]) {
        const int width = 16 / p.snK;   // lanes of a chunk
        float s = 0.0f;
#pragma unroll 1
        for (int j = 0; j < p.sK; ++j) {
            int id[1];
            float cf[1], f[8], dot = 0.0f;
            IdxLoad<TI, 1>::ld(iK + t * p.snK * p.sK + j, id);
            CoefLoad<TC, 1>::ld(cK + t * p.snK * p.sK + j, cf);
            Piece<TD> row;
            fetch<ROPE == 1>(row, DKh + (int64_t)inside(id[0], last) * dcK);
            row.get(f);
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = fmaf(qg[e], f[e], dot);
            for (int x = 1; x < width; x <<= 1) dot += __shfl_xor(dot, x, 16);
            s = fmaf(cf[0], dot, s);
        }
        for (int x = width; x < 16; x <<= 1) s += __shfl_xor(s, x, 16);
        return s;
    };
    for (int64_t t = t0 + team; t < t_end; t += kTeams) {   // (the lanes of a team leave together)
        codes(t);
        // rows of the first 8 pairs of both codes in flight together
        Piece<TD> rk[8], rv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            rk[j].zero();
            if (j < p.sK) fetch<ROPE == 1>(rk[j], DKh + (int64_t)ik[j] * dcK);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            rv[j].zero();
            if (j < p.sV) fetch<false>(rv[j], DVh + (int64_t)iv[j] * dcV);
        }
        float k[8], v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) k[e] = v[e] = 0.0f;
        auto add = [&](float (&x)[8], const Piece<TD> (&rows)[8], const float (&cf)[8]) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float f[8];
                rows[j].get(f);
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = fmaf(cf[j], f[e], x[e]);
            }
        };
        add(k, rk, ck);
        for (int j0 = 8; j0 < p.sK; j0 += 8) {       // longer codes: the rest, 8 pairs at a time
            int id[8];
            float cf[8];
            load_pairs<TI, TC, PV>(iK + t * p.snK * p.sK + j0, cK + t * p.snK * p.sK + j0, p.sK - j0, last, id, cf);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                rk[j].zero();
                if (j0 + j < p.sK) fetch<ROPE == 1>(rk[j], DKh + (int64_t)id[j] * dcK);
            }
            add(k, rk, cf);
        }
        if constexpr (ROPE != 0) {
            const double pos = (double)(p.rope_pos0 + t);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double r = pos * turns[e];
                const float f = (float)(r - rint(r));   // revolutions in [-1/2, 1/2]
                const float co = __builtin_amdgcn_cosf(f), si = __builtin_amdgcn_sinf(f);
                float &x = ROPE == 1 ? k[e] : k[2 * e], &y = ROPE == 1 ? k[e + 4] : k[2 * e + 1];
                const float a = x * co - y * si, bb = y * co + x * si;
                x = a;
                y = bb;
            }
        }
        float sc[GM], pw[GM];
        bool odd = false;
#pragma unroll
        for (int g = 0; g < GM; ++g) {
            float s = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) s = fmaf(q[g][e], k[e], s);
            // as in the streaming kernels a score that is no number counts like minus infinity: weight zero
            sc[g] = row_reduce<16>(s, OpAdd());
            if constexpr (ROPE == 0) odd = odd || !(fabsf(sc[g]) < INFINITY);
            else sc[g] = sc[g] > -INFINITY ? sc[g] : -INFINITY;
        }
        if (odd) {
#pragma unroll
            for (int g = 0; g < GM; ++g) {
                const float s = score_by_pairs(t, q[g]);
                sc[g] = s > -INFINITY ? s : -INFINITY;
            }
        }
#pragma unroll
        for (int g = 0; g < GM; ++g) {
            const float mn = fmaxf(m[g], sc[g]), old = __expf(m[g] - mn);   // (mn is finite or +infinity, see m)
            pw[g] = __expf(sc[g] - mn);
            m[g] = mn;
            l[g] = l[g] * old + pw[g];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] *= old;
        }
        add(v, rv, cv);
        for (int j0 = 8; j0 < p.sV; j0 += 8) {
            int id[8];
            float cf[8];
            load_pairs<TI, TC, PV>(iV + t * p.snV * p.sV + j0, cV + t * p.snV * p.sV + j0, p.sV - j0, last, id, cf);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                rv[j].zero();
                if (j0 + j < p.sV) fetch<false>(rv[j], DVh + (int64_t)id[j] * dcV);
            }
            add(v, rv, cf);
        }
#pragma unroll
        for (int g = 0; g < GM; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(pw[g], v[e], acc[g][e]);
    }

    // ---- the four teams of a wave, then the four waves -------------------------------------------------------------------
#pragma unroll
    for (int g = 0; g < GM; ++g) {
        const float M = fmaxf(fmaxf(lane_read(m[g], 0), lane_read(m[g], 16)), fmaxf(lane_read(m[g], 32), lane_read(m[g], 48)));
        const float w = __expf(m[g] - M);
        float ls = l[g] * w;
        ls = fold32(ls, ls);
        ls = fold16(ls, ls);
        float x4[4], x2[2];   // of dimensions 8 sub + 4 (upper half of the wave) + 2 (odd row) + 0, 1
#pragma unroll
        for (int e = 0; e < 4; ++e) x4[e] = fold32(acc[g][e] * w, acc[g][e + 4] * w);
#pragma unroll
        for (int e = 0; e < 2; ++e) x2[e] = fold16(x4[e], x4[e + 2]);
        *reinterpret_cast<float2 *>(&acc_s[wave][g][8 * sub + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1)]) = make_float2(x2[0], x2[1]);
        if (lane == 0) ml_s[wave][g] = make_float2(M, ls);
    }
    __syncthreads();
    for (int e = tid; e < p.G * 16; e += kThreads) {
        const int g = e >> 4;
        float M = -INFINITY, L = 0.0f, w[4], o[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) M = fmaxf(M, ml_s[i][g].x);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = __expf(ml_s[i][g].x - M);
            L = fmaf(w[i], ml_s[i][g].y, L);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            o[x] = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[x] = fmaf(w[i], acc_s[i][g][8 * sub + x], o[x]);
        }
        if (p.nchunks > 1) {
            float *dst = p.part + ((oq + g) * p.nchunks + c) * 128 + 8 * sub;
            *reinterpret_cast<float4 *>(dst) = make_float4(o[0], o[1], o[2], o[3]);
            *reinterpret_cast<float4 *>(dst + 4) = make_float4(o[4], o[5], o[6], o[7]);
            if (sub == 0) p.ml[(oq + g) * p.nchunks + c] = make_float2(M, L);
        } else {
#pragma unroll
            for (int x = 0; x < 8; ++x) o[x] = L > 0.0f ? o[x] / L : 0.0f;   // (no token with a weight)
            store8(p, (oq + g) * 128 + 8 * sub, o);
        }
    }
}

// One workgroup per (sequence, query head): thread (chunk group cg, dimensions 8 sub ..): every 16th chunk, U of them
// requested at once, and the first ones' outputs before the largest score is known: the launch is the latency of its
// requests.  With the maxima read one after the other, ahead of the rest, attention over 4096 fp32 tokens of one head (256 chunks)
// took 12.3 us, 9.9 now; 16384 fp16 tokens (1024 chunks) 32.3 and 21.6; 517 tokens, 8 x 4 heads (33 chunks) 9.8 and 9.1.
template <int U>
__global__ __launch_bounds__(256) void direct_combine_kernel(const DirectParams p)
{
    __shared__ float red_s[16][128];
    __shared__ float2 ml_s[16];
    const int tid = threadIdx.x, sub = tid & 15, cg = tid >> 4;
    const int64_t oq = blockIdx.x;
    const float2 *ml = p.ml + oq * p.nchunks;
    const float *part = p.part + oq * p.nchunks * 128 + 8 * sub;
    float2 v[U];
    float f[U][8];
    // a chunk without tokens never wrote its partial output, and past the last chunk that one is read again: weight zero, value dropped
    auto weights_of = [&](int c0) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            v[i] = ml[min(c0 + 16 * i, p.nchunks - 1)];
            if (c0 + 16 * i >= p.nchunks) v[i].x = -INFINITY;
        }
    };
    auto outputs_of = [&](int c0) {
#pragma unroll
        for (int i = 0; i < U; ++i) load8<float>(part + (int64_t)min(c0 + 16 * i, p.nchunks - 1) * 128, f[i]);
    };
    float M = -INFINITY;
    for (int c0 = cg + 16 * U; c0 < p.nchunks; c0 += 16 * U) {
        weights_of(c0);
#pragma unroll
        for (int i = 0; i < U; ++i) M = fmaxf(M, v[i].x);
    }
    weights_of(cg);
    outputs_of(cg);
#pragma unroll
    for (int i = 0; i < U; ++i) M = fmaxf(M, v[i].x);
    float L = 0.0f, o[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) o[x] = 0.0f;
    for (int c0 = cg;;) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const bool have = v[i].x > -INFINITY;
            const float w = have ? __expf(v[i].x - M) : 0.0f;
            L = have ? fmaf(w, v[i].y, L) : L;
#pragma unroll
            for (int x = 0; x < 8; ++x) o[x] = have ? fmaf(w, f[i][x], o[x]) : o[x];
        }
        c0 += 16 * U;
        if (c0 >= p.nchunks) break;
        weights_of(c0);
        outputs_of(c0);
    }
    *reinterpret_cast<float4 *>(&red_s[cg][8 * sub]) = make_float4(o[0], o[1], o[2], o[3]);
    *reinterpret_cast<float4 *>(&red_s[cg][8 * sub + 4]) = make_float4(o[4], o[5], o[6], o[7]);
    if (sub == 0) ml_s[cg] = make_float2(M, L);
    __syncthreads();
    if (tid < 128) {
        float Mt = -INFINITY, Lt = 0.0f, v = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) Mt = fmaxf(Mt, ml_s[i].x);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float w = ml_s[i].x > -INFINITY ? __expf(ml_s[i].x - Mt) : 0.0f;
            Lt = fmaf(w, ml_s[i].y, Lt);
            v = fmaf(w, red_s[i][tid], v);
        }
        v = Lt > 0.0f ? v / Lt : 0.0f;
        if (p.out16) reinterpret_cast<__half *>(p.out)[oq * 128 + tid] = __float2half_rn(v);
        else reinterpret_cast<float *>(p.out)[oq * 128 + tid] = v;
    }
}

int64_t pairs_of(int32_t sK, int32_t snK, int32_t sV, int32_t snV) { return (int64_t)sK * snK + (int64_t)sV * snV; }

size_t r256(size_t v) { return (v + 255) & ~size_t(255); }

template <int GM, typename TD, typename TI, typename TC, int PV>
void launch_r(const DecodeArgs &a, const DirectParams &p, unsigned groups)
{
    if constexpr (sizeof(TD) == 2) {
        if (a.rope_base > 0.0f) {
            if (a.rope_layout == 0) hipLaunchKernelGGL((direct_kernel<GM, TD, TI, TC, PV, 1>), dim3(groups), dim3(kThreads), 0, a.stream, p);
            else hipLaunchKernelGGL((direct_kernel<GM, TD, TI, TC, PV, 2>), dim3(groups), dim3(kThreads), 0, a.stream, p);
            return;
        }
    }
    hipLaunchKernelGGL((direct_kernel<GM, TD, TI, TC, PV, 0>), dim3(groups), dim3(kThreads), 0, a.stream, p);
}
template <int GM, typename TD, typename TI, typename TC>
void launch_v(const DecodeArgs &a, const DirectParams &p, unsigned groups)
{
    if (a.sK % 8 == 0 && a.sV % 8 == 0) launch_r<GM, TD, TI, TC, 8>(a, p, groups);
    else if (a.sK % 4 == 0 && a.sV % 4 == 0) launch_r<GM, TD, TI, TC, 4>(a, p, groups);
    else if (a.sK % 2 == 0 && a.sV % 2 == 0) launch_r<GM, TD, TI, TC, 2>(a, p, groups);
    else launch_r<GM, TD, TI, TC, 1>(a, p, groups);
}
template <typename TD, typename TI, typename TC>
void launch_g(const DecodeArgs &a, const DirectParams &p, unsigned groups)
{
    if (a.G <= 1) launch_v<1, TD, TI, TC>(a, p, groups);
    else if (a.G <= 2) launch_v<2, TD, TI, TC>(a, p, groups);
    else if (a.G <= 4) launch_v<4, TD, TI, TC>(a, p, groups);
    else launch_v<8, TD, TI, TC>(a, p, groups);
}

}  // namespace

bool plan_decode_direct(const csr_decode_desc &d, DecodePlan *p)
{
    const bool paper = d.q_dtype == CSR_F16 && d.dict_dtype == CSR_F16 && d.coef_dtype == CSR_F16 && d.idx_dtype == CSR_I16;
    const bool full = d.q_dtype == CSR_F32 && d.dict_dtype == CSR_F32 && d.coef_dtype == CSR_F32 && d.idx_dtype == CSR_I32;
    p->direct = false;
    if (!(paper || full) || d.T < 1 || d.B < 1) return false;
    const int32_t snK = d.snK ? d.snK : 1, snV = d.snV ? d.snV : 1;
    const int64_t heads = (int64_t)d.B * d.Hkv;
    const int64_t gathers = heads * d.T * pairs_of(d.sK, snK, d.sV, snV);   // each a row of up to 256 (512) bytes
    if (gathers * (full ? 2 : 1) > kMostGathers) return false;
    // as many workgroups as are resident at a time (their registers allow four per CU for one query head, else two), of at
    // least one token per team
    int64_t want = (d.Hq == d.Hkv ? 1024 : 512) / heads;
    if (want < 1) want = 1;
    int64_t ct = (d.T + want - 1) / want;
    ct = (ct + kTeams - 1) / kTeams * kTeams;
    p->direct = true;
    p->direct_tokens = (int32_t)ct;
    p->direct_chunks = (int32_t)((d.T + ct - 1) / ct);
    const size_t BHq = (size_t)d.B * d.Hq;
    p->off_direct_ml = r256(BHq * p->direct_chunks * 128 * sizeof(float));
    const size_t total = p->off_direct_ml + r256(BHq * p->direct_chunks * sizeof(float2));
    if (total > p->total_bytes) p->total_bytes = total;
    return true;
}

hipError_t launch_decode_direct(const DecodeArgs &a, const DecodePlan &pl)
{
    DirectParams p{};
    char *ws = static_cast<char *>(a.workspace);
    p.q = a.q; p.DK = a.DK; p.DV = a.DV; p.idxK = a.idxK; p.coefK = a.coefK; p.idxV = a.idxV; p.coefV = a.coefV;
    p.seq_lens = a.seq_lens; p.out = a.out;
    p.part = reinterpret_cast<float *>(ws);
    p.ml = reinterpret_cast<float2 *>(ws + pl.off_direct_ml);
    p.T = a.T; p.rope_pos0 = a.rope_pos0; p.Hq = a.Hq; p.Hkv = a.Hkv; p.G = a.G; p.N = a.N; p.sK = a.sK; p.sV = a.sV;
    p.snK = a.snK; p.snV = a.snV; p.chunk_tokens = pl.direct_tokens; p.nchunks = pl.direct_chunks; p.out16 = a.out16;
    p.scale = a.scale; p.rope_base = a.rope_base;
    const unsigned groups = (unsigned)((int64_t)a.B * a.Hkv * pl.direct_chunks);
    if (a.q16) launch_g<__half, uint16_t, __half>(a, p, groups);
    else launch_g<float, int32_t, float>(a, p, groups);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || pl.direct_chunks == 1) return e;
    // a thread's chunks at once, as far as registers go, and no more requests than it has chunks
    const dim3 grid((unsigned)(a.B * a.Hq));
    if (pl.direct_chunks <= 16) hipLaunchKernelGGL(direct_combine_kernel<1>, grid, dim3(256), 0, a.stream, p);
    else if (pl.direct_chunks <= 64) hipLaunchKernelGGL(direct_combine_kernel<4>, grid, dim3(256), 0, a.stream, p);
    else if (pl.direct_chunks <= 128) hipLaunchKernelGGL(direct_combine_kernel<8>, grid, dim3(256), 0, a.stream, p);
    else hipLaunchKernelGGL(direct_combine_kernel<16>, grid, dim3(256), 0, a.stream, p);
    return hipGetLastError();
}

}  // namespace csr
