// Matching Pursuit encoder for launches too small to fill the chip with the prefill encoders' shapes, and for fp32 vectors
// and dictionaries of any launch size (gfx950).  Any N up to 65536, chunks of 32, 64 or 128 dimensions.
//
// The prefill encoder (encode_mfma.hip) gives a wave 64 vectors and the WHOLE dictionary: with some thousand vectors
// per dictionary that is one wave per SIMD on a part of the chip, and a wave alone is a chain of LDS reads, matrix
// instructions and bookkeeping that leaves the matrix cores idle two thirds of the time.  Here a workgroup of 8 waves
// owns 32 P vectors (of 128 dimensions) and the waves split the ATOMS: every wave screens all of the workgroup's
// vectors against every eighth 32-atom tile, so that an iteration's sweep is an eighth as long and small launches still
// have two waves on every SIMD of the CUs they use.
//
//   prepare   the dictionary as fp16 in the order the matrix instructions take it - [tile][fragment][lane][8 halves],
//             rows past N zero - so that every request of the sweep is one contiguous KiB; per slice of atoms the
//             largest norm and the largest |d_n - fp16(d_n)| (0 for fp16 dictionaries): the screening bound needs both.
//             A dictionary of at most 128 KB needs none of this: its tiles stay in the waves' registers (HELD).  One of at most
//             256 KB is prepared, and with one pass of vectors read once, three quarters into registers and a quarter into LDS.
//   sweep     hi . d^_n on the matrix cores, hi = fp16(R), d^ = fp16(d); atoms straight from L2 into registers, the next
//             tile requested while the present one is multiplied; no barrier.  Per lane (a vector's column, half of the
//             tile's rows) the three largest 16-atom groups with their tile in the low mantissa bits, and the 16
//             magnitudes of the best one as fp16, as in encode_mfma.hip.
//   select    the 16 lists of a vector (8 waves x 2 halves) meet in LDS; a team of DC / 8 lanes takes them, one reduction
//             finds the best group and how many atoms lie within the bound.  Two candidates (5 % of the steps in fp32, 3 %
//             in fp16) are compared exactly by the team; more than that (below 1 %) by the whole wave: every atom of
//             every candidate group (of a list whose third group is a candidate: every atom of the list), lowest atom on
//             ties.
//   update    the coefficient exactly on the atom itself, Eq.4 by the team (8 dimensions a lane), the residual back into LDS.
// Two barriers an iteration.  The bound: |hi . d^ - R . d| <= |lo||d| + |hi||d - d^| + accumulation =: delta / 2 with
// R = hi + lo; the decision is thus the fp32 one of Eq.2-3 whatever fp16 loses.
//
// CSR_ENCODE_AUTO chooses between this encoder and the one of the larger launches by size, so both have to give the same
// codes, also where two correlations agree to the last bits.  MODE says whose arithmetic the exact comparisons, the
// coefficient and the residual follow, operation by operation:
//   kValu   encode_valu.hip: fp32 residual, four chains over the dimensions (k mod 4)
//   kMfma   encode_mfma.hip: residual as hi + lo (two fp16), packed dot products; comparisons sum quarters of the vector,
//           coefficients halves
//   kRes    encode_resident.hip: fp32 residual; comparisons as kMfma on its hi and lo, coefficients in four chains per half
// The chains of a sum are spread over lanes (each chain keeps its order; the tree that joins them is the same).
//
// Bound by the sweep, which runs at the rate of a large library product (1.38 against 1.32 PFLOP/s), and behind it by the select phase, in
// which the matrix cores stand still: three prompts of 1571 tokens on 8 KV heads, 4096 atoms, spend 250 of a call's 329 us in the sweeps (160
// vectors a workgroup; 8 iterations of 31 us, 1.38 PFLOP/s) and 9 us an iteration in lists, select and update (10 with IEEE square roots for the
// bound, fp16 operands converted first and an undecided vector's reductions through the LDS; 2 x 4096 fp32 vectors, 1024 atoms 58.7 us a call, 56.0
// without).  With 64
// vectors a workgroup the same call made three generations and took 420 us.  Two vectors of a team selected together, so that
// their chains overlap, is slower (356): the select phase is bound by its instructions.  The rules in csr_api.hip say what
// this encoder replaces, with figures.
#include <atomic>

#include "csr_internal.h"
#include "encode_common.h"
#include "lane_ops.h"

namespace csr {
namespace {

using namespace enc;
using namespace lane;

enum Mode { kValu, kMfma, kRes };

constexpr int kTrack = 3;            // groups a list tracks
constexpr int kMaxSlices = 64;       // workgroups per dictionary in the preparation, at most

template <typename TE> __device__ __forceinline__ void load8e(const TE *p, float (&f)[8]);
template <> __device__ __forceinline__ void load8e<__half>(const __half *p, float (&f)[8]) { unpack8(*reinterpret_cast<const uint4 *>(p), f); }
template <> __device__ __forceinline__ void load8e<float>(const float *p, float (&f)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}

// Fragment-ordered fp16 copy of one dictionary and the slices' bounds: bound[dct][slice] = (max |d_n|, max |d_n - d^_n|).
// A group of DC / 8 lanes handles an atom, 8 dimensions a lane: piece p of the row is fragment p / 2, lane half p % 2.
template <typename TE, int DC>
__global__ __launch_bounds__(256) void wide_prepare_kernel(const TE *__restrict__ Dict, __half *__restrict__ frag,
                                                           float2 *__restrict__ bound, int32_t N, int32_t ntiles, int32_t slices)
{
    constexpr int L = DC / 8, kAtoms = 256 / L;
    __shared__ float2 red[4];
    const int dct = blockIdx.x, sl = blockIdx.y, tid = threadIdx.x;
    const int sub = tid % L;
    float n2 = 0.0f, e2 = 0.0f;
    for (int n = sl * kAtoms + tid / L; n < ntiles * 32; n += kAtoms * slices) {
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = 0.0f;
        if (n < N) load8e<TE>(Dict + ((int64_t)dct * N + n) * DC + sub * 8, f);
        half8 h;
        float a = 0.0f, b = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h[e] = (_Float16)f[e];
            const float d = f[e] - (float)h[e];   // beyond the fp16 range this is infinite: every vector is then undecided
            a = fmaf(f[e], f[e], a);
            b = fmaf(d, d, b);
        }
        const int64_t at = (((int64_t)dct * ntiles + (n >> 5)) * (DC / 16) + (sub >> 1)) * 64 + (n & 31) + 32 * (sub & 1);
        *reinterpret_cast<half8 *>(frag + at * 8) = h;
        n2 = fmaxf(n2, row_reduce<L>(a, OpAdd()));
        const float err = row_reduce<L>(b, OpAdd());
        e2 = fmaxf(e2, err >= 0.0f ? err : INFINITY);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        n2 = fmaxf(n2, __shfl_xor(n2, m, 64));
        e2 = fmaxf(e2, __shfl_xor(e2, m, 64));
    }
    if ((tid & 63) == 0) red[tid >> 6] = make_float2(n2, e2);
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            n2 = fmaxf(n2, red[w].x);
            e2 = fmaxf(e2, red[w].y);
        }
        bound[dct * kMaxSlices + sl] = make_float2(sqrtf(n2), sqrtf(e2));
    }
}

struct WideParams {
    const void *X, *Dict;
    const __half *frag;
    const float2 *bound;
    void *idx_out, *coef_out;
    float *res_norm2;
    int64_t T, m_first, M, x_stride_h, x_stride_t, code_stride_h;
    int32_t N, s, sn, dict_count, tiles_per_h, n_groups, ntiles, slices, idx16, coef_mode;
    uint32_t code_mask;
};

// What stands in LDS about a vector besides its residual
struct VectorState {
    float r2, delta;   // |R|^2, screening bound
    int32_t sexp, pad; // the residual is the vector's times 2^sexp
    int64_t code_at;   // first pair of its code; negative past the last vector
};

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b)   // the larger of each 16-bit half
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2v, a), __builtin_bit_cast(ushort2v, b)));
}
struct OpPkMax { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return pk_max(a, b); } };

// The residuals of a workgroup in LDS, [vector][dimension]: kMfma two fp16 planes (hi, lo), else fp32.  16-byte pieces are
// XOR-swizzled by the vector: the 32 columns of a fragment read have to spread over the banks.
template <int DC, int MODE, int TOK> struct Residuals {
    unsigned char *s;
    float unit;   // see opaque_one
    static constexpr int kBytes = TOK * DC * 4;
    static __device__ __forceinline__ int half_at(int tok, int p)    // piece of 8 halves
    {
        const int swz = DC == 128 ? (tok & 15) : DC == 64 ? ((tok >> 1) & 7) : ((tok >> 2) & 3);
        return tok * (DC * 2) + ((p ^ swz) << 4);
    }
    static __device__ __forceinline__ int word_at(int tok, int p)    // piece of 4 floats
    {
        const int swz = DC == 32 ? ((tok >> 1) & 7) : (tok & 15);
        return tok * (DC * 4) + ((p ^ swz) << 4);
    }
    // the fp16 operand, 8 dimensions
    __device__ __forceinline__ half8 hi8(int tok, int p) const
    {
        if constexpr (MODE == kMfma) {
            return *reinterpret_cast<const half8 *>(s + half_at(tok, p));
        } else {
            float v[8];
            full8(tok, p, v);
            return to_half8(v);
        }
    }
    // hi (part 0) or lo (part 1) as fp16
    __device__ __forceinline__ half8 part8(int tok, int p, int part) const
    {
        if constexpr (MODE == kMfma) {
            return *reinterpret_cast<const half8 *>(s + part * (TOK * DC * 2) + half_at(tok, p));
        } else {
            float v[8], l[8];
            full8(tok, p, v);
            const half8 h = to_half8(v);
            if (!part) return h;
#pragma unroll
            for (int e = 0; e < 8; ++e) l[e] = minus_half(v[e], h[e], unit);
            return to_half8(l);
        }
    }
    __device__ __forceinline__ void full8(int tok, int p, float (&v)[8]) const
    {
        if constexpr (MODE == kMfma) {
            const half8 h = part8(tok, p, 0), l = part8(tok, p, 1);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = plus_halves(h[e], l[e], unit);   // exact: 22 significant bits
        } else {
            const float4 x = *reinterpret_cast<const float4 *>(s + word_at(tok, 2 * p));
            const float4 y = *reinterpret_cast<const float4 *>(s + word_at(tok, 2 * p + 1));
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
        }
    }
    __device__ __forceinline__ float one(int tok, int k) const   // fp32 modes
    {
        return *reinterpret_cast<const float *>(s + word_at(tok, k >> 2) + ((k & 3) << 2));
    }
    // stores 8 dimensions; returns their share of |R - hi|^2
    __device__ __forceinline__ float put8(int tok, int p, const float (&v)[8]) const
    {
        const half8 h = to_half8(v);
        float d[8], l2 = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            d[e] = minus_half(v[e], h[e], unit);
            l2 = fmaf(d[e], d[e], l2);
        }
        if constexpr (MODE == kMfma) {
            *reinterpret_cast<half8 *>(s + half_at(tok, p)) = h;
            *reinterpret_cast<half8 *>(s + TOK * DC * 2 + half_at(tok, p)) = to_half8(d);
        } else {
            *reinterpret_cast<float4 *>(s + word_at(tok, 2 * p)) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4 *>(s + word_at(tok, 2 * p + 1)) = make_float4(v[4], v[5], v[6], v[7]);
        }
        return l2;
    }
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(__half v) { return __half2float(v); }

// kValu: R . d, one chain per k mod 4, by four neighbouring lanes (r = lane % 4); every one of them gets the sum
template <typename TE, int DC, typename RES>
__device__ __forceinline__ float dot_valu(const RES &res, int tok, const TE *__restrict__ row, int r)
{
    constexpr int K = DC / 4;
    TE d[K];
#pragma unroll
    for (int i = 0; i < K; ++i) d[i] = row[4 * i + r];
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) a = fmaf(res.one(tok, 4 * i + r), to_f32(d[i]), a);
    return row_reduce<4>(a, OpAdd());
}

// kMfma, kRes, comparison: quarters of the vector, hi and lo, two chains each; by eight neighbouring lanes (x: part,
// q: quarter), all of which get the sum
template <int DC, typename RES>
__device__ __forceinline__ float dot_compare(const RES &res, int tok, const __half *__restrict__ row, int x, int q)
{
    constexpr int kQ = DC / 32;
    float s0 = 0.0f, s1 = 0.0f;
    uint4 raw[kQ];
#pragma unroll
    for (int j = 0; j < kQ; ++j) raw[j] = *reinterpret_cast<const uint4 *>(row + (q * kQ + j) * 8);
#pragma unroll
    for (int j = 0; j < kQ; ++j) dot8(res.part8(tok, q * kQ + j, x), *reinterpret_cast<const half8 *>(&raw[j]), s0, s1);
    return row_reduce<8>(s0 + s1, OpAdd());
}

// kMfma, coefficient: halves of the vector, hi and lo, two chains each; by four neighbouring lanes (x: part, h: half)
template <int DC, typename RES>
__device__ __forceinline__ float dot_coef_mfma(const RES &res, int tok, const __half *__restrict__ row, int x, int h)
{
    constexpr int kF = DC / 16;
    float s0 = 0.0f, s1 = 0.0f;
    uint4 raw[kF];
#pragma unroll
    for (int j = 0; j < kF; ++j) raw[j] = *reinterpret_cast<const uint4 *>(row + (h * kF + j) * 8);
#pragma unroll
    for (int j = 0; j < kF; ++j) dot8(res.part8(tok, h * kF + j, x), *reinterpret_cast<const half8 *>(&raw[j]), s0, s1);
    return row_reduce<4>(s0 + s1, OpAdd());
}

// kRes, coefficient: halves of the vector, four chains each (dimension mod 4); by eight neighbouring lanes (r, h)
template <int DC, typename RES>
__device__ __forceinline__ float dot_coef_res(const RES &res, int tok, const __half *__restrict__ row, int r, int h)
{
    constexpr int K = DC / 8;
    __half d[K];
#pragma unroll
    for (int i = 0; i < K; ++i) d[i] = row[h * (DC / 2) + 4 * i + r];
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) a = fmaf(res.one(tok, h * (DC / 2) + 4 * i + r), __half2float(d[i]), a);
    return row_reduce<8>(a, OpAdd());
}

// The whole wave resolves ONE undecided vector: exact arg-max (lowest atom on ties) over the atoms of its candidate groups
// - of a list whose last tracked group is a candidate, over all atoms the list stands for.  Four lanes (q) take an atom of
// a 16-atom group.  `ls`: the lists as the vector's team holds them, first lane `lead`.
template <typename TE, int DC, int MODE, int W, int LL, typename RES>
__device__ __forceinline__ int resolve(const TE *__restrict__ Dh, int32_t N, int32_t ntiles, uint32_t code_mask, const RES &res,
                                       int tok, const uint4 (&ls)[LL], uint32_t thr_bits, int lead, int lane)
{
    constexpr int L = DC / 8, kLists = 2 * W;
    const int a = lane >> 2, q = lane & 3;
    constexpr int kQ = DC >= 32 ? DC / 32 : 1;
    half8 th[kQ], tl[kQ];
    if constexpr (MODE != kValu) {
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            th[j] = res.part8(tok, q * kQ + j, 0);
            tl[j] = res.part8(tok, q * kQ + j, 1);
        }
    }
    unsigned long long best = 0xffffffffull;   // (best_atom)
    auto take = [&](unsigned long long o) { best = o > best ? o : best; };
    auto eval_group = [&](int list, int code) {
        const int na = ((list >> 1) + W * code) * 32 + 4 * (list & 1) + 8 * (a >> 2) + (a & 3);
        const TE *row = Dh + (int64_t)min(na, N - 1) * DC;
        float c;
        if constexpr (MODE == kValu) {
            c = dot_valu<TE, DC>(res, tok, row, q);
        } else {
            uint4 raw[kQ];
#pragma unroll
            for (int j = 0; j < kQ; ++j) raw[j] = *reinterpret_cast<const uint4 *>(row + (q * kQ + j) * 8);
            float s0 = 0.0f, s1 = 0.0f, l0 = 0.0f, l1 = 0.0f;
#pragma unroll
            for (int j = 0; j < kQ; ++j) {
                dot8(th[j], *reinterpret_cast<const half8 *>(&raw[j]), s0, s1);
                dot8(tl[j], *reinterpret_cast<const half8 *>(&raw[j]), l0, l1);
            }
            c = row_reduce<4>((s0 + s1) + (l0 + l1), OpAdd());
        }
        const float ab = fabsf(c);
        if (na < N && ab >= 0.0f) take(((unsigned long long)__float_as_uint(ab) << 32) | (uint32_t)~na);   // (not a number: never)
    };
    const uint32_t team_mask = (uint32_t)((1ull << L) - 1);
#pragma unroll
    for (int k = 0; k < LL; ++k) {
        if (L * k >= kLists) continue;
        // a team may have more lanes than there are lists: the excess lanes hold none
        const uint32_t have = kLists - L * k >= L ? team_mask : (1u << (kLists - L * k)) - 1u;
        uint32_t todo = (uint32_t)(__ballot(ls[k].x >= thr_bits) >> lead) & have;
        const uint32_t two = (uint32_t)(__ballot(ls[k].y >= thr_bits) >> lead), whole = (uint32_t)(__ballot(ls[k].z >= thr_bits) >> lead);
        while (todo) {
            const int src = __ffs((int)todo) - 1;
            todo &= todo - 1;
            const int list = src + L * k;
            if ((whole >> src) & 1u) {
                const int w = list >> 1;
                const int tiles = w < ntiles ? (ntiles - w + W - 1) / W : 0;
#pragma unroll 1
                for (int c = 0; c < tiles; ++c) eval_group(list, c);
            } else {
                const int n_grp = 1 + ((two >> src) & 1u);
#pragma unroll 1
                for (int i = 0; i < n_grp; ++i) {
                    const uint32_t u = (uint32_t)__builtin_amdgcn_readlane((int)(i ? ls[k].y : ls[k].x), lead + src);
                    eval_group(list, (int)(u & code_mask));
                }
            }
        }
    }
    return best_atom(best);
}

// What a workgroup of P * 128 / DC blocks keeps in LDS: residuals | lists | state | HELD's bounds of the waves
template <int DC, int W, int P, int LDS_TILES> struct WideLds {
    static constexpr int kTok = 32 * (P * 128 / DC);
    static constexpr int kList = kTok * DC * 4, kState = kList + kTok * 2 * W * 16, kHeld = kState + kTok * (int)sizeof(VectorState);
    static constexpr int kTiles = kHeld + W * 8;
    static constexpr int kBytes = kTiles + W * LDS_TILES * DC * 64;
    static_assert(kBytes <= 160 * 1024, "a CU's LDS");
};

// Blocks whose fp16 operand a wave holds in registers for the whole sweep (the others are read from LDS for every tile): with
// five or six of them 256 registers take three or two.  (Four blocks of 128 dimensions spill 17 registers, 14 in the vector
// ALU's order, five of which three are held 11.)
template <int DC, int P> constexpr int blocks_held() { return P <= 4 ? P * 128 / DC : P == 5 ? 3 : 2; }

// W waves; P * 128 / DC blocks of 32 vectors.  HELD: the dictionary's first HELD tiles of every wave are read once and stay in
// registers for all iterations, the next LDS_TILES in the wave's part of the LDS: no dictionary traffic in the sweeps.
//   128 KB of fp16, 16 / (DC / 16) tiles in registers: read from the dictionary itself, no prepared copy, no scratch.
//   256 KB, 24 / (DC / 16) in registers and 8 / (DC / 16) in LDS, one pass of vectors: read from the prepared copy (every workgroup
//   would spend 10 us on the conversion of 512 KB of fp32).  With L1 and L2 in the way a sweep of 1024 atoms took 3.6 us, 2.7 now
//   (all four tiles of 128 dimensions in registers spill 59 of them): 2 x 4096 fp32 vectors, 1024 atoms, s = 8, with the attention that
//   follows 59.7 -> 56.1 us, 8 x 1024, s = 16 106 -> 91.5, fp16 8 x 1024, s = 8 45.9 -> 39.7, with 640 atoms 37.8 -> 34.0.
template <typename TE, int DC, int MODE, int W, int P, int HELD, int LDS_TILES>
__global__ __launch_bounds__(64 * W) void encode_wide_kernel(const WideParams p)
{
    constexpr int L = DC / 8;                    // lanes per team = 8-dimension pieces of a vector
    constexpr int kTeams = 64 * W / L;           // vectors per pass of the select phase
    constexpr int kBlk = P * 128 / DC;           // 32-vector blocks
    constexpr int kTok = 32 * kBlk;              // vectors per workgroup
    constexpr int kPass = kTok / kTeams;
    constexpr int kFrags = DC / 16;
    constexpr int kLists = 2 * W;                // lists of tracked groups per vector
    constexpr int kLl = kLists > L ? kLists / L : 1;   // lists a lane of a team takes (with fewer lists than lanes some take none)
    static_assert(kTok % kTeams == 0, "whole passes");
    static_assert(MODE == kValu || DC >= 64, "the teams' exact dot products");
    static_assert(P <= 4 || (MODE == kMfma && DC == 128), "operands from LDS: the residual's fp16 plane, whole vectors");
    constexpr int kInRegs = blocks_held<DC, P>();
    using RES = Residuals<DC, MODE, kTok>;
    using LDS = WideLds<DC, W, P, LDS_TILES>;
    static_assert(RES::kBytes == LDS::kList, "layout");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_s[];
    uint4(*list_s)[kLists] = reinterpret_cast<uint4(*)[kLists]>(lds_s + LDS::kList);   // (tracked groups, best group: atom << 16 | place of the second << 2 | flags)
    VectorState *state_s = reinterpret_cast<VectorState *>(lds_s + LDS::kState);
    float2 *held_s = reinterpret_cast<float2 *>(lds_s + LDS::kHeld);
    const RES res{lds_s, opaque_one()};

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hf = lane >> 5;
    const int sub = tid % L, team = tid / L;
    // each XCD gets a contiguous run of workgroups: those of one dictionary share an L2 (see encode_mfma.hip)
    int work = blockIdx.x;
    if ((int)blockIdx.x < (p.n_groups & ~7)) work = (blockIdx.x & 7) * (p.n_groups >> 3) + (blockIdx.x >> 3);
    const int dct = work / p.tiles_per_h, tile_wg = work - dct * p.tiles_per_h;
    const int dict = dct / p.sn, ch = dct - dict * p.sn;
    const TE *Dh = reinterpret_cast<const TE *>(p.Dict) + (int64_t)dct * p.N * DC;
    const uint4 *frag = reinterpret_cast<const uint4 *>(p.frag) + (int64_t)dct * p.ntiles * (kFrags * 64) + lane;

    uint32_t keep_mask;   // ~code_mask in a vector register: packing is then one v_and_or_b32
    asm volatile("v_mov_b32 %0, %1" : "=v"(keep_mask) : "s"(~p.code_mask));
    const float pack_q = (float)(p.code_mask + 1) * 1.1920929e-7f;

    const int my_tiles = wave < p.ntiles ? (p.ntiles - wave + W - 1) / W : 0;
    auto load_tile = [&](int i, uint4 (&a)[kFrags]) {
        const uint4 *src = frag + (int64_t)(wave + W * i) * (kFrags * 64);
#pragma unroll
        for (int j = 0; j < kFrags; ++j) a[j] = src[j * 64];
    };
    constexpr int kHeld = HELD ? HELD : 1;
    // this lane's first fragment of the wave's tiles in LDS; not known from one iteration to the next, or they would be read once, into
    // registers that are not there
    uint32_t lds_at = (uint32_t)(LDS::kTiles + wave * (LDS_TILES * kFrags * 1024) + lane * 16);
    uint4 a0[kHeld][kFrags];   // HELD: the wave's tiles; else the first of the two buffers of the sweep
    float dmax = 0.0f, derr = 0.0f;
    if constexpr (HELD > 0 && LDS_TILES == 0) {
#pragma unroll
        for (int i = 0; i < kHeld; ++i) {
            const int n = (wave + W * i) * 32 + col;
            float n2 = 0.0f, e2 = 0.0f;
#pragma unroll
            for (int j = 0; j < kFrags; ++j) {
                float f[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = 0.0f;
                if (n < p.N) load8e<TE>(Dh + (int64_t)n * DC + (2 * j + hf) * 8, f);
                half8 h;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    h[e] = (_Float16)f[e];
                    const float d = f[e] - (float)h[e];
                    n2 = fmaf(f[e], f[e], n2);
                    e2 = fmaf(d, d, e2);
                }
                a0[i][j] = *reinterpret_cast<const uint4 *>(&h);
            }
            n2 += xchg32f(n2, hf);
            e2 += xchg32f(e2, hf);
            dmax = fmaxf(dmax, n2);
            derr = fmaxf(derr, e2 >= 0.0f ? e2 : INFINITY);
        }
        dmax = wave_max(dmax);
        derr = wave_max(derr);
        if (lane == 0) held_s[wave] = make_float2(dmax, derr);
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) {
            dmax = fmaxf(dmax, held_s[w].x);
            derr = fmaxf(derr, held_s[w].y);
        }
        dmax = sqrtf(dmax);
        derr = sqrtf(derr) * 1.001f;
    } else {
#pragma unroll
        for (int i = 0; i < kHeld; ++i)
            if (i < my_tiles) load_tile(i, a0[i]);
#pragma unroll
        for (int i = 0; i < LDS_TILES; ++i)
            if (kHeld + i < my_tiles) {
                uint4 a1[kFrags];
                load_tile(kHeld + i, a1);
#pragma unroll
                for (int j = 0; j < kFrags; ++j) *reinterpret_cast<uint4 *>(lds_s + lds_at + (i * kFrags + j) * 1024) = a1[j];   // only this lane reads it
            }
        if (lane < p.slices) {
            const float2 b = p.bound[dct * kMaxSlices + lane];
            dmax = b.x;
            derr = b.y;
        }
        dmax = wave_max(dmax);
        derr = wave_max(derr) * 1.001f;   // |hi| <= 1.001 |R|
    }

    // ---- the vectors: scaled by a power of two that brings max |x_k| into [2^11, 2^12) ----------------------------------
    auto bound_of = [&](float lo2, float n2) { return screen_delta(dmax, lo2, n2) + 2.000002f * derr * __builtin_amdgcn_sqrtf(n2); };
#pragma unroll 1
    for (int q = 0; q < kPass; ++q) {
        const int tok = q * kTeams + team;
        const int64_t m = p.m_first + (int64_t)tile_wg * kTok + tok;
        const bool valid = m < p.M;
        const int64_t mc = valid ? m : p.M - 1;   // past the end: a zero vector, for which nothing is resolved, and never stored
        const int rep = (int)(mc / p.T);
        const int64_t t = mc - rep * p.T, h = (int64_t)rep * p.dict_count + dict;
        float R[8];
        load8e<TE>(reinterpret_cast<const TE *>(p.X) + h * p.x_stride_h + t * p.x_stride_t + ch * DC + sub * 8, R);
#pragma unroll
        for (int e = 0; e < 8; ++e) R[e] = valid ? R[e] : 0.0f;
        float amax = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(R[e]));
        amax = row_reduce<L>(amax, OpMax());
        int ex = 0;
        if (amax > 0.0f && amax < INFINITY) {
            (void)frexpf(amax, &ex);
            ex = 12 - ex;
        }
        float n2 = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            R[e] = ldexpf(R[e], ex);
            n2 = fmaf(R[e], R[e], n2);
        }
        n2 = row_reduce<L>(n2, OpAdd());
        const float lo2 = row_reduce<L>(res.put8(tok, sub, R), OpAdd());
        if (sub == 0) {
            VectorState v;
            v.r2 = n2; v.delta = bound_of(lo2, n2); v.sexp = ex; v.pad = 0;
            v.code_at = valid ? h * p.code_stride_h + (t * p.sn + ch) * p.s : -1;
            state_s[tok] = v;
        }
    }
    __syncthreads();

#pragma unroll 1
    for (int g = 0; g < p.s; ++g) {
        // ---- screen ------------------------------------------------------------------------------------------------
        {
            half8 hi[kInRegs][kFrags];
            uint32_t u[kBlk][kTrack], keep[kBlk][8];
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
                if (b < kInRegs) {
#pragma unroll
                    for (int j = 0; j < kFrags; ++j) hi[b < kInRegs ? b : 0][j] = res.hi8(b * 32 + col, 2 * j + hf);
                }
#pragma unroll
                for (int k = 0; k < kTrack; ++k) u[b][k] = 0u;
#pragma unroll
                for (int r = 0; r < 8; ++r) keep[b][r] = 0u;
            }
            // `used(j)`: called once fragment j of the tile is multiplied for the last time
            auto sweep = [&](int i, const uint4 (&a)[kFrags], auto used) {
                const uint32_t code = (uint32_t)i;
                // where the first fragment of this lane's column stands; not known from one tile to the next, or the compiler
                // would read the blocks' operands once, ahead of all tiles, into registers that are not there
                uint32_t hi_at = (uint32_t)RES::half_at(col, hf);
                if constexpr (kInRegs < kBlk) asm volatile("" : "+v"(hi_at));
#pragma unroll
                for (int b = 0; b < kBlk; ++b) {
                    floatx16 acc;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
                    for (int j = 0; j < kFrags; ++j) {
                        half8 v;
                        if (b < kInRegs) v = hi[b < kInRegs ? b : 0][j];
                        else v = *reinterpret_cast<const half8 *>(lds_s + b * (32 * DC * 2) + (hi_at ^ (uint32_t)(j << 5)));
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const half8 *>(&a[j]), v, acc, 0, 0, 0);
                        if (b == kBlk - 1) used(j);
                    }
                    float m = 0.0f;
#pragma unroll
                    for (int r = 0; r < 16; r += 2) m = fmaxf(fmaxf(m, fabsf(acc[r])), fabsf(acc[r + 1]));
                    const uint32_t v = (__float_as_uint(m) & keep_mask) | code;
                    if (v > u[b][0]) {
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const auto pk = __builtin_amdgcn_cvt_pkrtz(fabsf(acc[2 * r]), fabsf(acc[2 * r + 1]));
                            keep[b][r] = *reinterpret_cast<const uint32_t *>(&pk);
                        }
                    }
                    const uint32_t n2 = umed3(u[b][1], u[b][2], v), n1 = umed3(u[b][0], u[b][1], v);
                    u[b][0] = max(u[b][0], v);
                    u[b][1] = n1;
                    u[b][2] = n2;
                }
            };
            auto none = [](int) {};
            if constexpr (HELD > 0) {
#pragma unroll
                for (int i = 0; i < kHeld; ++i) {
                    if (i < my_tiles) sweep(i, a0[i], none);
                    if constexpr (LDS_TILES > 0) __builtin_amdgcn_sched_barrier(0);   // accumulators of one tile at a time
                }
                asm volatile("" : "+v"(lds_at));
#pragma unroll
                for (int i = 0; i < LDS_TILES; ++i)
                    if (kHeld + i < my_tiles) {
                        uint4 a1[kFrags];
#pragma unroll
                        for (int j = 0; j < kFrags; ++j) a1[j] = *reinterpret_cast<const uint4 *>(lds_s + lds_at + (i * kFrags + j) * 1024);
                        sweep(kHeld + i, a1, none);
                    }
            } else if constexpr (P > 2) {
                // a tile's fragments make room for the next tile's one by one (behind the last tile the next sweep's first):
                // a wave waits for them a little, while the other one of its SIMD multiplies
                for (int i = 0; i < my_tiles; ++i) {
                    const uint4 *next = frag + (int64_t)(wave + W * (i + 1 < my_tiles ? i + 1 : 0)) * (kFrags * 64);
                    sweep(i, a0[0], [&](int j) { a0[0][j] = next[j * 64]; });
                }
            } else {
                uint4 a1[kFrags];
                for (int i = 0; i < my_tiles; i += 2) {
                    if (i + 1 < my_tiles) load_tile(i + 1, a1);
                    sweep(i, a0[0], none);
                    if (i + 1 < my_tiles) {
                        if (i + 2 < my_tiles) load_tile(i + 2, a0[0]);
                        sweep(i + 1, a1, none);
                    }
                }
                if (my_tiles > 0) load_tile(0, a0[0]);   // the next sweep's first tile, behind the select phase
            }
            // the best group as it was kept: where its two largest values stand, whether the second (1) and the third (2)
            // are too close to the first to tell
#pragma unroll
            for (int b = 0; b < kBlk; ++b) {
                uint32_t k1 = 0u, k2 = 0u, k3 = 0u;   // three largest kept values (fp16 bits), their places in the low half
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const uint32_t w = keep[b][r >> 1];
                    const uint32_t v = ((r & 1) ? (w & 0xffff0000u) : (w << 16)) | (uint32_t)r;
                    k3 = umed3(k2, k3, v);
                    k2 = umed3(k1, k2, v);
                    k1 = max(k1, v);
                }
                auto kept = [](uint32_t k) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(k >> 16)); };
                const int tok = b * 32 + col, li = wave * 2 + hf;
                // kept values were rounded toward zero to 11 bits
                const float ba = kept(k1), least = ba - state_s[tok].delta - ba * 9.765625e-4f;
                const uint32_t p1 = k1 & 15u, p2 = k2 & 15u;
                const uint32_t n = (uint32_t)(wave + W * (int)(u[b][0] & p.code_mask)) * 32 + 8 * (p1 >> 2) + (p1 & 3) + 4 * hf;
                list_s[tok][li ^ (tok & (kLists - 1))] =
                    make_uint4(u[b][0], u[b][1], u[b][2],
                               (n << 16) | (p2 << 2) | (!(kept(k2) < least) ? 1u : 0u) | (!(kept(k3) < least) ? 2u : 0u));
            }
        }
        __syncthreads();

        // ---- select and update ---------------------------------------------------------------------------------------
#pragma unroll 1
        for (int q = 0; q < kPass; ++q) {
            const int tok = q * kTeams + team;
            const VectorState st = state_s[tok];
            uint4 ls[kLl];
            uint32_t bu = 0u;
#pragma unroll
            for (int k = 0; k < kLl; ++k) {
                ls[k] = sub + L * k < kLists ? list_s[tok][((sub + L * k) ^ tok) & (kLists - 1)] : make_uint4(0u, 0u, 0u, 0u);
                bu = max(bu, ls[k].x);
            }
            bu = row_reduce<L>(bu, OpMaxU());
            const float A = __uint_as_float(bu & ~p.code_mask);
            const float thr = (A - st.delta) * (1.0f - 2.0f * pack_q);
            const uint32_t thr_bits = thr > 0.0f ? (__float_as_uint(thr) & ~p.code_mask) : 0u;
            const bool zero = !(st.r2 > 0.0f);
            // Candidates: the best group's largest atom of every list within the bound, its second one if that is too close
            // to tell.  Up to two of them are decided by the team; count: how many, + 256 if more than these could matter.
            uint32_t count = 0u, ends = 0u;   // ends: largest candidate << 16 | 65535 - smallest candidate
#pragma unroll
            for (int k = 0; k < kLl; ++k) {
                if (sub + L * k < kLists && ls[k].x >= thr_bits) {
                    const uint32_t w = ls[k].w, n1 = w >> 16, p2 = (w >> 2) & 15u;
                    const uint32_t n2 = (w & 1u) ? (n1 & ~27u) + 8 * (p2 >> 2) + (p2 & 3) : n1;
                    count += 1u + (w & 1u) + (((w & 2u) || ls[k].y >= thr_bits) ? 256u : 0u);
                    ends = pk_max(ends, (max(n1, n2) << 16) | (65535u - min(n1, n2)));
                }
            }
            ends = row_reduce<L>(ends, OpPkMax());
            count = row_reduce<L>(count, OpAdd());
            int n_lo = min(65535 - (int)(ends & 0xffffu), p.N - 1), n_hi = min((int)(ends >> 16), p.N - 1);
            // vectors with more candidates, one at a time, by the whole wave
            unsigned long long todo = __ballot(!zero && count != 1u && count != 2u && sub == 0);
            while (todo) {
                const int lead = __ffsll((long long)todo) - 1;   // first lane of the vector's team
                todo &= todo - 1;
                const int n_res = resolve<TE, DC, MODE, W>(Dh, p.N, p.ntiles, p.code_mask, res, q * kTeams + wave * (64 / L) + lead / L, ls,
                                                           (uint32_t)__builtin_amdgcn_readlane((int)thr_bits, lead), lead, lane);
                if (lane / L == lead / L) n_lo = n_hi = n_res;
            }
            if (zero) n_lo = n_hi = 0;
            // this lane's piece of both rows, for Eq.4
            float d[8], d_hi[8];
            load8e<TE>(Dh + (int64_t)n_lo * DC + sub * 8, d);
            load8e<TE>(Dh + (int64_t)n_hi * DC + sub * 8, d_hi);
            const TE *row_lo = Dh + (int64_t)n_lo * DC, *row_hi = Dh + (int64_t)n_hi * DC;
            // coefficients of both, by one half of the team each (32-dimensional vectors: one after the other)
            const bool upper = sub >= L / 2;
            float c, c_hi;
            bool take_hi;
            if constexpr (MODE == kValu) {
                if constexpr (L == 4) {
                    c = dot_valu<TE, DC>(res, tok, row_lo, sub);
                    c_hi = dot_valu<TE, DC>(res, tok, row_hi, sub);
                } else {
                    const float own = dot_valu<TE, DC>(res, tok, upper ? row_hi : row_lo, sub & 3);
                    const float oth = L == 16 ? dpp_mov<0x140>(own) : dpp_mov<0x141>(own);
                    c = upper ? oth : own;
                    c_hi = upper ? own : oth;
                }
                take_hi = fabsf(c_hi) > fabsf(c);   // the lower atom on ties
            } else {
                take_hi = false;
                if (__ballot(n_lo != n_hi)) {
                    float v_lo, v_hi;
                    if constexpr (L == 16) {
                        const float own = dot_compare<DC>(res, tok, upper ? row_hi : row_lo, sub & 1, (sub >> 1) & 3);
                        const float oth = dpp_mov<0x140>(own);
                        v_lo = upper ? oth : own;
                        v_hi = upper ? own : oth;
                    } else {
                        v_lo = dot_compare<DC>(res, tok, row_lo, sub & 1, (sub >> 1) & 3);
                        v_hi = dot_compare<DC>(res, tok, row_hi, sub & 1, (sub >> 1) & 3);
                    }
                    take_hi = fabsf(v_hi) > fabsf(v_lo);
                }
                if constexpr (MODE == kMfma) {
                    const float own = dot_coef_mfma<DC>(res, tok, upper ? row_hi : row_lo, sub & 1, (sub >> 1) & 1);
                    const float oth = L == 16 ? dpp_mov<0x140>(own) : dpp_mov<0x141>(own);
                    c = upper ? oth : own;
                    c_hi = upper ? own : oth;
                } else {
                    c = c_hi = dot_coef_res<DC>(res, tok, take_hi ? row_hi : row_lo, sub & 3, (sub >> 2) & 1);
                }
            }
            const int n = take_hi ? n_hi : n_lo;
            c = take_hi ? c_hi : c;
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e] = take_hi ? d_hi[e] : d[e];
            if (zero) c = 0.0f;
            // closed loop: what Eq.4 subtracts is the coefficient as it will be stored (rounded in the input's scale)
            if (coef_rounds_in_loop(p.coef_mode)) c = ldexpf(__half2float(__float2half_rn(ldexpf(c, -st.sexp))), st.sexp);
            if (st.code_at >= 0) {
                const int64_t o = st.code_at + g;
                if (sub == 0) {
                    if (p.idx16) reinterpret_cast<uint16_t *>(p.idx_out)[o] = (uint16_t)n;
                    else reinterpret_cast<int32_t *>(p.idx_out)[o] = n;
                } else if (sub == 1) {
                    const float co = ldexpf(c, -st.sexp);
                    if (coef_is_f16(p.coef_mode)) reinterpret_cast<__half *>(p.coef_out)[o] = __float2half_rn(co);
                    else reinterpret_cast<float *>(p.coef_out)[o] = co;
                }
            }
            float R[8], n2 = 0.0f;
            res.full8(tok, sub, R);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                R[e] = fmaf(-c, d[e], R[e]);   // Eq.4
                n2 = fmaf(R[e], R[e], n2);
            }
            n2 = row_reduce<L>(n2, OpAdd());
            int sexp = st.sexp;
            // a residual that shrank or grew a lot is scaled again, so that hi and its remainder stay normal fp16 numbers
            if ((n2 < 65536.0f && n2 > 0.0f) || (n2 >= 1073741824.0f && n2 < INFINITY)) {
                int e2 = 0;
                (void)frexpf(n2, &e2);
                const int k2 = 14 - (e2 + 1) / 2;
                const float sc = ldexpf(1.0f, k2);
#pragma unroll
                for (int e = 0; e < 8; ++e) R[e] *= sc;
                n2 *= sc * sc;
                sexp += k2;
            }
            wave_lds_fence();   // every lane of the team has read the old residual
            const float lo2 = row_reduce<L>(res.put8(tok, sub, R), OpAdd());
            if (sub == 0) {
                state_s[tok].r2 = n2;
                state_s[tok].delta = bound_of(lo2, n2);
                state_s[tok].sexp = sexp;
            }
        }
        __syncthreads();
    }
    if (p.res_norm2) {
#pragma unroll 1
        for (int tok = tid; tok < kTok; tok += 64 * W) {
            const int64_t m = p.m_first + (int64_t)tile_wg * kTok + tok;
            if (m >= p.M) break;
            const int rep = (int)(m / p.T);
            p.res_norm2[(((int64_t)rep * p.dict_count + dict) * p.T + (m - rep * p.T)) * p.sn + ch] =
                ldexpf(state_s[tok].r2, -2 * state_s[tok].sexp);
        }
    }
}

size_t r256(size_t v) { return (v + 255) & ~size_t(255); }

struct WidePlan {
    int32_t ntiles, slices;
    size_t off_bound, total;
};

// The encoder whose arithmetic CSR_ENCODE_AUTO's codes follow at this shape (see MODE)
Mode wide_mode(const EncodeArgs &a)
{
    if (encode_resident_supported(a)) return kRes;
    return encode_mfma_supported(a) && a.d >= 64 ? kMfma : kValu;
}

// How many passes P of 4096 / d vectors a workgroup takes.  A generation of workgroups (one per CU) costs about P + 0.4 passes
// (16 dictionaries, s = 8, 4096 atoms, one full generation with the preparation: 107, 161, 221, 298, 360, 423 us for P = 1 .. 6; 1024 atoms,
// which one pass holds on the CU (a pass is then 34 of them, two are 62), 44, 72, 97, 122, 142, 164; fp32 114, 170, 232, 307 and 44, 73, 98, 131 for P = 1 .. 4; 64 dimensions, 2048 atoms
// 48, 89, 128 and 54, 98, 141), so what counts is how many generations a launch
// makes: three prompts of 1571 tokens on 8 KV heads are 592 workgroups of 64 vectors, three generations, or 240 of 160, one.
struct WidePasses {
    int P;
    float cost;
};
WidePasses wide_passes(const EncodeArgs &a, int64_t vectors)
{
    const Mode mode = wide_mode(a);
    const int most = a.d == 32 ? 1 : mode == kRes ? 2 : a.d == 64 ? 3 : mode == kMfma ? 6 : 4;
    const int64_t dicts = (int64_t)a.dict_count * a.sn;
    WidePasses best{1, 0.0f};
    for (int P = 1; P <= most; ++P) {
        const int64_t tok = (int64_t)P * 4096 / a.d, groups = (vectors + tok - 1) / tok * dicts;
        const float cost = (float)((groups + kCus - 1) / kCus) * ((float)P + 0.4f);
        if (P == 1 || cost < best.cost) best = {P, cost};
    }
    return best;
}

// Whether a workgroup holds the dictionary (see HELD); with more than one pass of vectors there are no registers for it.  What is held is read
// ahead of the first sweep instead of during it, so that it takes a few iterations to pay, more of them with tiles in LDS (above 192 KB).
// us, not held -> held: one pair, 1024 atoms, 2 x 200 vectors fp16 11.1 -> 13.0, fp32 11.9 -> 13.6; 300 x 33 fp16 56 -> 63; 544 atoms 10.0 -> 9.8
// and 36.5 -> 37.0.  Two, 1024 atoms 16.2 -> 16.8, 16.8 -> 17.8, 71.0 -> 73.4; 544 atoms 13.6 -> 12.6, 14.6 -> 13.5, 47.9 -> 46.1.  Three, 1024
// atoms 20.9 -> 20.2, 21.6 -> 21.3, 85.3 -> 84.6; 544 atoms 17.4 -> 15.4, 16.4 -> 15.2, 58.0 -> 54.6.
bool held_on_the_cu(const EncodeArgs &a)
{
    const int64_t bytes = (int64_t)((a.N + 31) / 32) * (a.d * 64);
    return bytes <= (a.s >= 3 ? 256 : a.s == 2 ? 192 : 0) * 1024;
}

WidePlan plan_wide(const EncodeArgs &a)
{
    WidePlan pl{};
    const size_t dicts = (size_t)a.dict_count * a.sn;
    pl.ntiles = (a.N + 31) / 32;
    const int atoms_per_pass = 2048 / a.d;   // of one workgroup of the preparation
    const int passes = (pl.ntiles * 32 + atoms_per_pass - 1) / atoms_per_pass;
    pl.slices = passes < kMaxSlices ? passes : kMaxSlices;
    pl.off_bound = r256(dicts * pl.ntiles * 32 * a.d * sizeof(__half));
    pl.total = pl.off_bound + r256(dicts * kMaxSlices * sizeof(float2));
    return pl;
}

template <typename TE, int DC, int MODE, int P, int HELD = 0, int LDS_TILES = 0>
hipError_t launch_p(const EncodeArgs &a, WideParams &p)
{
    constexpr int W = 8, kTok = 32 * (P * 128 / DC);
    const int64_t tiles = (p.M - p.m_first + kTok - 1) / kTok, groups = tiles * a.dict_count * a.sn;
    if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
    p.tiles_per_h = (int32_t)tiles;
    p.n_groups = (int32_t)groups;
    int bits = 0;
    while ((1 << bits) < (p.ntiles + W - 1) / W) ++bits;
    p.code_mask = (1u << bits) - 1u;
    constexpr int kLds = WideLds<DC, W, P, LDS_TILES>::kBytes;
    const int lds = p.ntiles <= HELD * W ? WideLds<DC, W, P, 0>::kBytes : kLds;   // no wave has a tile there
    if constexpr (kLds > 64 * 1024) {   // above the default limit: per device, once
        static std::atomic<bool> attr_set[64];
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        if (!attr_set[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(encode_wide_kernel<TE, DC, MODE, W, P, HELD, LDS_TILES>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
            if (e != hipSuccess) return e;
            attr_set[dev].store(true, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL((encode_wide_kernel<TE, DC, MODE, W, P, HELD, LDS_TILES>), dim3((unsigned)groups), dim3(64 * W), lds, a.stream, p);
    return hipGetLastError();
}

template <typename TE, int DC, int MODE>
hipError_t launch_m(const EncodeArgs &a)
{
    constexpr int kTileRegs = DC / 16;   // 16-byte registers of a tile
    const WidePlan pl = plan_wide(a);
    char *ws = static_cast<char *>(a.workspace);
    __half *frag = reinterpret_cast<__half *>(ws);
    float2 *bound = reinterpret_cast<float2 *>(ws + pl.off_bound);
    const int dicts = a.dict_count * a.sn;
    WideParams p{};
    p.X = a.X; p.Dict = a.D; p.frag = frag; p.bound = bound; p.idx_out = a.idx; p.coef_out = a.coef; p.res_norm2 = a.res_norm2;
    p.T = a.T; p.m_first = a.m_first; p.M = a.m_end;
    p.x_stride_h = a.x_stride_h; p.x_stride_t = a.x_stride_t; p.code_stride_h = a.code_stride_h;
    p.N = a.N; p.s = a.s; p.sn = a.sn; p.dict_count = a.dict_count; p.ntiles = pl.ntiles; p.slices = pl.slices;
    p.idx16 = a.idx16; p.coef_mode = (a.coef16 ? kCoefF16 : 0) | (a.closed_loop ? kCoefClosed : 0);
    const int P = wide_passes(a, a.m_end - a.m_first).P;
    if constexpr (MODE == kRes) {
        return P == 2 ? launch_p<TE, DC, MODE, 2, 16 / kTileRegs>(a, p) : launch_p<TE, DC, MODE, 1, 16 / kTileRegs>(a, p);
    } else {
        hipLaunchKernelGGL((wide_prepare_kernel<TE, DC>), dim3((unsigned)dicts, (unsigned)pl.slices), dim3(256), 0, a.stream,
                           (const TE *)a.D, frag, bound, a.N, pl.ntiles, pl.slices);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if constexpr (MODE == kMfma && DC == 128) {
            if (P == 6) return launch_p<TE, DC, MODE, 6>(a, p);
            if (P == 5) return launch_p<TE, DC, MODE, 5>(a, p);
        }
        if constexpr (DC == 128) {
            if (P == 4) return launch_p<TE, DC, MODE, 4>(a, p);
        }
        if constexpr (DC > 32) {
            if (P == 3) return launch_p<TE, DC, MODE, 3>(a, p);
            if (P == 2) return launch_p<TE, DC, MODE, 2>(a, p);
        }
        if (held_on_the_cu(a)) return launch_p<TE, DC, MODE, 1, 24 / kTileRegs, 8 / kTileRegs>(a, p);
        return launch_p<TE, DC, MODE, 1>(a, p);
    }
}

template <typename TE>
hipError_t launch_valu_order(const EncodeArgs &a)
{
    return a.d == 32 ? launch_m<TE, 32, kValu>(a) : a.d == 64 ? launch_m<TE, 64, kValu>(a) : launch_m<TE, 128, kValu>(a);
}

}  // namespace

bool encode_wide_supported(const EncodeArgs &a)
{
    return (a.d == 32 || a.d == 64 || a.d == 128) && a.N >= 1 && a.N <= 65536 && a.dict_count >= 1;
}

size_t encode_wide_workspace_bytes(const EncodeArgs &a) { return wide_mode(a) == kRes ? 0 : plan_wide(a).total; }

// 0.4: the preparation of the dictionary, where there is one
float encode_wide_cost(const EncodeArgs &a, int64_t vectors) { return (wide_mode(a) == kRes ? 0.0f : 0.4f) + wide_passes(a, vectors).cost; }

hipError_t launch_encode_wide(const EncodeArgs &a)
{
    switch (wide_mode(a)) {
        case kRes: return a.d == 64 ? launch_m<__half, 64, kRes>(a) : launch_m<__half, 128, kRes>(a);
        case kMfma: return a.d == 64 ? launch_m<__half, 64, kMfma>(a) : launch_m<__half, 128, kMfma>(a);
        default: return a.f16 ? launch_valu_order<__half>(a) : launch_valu_order<float>(a);
    }
}

}  // namespace csr
