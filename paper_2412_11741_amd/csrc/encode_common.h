// Device helpers and the screening bound shared by the matrix-core Matching Pursuit encoders (encode_mfma.hip,
// encode_resident.hip, encode_split.hip, encode_gram.hip, encode_gramstep.hip).
#pragma once
#include "csr_internal.h"
#include "lane_ops.h"

namespace csr {
namespace enc {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// fp32 accumulation error of a 128-term dot product of exact fp16 products, relative to |hi||d|:
// 129 roundings of at most 2^-23 each (this also covers accumulators that truncate).
constexpr float kGammaAcc = 1.6e-5f;

// The bound of the screening sweep (Eq.2-3 decided on hi . d_n instead of R . d_n, R = hi + lo):
//   |hi . d_n - R . d_n| <= |lo| |d_n| + kGammaAcc |R| |d_n|  =: delta / 2  for every atom n,
// so the atom of largest true |correlation| lies within delta of the largest screened value.  dmax: the largest
// atom norm of the dictionary; lo2 = |lo|^2, r2 = |R|^2.
// The hardware's square roots (1 ulp), and |R|^2 need only be known to 2^-8: the factors cover both.
__device__ __forceinline__ float screen_delta(float dmax, float lo2, float r2)
{
    return 2.0f * dmax * (1.000001f * __builtin_amdgcn_sqrtf(lo2) + 1.01f * kGammaAcc * __builtin_amdgcn_sqrtf(r2));
}

// fp16 operands of an fp32 sum in one instruction (v_fma_mix_f32), by a product with a one that the compiler does not know to be one: it
// would convert them first.  The sums are the same: a product with one is exact.
__device__ __forceinline__ float opaque_one()
{
    float one;
    asm volatile("s_mov_b32 %0, 1.0" : "=s"(one));
    return one;
}
__device__ __forceinline__ float minus_half(float r, _Float16 h, float one) { return fmaf(-(float)h, one, r); }
__device__ __forceinline__ float plus_halves(_Float16 h, _Float16 l, float one) { return fmaf((float)h, one, (float)l); }

__device__ __forceinline__ half8 to_half8(const float (&f)[8])   // v_cvt_pk_f16_f32, two at a time
{
    typedef float float2v __attribute__((ext_vector_type(2)));
    half8 h;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const half2v p = __builtin_convertvector((float2v{f[e], f[e + 1]}), half2v);
        h[e] = p[0];
        h[e + 1] = p[1];
    }
    return h;
}

__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c)
{
    return max(min(a, b), min(max(a, b), c));
}

// value of the other lane of the pair (lane ^ 32)
__device__ __forceinline__ uint32_t xchg32(uint32_t v, int hf)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return hf ? r[0] : r[1];
}
__device__ __forceinline__ float xchg32f(float v, int hf) { return __uint_as_float(xchg32(__float_as_uint(v), hf)); }

__device__ __forceinline__ void unpack8(const uint4 &raw, float (&f)[8])
{
    const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 v = __half22float2(h2[j]);
        f[2 * j] = v.x;
        f[2 * j + 1] = v.y;
    }
}

// 8 dimensions of a dot product: a (fp16 x 8) . d (fp16 x 8), two fp32 accumulators; the products of fp16 pairs
// are exact in fp32
__device__ __forceinline__ void dot8(const half8 &a, const half8 &d, float &s0, float &s1)
{
    s0 = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(d, d, 0, 1), s0, false);
    s1 = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(d, d, 2, 3), s1, false);
    s0 = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(d, d, 4, 5), s0, false);
    s1 = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(d, d, 6, 7), s1, false);
}

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// waits until at most `n` of this wave's vector memory operations are still in flight
template <int N_LEFT>
__device__ __forceinline__ void wait_vmem_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N_LEFT) : "memory"); }

// LDS traffic inside one wave needs no barrier (the LDS executes a wave's instructions in order),
// only that the compiler keeps the order and waits for the data.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// (|c|, atom, c) candidates: larger |c| wins, the lower atom on equal |c| (the tie rule of Eq.3)
__device__ __forceinline__ void take_better(float &ba, int &bi, float &bc, float oa, int oi, float oc)
{
    if (oa > ba || (oa == ba && oi < bi)) { ba = oa; bi = oi; bc = oc; }
}

// Of the 16 atoms that a wave's quads have evaluated, the one with the largest key: |correlation|, then the lower atom, bits << 32 | ~atom.
__device__ __forceinline__ int best_atom(unsigned long long best)
{
    using namespace lane;
    auto take = [&](unsigned long long o) { best = o > best ? o : best; };
    take(dpp_mov<0x141>(best));   // row_half_mirror: the four quads of a row
    take(dpp_mov<0x140>(best));   // row_mirror
    const unsigned long long r0 = lane_read(best, 0), r1 = lane_read(best, 16), r2 = lane_read(best, 32), r3 = lane_read(best, 48);
    take(r0);
    take(r1);
    take(r2);
    take(r3);
    return ~__builtin_amdgcn_readfirstlane((int)(uint32_t)best);
}

// The whole wave resolves ONE vector whose pick the kept values of a sweep could not decide (encode_mfma.hip, encode_resident.hip).
// `scr` holds that vector's residual, written by its two owner lanes:
//   [0, 256)    hi, dimensions in order        [256, 512)  lo
// `own`: the tracked group values of this lane's vector and half; the vector's are those of lanes v and v + 32.  rows(n, q, d): quarter q of
// atom n; kFar: from L2, so that the first two candidate groups' are requested together.  Lane (a = lane / 4, q = lane % 4) evaluates
// atom a of a 16-atom group over a quarter of the dimensions.
// Returns the arg-max of |hi . d + lo . d| (lowest index on ties) over the groups that reach thr_bits, or over all atoms
// when a lane's last tracked group does.
// (The group values through LDS, one at a time, each group's rows only then, and the reductions by ds_bpermute were a chain of two dozen LDS
// trips: 10 of the 33 us of an iteration of the resident encoder with 64 x 4096 vectors, 256 atoms.)
constexpr int kResolveTrack = 4;   // group maxima tracked per lane
template <int DC, typename Rows>
__device__ __forceinline__ int resolve_vector(const Rows &rows, int32_t N, int ntiles, uint32_t code_mask, const unsigned char *scr,
                                              const uint32_t (&own)[kResolveTrack], uint32_t thr_own, int v, int lane)
{
    using namespace lane;
    constexpr int kQ = DC / 32;  // 8-element pieces of a quarter vector
    const int a = lane >> 2, q = lane & 3;
    const uint32_t thr_bits = lane_read(thr_own, v);
    const int at = 8 * (a >> 2) + (a & 3);
    // tracked group values, lane half 0 then half 1 (scalars); the first two candidates' first atoms, a mask of the others
    uint32_t group[2 * kResolveTrack], more = 0u;
    int first = -1, second = -1;
    bool overflow = false;
#pragma unroll
    for (int e = 0; e < 2 * kResolveTrack; ++e) {
        group[e] = lane_read(own[e % kResolveTrack], v + 32 * (e / kResolveTrack));
        if (group[e] < thr_bits) continue;
        const int n = (ntiles - 1 - (int)(group[e] & code_mask)) * 32 + 4 * (e / kResolveTrack);
        overflow = overflow || e % kResolveTrack == kResolveTrack - 1;
        if (first < 0) first = n;
        else if (second < 0) second = n;
        else more |= 1u << e;
    }
    unsigned long long best = 0xffffffffull;   // (best_atom)
    half8 th[kQ], tl[kQ];
    auto take = [&](unsigned long long o) { best = o > best ? o : best; };
    auto eval = [&](int n, const half8 (&d)[kQ]) {
        float s0 = 0.0f, s1 = 0.0f, l0 = 0.0f, l1 = 0.0f;
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            dot8(th[j], d[j], s0, s1);
            dot8(tl[j], d[j], l0, l1);
        }
        const float ab = fabsf(row_reduce<4>((s0 + s1) + (l0 + l1), OpAdd()));
        const unsigned long long key = ((unsigned long long)__float_as_uint(ab) << 32) | (uint32_t)~n;
        if (ab >= 0.0f) take(key);   // (not a number: never the best)
    };
    auto residual = [&]() {
#pragma unroll
        for (int j = 0; j < kQ; ++j) {
            th[j] = *reinterpret_cast<const half8 *>(scr + q * (DC / 2) + j * 16);
            tl[j] = *reinterpret_cast<const half8 *>(scr + 256 + q * (DC / 2) + j * 16);
        }
    };
    if (!overflow && !Rows::kFar) {
        residual();
        half8 d[kQ];
#pragma unroll
        for (int e = 0; e < 2 * kResolveTrack; ++e) {
            if (group[e] < thr_bits) continue;
            const int n = (ntiles - 1 - (int)(group[e] & code_mask)) * 32 + 4 * (e / kResolveTrack) + at;
            rows(n, q, d);
            eval(n, d);
        }
    } else if (!overflow) {
        const int n0 = max(first, 0) + at, n1 = (second < 0 ? max(first, 0) : second) + at;
        half8 d0[kQ], d1[kQ];
        rows(n0, q, d0);
        rows(n1, q, d1);
        residual();
        eval(n0, d0);
        eval(n1, d1);
        if (more) {
#pragma unroll
            for (int e = 2; e < 2 * kResolveTrack; ++e) {
                if (!((more >> e) & 1u)) continue;
                const int n = (ntiles - 1 - (int)(group[e] & code_mask)) * 32 + 4 * (e / kResolveTrack) + at;
                rows(n, q, d0);
                eval(n, d0);
            }
        }
    } else {
        residual();
#pragma unroll 1
        for (int n0 = 0; n0 < N; n0 += 32) {   // N is a multiple of 32
            half8 d0[kQ], d1[kQ];
            rows(n0 + a, q, d0);
            rows(n0 + 16 + a, q, d1);
            eval(n0 + a, d0);
            eval(n0 + 16 + a, d1);
        }
    }
    return best_atom(best);
}

}  // namespace enc
}  // namespace csr
