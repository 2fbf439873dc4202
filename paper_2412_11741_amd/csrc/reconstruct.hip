// De-sparse restore, Eq.12 of the paper's Section "De-Sparse to restore": X~ = D r, i.e. every coded vector
// is rebuilt as the sum of its s coefficient-weighted atoms (per chunk with chunked codes).  This is the step the
// paper puts in front of ordinary attention; the code-domain decode kernel never needs it, but callers that must
// touch the dense vectors (a position embedding applied to rebuilt keys, inspection, a loss on X - X~) do.
//
// Bound: the texture path, 64 bytes a cycle and CU, and behind it the L1 misses of the atom rows, which come from L2 (32 x 4096 vectors, 8
// pairs: 19.5 thousand cycles of accesses per CU; its data unit is busy 22.9 of the 26.1 thousand cycles in which waves run with 256
// atoms, 30.7 of 33.8 with 4096, where 1.6 times the lines miss).  HBM sees 2 d bytes per vector written and 4 s read.
// Lane (vector, chunk, 8-dimension piece): all lanes of a vector's chunk read the same s pairs (one broadcast
// load each) and gather 16 bytes of each of the s atom rows, so a chunk's rows are fetched as whole lines.
#include <utility>

#include "csr_internal.h"

namespace csr {
namespace {

template <typename T> __device__ __forceinline__ void load8f(const T *p, float (&f)[8]);
template <> __device__ __forceinline__ void load8f<__half>(const __half *p, float (&f)[8])
{
    const uint4 raw = *reinterpret_cast<const uint4 *>(p);
    const __half2 *h2 = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float2 v = __half22float2(h2[j]);
        f[2 * j] = v.x;
        f[2 * j + 1] = v.y;
    }
}
template <> __device__ __forceinline__ void load8f<float>(const float *p, float (&f)[8])
{
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}
// From 4 MB of output on the stores are non-temporal: the vectors do not push atom rows out of the L2s and the cache behind them, and nothing
// is dirty when the kernel ends.  That is for the call itself and for what runs between it and the vectors' use; a kernel right behind it that
// reads them all finds fewer of them cached, and between 16 and 270 MB the two together are up to 9 % slower for it.  us, plain -> non-temporal: the
// call alone; with such a kernel behind it, x + 1; with another, the maximum over d.
//   32 x 4096 vectors, 4096 atoms, 8 pairs (33.5 MB), keys and values in turn (two calls)
//     three layers, all of whose dictionaries and codes stay in the 256 MB behind the L2s: 50.4 -> 32.9; 68.0 -> 73.8; 91.3 -> 92.3
//     eight layers: 47.0 -> 49.3; 67.9 -> 74.4; 87.9 -> 94.5
//   one call, dictionaries, codes and outputs in turn through 1.5 GB
//     4.1 MB, 4096 atoms 7.8 -> 7.0; 10.3 -> 9.9; 12.4 -> 12.0         16 MB 16.1 -> 15.4; 21.4 -> 22.6; 27.0 -> 28.0
//     34 MB, 256 atoms 20.6 -> 14.3; 30.7 -> 32.2; 40.0 -> 42.0        131 MB, 1024 atoms 73 -> 51; 113 -> 110; 141 -> 149
//     268 MB, 4096 atoms 157 -> 148; 243 -> 244; 300 -> 309            537 MB, 2048 atoms 290 -> 274; 463 -> 456; 599 -> 596
//   one call, everything cached
//     8.2 MB 6.4 -> 5.8; 11.4 -> 11.4; 14.5 -> 14.7                    4.1 MB 4.7 -> 4.4; 7.5 -> 7.7; 9.4 -> 9.5
//     1.0 MB 2.5 -> 2.5; 4.7 -> 4.9; 5.8 -> 6.1                        0.5 MB 2.4 -> 2.4; 4.6 -> 4.7; 5.7 -> 5.9
// Below 4 MB they stay plain.  (The code words as non-temporal loads, too, on codes already seen: 36.2 -> 43; a line of them serves eight vectors.)
constexpr uint64_t kPastBytes = 4u << 20;
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
template <bool PAST, typename V> __device__ __forceinline__ void store16(void *p, const V &v)
{
    if constexpr (PAST) __builtin_nontemporal_store(__builtin_bit_cast(uint4v, v), reinterpret_cast<uint4v *>(p));
    else *reinterpret_cast<uint4v *>(p) = __builtin_bit_cast(uint4v, v);
}
template <bool PAST> __device__ __forceinline__ void store8f(__half *p, const float (&f)[8])
{
    uint4 raw;
    __half2 *h2 = reinterpret_cast<__half2 *>(&raw);
#pragma unroll
    for (int j = 0; j < 4; ++j) h2[j] = __floats2half2_rn(f[2 * j], f[2 * j + 1]);
    store16<PAST>(p, raw);
}
template <bool PAST> __device__ __forceinline__ void store8f(float *p, const float (&f)[8])
{
    store16<PAST>(p, make_float4(f[0], f[1], f[2], f[3]));
    store16<PAST>(p + 4, make_float4(f[4], f[5], f[6], f[7]));
}
__device__ __forceinline__ int load_idx(const uint16_t *p) { return *p; }
__device__ __forceinline__ int load_idx(const int32_t *p) { return *p; }
__device__ __forceinline__ float load_coef(const __half *p) { return __half2float(*p); }
__device__ __forceinline__ float load_coef(const float *p) { return *p; }

// Workgroups are dealt to the 8 XCDs round-robin, and each XCD has an L2 of its own (4 MB).  Numbered plainly, the
// workgroups in flight span several dictionaries and every L2 would have to hold all of them; give each XCD a
// contiguous eighth of the elements instead, so that at any time it gathers from one or two dictionaries.
__device__ __forceinline__ int64_t xcd_contiguous_block()
{
    const unsigned b = blockIdx.x, per = gridDim.x >> 3;
    return b < per * 8u ? (int64_t)(b & 7u) * per + (b >> 3) : (int64_t)b;
}

struct Where {
    int64_t h, t, code;
    int ch, pc;
};
// element e = (vector h * T + t, piece): its block, token, chunk, piece inside the chunk, first pair of its code
__device__ __forceinline__ Where locate(int64_t e, int pieces, int ppc, int64_t T, int sn, int s, int64_t code_stride_h)
{
    Where w;
    const int piece = (int)(e % pieces);
    const int64_t v = e / pieces;
    w.h = v / T;
    w.t = v - w.h * T;
    w.ch = piece / ppc;
    w.pc = piece - w.ch * ppc;
    w.code = w.h * code_stride_h + (w.t * sn + w.ch) * s;
    return w;
}

// Any types, any s, any alignment: one pair at a time.
template <bool PAST, typename TD, typename TI, typename TC, typename TO>
__global__ __launch_bounds__(256) void reconstruct_kernel(const TD *__restrict__ Dict, const TI *__restrict__ idx,
                                                          const TC *__restrict__ coef, TO *__restrict__ out, int64_t T,
                                                          int32_t d, int32_t N, int32_t s, int32_t sn, int32_t dict_count,
                                                          int64_t code_stride_h, int64_t out_stride_h,
                                                          int64_t out_stride_t, int64_t total)
{
    const int pieces = d >> 3;             // lanes per vector
    const int dc = d / sn, ppc = dc >> 3;  // dimensions / pieces per chunk
    const int64_t e = xcd_contiguous_block() * 256 + threadIdx.x;
    if (e >= total) return;
    const Where w = locate(e, pieces, ppc, T, sn, s, code_stride_h);
    const TD *Dh = Dict + ((int64_t)(w.h % dict_count) * sn + w.ch) * N * dc + w.pc * 8;
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
    for (int j = 0; j < s; ++j) {
        const int n = load_idx(idx + w.code + j);
        const float c = load_coef(coef + w.code + j);
        float row[8];
        load8f<TD>(Dh + (int64_t)n * dc, row);
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = fmaf(c, row[k], acc[k]);
    }
    store8f<PAST>(out + w.h * out_stride_h + w.t * out_stride_t + (w.ch * ppc + w.pc) * 8, acc);
}

// The paper's storage (16-bit indices, fp16 coefficients) with s = 8 G pairs: a lane reads eight pairs with one
// 16-byte load per stream and has the eight atom-row pieces of a group in flight together; same sum order.
template <bool PAST, typename TD, typename TO, int G>
__global__ __launch_bounds__(256) void reconstruct_vec_kernel(const TD *__restrict__ Dict, const uint16_t *__restrict__ idx,
                                                              const __half *__restrict__ coef, TO *__restrict__ out,
                                                              int64_t T, int32_t d, int32_t N, int32_t sn,
                                                              int32_t dict_count, int64_t code_stride_h,
                                                              int64_t out_stride_h, int64_t out_stride_t, int64_t total)
{
    const int pieces = d >> 3;
    const int dc = d / sn, ppc = dc >> 3;
    const int64_t e = xcd_contiguous_block() * 256 + threadIdx.x;
    if (e >= total) return;
    const Where w = locate(e, pieces, ppc, T, sn, 8 * G, code_stride_h);
    uint4 qi[G], qc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        qi[g] = *reinterpret_cast<const uint4 *>(idx + w.code + 8 * g);
        qc[g] = *reinterpret_cast<const uint4 *>(coef + w.code + 8 * g);
    }
    const TD *Dh = Dict + ((int64_t)(w.h % dict_count) * sn + w.ch) * N * dc + w.pc * 8;
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint32_t iw[4] = {qi[g].x, qi[g].y, qi[g].z, qi[g].w};
        const __half2 *h2 = reinterpret_cast<const __half2 *>(&qc[g]);
        float row[8][8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = (j & 1) ? (int)(iw[j >> 1] >> 16) : (int)(iw[j >> 1] & 0xffffu);
            load8f<TD>(Dh + (int64_t)n * dc, row[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float2 cf = __half22float2(h2[j >> 1]);
            const float c = (j & 1) ? cf.y : cf.x;
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] = fmaf(c, row[j][k], acc[k]);
        }
    }
    store8f<PAST>(out + w.h * out_stride_h + w.t * out_stride_t + (w.ch * ppc + w.pc) * 8, acc);
}

// The paper's storage with 1 to 7 pairs: the code is requested as a whole (in 32-bit words, or for odd NP pair by pair),
// then all its rows; same sum order.  One pair at a time every row waits for its own index: 32 x 4096 vectors, 4096 atoms
// (us) 4 pairs 20.3 -> 15.2, 6 pairs 22.7 -> 17.9, 2 x 2 15.9 -> 12.9, 2 x 3 16.7 -> 13.8, 2 x 4 18.5 -> 14.2.
template <bool PAST, typename TD, typename TO, int NP>
__global__ __launch_bounds__(256) void reconstruct_few_kernel(const TD *__restrict__ Dict, const uint16_t *__restrict__ idx,
                                                              const __half *__restrict__ coef, TO *__restrict__ out,
                                                              int64_t T, int32_t d, int32_t N, int32_t sn,
                                                              int32_t dict_count, int64_t code_stride_h,
                                                              int64_t out_stride_h, int64_t out_stride_t, int64_t total)
{
    const int pieces = d >> 3;
    const int dc = d / sn, ppc = dc >> 3;
    const int64_t e = xcd_contiguous_block() * 256 + threadIdx.x;
    if (e >= total) return;
    const Where w = locate(e, pieces, ppc, T, sn, NP, code_stride_h);
    int n[NP];
    float c[NP];
    if constexpr (NP % 2 == 0) {
        uint32_t wi[NP / 2], wc[NP / 2];
#pragma unroll
        for (int j = 0; j < NP / 2; ++j) {
            wi[j] = reinterpret_cast<const uint32_t *>(idx + w.code)[j];
            wc[j] = reinterpret_cast<const uint32_t *>(coef + w.code)[j];
        }
#pragma unroll
        for (int j = 0; j < NP / 2; ++j) {
            n[2 * j] = (int)(wi[j] & 0xffffu);
            n[2 * j + 1] = (int)(wi[j] >> 16);
            const float2 cf = __half22float2(*reinterpret_cast<const __half2 *>(&wc[j]));
            c[2 * j] = cf.x;
            c[2 * j + 1] = cf.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            n[j] = load_idx(idx + w.code + j);
            c[j] = load_coef(coef + w.code + j);
        }
    }
    const TD *Dh = Dict + ((int64_t)(w.h % dict_count) * sn + w.ch) * N * dc + w.pc * 8;
    float row[NP][8];
#pragma unroll
    for (int j = 0; j < NP; ++j) load8f<TD>(Dh + (int64_t)n[j] * dc, row[j]);
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = fmaf(c[j], row[j][k], acc[k]);
    }
    store8f<PAST>(out + w.h * out_stride_h + w.t * out_stride_t + (w.ch * ppc + w.pc) * 8, acc);
}

// The paper's storage, whole vectors of 128 dimensions or a multiple: the 16 lanes of a row share one code.  A lane requests ONE
// 32-bit word of it (S words in all, indices before coefficients; two words with more than 16 pairs) and the row hands them
// round; with every lane requesting the whole code, pairs were a fifth of the bytes that the texture path delivered.
// Divisions are in 32 bits.  Same sum order.  32 x 4096 vectors (us): 4096 atoms, 8
// pairs 19.2 -> 18.4, 6 pairs 17.8 -> 17.1, 8192 atoms, 16 pairs 40.5 -> 39.2; 256 atoms, 8 pairs 16.1 -> 14.9, twice the vectors with 4 pairs
// 22.5 -> 18.7; 4 pairs of 256 to 2048 atoms 13.2 -> 10.9 and 12.5 -> 11.5, of 3072 and 8192
// level, of 4096 13.7 -> 14.2.  Workgroups that stay and request the next tile's words ahead are slower (8 pairs 18.9).
template <int S, int W, int... K>
__device__ __forceinline__ void hand_round(uint32_t (&code)[S], const uint32_t (&w)[W], std::integer_sequence<int, K...>)
{
    ((code[K] = (uint32_t)__builtin_amdgcn_mov_dpp((int)w[K / 16], 0x150 + K % 16, 0xf, 0xf, true)), ...);   // row_newbcast
}

template <bool PAST, typename TD, typename TO, int S>
__global__ __launch_bounds__(256) void reconstruct_row_kernel(const TD *__restrict__ Dict, const uint32_t *__restrict__ idx,
                                                              const uint32_t *__restrict__ coef, TO *__restrict__ out,
                                                              uint32_t T, int32_t d, int32_t N, uint32_t sn, uint32_t dict_count,
                                                              int64_t code_stride_h, int64_t out_stride_h,
                                                              int64_t out_stride_t, uint32_t rows)
{
    constexpr int kWords = (S + 15) / 16, kHalf = S / 2;
    const uint32_t rows_per_vec = (uint32_t)d >> 7, sub = threadIdx.x & 15;
    const uint32_t r = (uint32_t)xcd_contiguous_block() * 16 + (threadIdx.x >> 4);   // row of lanes: (vector, 128 dimensions)
    if (r >= rows) return;   // whole rows: the words below come from lanes that are there
    const uint32_t v = rows_per_vec == 1 ? r : r / rows_per_vec, col = (r - v * rows_per_vec) * 128 + sub * 8;   // first dimension
    const uint32_t dc = (uint32_t)d / sn, ch = sn == 1 ? 0 : col / dc, h = v / T, t = v - h * T;
    const int64_t code = ((int64_t)h * code_stride_h + ((int64_t)t * sn + ch) * S) >> 1;   // in words: S is even
    uint32_t w[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
        const int k = min((int)sub + 16 * i, S - 1);
        w[i] = (k < kHalf ? idx + k : coef + (k - kHalf))[code];
    }
    uint32_t words[S];
    hand_round(words, w, std::make_integer_sequence<int, S>());
    const TD *Dh = Dict + ((int64_t)(h % dict_count) * sn + ch) * N * dc + (col - ch * dc);
    float acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
#pragma unroll
    for (int j0 = 0; j0 < S; j0 += 8) {   // the rows of eight pairs in flight together
        float row[8][8];
#pragma unroll
        for (int j = 0; j < 8 && j0 + j < S; ++j) {
            const uint32_t n2 = words[(j0 + j) >> 1];
            load8f<TD>(Dh + (int64_t)(j & 1 ? n2 >> 16 : n2 & 0xffffu) * dc, row[j]);
        }
#pragma unroll
        for (int j = 0; j < 8 && j0 + j < S; ++j) {
            const float2 cf = __half22float2(*reinterpret_cast<const __half2 *>(&words[kHalf + ((j0 + j) >> 1)]));
            const float c = j & 1 ? cf.y : cf.x;
#pragma unroll
            for (int k = 0; k < 8; ++k) acc[k] = fmaf(c, row[j][k], acc[k]);
        }
    }
    store8f<PAST>(out + (int64_t)h * out_stride_h + (int64_t)t * out_stride_t + col, acc);
}

template <bool PAST, typename TD, typename TI, typename TC, typename TO>
hipError_t launch_t(const ReconstructArgs &a)
{
    const int64_t total = (int64_t)a.H * a.T * (a.d / 8);
    const int64_t blocks = (total + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    if constexpr (sizeof(TI) == 2 && sizeof(TC) == 2) {
        // even s: every code starts at a 32-bit word
        const bool words = a.code_stride_h % 2 == 0 && (reinterpret_cast<uintptr_t>(a.idx) % 4) == 0 &&
                           (reinterpret_cast<uintptr_t>(a.coef) % 4) == 0;
        if (words && a.s % 2 == 0 && (a.d / a.sn) % 128 == 0 && total / 16 < 0x7fffffffLL) {
#define CSR_REC_ROW(S)                                                                                              \
    case S:                                                                                                         \
        hipLaunchKernelGGL((reconstruct_row_kernel<PAST, TD, TO, S>), grid, dim3(256), 0, a.stream, (const TD *)a.D,      \
                           (const uint32_t *)a.idx, (const uint32_t *)a.coef, (TO *)a.out, (uint32_t)a.T, a.d, a.N, \
                           (uint32_t)a.sn, (uint32_t)a.dict_count, a.code_stride_h, a.out_stride_h, a.out_stride_t, \
                           (uint32_t)(total / 16));                                                                 \
        return hipGetLastError()
            switch (a.s) {
                CSR_REC_ROW(2);
                CSR_REC_ROW(4);
                CSR_REC_ROW(6);
                CSR_REC_ROW(8);
                CSR_REC_ROW(16);
                CSR_REC_ROW(24);
                CSR_REC_ROW(32);
                default: break;
            }
#undef CSR_REC_ROW
        }
        const bool vec = a.s % 8 == 0 && a.code_stride_h % 8 == 0 && (reinterpret_cast<uintptr_t>(a.idx) % 16) == 0 &&
                         (reinterpret_cast<uintptr_t>(a.coef) % 16) == 0;
        if (vec) {
#define CSR_REC_VEC(G)                                                                                              \
    hipLaunchKernelGGL((reconstruct_vec_kernel<PAST, TD, TO, G>), grid, dim3(256), 0, a.stream, (const TD *)a.D,          \
                       (const uint16_t *)a.idx, (const __half *)a.coef, (TO *)a.out, a.T, a.d, a.N, a.sn,           \
                       a.dict_count, a.code_stride_h, a.out_stride_h, a.out_stride_t, total)
            switch (a.s / 8) {
                case 1: CSR_REC_VEC(1); break;
                case 2: CSR_REC_VEC(2); break;
                case 3: CSR_REC_VEC(3); break;
                default: CSR_REC_VEC(4); break;
            }
#undef CSR_REC_VEC
            return hipGetLastError();
        }
        if (a.s < 8 && (a.s % 2 == 1 || words)) {
#define CSR_REC_FEW(NP)                                                                                             \
    hipLaunchKernelGGL((reconstruct_few_kernel<PAST, TD, TO, NP>), grid, dim3(256), 0, a.stream, (const TD *)a.D,         \
                       (const uint16_t *)a.idx, (const __half *)a.coef, (TO *)a.out, a.T, a.d, a.N, a.sn,           \
                       a.dict_count, a.code_stride_h, a.out_stride_h, a.out_stride_t, total)
            switch (a.s) {
                case 1: CSR_REC_FEW(1); break;
                case 2: CSR_REC_FEW(2); break;
                case 3: CSR_REC_FEW(3); break;
                case 4: CSR_REC_FEW(4); break;
                case 5: CSR_REC_FEW(5); break;
                case 6: CSR_REC_FEW(6); break;
                default: CSR_REC_FEW(7); break;
            }
#undef CSR_REC_FEW
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((reconstruct_kernel<PAST, TD, TI, TC, TO>), grid, dim3(256), 0, a.stream, (const TD *)a.D,
                       (const TI *)a.idx, (const TC *)a.coef, (TO *)a.out, a.T, a.d, a.N, a.s, a.sn, a.dict_count,
                       a.code_stride_h, a.out_stride_h, a.out_stride_t, total);
    return hipGetLastError();
}

template <typename TD, typename TI, typename TC>
hipError_t launch_o(const ReconstructArgs &a)
{
    const bool past = (uint64_t)a.H * (uint64_t)a.T * (uint64_t)a.d * (a.out16 ? 2 : 4) >= kPastBytes;
    if (past) return a.out16 ? launch_t<true, TD, TI, TC, __half>(a) : launch_t<true, TD, TI, TC, float>(a);
    return a.out16 ? launch_t<false, TD, TI, TC, __half>(a) : launch_t<false, TD, TI, TC, float>(a);
}
template <typename TD, typename TI>
hipError_t launch_c(const ReconstructArgs &a)
{
    return a.coef16 ? launch_o<TD, TI, __half>(a) : launch_o<TD, TI, float>(a);
}
template <typename TD>
hipError_t launch_i(const ReconstructArgs &a)
{
    return a.idx16 ? launch_c<TD, uint16_t>(a) : launch_c<TD, int32_t>(a);
}

}  // namespace

hipError_t launch_reconstruct(const ReconstructArgs &a)
{
    return a.dict16 ? launch_i<__half>(a) : launch_i<float>(a);
}

}  // namespace csr
