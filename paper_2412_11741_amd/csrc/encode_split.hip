// Matching Pursuit encoder for FEW vectors per dictionary (gfx950): the tokens generated in one decoding step,
// which Section "KV Decomposition and Sparse Storage" encodes like the prompt's (Eq.2-4, s iterations).
//
// With a handful of vectors per dictionary the work is a matrix-vector product per iteration: every iteration must look
// at the whole dictionary (1 MB at N = 4096) for a few dot products per atom.  One workgroup per dictionary - the shape of
// the prefill encoder - leaves most of the chip idle while a single CU streams it.  Here the ATOMS of every dictionary are
// split over k workgroups, one per CU, and ONE launch runs all iterations: a workgroup reads its slice once, into registers
// (the dictionaries of a layer's 32 heads, 33 MB, are 128 KB per CU, a quarter of its registers), and the k workgroups of a
// dictionary exchange their slices' candidates through device memory after every iteration.
//
//   sweep    each wave: c[n] = hi . d_n + lo . d_n for its tiles on the matrix cores (v_mfma_f32_32x32x16_f16, atoms as
//            rows, vectors as columns; R = hi + lo, two fp16, 22 significant bits; products of fp16 pairs are exact,
//            accumulation is fp32), the wave's best (|c|, n, c) per vector
//   publish  the slice's best per vector as ONE 64-bit word - |c|, atom, sign and the iteration's tag - in a slot of its own
//            (iteration, vector, slice), with a relaxed device-scope store: the word says by itself whether it has arrived
//   collect  the other slices' words, polled with relaxed device-scope loads
//   update   every workgroup of the dictionary applies Eq.4 to its own copy of the residuals (fp32, in LDS) with identical
//            arithmetic, so the copies never diverge; slice 0 stores the pair
//
// The workgroups need not run at the same time: one that starts late finds the others' words and catches up, and one that
// waits in vain for kPatience (its partners hold no CU, because other work does) goes on alone: each of its waves sweeps the
// whole dictionary, from device memory, for the vectors whose words are missing, and waits an eighth of the time from then on
// (46 us in a call, all in all).  The arithmetic is the same, so every wait ends and the result does not depend on it.
// CSR_FLAG_NO_WAIT goes that way from the start.  (The lone workgroup's waves sharing that work would be faster there, but asking whether to, once an
// iteration, costs every call 1.5 %.)  The slots
// are cleared by a launch of their own before (a workspace's contents are undefined); a slot is written once per call.
//
// Bound: reading the dictionaries once (11 us of a call with one iteration), then a dependent chain per iteration, 2.4 us: hi and lo from LDS, 16
// dependent matrix instructions per tile (8 with at most 16 vectors; 0.24 us), the tournament over the accumulators and the waves, publish and
// poll (one trip each to where the chip's L2s meet, 0.8 us together), the row of the chosen atom (hidden), the update.  32 dictionaries of 4096
// atoms, s = 8, one vector each: 28 us a call; 33 before the tournament's winner was numbered bit by bit and the state stayed in registers; a
// whole decoding step with them 94.8 -> 84.9, with 8192 atoms and s = 16 183 -> 150, 60 vectors for each of 8 dictionaries 131 -> 122.
#include <atomic>
#include <cmath>

#include "csr_internal.h"
#include "encode_common.h"
#include "lane_ops.h"

namespace csr {
namespace {

using namespace enc;
using namespace lane;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kMaxVectors = 128;   // per dictionary; beyond that the prefill encoders' shapes are the better ones
constexpr int kNarrowVectors = 16; // ... and up to here half a block is enough (kNarrow)
constexpr int kMaxSlices = 16;
constexpr int kTargetGroups = 256; // one workgroup per CU
constexpr int kPatience = 4000;    // ticks of the 100 MHz counter a wave waits for the partners, 40 us: a whole call's time

struct SplitParams {
    const __half *X;
    const __half *Dict;
    void *idx_out;
    void *coef_out;
    unsigned long long *slots;   // [s][V][k]
    int64_t V;                   // vectors in all
    int64_t T;
    int64_t x_stride_h, x_stride_t, code_stride_h;
    int32_t N, s, sn, dict_count, n_dicts, M, k, idx16, coef_mode, patience;   // patience: kPatience, or -1: not even look
    float *res_norm2;            // optional [H][T][sn]
};

// A candidate as an integer whose maximum is the tie rule of Eq.3 (largest |c|, then the lowest atom):
// |c| | 0xffffff - n | tag (7 bits) | sign of c
__device__ __forceinline__ unsigned long long pack_candidate(float c, int n, int tag)
{
    const uint32_t b = __float_as_uint(c);
    return ((unsigned long long)(b & 0x7fffffffu) << 32) | ((uint32_t)(0xffffff - n) << 8) | ((uint32_t)tag << 1) | (b >> 31);
}
__device__ __forceinline__ int candidate_atom(unsigned long long w) { return 0xffffff - (int)((uint32_t)w >> 8); }
__device__ __forceinline__ int candidate_tag(unsigned long long w) { return (int)(((uint32_t)w >> 1) & 127u); }
__device__ __forceinline__ float candidate_coef(unsigned long long w)
{
    return __uint_as_float((uint32_t)(w >> 32) | ((uint32_t)w << 31));
}
struct OpMaxU64 { __device__ __forceinline__ unsigned long long operator()(unsigned long long a, unsigned long long b) const { return a > b ? a : b; } };

__global__ __launch_bounds__(256) void clear_slots_kernel(ulonglong2 *__restrict__ slots, int64_t n2)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n2) slots[i] = make_ulonglong2(0ull, 0ull);
}

// the value of the lane whose number differs in bit 4 (`up`: this lane's bit 4)
__device__ __forceinline__ uint32_t xchg16(uint32_t v, bool up)
{
    const auto x = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // rows (0, 0, 2, 2) and (1, 1, 3, 3)
    return up ? x[0] : x[1];
}

// LDS byte offset of dimensions 4 pc .. 4 pc + 3 of vector v's residual: 32 vectors' rows are read at the same piece
template <int DC> __device__ __forceinline__ int res_at(int v, int pc) { return v * (DC * 4) + ((pc ^ (v & 15)) << 4); }

// ... of dimensions 8 p .. 8 p + 7 in its fp16 copies
template <int DC> __device__ __forceinline__ int half_at(int v, int p) { return v * (DC * 2) + ((p ^ (DC == 128 ? (v & 15) : ((v >> 1) & 7))) << 4); }

struct SplitState { int32_t sexp, pad; int64_t vid, code_at; };   // scale of a vector's residual, its number, its code's first pair

// HELD: tiles of 32 atoms a wave keeps in registers.  A workgroup is two waves per SIMD, and with 128 dimensions there is no
// room for a second one: the compiler is told so, or it spends instructions on registers that nobody can use.  With 64 dimensions and up to two
// tiles it has to stay within 128 registers, so that two workgroups share a CU where a launch has more of them than there are CUs (512
// dictionaries of 512 atoms, s = 8, one vector each: 31.3 us with 132 registers, 23.2 with 128; 40 vectors each 55.5 and 42.2; one workgroup per CU level).
template <int DC, int HELD, bool kNarrow>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(DC == 64 && HELD <= 2 ? 4 : 2, DC == 128 ? 2 : 4))) void encode_split_kernel(const SplitParams p)
{
    constexpr int kFrags = DC / 16;
    constexpr int L = DC / 8;                  // lanes of a vector's team in the update, 8 dimensions each
    constexpr int kTeams = kThreads / L;
    constexpr int kSlots = kMaxSlices / L;     // slices a lane of a team waits for, at most: 1 or 2
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int m_pad = (p.M + 31) & ~31;        // vectors, whole blocks of 32
    unsigned char *res = lds;                        // [m_pad][DC] fp32: the residuals (kNarrow: none, nor states)
    unsigned char *hi_s = res + (kNarrow ? 0 : m_pad * DC * 4);                                   // [m_pad][DC] fp16: hi, and behind it lo
    unsigned char *lo_s = hi_s + m_pad * DC * 2;
    unsigned long long *red = reinterpret_cast<unsigned long long *>(lo_s + m_pad * DC * 2);      // [kWaves][m_pad]
    SplitState *state = reinterpret_cast<SplitState *>(red + kWaves * m_pad);                     // [M]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hf = lane >> 5;
    const int sub = tid % L, team = tid / L;
    // Workgroups are dealt to the 8 XCDs round-robin: the slices of a dictionary sit on one XCD, whose L2 then has the rows
    // the update gathers.
    int sl, dct;                               // dct = dictionary * sn + chunk
    if (p.n_dicts % 8 == 0) {
        const int i = blockIdx.x >> 3;
        dct = (blockIdx.x & 7) * (p.n_dicts >> 3) + i / p.k;
        sl = i % p.k;
    } else {
        dct = blockIdx.x / p.k;
        sl = blockIdx.x % p.k;
    }
    const int dict = dct / p.sn, ch = dct - dict * p.sn;
    const __half *Dh = p.Dict + (int64_t)dct * p.N * DC;
    const int tiles = p.N >> 5;
    const int per_slice = (tiles + p.k - 1) / p.k;
    const int t_begin = sl * per_slice, t_end = min(tiles, t_begin + per_slice);

    auto load_tile = [&](int tile, uint4 (&a)[kFrags]) {
        const __half *row = Dh + ((int64_t)tile * 32 + col) * DC + hf * (DC / 2);
#pragma unroll
        for (int j = 0; j < kFrags; ++j) a[j] = *reinterpret_cast<const uint4 *>(row + 8 * j);
    };
    uint4 held[HELD][kFrags];
#pragma unroll
    for (int q = 0; q < HELD; ++q)
        if (t_begin + wave + q * kWaves < t_end) load_tile(t_begin + wave + q * kWaves, held[q]);

    // this lane's 8 dimensions of a residual: fp32 and the split into hi + lo
    auto put = [&](int v, const float (&R)[8]) {
        half8 h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const _Float16 hh = (_Float16)R[e];
            h[e] = hh;
            l[e] = (_Float16)(R[e] - (float)hh);
        }
        if constexpr (!kNarrow) {
            *reinterpret_cast<float4 *>(res + res_at<DC>(v, 2 * sub)) = make_float4(R[0], R[1], R[2], R[3]);
            *reinterpret_cast<float4 *>(res + res_at<DC>(v, 2 * sub + 1)) = make_float4(R[4], R[5], R[6], R[7]);
        }
        *reinterpret_cast<half8 *>(hi_s + half_at<DC>(v, sub)) = h;
        *reinterpret_cast<half8 *>(lo_s + half_at<DC>(v, sub)) = l;
    };

    // kNarrow: a team has one vector at most, and what it needs of it from one iteration to the next is in its registers (out of LDS it
    // is a chain of trips in every one: 0.1 of an iteration's 3.1 us)
    static_assert(!kNarrow || kTeams >= 32, "a team for every column");
    float own_R[8];
    SplitState own{};
    // ---- the vectors, scaled by a power of two that brings max |x_k| into [2^11, 2^12): hi and lo stay normal ----------
    for (int v = team; v < m_pad; v += kTeams) {
        // vector m of this dictionary: block h = (m / T) dict_count + dict, its token m % T
        const int m = min(v, p.M - 1);         // the last block's missing columns recompute the last vector
        const int rep = (int)(m / p.T);
        const int64_t t = m - rep * p.T, h = (int64_t)rep * p.dict_count + dict;
        float R[8];
        unpack8(*reinterpret_cast<const uint4 *>(p.X + h * p.x_stride_h + t * p.x_stride_t + ch * DC + sub * 8), R);
        float amax = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(R[e]));
        amax = row_reduce<L>(amax, OpMax());
        int ex = 0;
        if (amax > 0.0f && amax < INFINITY) {
            (void)frexpf(amax, &ex);           // amax = f 2^ex, f in [0.5, 1)
            ex = 12 - ex;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) R[e] = ldexpf(R[e], ex);
        put(v, R);
        SplitState st;
        st.sexp = ex; st.pad = 0;
        st.vid = (h * p.T + t) * p.sn + ch;
        st.code_at = h * p.code_stride_h + (t * p.sn + ch) * p.s;
        if constexpr (kNarrow) {
            own = st;
#pragma unroll
            for (int e = 0; e < 8; ++e) own_R[e] = R[e];
        } else if (sub == 0 && v < p.M) {
            state[v] = st;
        }
    }
    __syncthreads();

    // The best candidate of vectors m0 .. m0 + 31 over the tiles first, first + step .. below last, as a packed word with
    // `tag` (lanes col of either half); `own`: this wave's tiles of the workgroup's slice, the first ones in registers.
    // kNarrow (at most 16 vectors): hi takes columns 0 - 15 and lo columns 16 - 31: one pass of matrix instructions instead of two, and
    // half the values per lane behind it.  hi . d and lo . d are then sums of their own instead of one chain: the low bits of a
    // coefficient, and at a tie the atom, are not those of a launch with more vectors.  Error of a coefficient against 64 bits, over |R| (128
    // dimensions, 4096 atoms, s = 8): 2.4e-8 on average and 1.1e-7 at most, with more vectors 3.0e-8 and 1.5e-7.
    auto sweep = [&](int m0, int first, int last, int step, bool own, int tag) {
        half8 hi[kFrags], lo[kNarrow ? 1 : kFrags];
        // columns past the last vector repeat it: one LDS address for them all
        const int mine = min(kNarrow ? (col & 15) : m0 + col, p.M - 1);
#pragma unroll
        for (int j = 0; j < kFrags; ++j) {
            if constexpr (kNarrow) {
                hi[j] = *reinterpret_cast<const half8 *>((col < 16 ? hi_s : lo_s) + half_at<DC>(mine, hf * kFrags + j));
            } else {
                hi[j] = *reinterpret_cast<const half8 *>(hi_s + half_at<DC>(mine, hf * kFrags + j));
                lo[j] = *reinterpret_cast<const half8 *>(lo_s + half_at<DC>(mine, hf * kFrags + j));
            }
        }
        float ba = -1.0f, bc = 0.0f;
        int bi = 0;
        auto tile_best = [&](int tile, const uint4 (&a)[kFrags]) {
            floatx16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int j = 0; j < kFrags; ++j) {
                const half8 av = *reinterpret_cast<const half8 *>(&a[j]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, hi[j], acc, 0, 0, 0);
                if constexpr (!kNarrow) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, lo[j], acc, 0, 0, 0);
            }
            // accumulator r of lane half hf is atom 8 (r / 4) + (r % 4) + 4 hf of the tile, ascending in r: a tournament in
            // which the left side wins ties
            float c[8];
            int at[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                if constexpr (kNarrow) {   // lanes 0 - 15 of a half get the sum of accumulator 2 r, lanes 16 - 31 of 2 r + 1
                    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[2 * r]), __float_as_uint(acc[2 * r + 1]), false, false);
                    c[r] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
                    at[r] = 0;
                } else {
                    const bool right = fabsf(acc[2 * r + 1]) > fabsf(acc[2 * r]);
                    c[r] = right ? acc[2 * r + 1] : acc[2 * r];
                    at[r] = right ? 1 : 0;
                }
            }
#pragma unroll
            for (int m = 4; m >= 1; m >>= 1) {
#pragma unroll
                for (int r = 0; r < m; ++r) {
                    const bool right = fabsf(c[2 * r + 1]) > fabsf(c[2 * r]);
                    c[r] = right ? c[2 * r + 1] : c[2 * r];
                    // the winner's number, a bit a round (chosen from ready numbers, the compiler turns the choice into a search
                    // through a table, a hundred instructions a tile)
                    at[r] = right ? (at[2 * r + 1] | (8 / m)) : at[2 * r];
                }
            }
            if constexpr (kNarrow) at[0] += col >> 4;
            if (fabsf(c[0]) > ba) {
                ba = fabsf(c[0]);
                bi = tile * 32 + 8 * (at[0] >> 2) + (at[0] & 3) + 4 * hf;
                bc = c[0];
            }
        };
        if (own) {
#pragma unroll
            for (int q = 0; q < HELD; ++q)
                if (first + q * kWaves < last) tile_best(first + q * kWaves, held[q]);
        }
        for (int tile = first + (own ? HELD * kWaves : 0); tile < last; tile += step) {
            uint4 a[kFrags];
            load_tile(tile, a);
            tile_best(tile, a);
        }
        take_better(ba, bi, bc, xchg32f(ba, hf), (int)xchg32((uint32_t)bi, hf), xchg32f(bc, hf));
        if constexpr (kNarrow) {
            const bool up = col >= 16;
            take_better(ba, bi, bc, __uint_as_float(xchg16(__float_as_uint(ba), up)), (int)xchg16((uint32_t)bi, up),
                        __uint_as_float(xchg16(__float_as_uint(bc), up)));
        }
        // a wave without tiles: below every candidate
        return ba >= 0.0f ? pack_candidate(bc, bi, tag) : (unsigned long long)((uint32_t)tag << 1);
    };
    int patience = p.patience;   // this wave's: an eighth of it is left each time it has waited in vain
#pragma unroll 1
    for (int g = 0; g < p.s; ++g) {
        const int tag = g + 1;
        for (int m0 = 0; m0 < p.M; m0 += 32) {
            const unsigned long long w = sweep(m0, t_begin + wave, t_end, kWaves, true, tag);
            if (hf == 0) red[wave * m_pad + m0 + col] = w;
        }
        __syncthreads();
        // From here to the next barrier a vector is its team's affair.  The slice's best of every vector, published:
        unsigned long long *slot = p.slots + (int64_t)g * p.V * p.k;
        unsigned long long own_w = 0ull;
        if constexpr (kNarrow) {
            if (team < p.M) {
                own_w = row_reduce<kWaves>(red[(sub & (kWaves - 1)) * m_pad + team], OpMaxU64());
                if (sub == 0 && p.k > 1) __hip_atomic_store(slot + own.vid * p.k + sl, own_w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            for (int v = team; v < p.M; v += kTeams) {
                unsigned long long w = red[(sub & (kWaves - 1)) * m_pad + v];
                w = row_reduce<kWaves>(w, OpMaxU64());
                if (sub == 0) {
                    red[v] = w;
                    if (p.k > 1) __hip_atomic_store(slot + state[v].vid * p.k + sl, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            wave_lds_fence();
        }
        // ---- the other slices' candidates, the pick, Eq.4 -----------------------------------------------------------------
        for (int v0 = wave * (64 / L); v0 < p.M; v0 += kTeams) {   // (uniform over the wave)
            const int v = v0 + lane / L;
            const int vc = min(v, p.M - 1);   // a team past the last vector idles along: it waits for nobody
            const int slices = v < p.M ? p.k : 0;
            const SplitState &st = kNarrow ? own : state[vc];   // (in LDS: what is used late is read late)
            unsigned long long w = kNarrow ? own_w : vc == v ? red[v] : 0ull;
            if (p.k > 1) {
                unsigned long long *mine = slot + st.vid * p.k;
                unsigned long long got[kSlots];
                bool ok = true;
#pragma unroll
                for (int i = 0; i < kSlots; ++i) {
                    const int j = sub + i * L;
                    got[i] = 0ull;
                    if (j < slices && j != sl) {
                        if (p.patience >= 0) got[i] = __hip_atomic_load(mine + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok = ok && candidate_tag(got[i]) == tag;
                    }
                }
                if (__ballot(!ok)) {
                    const uint64_t began = wall_clock64();
                    while (patience >= 0) {
                        __builtin_amdgcn_s_sleep(1);
                        ok = true;
#pragma unroll
                        for (int i = 0; i < kSlots; ++i) {
                            const int j = sub + i * L;
                            if (j < slices && j != sl && candidate_tag(got[i]) != tag) {
                                got[i] = __hip_atomic_load(mine + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                ok = ok && candidate_tag(got[i]) == tag;
                            }
                        }
                        if (!__ballot(!ok) || wall_clock64() - began > (uint64_t)patience) break;
                    }
                    if (__ballot(!ok)) {
                        // partners that hold no CU: the candidates of this wave's vectors - they are of one block of 32 -
                        // over the whole dictionary, in one sweep for all of them (their slices' words would lead to the same)
                        patience >>= 3;
                        const unsigned long long o = sweep(v0 & ~31, 0, tiles, 1, false, tag);
                        const unsigned long long theirs = __shfl(o, v & 31, 64);
                        w = theirs > w ? theirs : w;
                    }
                }
#pragma unroll
                for (int i = 0; i < kSlots; ++i) w = candidate_tag(got[i]) == tag && got[i] > w ? got[i] : w;
                w = row_reduce<L>(w, OpMaxU64());
            }
            // (no candidate at all - correlations that are not numbers - counts as atom 0 with coefficient 0)
            const int n = candidate_atom(w) < p.N ? candidate_atom(w) : 0;
            float c = candidate_coef(w);
            float d[8];
            unpack8(*reinterpret_cast<const uint4 *>(Dh + (int64_t)n * DC + sub * 8), d);
            const int sexp = st.sexp;
            // closed loop: what Eq.4 subtracts is the coefficient as it will be stored (rounded in the input's scale)
            if (coef_rounds_in_loop(p.coef_mode)) c = ldexpf(__half2float(__float2half_rn(ldexpf(c, -sexp))), sexp);
            if (sl == 0 && v < p.M) {
                const int64_t o = st.code_at + g;
                if (sub == 0) {
                    if (p.idx16) reinterpret_cast<uint16_t *>(p.idx_out)[o] = (uint16_t)n;
                    else reinterpret_cast<int32_t *>(p.idx_out)[o] = n;
                } else if (sub == 1) {
                    const float c_out = ldexpf(c, -sexp);
                    if (coef_is_f16(p.coef_mode)) reinterpret_cast<__half *>(p.coef_out)[o] = __float2half_rn(c_out);
                    else reinterpret_cast<float *>(p.coef_out)[o] = c_out;
                }
            }
            float R[8];
            if constexpr (kNarrow) {
#pragma unroll
                for (int e = 0; e < 8; ++e) R[e] = own_R[e];
            } else {
                const float4 x = *reinterpret_cast<const float4 *>(res + res_at<DC>(v, 2 * sub));
                const float4 y = *reinterpret_cast<const float4 *>(res + res_at<DC>(v, 2 * sub + 1));
                R[0] = x.x; R[1] = x.y; R[2] = x.z; R[3] = x.w; R[4] = y.x; R[5] = y.y; R[6] = y.z; R[7] = y.w;
            }
            float r2 = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                R[e] = fmaf(-c, d[e], R[e]);   // Eq.4 with the unrounded coefficient
                r2 = fmaf(R[e], R[e], r2);
            }
            r2 = row_reduce<L>(r2, OpAdd());
            if (g + 1 == p.s) {
                if (p.res_norm2 && sl == 0 && sub == 0 && v < p.M) p.res_norm2[st.vid] = ldexpf(r2, -2 * sexp);
                continue;
            }
            // A residual that has shrunk a lot (a vector that is nearly a multiple of an atom) is scaled up again
            // before the split, or lo would sink into the fp16 subnormals; one that has grown (atoms of norm above
            // sqrt(2) make Eq.4 expand it) is scaled down before hi could leave the fp16 range.
            if ((r2 < 65536.0f && r2 > 0.0f) || (r2 >= 1073741824.0f && r2 < INFINITY)) {
                int e2 = 0;
                (void)frexpf(r2, &e2);                // |R| in [2^((e2-1)/2), 2^(e2/2))
                const int k2 = 14 - (e2 + 1) / 2;     // brings |R| into [2^12.5, 2^14.5)
                const float sc = ldexpf(1.0f, k2);
#pragma unroll
                for (int e = 0; e < 8; ++e) R[e] *= sc;
                if constexpr (kNarrow) {
                    own.sexp = sexp + k2;
                } else {
                    wave_lds_fence();                 // the team has read the old exponent
                    if (sub == 0 && v < p.M) state[v].sexp = sexp + k2;
                }
            }
            if (v < p.M) put(v, R);
            if constexpr (kNarrow) {
#pragma unroll
                for (int e = 0; e < 8; ++e) own_R[e] = R[e];
            }
        }
        __syncthreads();
    }
}

size_t r256(size_t v) { return (v + 255) & ~size_t(255); }

struct SplitPlan {
    int32_t k, M, held;
    int64_t V;
    size_t lds, total;
};

SplitPlan plan_split(const EncodeArgs &a)
{
    SplitPlan pl{};
    const int n_dicts = a.dict_count * a.sn;
    pl.M = (int32_t)((int64_t)(a.H / a.dict_count) * a.T);
    pl.V = (int64_t)a.H * a.T * a.sn;
    const int tiles = a.N / 32;
    int k = kTargetGroups / (n_dicts > 0 ? n_dicts : 1);
    if (k > tiles / kWaves) k = tiles / kWaves;  // at least one tile per wave
    if (k > kMaxSlices) k = kMaxSlices;
    if (k < 1) k = 1;
    pl.k = k;
    const int per_wave = ((tiles + k - 1) / k + kWaves - 1) / kWaves;
    pl.held = per_wave <= 1 ? 1 : per_wave <= 2 ? 2 : 4;   // of 128 dimensions: 32, 64 or 128 registers
    const int m_pad = (pl.M + 31) & ~31;
    pl.lds = (size_t)m_pad * a.d * 4 + (size_t)kWaves * m_pad * 8;
    if (pl.M > kNarrowVectors) pl.lds += (size_t)m_pad * a.d * 4 + (size_t)pl.M * sizeof(SplitState);
    pl.total = r256((size_t)a.s * pl.V * k * sizeof(unsigned long long));
    return pl;
}

template <int DC, int HELD, bool kNarrow>
hipError_t launch_split_t(const EncodeArgs &a, const SplitPlan &pl, const SplitParams &p)
{
    static std::atomic<bool> attr_set[64];   // per device, once: many vectors need more LDS than the default limit
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(encode_split_kernel<DC, HELD, kNarrow>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                159 * 1024);   // (plan_split: at most 139 KB)
        if (e != hipSuccess) return e;
        attr_set[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((encode_split_kernel<DC, HELD, kNarrow>), dim3((unsigned)(pl.k * p.n_dicts)), dim3(kThreads), pl.lds, a.stream, p);
    return hipGetLastError();
}

template <int DC>
hipError_t launch_split_held(const EncodeArgs &a, const SplitPlan &pl, const SplitParams &p)
{
    if (pl.M <= kNarrowVectors)
        return pl.held == 1 ? launch_split_t<DC, 1, true>(a, pl, p) : pl.held == 2 ? launch_split_t<DC, 2, true>(a, pl, p) : launch_split_t<DC, 4, true>(a, pl, p);
    return pl.held == 1 ? launch_split_t<DC, 1, false>(a, pl, p) : pl.held == 2 ? launch_split_t<DC, 2, false>(a, pl, p) : launch_split_t<DC, 4, false>(a, pl, p);
}

}  // namespace

bool encode_split_supported(const EncodeArgs &a)
{
    if (!(a.f16 && (a.d == 128 || a.d == 64) && a.N >= 32 && a.N % 32 == 0 && a.N <= (1 << 24))) return false;
    if (a.dict_count < 1 || a.H % a.dict_count != 0) return false;
    if ((int64_t)a.dict_count * a.sn > 65535) return false;
    return (int64_t)(a.H / a.dict_count) * a.T <= kMaxVectors;
}

size_t encode_split_workspace_bytes(const EncodeArgs &a) { return plan_split(a).total; }

hipError_t launch_encode_split(const EncodeArgs &a)
{
    const SplitPlan pl = plan_split(a);
    SplitParams p{};
    p.X = (const __half *)a.X; p.Dict = (const __half *)a.D; p.idx_out = a.idx; p.coef_out = a.coef;
    p.slots = reinterpret_cast<unsigned long long *>(a.workspace);
    p.V = pl.V; p.T = a.T; p.x_stride_h = a.x_stride_h; p.x_stride_t = a.x_stride_t; p.code_stride_h = a.code_stride_h;
    p.N = a.N; p.s = a.s; p.sn = a.sn; p.dict_count = a.dict_count; p.n_dicts = a.dict_count * a.sn; p.M = pl.M; p.k = pl.k;
    p.idx16 = a.idx16; p.coef_mode = (a.coef16 ? kCoefF16 : 0) | (a.closed_loop ? kCoefClosed : 0); p.res_norm2 = a.res_norm2;
    p.patience = a.no_wait ? -1 : kPatience;
    if (pl.k > 1) {
        const int64_t n2 = (int64_t)(pl.total / 16);
        hipLaunchKernelGGL(clear_slots_kernel, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, a.stream,
                           reinterpret_cast<ulonglong2 *>(a.workspace), n2);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return a.d == 64 ? launch_split_held<64>(a, pl, p) : launch_split_held<128>(a, pl, p);
}

}  // namespace csr
