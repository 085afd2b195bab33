// Router and gating for gfx950 (paper Sec. 3.1 Eq. (1); Sec. 3.2 Eqs. (4)-(5)
// sigmoid gating with renormalisation; Sec. 3.2 "Load Balancing" Eq. (7):
// the bias b is added to the sigmoid score for selection only).
//
// Routing decides integers, so it is computed reproducibly in fp32:
//   logit  = one fused multiply-add chain over i = 0..d-1, ascending, from +0
//   sigmoid = 1 / (1 + exp(-s)), exp by Cody-Waite reduction and a degree-7
//             Taylor polynomial, using only correctly rounded operations.
// This file is compiled with -ffp-contract=off so the compiler cannot fuse or
// reorder any of these steps.
#include "gemm_device.h"
#include "moe_internal.h"

#include <math.h>

#include <type_traits>
#include <utility>

namespace moe {
namespace {

// exp(z) = 2^n * exp(r), n = rint(z / ln 2), r = z - n ln 2 in two steps with
// ln 2 split into a 15-bit head (22713 * 2^-15, so n * head is exact for
// |n| <= 126) and the fp32-rounded remainder.
constexpr float kLog2e = 0x1.715476p+0f;   // fl32(1 / ln 2)
constexpr float kLn2Head = 0x1.62e4p-1f;   // 22713 * 2^-15
constexpr float kLn2Tail = 0x1.7f7d1cp-20f;  // fl32(ln 2 - head)

__device__ __forceinline__ float sigmoid_fp32(float s) {
    // Taylor coefficients 1/k!, each the correctly rounded fp32 quotient.
    const float q2 = 1.0f / 2.0f, q3 = 1.0f / 6.0f, q4 = 1.0f / 24.0f;
    const float q5 = 1.0f / 120.0f, q6 = 1.0f / 720.0f, q7 = 1.0f / 5040.0f;
    float z = -s;
    // Clamp so exp(z) and the quotient stay normal numbers (|z| <= 87).
    z = z > 87.0f ? 87.0f : z;
    z = z < -87.0f ? -87.0f : z;
    const float n = rintf(z * kLog2e);
    float r = fmaf(-n, kLn2Head, z);
    r = fmaf(-n, kLn2Tail, r);
    float p = fmaf(q7, r, q6);
    p = fmaf(p, r, q5);
    p = fmaf(p, r, q4);
    p = fmaf(p, r, q3);
    p = fmaf(p, r, q2);
    p = fmaf(p, r, 1.0f);
    p = fmaf(p, r, 1.0f);
    const float ez = ldexpf(p, (int)n);
    return 1.0f / (1.0f + ez);
}

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }

// Eight consecutive elements starting at p (16-byte aligned for bf16, two
// 16-byte loads for fp32), widened to fp32.
__device__ __forceinline__ void load8(const bf16_t* p, float* v) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        v[2 * q] = __uint_as_float(w[q] << 16);
        v[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
    }
}
__device__ __forceinline__ void load8(const float* p, float* v) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Rank of a selection key as an unsigned integer of the same order, from
// 0x007fffff for -inf up; a NaN counts as -inf (fmaxf returns the number).
// Every selection below compares ranks, with 0 for an unused or taken place,
// so a damaged key never displaces a sound one and K distinct experts in range
// come out whatever the keys are. (A key of -0 cannot occur: the sigmoid is
// positive, and a sum that cancels rounds to +0.)
__device__ __forceinline__ uint32_t key_rank(float key) {
    const uint32_t u = __float_as_uint(fmaxf(key, -INFINITY));
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Top-K selection and gates, one wavefront per token. Lane l holds experts
// l, l + 64, ...; each of the K rounds takes the wave-wide best (key
// descending, expert index ascending on equal keys) with a butterfly of
// cross-lane exchanges, then the owner lane marks it taken.
constexpr int kPerLane = kMaxE / kWave;

__global__ __launch_bounds__(256) void k_topk(const float* __restrict__ logits, int ld,
                                             const float* __restrict__ bias, int T, int E, int K,
                                             int32_t* __restrict__ topk_idx,
                                             float* __restrict__ topk_gate) {
    const int lane = threadIdx.x & (kWave - 1);
    const int t = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (t >= T) return;  // uniform per wave
    const int per = (E + kWave - 1) / kWave;
    float sig[kPerLane];
    uint32_t key[kPerLane];
#pragma unroll
    for (int m = 0; m < kPerLane; ++m) {
        const int e = lane + kWave * m;
        const bool ok = m < per && e < E;
        sig[m] = ok ? sigmoid_fp32(logits[(size_t)t * ld + e]) : 0.0f;
        key[m] = ok ? key_rank(bias ? sig[m] + bias[e] : sig[m]) : 0u;
    }
    uint32_t taken = 0;
    float csig[kMaxK];
    int cidx[kMaxK];
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        csig[j] = 0.0f;
        cidx[j] = 0;
        if (j >= K) continue;
        uint32_t bk = 0u;
        int be = 0x7fffffff;
        float bs = 0.0f;
#pragma unroll
        for (int m = 0; m < kPerLane; ++m) {
            const int e = lane + kWave * m;
            if (m < per && e < E && !((taken >> m) & 1u)) {
                if (key[m] > bk || (key[m] == bk && e < be)) {
                    bk = key[m];
                    be = e;
                    bs = sig[m];
                }
            }
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const uint32_t ok = __shfl_xor(bk, off);
            const int oe = __shfl_xor(be, off);
            const float os = __shfl_xor(bs, off);
            if (ok > bk || (ok == bk && oe < be)) {
                bk = ok;
                be = oe;
                bs = os;
            }
        }
        if ((be & (kWave - 1)) == lane) taken |= 1u << (be / kWave);
        csig[j] = bs;
        cidx[j] = be;
    }
    float den = csig[0];
#pragma unroll
    for (int j = 1; j < kMaxK; ++j)
        if (j < K) den = den + csig[j];
    int my_e = 0;
    float my_g = 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        if (j == lane && j < K) {
            my_e = cidx[j];
            my_g = csig[j] / den;
        }
    }
    if (lane < K) {
        topk_idx[(size_t)t * K + lane] = my_e;
        topk_gate[(size_t)t * K + lane] = my_g;
    }
}

// ---------------------------------------------------------------- fast path
//
// bf16 layers: the logits are first computed with the bf16 MFMA GEMM (every
// product of two bf16 values is exact in fp32; only the accumulation order
// differs from the FMA chain). For each (token, expert) the difference to the
// chain is bounded by (gamma_d + 4 d u) * ||x_t|| * ||w_e|| (u = 2^-24; the
// chain's own error is at most gamma_d * sum |x_i w_i|, the MFMA's at most
// 4 d u * sum |x_i w_i| under any accumulation order with per-addition error
// of 2u or less, and sum |x_i w_i| <= ||x|| ||w||). Through the sigmoid
// (1/4-Lipschitz, plus the recipe's own few-ulp error) and the bias addition
// this gives an interval around every key. The K-th largest lower end L is a
// lower bound of the true K-th key, so any expert whose upper end is below L
// cannot be selected. The remaining candidates (a dozen or so per token) are
// recomputed with the exact chain and selected exactly as on the exact path:
// indices and gates are identical bit for bit. A token with more candidates
// than its slots (16, or 32 when K > 8) is queued and routed by the exact
// all-experts kernel.
//
// The interval test itself uses a cheap sigmoid (hardware exp2 and
// reciprocal, absolute error below 1e-6 for every input, covered by extra
// slack in the half-width); only the candidates go through recipe S.

__device__ __forceinline__ float sigmoid_fast(float s) {
    return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-s * kLog2e));
}

// Upper bound of the 2-norm of every row of a [rows, d] bf16 matrix (fp32 sum
// of squares, inflated to cover its rounding). One wave per row. Block 0 also
// clears the overflow counter used by the repair kernel.
__global__ __launch_bounds__(256) void k_row_norms(const bf16_t* __restrict__ a, int rows, float* __restrict__ out,
                                                   int d, int32_t* __restrict__ clear, float* __restrict__ a32) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;
    const int lane = threadIdx.x & (kWave - 1);
    const int row = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (row >= rows) return;
    const bf16_t* p = a + (size_t)row * d;
    float acc = 0.0f;
    // a32 (optional): the rows of a widened to fp32 (exact), for the
    // small-batch chain kernel.
    float* const r32 = a32 ? a32 + (size_t)row * d : nullptr;
    for (int i = lane * 8; i < d; i += kWave * 8) {
        float v[8];
        load8(p + i, v);
#pragma unroll
        for (int q = 0; q < 8; ++q) acc = fmaf(v[q], v[q], acc);
        if (r32) {
            *reinterpret_cast<float4*>(r32 + i) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4*>(r32 + i + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) out[row] = sqrtf(acc) * 1.001f + 1e-30f;
}

// Maximum over each aligned group of 16 lanes (a DPP row), in every lane of
// the group: swaps inside quads (xor 1, xor 2), then the mirror inside each
// half row and the mirror of the whole row.
template <int CTRL>
__device__ __forceinline__ float dpp_max(float a) {
    return fmaxf(a, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), CTRL, 0xF, 0xF, false)));
}
__device__ __forceinline__ float row16_max(float v) {
    v = dpp_max<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_max<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = dpp_max<0x141>(v);  // row_half_mirror
    v = dpp_max<0x140>(v);  // row_mirror
    return v;
}

// Maximum over each aligned group of LPA lanes (16 or 64).
template <int LPA>
__device__ __forceinline__ float group_max(float v) {
    static_assert(LPA == 16 || LPA == 64, "groups of 16 or 64 lanes");
    v = row16_max(v);
    if constexpr (LPA == 64) {
        v = fmaxf(v, __shfl_xor(v, 16));
        v = fmaxf(v, __shfl_xor(v, 32));
    }
    return v;
}

// PER consecutive floats from a 16-byte aligned address.
template <int PER>
__device__ __forceinline__ void load_row(const float* p, float (&v)[PER]) {
#pragma unroll
    for (int i = 0; i < PER / 4; ++i) {
        const float4 q = *reinterpret_cast<const float4*>(p + 4 * i);
        v[4 * i] = q.x;
        v[4 * i + 1] = q.y;
        v[4 * i + 2] = q.z;
        v[4 * i + 3] = q.w;
    }
}

// ------------------------------------------------- exact logits on the matrix cores
//
// v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32 add their 2 or 4 products
// to the accumulator one after another in ascending k, each step one fused
// multiply-add rounded to fp32 (measured: bit-identical to a host fmaf chain
// for ordinary, cancelling, denormal, overflowing and non-finite sums). A K
// loop over ascending columns from a zero accumulator is therefore the logit's
// defined chain itself, at up to 141 TFLOP/s of the card's fp32 matrix rate,
// with no approximate pass and nothing to repair.
//
// Blocks of four waves, W_T x W_E wave tiles of TS tokens x TS experts (TS = 32
// or 16). Experts are the MFMA's rows and tokens its columns, so each lane
// holds runs of four experts of one token. Row pieces of 2 CH 16-byte chunks
// of the block's tokens and experts stream into a ring of ST slabs with
// direct-to-LDS copies, the chunks swizzled by row so that the 16 rows read
// together fall on distinct banks. The barrier of a slab sits before its
// second half's MFMAs, so the first words of the next slab are read behind
// them. What bounds it: few waves (one image and less) wait on their own
// chain, about 45 cycles per 16x16x4 step; many waves reach 115 of the 141
// TFLOP/s, the fp32 MFMAs and the permutes not overlapping fully. Measured,
// whole route, before (bf16 pre-pass GEMM and exact repair of the candidates)
// and after: 5 tokens d 1024 E 128 20.6 -> 15 us, 7175 tokens 73 -> 33 us,
// 18432 tokens d 768 E 64 49 -> 38 us, 65536 tokens d 1280 E 31 129 -> 65 us;
// kernels of one image (1025 tokens, d 1536, E 256) 32.1 -> 26.7 us; fp32 2304
// tokens d 768 E 64 61 -> 13.5 us (VALU chains before).
// The MFMA operands of this lane (row lane % TS, k index q = lane / TS) from a
// 16-byte row chunk in LDS: N words, one for each of the chunk's MFMAs,
// holding column q of its 2 (TS 32) or 4 (TS 16) columns. 32 x 32 tiles read
// bf16 chunks whole and widen by a byte permute (PERM); 16 x 16 tiles, whose
// waves wait on their own chain, read each bf16 value straight into the high
// half of its word (the low half stays 0) and leave no vector work between
// the MFMAs.
template <typename TIn, int TS>
struct ChainFrag {
    static constexpr int KM = TS == 32 ? 2 : 4;
    static constexpr int N = 16 / (int)sizeof(TIn) / KM;
    static constexpr bool BF16 = sizeof(TIn) == 2;
    static constexpr bool PERM = BF16 && TS == 32;
    // Byte offset of the lane's first value in the chunk.
    __device__ static uint32_t offset(int q) { return PERM ? 0u : (uint32_t)sizeof(TIn) * q; }
    __device__ static uint32_t selector(int q) {  // bytes of column q's half into the high half, 0 below
        return (q & 1) ? 0x03020c0cu : 0x01000c0cu;
    }
    // Reads of whole chunks fill a vector, which is split into words only after
    // the wait: a copy of a word before it could carry the register's old value.
    static constexpr bool VEC = PERM || (!BF16 && N == 2);
    typedef uint32_t vec_t __attribute__((ext_vector_type(PERM ? 4 : 2)));
    __device__ static void read(vec_t& v, uint32_t (&w)[N], uint32_t addr) {
        if constexpr (PERM) {
            v = lds_read16u_asm(addr);
        } else if constexpr (VEC) {
            lds_read2_asm(v, addr);
        } else if constexpr (BF16) {
            asm volatile("ds_read_u16_d16_hi %0, %1" : "+v"(w[0]) : "v"(addr));
            asm volatile("ds_read_u16_d16_hi %0, %1 offset:8" : "+v"(w[1]) : "v"(addr));
        } else {
            asm volatile("ds_read_b32 %0, %1" : "=v"(w[0]) : "v"(addr));
        }
    }
    // The words of a read that has been waited for.
    __device__ static void landed(vec_t& v, uint32_t (&w)[N]) {
        if constexpr (VEC) {
            tie(v);
#pragma unroll
            for (int m = 0; m < N; ++m) w[m] = v[m];
        } else {
#pragma unroll
            for (int m = 0; m < N; ++m) tie(w[m]);
        }
    }
};

template <typename TIn, int TS, int W_T, int W_E, int CH, int ST>
__global__ __launch_bounds__(256) void k_router_logits(const TIn* __restrict__ x, const TIn* __restrict__ wr,
                                                      float* __restrict__ logits, int T, int d, int E, int ld) {
    static_assert(W_T * W_E == 4, "four waves");
    constexpr int TR = W_T * TS, ER = W_E * TS;  // token and expert rows of the block
    constexpr int CPR = 2 * CH, ROWB = CPR * 16;  // 16-byte chunks and bytes of a row piece
    constexpr int SLAB = (TR + ER) * ROWB;
    constexpr int RPP = kWave / CPR;  // rows per 1 KB copy piece
    constexpr int P = (TR + ER) / RPP / 4;  // 1 KB copy pieces per wave and slab
    static_assert((TR + ER) % (4 * RPP) == 0 && TR % RPP == 0 && (ST - 2) * P <= 63, "even pieces, counted in vmcnt");
    constexpr int KB = ROWB / (int)sizeof(TIn);
    using Frag = ChainFrag<TIn, TS>;
    constexpr int NF = Frag::N;
    constexpr int NA = TS == 32 ? 16 : 4;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[ST * SLAB];
    // XCD-aware order, the expert tiles of one token tile adjacent (they
    // share its x rows in one L2).
    const int n_e = (E + ER - 1) / ER;
    const int total = (T + TR - 1) / TR * n_e;
    const int per = (total + kNumXcd - 1) / kNumXcd;
    const int j8 = (int)blockIdx.x / kNumXcd;
    const int lid = ((int)blockIdx.x % kNumXcd) * per + j8;
    if (j8 >= per || lid >= total) return;
    const int t0 = lid / n_e * TR, e0 = lid % n_e * ER;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wt = wave / W_E, we = wave % W_E;
    const uint32_t rowb = (uint32_t)d * sizeof(TIn);
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(x, (uint32_t)T * rowb);
    const __amdgpu_buffer_rsrc_t wres = make_rsrc(wr, (uint32_t)E * rowb);
    // Copy piece i of this wave: RPP rows (8, or 4 of 256 bytes), tokens first; token rows past T repeat
    // the last one (not stored), expert rows past E read as zeros.
    auto swz = [](int r) { return CPR == 8 ? (r >> 1) & 7 : r & 15; };
    uint32_t off[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int r = (wave + 4 * i) * RPP + lane / CPR;
        const int c = (lane % CPR) ^ swz(r);
        const uint32_t row = r < TR ? (uint32_t)min(t0 + r, T - 1) : (uint32_t)(e0 + r - TR);
        off[i] = row * rowb + c * 16;
    }
    auto issue = [&](int slot, int kt) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const bool tok = (wave + 4 * i) * RPP < TR;  // uniform per wave
            copy16_to_lds(tok ? xres : wres, off[i], (uint32_t)kt * (uint32_t)ROWB, smem + slot * SLAB + (wave + 4 * i) * 1024);
        }
    };
    // Fragment chunk c of a row: tokens at xo, experts at eo.
    const int fr = lane % TS, q = lane / TS;
    const uint32_t base = lds_address(smem);
    const uint32_t xo = base + (uint32_t)((wt * TS + fr) * ROWB) + Frag::offset(q);
    const uint32_t eo = base + (uint32_t)((TR + we * TS + fr) * ROWB) + Frag::offset(q);
    const int sw = swz(fr);  // rows of a fragment start at multiples of 16
    uint32_t sel = Frag::selector(q);
    asm volatile("" : "+v"(sel));
    uint32_t xf[2][CH][NF] = {}, wf[2][CH][NF] = {};
    typename Frag::vec_t xv[2][CH], wv[2][CH];
    auto read_chunk = [&](int slot, auto HC, int c) {
        constexpr int h = decltype(HC)::value;
        const uint32_t o = (uint32_t)slot * SLAB + (uint32_t)(((CH * h + c) ^ sw) << 4);
        Frag::read(xv[h][c], xf[h][c], xo + o);
        Frag::read(wv[h][c], wf[h][c], eo + o);
    };
    // Half h's words have landed; widen them (PERM). All of it before the
    // half's first MFMA: a vector operation between two dependent MFMAs costs
    // 8 to 20 cycles of the chain (16x16x4: 54 instead of 33 cycles per step
    // with two permutes between).
    auto take_half = [&](auto HC) {
        constexpr int h = decltype(HC)::value;
        wait_lgkmcnt0();
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            Frag::landed(wv[h][c], wf[h][c]);
            Frag::landed(xv[h][c], xf[h][c]);
            if constexpr (Frag::PERM)
#pragma unroll
                for (int m = 0; m < NF; ++m) {
                    wf[h][c][m] = __builtin_amdgcn_perm(0u, wf[h][c][m], sel);
                    xf[h][c][m] = __builtin_amdgcn_perm(0u, xf[h][c][m], sel);
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    typedef float acc_t __attribute__((ext_vector_type(NA)));
    acc_t acc;
#pragma unroll
    for (int v = 0; v < NA; ++v) acc[v] = 0.0f;
    // Half h's MFMAs, the words of half RC of slab `slot` read between them
    // (READ): LDS reads, unlike vector operations, do not delay the chain.
    auto mul_half = [&](auto HC, auto RC, int slot, bool read) {
        constexpr int h = decltype(HC)::value;
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int m = 0; m < NF; ++m) {
                const float w = __uint_as_float(wf[h][c][m]), v = __uint_as_float(xf[h][c][m]);
                if constexpr (TS == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w, v, acc, 0, 0, 0);
                else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w, v, acc, 0, 0, 0);
                if (m == 0 && read) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_chunk(slot, RC, c);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    // Slab kt's copies have landed for this wave, `ahead` younger slabs in flight.
    auto wait_slab = [&](int ahead) {
        static_for<ST - 1>([&](auto AC) {
            constexpr int A = decltype(AC)::value;
            if (ahead == A) wait_vmcnt<A * P>();
        });
    };
    const int nk = d / KB;
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
        if (s < nk) issue(s, s);
    wait_slab(min(nk, ST - 1) - 1);
    barrier_no_fence();
    const std::integral_constant<int, 0> H0;
    const std::integral_constant<int, 1> H1;
#pragma unroll
    for (int c = 0; c < CH; ++c) read_chunk(0, H0, c);
    int slot = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // Slab kt + ST - 1 goes to the slot of slab kt - 1, which every wave
        // finished reading before the last barrier.
        if (kt + ST - 1 < nk) issue(slot == 0 ? ST - 1 : slot - 1, kt + ST - 1);
        take_half(H0);
        mul_half(H0, H1, slot, true);
        take_half(H1);
        slot = slot == ST - 1 ? 0 : slot + 1;
        if (kt + 1 < nk) {
            wait_slab(min(nk - 1, kt + ST - 1) - (kt + 1));
            barrier_no_fence();
            mul_half(H1, H0, slot, true);
        } else {
            mul_half(H1, H0, slot, false);
        }
    }
    // D rows (experts) of lane l: TS == 32: 8 g + 4 (l / 32) + v; 16: 4 (l / 16) + v.
    const int t = t0 + wt * TS + fr;
    if (t >= T) return;
    float* const row = logits + (size_t)t * ld + e0 + we * TS + 4 * q;
#pragma unroll
    for (int g = 0; g < NA / 4; ++g)
        *reinterpret_cast<float4*>(row + 8 * g) = make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
}

// Maximum of an unsigned key over each aligned group of 16 lanes, in every lane.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_umax(uint32_t a) {
    return max(a, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a, CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ uint32_t row16_umax(uint32_t v) {
    v = dpp_umax<0xB1>(v);
    v = dpp_umax<0x4E>(v);
    v = dpp_umax<0x141>(v);
    return dpp_umax<0x140>(v);
}

// Sigmoids, top-K and gates from exact logits for up to 16 PER experts: 16
// lanes per token (lane g holds experts g PER ..), 4 tokens per wave. Each of
// the K rounds takes the group's largest key rank, lowest lane and then lowest
// expert on ties. The winners' experts and the token's sigmoids meet in LDS
// for the denominator in slot order.
template <int PER>
__global__ __launch_bounds__(256) void k_topk16(const float* __restrict__ logits, int ld,
                                               const float* __restrict__ bias, int T, int E, int K,
                                               int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate) {
    static_assert(PER % 4 == 0, "whole 16-byte loads");
    __shared__ __attribute__((aligned(16))) float ssig[16][16 * PER + 4];
    __shared__ int32_t sidx[16][kMaxK];
    const int lane = threadIdx.x & (kWave - 1);
    const int g = lane & 15;
    const int tl = threadIdx.x / 16;
    const int t = blockIdx.x * (blockDim.x / 16) + tl;
    const int e0 = g * PER;
    float s[PER], b[PER];
    load_row<PER>(logits + (size_t)min(t, T - 1) * ld + (e0 < ld ? e0 : 0), s);
#pragma unroll
    for (int m = 0; m < PER; ++m) b[m] = bias ? bias[min(e0 + m, E - 1)] : 0.0f;
    uint32_t key[PER];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        s[m] = sigmoid_fp32(s[m]);
        key[m] = e0 + m < E ? key_rank(bias ? s[m] + b[m] : s[m]) : 0u;
    }
#pragma unroll
    for (int m = 0; m < PER; m += 4)
        *reinterpret_cast<float4*>(&ssig[tl][e0 + m]) = make_float4(s[m], s[m + 1], s[m + 2], s[m + 3]);
    for (int j = 0; j < K; ++j) {
        uint32_t mine = key[0];
#pragma unroll
        for (int m = 1; m < PER; ++m) mine = max(mine, key[m]);
        const uint32_t best = row16_umax(mine);
        const uint32_t holders = (uint32_t)(__ballot(mine == best) >> (lane & 48)) & 0xffffu;
        if (g == __ffs(holders) - 1) {
            int mi = PER - 1;
#pragma unroll
            for (int m = PER - 2; m >= 0; --m) mi = key[m] == best ? m : mi;
#pragma unroll
            for (int m = 0; m < PER; ++m) key[m] = m == mi ? 0u : key[m];
            sidx[tl][j] = e0 + mi;
        }
    }
    __syncthreads();
    if (t >= T) return;
    // Gate denominator in slot order.
    const int my = g < K ? sidx[tl][g] : 0;
    float den = ssig[tl][sidx[tl][0]];
    for (int j = 1; j < K; ++j) den = den + ssig[tl][sidx[tl][j]];
    if (g < K) {
        topk_idx[(size_t)t * K + g] = my;
        topk_gate[(size_t)t * K + g] = ssig[tl][my] / den;
    }
}

// Candidates of each token: LPA lanes per token, lane g holding experts
// g PER .. g PER + PER - 1 (contiguous, so that its logits are PER / 4
// 16-byte loads); the MFMA logits have rows of ld >= E (a multiple of 64), in
// nsplit partial arrays (split K) sstride floats apart. L = the K-th largest
// lower end of the key intervals; the candidates are the experts whose upper
// end reaches L, written to cand[t][0 .. NS) (in no particular order) with
// their count in ncand[t]. A token with more than NS candidates gets
// ncand = -1 and is appended to the overflow queue. An interval without
// numbers (a NaN logit, norm or bias) reaches from -inf to +inf: it raises no
// L, and its expert is a candidate, whose exact key decides; the interval of
// a -inf bias is that one point.
template <int LPA, int PER, int NS, bool SPLIT>
__global__ __launch_bounds__(256) void k_router_cand(const float* __restrict__ s_fast,
                                                    const bf16_t* __restrict__ x,
                                                    const float* __restrict__ xnorm2, int d,
                                                    const float* __restrict__ wnorm,
                                                    const float* __restrict__ bias, int T, int E, int ld,
                                                    int K, float cst, uint16_t* __restrict__ cand,
                                                    int32_t* __restrict__ ncand, int32_t* __restrict__ ovf_count,
                                                    int32_t* __restrict__ ovf_list, int nsplit, size_t sstride) {
    static_assert(LPA <= kWave && kWave % LPA == 0, "token groups inside a wave");
    static_assert(PER % 4 == 0 && 64 % PER == 0, "whole 16-byte loads inside a row of a multiple of 64");
    const int lane = threadIdx.x & (kWave - 1);
    const int g = lane % LPA;
    const int t = blockIdx.x * (blockDim.x / LPA) + threadIdx.x / LPA;
    const bool live = t < T;  // uniform within the group: dead groups compute on -inf
    const uint64_t grp = (LPA == kWave ? ~0ull : ((1ull << LPA) - 1ull)) << (lane - g);

    // Selection biases and weight-row norms of all experts, in LDS.
    static_assert(LPA * PER <= kMaxE, "the lanes' experts inside the arrays");
    __shared__ __attribute__((aligned(16))) float sb[kMaxE];
    __shared__ __attribute__((aligned(16))) float swn[kMaxE];
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        sb[e] = bias ? bias[e] : 0.0f;
        swn[e] = wnorm[e];
    }

    // ||x_t||, raised by 0.1 % as k_row_norms does for the weight rows (an
    // upper bound is all the interval needs; the rounding of the sum of
    // squares, in any order, is far inside that margin). The sum of squares
    // comes from the logits GEMM (xnorm2) or, without it, from the token's
    // LPA lanes reading its row in 16-byte pieces and adding their partial
    // sums.
    float ss = 0.0f;
    if (xnorm2) {
        ss = live ? xnorm2[t] : 0.0f;
    } else {
        if (live) {
            // Four pieces per round, all loaded before the adds.
            const bf16_t* xr = x + (size_t)t * d;
            for (int i = g * 8; i < d; i += 4 * LPA * 8) {
                float v[4][8];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i + u * LPA * 8 < d) load8(xr + i + u * LPA * 8, v[u]);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i + u * LPA * 8 < d)
#pragma unroll
                        for (int q = 0; q < 8; ++q) ss = fmaf(v[u][q], v[u][q], ss);
            }
        }
#pragma unroll
        for (int off = LPA / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    }
    const float xn = live ? sqrtf(ss) * 1.001f + 1e-30f : 0.0f;

    // Fast logits of the lane's experts. Split-K logits (SPLIT, up to 8
    // parts): the partial sums in part order (any order of the d products is
    // covered by the bound), with every part's loads issued before the first
    // add (parts past nsplit re-read part 0 and are not added).
    // Dead tokens read row 0 and lanes past the logit row column 0 (neither
    // is used), so the loads need no branch.
    const int e0 = g * PER;
    float sf[PER];
    {
        const float* row = s_fast + (size_t)(live ? t : 0) * ld + (e0 < ld ? e0 : 0);
        if constexpr (SPLIT) {
            float pv[8][PER];
#pragma unroll
            for (int q = 0; q < 8; ++q) load_row<PER>(row + (q < nsplit ? q * sstride : 0), pv[q]);
#pragma unroll
            for (int m = 0; m < PER; ++m) sf[m] = pv[0][m];
#pragma unroll
            for (int q = 1; q < 8; ++q)
#pragma unroll
                for (int m = 0; m < PER; ++m) sf[m] = q < nsplit ? sf[m] + pv[q][m] : sf[m];
        } else {
            load_row<PER>(row, sf);
        }
    }
    __syncthreads();
    // The lane's biases and norms in 16-byte LDS reads (entries past E are
    // read but not used), then every interval without a branch.
    float bv[PER], wn[PER];
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
        const float4 b4 = *reinterpret_cast<const float4*>(sb + e0 + 4 * q);
        const float4 n4 = *reinterpret_cast<const float4*>(swn + e0 + 4 * q);
        bv[4 * q] = b4.x, bv[4 * q + 1] = b4.y, bv[4 * q + 2] = b4.z, bv[4 * q + 3] = b4.w;
        wn[4 * q] = n4.x, wn[4 * q + 1] = n4.y, wn[4 * q + 2] = n4.z, wn[4 * q + 3] = n4.w;
    }
    float lo[PER], hi[PER];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const bool ok = live && e0 + m < E;
        const float key = sigmoid_fast(sf[m]) + bv[m];
        const float delta = 0.25f * (cst * xn * wn[m]) + 4e-6f + 1e-6f * fabsf(bv[m]);
        lo[m] = ok ? fmaxf(key - delta, -INFINITY) : -INFINITY;  // fmaxf: the number, if one is a NaN
        hi[m] = ok ? fmaxf(key + delta, key) : -INFINITY;
    }
    // L: the K-th largest of the lanes' three largest lower ends. These are a
    // subset of all lower ends, so L is at most the K-th largest lower end and
    // still a lower bound of the true K-th key; it equals it unless one lane
    // holds four or more of the K largest.
    float t1 = -INFINITY, t2 = -INFINITY, t3 = -INFINITY;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const float v = lo[m];
        t3 = fmaxf(t3, fminf(t2, v));
        t2 = fmaxf(t2, fminf(t1, v));
        t1 = fmaxf(t1, v);
    }
    float L = -INFINITY;
    int used = 0;  // how many of t1, t2, t3 (in that order) have been taken
    for (int j = 0; j < K; ++j) {
        const float mine = used == 0 ? t1 : (used == 1 ? t2 : (used == 2 ? t3 : -INFINITY));
        const float gmax = group_max<LPA>(mine);
        const uint64_t holders = __ballot(used < 3 && mine == gmax) & grp;
        if (holders && lane == __ffsll((unsigned long long)holders) - 1) ++used;
        L = gmax;
    }
    int nc = 0;
    if constexpr (LPA == 16) {
        // Lane g's candidates in expert order after those of lanes 0 .. g - 1
        // (an inclusive scan of the lanes' counts along the 16-lane DPP row).
        uint32_t cbits = 0;
#pragma unroll
        for (int m = 0; m < PER; ++m) cbits |= (live && !(hi[m] < L)) ? (1u << m) : 0u;
        const int cnt = __popc(cbits);
        int incl = cnt;
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x111, 0xF, 0xF, false);  // row_shr:1
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x112, 0xF, 0xF, false);  // row_shr:2
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x114, 0xF, 0xF, false);  // row_shr:4
        incl += __builtin_amdgcn_update_dpp(0, incl, 0x118, 0xF, 0xF, false);  // row_shr:8
        nc = __builtin_amdgcn_update_dpp(0, incl, 0x15F, 0xF, 0xF, false);     // row_newbcast:15
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const int pos = incl - cnt + __popc(cbits & ((1u << m) - 1u));
            if (((cbits >> m) & 1u) && pos < NS) cand[(size_t)t * NS + pos] = (uint16_t)(e0 + m);
        }
    } else {
        const uint64_t below = grp & ((1ull << lane) - 1ull);
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            const bool c = live && !(hi[m] < L);
            const uint64_t bal = __ballot(c) & grp;
            if (c) {
                const int pos = nc + __popcll(bal & below);
                if (pos < NS) cand[(size_t)t * NS + pos] = (uint16_t)(e0 + m);
            }
            nc += __popcll(bal);
        }
    }
    if (live && g == 0) {
        if (nc > NS) {
            const int slot = atomicAdd(ovf_count, 1);
            ovf_list[slot] = t;
            nc = -1;
        }
        ncand[t] = nc;
    }
}

// Exact top-K of a token's candidates and their gates, for the chain kernels
// (TPB tokens of LPT lanes, CPL chains per lane; candidate slot g + LPT c of
// token tl holds expert ec[c] with exact logit acc[c]). Every candidate's key
// (the rank of sigmoid plus selection bias), sigmoid and expert go to LDS; each
// lane ranks its own candidates among the token's in (key descending, expert
// ascending) order, the order of taking the K largest keys one by one; ranks
// below K are the slots. Then every lane of the token forms the gate
// denominator in slot order and writes its slots. Called by every thread of
// the block once its chains are done; lds holds at least
// TPB (12 LPT CPL + 8 kMaxK) bytes and is no longer read by the chains.
template <int TPB, int LPT, int CPL>
__device__ __forceinline__ void chain_select(uint8_t* lds, int tl, int g, int t, int T, int nc, int K,
                                             const bool (&on)[CPL], const int (&ec)[CPL], const float (&acc)[CPL],
                                             const float (&bc)[CPL], bool has_bias, int32_t* __restrict__ topk_idx,
                                             float* __restrict__ topk_gate) {
    constexpr int NS = LPT * CPL;
    uint32_t* skey = reinterpret_cast<uint32_t*>(lds);
    float* ssig = reinterpret_cast<float*>(skey + TPB * NS);
    int* sexp = reinterpret_cast<int*>(ssig + TPB * NS);
    float* osig = reinterpret_cast<float*>(sexp + TPB * NS);
    int* oexp = reinterpret_cast<int*>(osig + TPB * kMaxK);
    uint32_t kc[CPL];
    float sc[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int j = g + LPT * c;
        sc[c] = 0.0f;
        kc[c] = 0u;
        if (on[c]) {
            sc[c] = sigmoid_fp32(acc[c]);
            kc[c] = key_rank(has_bias ? sc[c] + bc[c] : sc[c]);
            skey[tl * NS + j] = kc[c];
            ssig[tl * NS + j] = sc[c];
            sexp[tl * NS + j] = ec[c];
        }
    }
    __syncthreads();
    // The token's NS keys and experts in 16-byte reads (slots from nc on are
    // read but not counted).
    static_assert(NS % 4 == 0, "whole 16-byte reads");
    uint32_t kq[NS];
    int eq[NS];
#pragma unroll
    for (int q = 0; q < NS; q += 4) {
        const uint4 k4 = *reinterpret_cast<const uint4*>(skey + tl * NS + q);
        const int4 e4 = *reinterpret_cast<const int4*>(sexp + tl * NS + q);
        kq[q] = k4.x, kq[q + 1] = k4.y, kq[q + 2] = k4.z, kq[q + 3] = k4.w;
        eq[q] = e4.x, eq[q + 1] = e4.y, eq[q + 2] = e4.z, eq[q + 3] = e4.w;
    }
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        if (!on[c]) continue;
        int rank = 0;  // the candidate itself compares neither greater nor lower
#pragma unroll
        for (int q = 0; q < NS; ++q)
            rank += (q < nc && (kq[q] > kc[c] || (kq[q] == kc[c] && eq[q] < ec[c]))) ? 1 : 0;
        if (rank < K) {
            osig[tl * kMaxK + rank] = sc[c];
            oexp[tl * kMaxK + rank] = ec[c];
        }
    }
    __syncthreads();
    if (t >= T || nc == 0) return;
    // Gate denominator in slot order 0 .. K - 1.
    float os[kMaxK];
#pragma unroll
    for (int j = 0; j < kMaxK; j += 4) {
        const float4 o4 = *reinterpret_cast<const float4*>(osig + tl * kMaxK + j);
        os[j] = o4.x, os[j + 1] = o4.y, os[j + 2] = o4.z, os[j + 3] = o4.w;
    }
    float den = os[0];
#pragma unroll
    for (int j = 1; j < kMaxK; ++j) den = j < K ? den + os[j] : den;
    for (int j = g; j < K; j += LPT) {
        topk_idx[(size_t)t * K + j] = oexp[tl * kMaxK + j];
        topk_gate[(size_t)t * K + j] = osig[tl * kMaxK + j] / den;
    }
}

// Exact top-K of token t from its E sigmoids (sig, in LDS) and gates, by one
// wave: each of the K rounds takes the wave-wide best key (descending, lower
// expert index first on equal keys) with a butterfly of cross-lane exchanges.
__device__ __forceinline__ void exact_select_wave(const float* sig, const float* __restrict__ bias, int E, int K,
                                                  int t, int lane, int32_t* __restrict__ topk_idx,
                                                  float* __restrict__ topk_gate) {
    const int per = (E + kWave - 1) / kWave;
    float sg[kPerLane];
    uint32_t key[kPerLane];
#pragma unroll
    for (int m = 0; m < kPerLane; ++m) {
        const int e = lane + kWave * m;
        const bool ok = m < per && e < E;
        sg[m] = ok ? sig[e] : 0.0f;
        key[m] = ok ? key_rank(bias ? sg[m] + bias[e] : sg[m]) : 0u;
    }
    uint32_t taken = 0;
    float csig[kMaxK];
    int cidx[kMaxK];
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        csig[j] = 0.0f;
        cidx[j] = 0;
        if (j >= K) continue;
        uint32_t bk = 0u;
        int be = 0x7fffffff;
        float bs = 0.0f;
#pragma unroll
        for (int m = 0; m < kPerLane; ++m) {
            const int e = lane + kWave * m;
            if (m < per && e < E && !((taken >> m) & 1u) && (key[m] > bk || (key[m] == bk && e < be))) {
                bk = key[m];
                be = e;
                bs = sg[m];
            }
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const uint32_t ok = __shfl_xor(bk, off);
            const int oe = __shfl_xor(be, off);
            const float os = __shfl_xor(bs, off);
            if (ok > bk || (ok == bk && oe < be)) {
                bk = ok;
                be = oe;
                bs = os;
            }
        }
        if ((be & (kWave - 1)) == lane) taken |= 1u << (be / kWave);
        csig[j] = bs;
        cidx[j] = be;
    }
    float den = csig[0];
#pragma unroll
    for (int j = 1; j < kMaxK; ++j)
        if (j < K) den = den + csig[j];
    int my_e = 0;
    float my_g = 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j)
        if (j == lane && j < K) {
            my_e = cidx[j];
            my_g = csig[j] / den;
        }
    if (lane < K) {
        topk_idx[(size_t)t * K + lane] = my_e;
        topk_gate[(size_t)t * K + lane] = my_g;
    }
}

// Exact routing of the queued tokens: all E logits by the FMA chain, then
// the same top-K. Blocks first, first + stride, ... walk the queue (fixed by
// the time this runs); every block exits once it is exhausted. Any block
// size that is a multiple of the wave works (the selection uses wave 0).
__device__ __forceinline__ void exact_list_run(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wr,
                               const float* __restrict__ bias, int d, int E, int K,
                               const int32_t* __restrict__ ovf_count, const int32_t* __restrict__ ovf_list,
                               int32_t* __restrict__ topk_idx, float* __restrict__ topk_gate, int first,
                               int stride) {
    __shared__ float sig[kMaxE];
    const int n = *ovf_count;
    const int lane = threadIdx.x & (kWave - 1);
    for (int it = first; it < n; it += stride) {
        const int t = ovf_list[it];
        const bf16_t* xt = x + (size_t)t * d;
        for (int e = threadIdx.x; e < E; e += blockDim.x) {
            const bf16_t* we = wr + (size_t)e * d;
            // The same fma sequence over i = 0..d-1; the loads of 32 columns
            // are issued before their multiply-adds (d is a multiple of 64).
            float a = 0.0f;
            for (int i = 0; i < d; i += 32) {
                float xv[4][8], wv[4][8];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    load8(xt + i + 8 * q, xv[q]);
                    load8(we + i + 8 * q, wv[q]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int u = 0; u < 8; ++u) a = fmaf(xv[q][u], wv[q][u], a);
            }
            sig[e] = sigmoid_fp32(a);
        }
        __syncthreads();
        if (threadIdx.x < kWave) exact_select_wave(sig, bias, E, K, t, lane, topk_idx, topk_gate);
        __syncthreads();
    }
}

// Exact logits of the candidates, recipe S, exact top-K and gates. LPT lanes
// per token, each running CPL candidate chains (slots g, g + LPT, ...) side by
// side: one fused multiply-add chain per candidate over the model width, in
// ascending order. The block's tokens stream their x rows from global memory;
// the router weights of every expert stream through LDS in chunks of DC
// columns (bf16, rows padded by 16 bytes against bank conflicts, widened to
// fp32 in registers), double-buffered with one barrier per chunk; DC must
// divide d. Tokens queued by the candidate kernel are skipped.
template <int TPB, int LPT, int CPL, int EMAX, int DC>
__global__ __launch_bounds__(TPB* LPT) void k_router_chain(const bf16_t* __restrict__ x,
                                                         const bf16_t* __restrict__ wr,
                                                         const float* __restrict__ bias,
                                                         const uint16_t* __restrict__ cand,
                                                         const int32_t* __restrict__ ncand, int T, int d, int E,
                                                         int K, int32_t* __restrict__ topk_idx,
                                                         float* __restrict__ topk_gate, int chain_blocks,
                                                         const int32_t* __restrict__ ovf_count,
                                                         const int32_t* __restrict__ ovf_list) {
    // Blocks from chain_blocks on route the tokens of the overflow queue (all
    // of it is written: the candidate kernel has finished); with an empty
    // queue they exit at once.
    if ((int)blockIdx.x >= chain_blocks) {
        exact_list_run(x, wr, bias, d, E, K, ovf_count, ovf_list, topk_idx, topk_gate,
                       (int)blockIdx.x - chain_blocks, (int)gridDim.x - chain_blocks);
        return;
    }
    constexpr int NT = TPB * LPT;
    constexpr int NS = LPT * CPL;
    constexpr int ROW = DC + 8;             // bf16 per LDS row (16 bytes of padding)
    constexpr int XQ = DC / 8;              // 16-byte x pieces per chunk
    constexpr int WP = EMAX * DC / 8;        // 16-byte router-weight pieces per chunk
    constexpr int WQ = (WP + NT - 1) / NT;   // per thread
    static_assert(NS <= 32, "at most 32 candidate slots");
    constexpr int RING = 2 * EMAX * ROW * 2, SEL = TPB * (NS * 12 + kMaxK * 8);
    __shared__ __attribute__((aligned(16))) uint8_t lds[RING > SEL ? RING : SEL];
    auto wsh = reinterpret_cast<bf16_t(*)[EMAX][ROW]>(lds);

    const int tid = threadIdx.x;
    const int g = tid % LPT;
    const int tl = tid / LPT;

    // Token slots grouped by the chains per lane each token needs (0..CPL).
    // A wave runs as many chains per lane as its busiest token; in token
    // order nearly every wave holds some token with a few extra candidates,
    // grouped most waves run only the chains of a token with K candidates.
    // The order is ascending token within a group; a token's results do not
    // depend on the lanes that compute it.
    static_assert(TPB % kWave == 0 && NT >= TPB, "token slots fill whole waves");
    constexpr int TW = TPB / kWave;
    __shared__ int32_t sperm[TPB];
    __shared__ int32_t sgrp[TW][CPL + 1];
    {
        const int lane = tid & (kWave - 1), wv = tid / kWave;
        int key = 0;
        uint64_t same = 0;
        if (tid < TPB) {  // whole waves
            const int u = blockIdx.x * TPB + tid;
            const int n = u < T ? ncand[u] : 0;
            key = n <= 0 ? 0 : min((n + LPT - 1) / LPT, CPL);
#pragma unroll
            for (int k = 0; k <= CPL; ++k) {
                const uint64_t m = __ballot(key == k);
                if (k == key) same = m;
                if (lane == 0) sgrp[wv][k] = __popcll(m);
            }
        }
        __syncthreads();
        if (tid < TPB) {
            int pos = __popcll(same & ((1ull << lane) - 1ull));
            for (int k = 0; k < key; ++k)
                for (int w = 0; w < TW; ++w) pos += sgrp[w][k];
            for (int w = 0; w < wv; ++w) pos += sgrp[w][key];
            sperm[pos] = tid;
        }
        __syncthreads();
    }
    const int t = blockIdx.x * TPB + sperm[tl];
    int nc = t < T ? ncand[t] : 0;
    nc = nc < 0 ? 0 : nc;  // queued tokens are routed by the exact-list kernel
    int ec[CPL];
    bool on[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int j = g + LPT * c;
        on[c] = j < nc;
        ec[c] = on[c] ? (int)cand[(size_t)t * NS + j] : 0;
    }
    const bf16_t* xt = x + (size_t)(t < T ? t : 0) * d;
    float bc[CPL];  // selection bias of each chain's expert, read while the chains run
#pragma unroll
    for (int c = 0; c < CPL; ++c) bc[c] = (bias && on[c]) ? bias[ec[c]] : 0.0f;

    u32x4_t xr[XQ], wrg[WQ];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < XQ; ++i) xr[i] = *reinterpret_cast<const u32x4_t*>(xt + k0 + 8 * i);
#pragma unroll
        for (int i = 0; i < WQ; ++i) {
            const int q = (tid + NT * i) * 8;  // element of the EMAX x DC chunk
            const int e = q / DC, c = q % DC;
            wrg[i] = (u32x4_t){0u, 0u, 0u, 0u};
            if (tid + NT * i < WP && e < E) wrg[i] = *reinterpret_cast<const u32x4_t*>(wr + (size_t)e * d + k0 + c);
        }
    };
    auto stash = [&](int b) {
#pragma unroll
        for (int i = 0; i < WQ; ++i) {
            if (tid + NT * i >= WP) continue;
            const int q = (tid + NT * i) * 8;
            *reinterpret_cast<u32x4_t*>(&wsh[b][q / DC][q % DC]) = wrg[i];
        }
    };

    float acc[CPL];
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = 0.0f;

    // One chunk: for every 8 columns, widen x once and advance each of the
    // first NC chains by 8 fused multiply-adds (ascending columns).
    auto chunk = [&](auto NCC, int b) {
        constexpr int NC = decltype(NCC)::value;
#pragma unroll
        for (int i = 0; i < XQ; ++i) {
            const u32x4_t u = xr[i];
            const float x0 = __uint_as_float(u.x << 16), x1 = __uint_as_float(u.x & 0xffff0000u);
            const float x2 = __uint_as_float(u.y << 16), x3 = __uint_as_float(u.y & 0xffff0000u);
            const float x4 = __uint_as_float(u.z << 16), x5 = __uint_as_float(u.z & 0xffff0000u);
            const float x6 = __uint_as_float(u.w << 16), x7 = __uint_as_float(u.w & 0xffff0000u);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const u32x4_t w = *reinterpret_cast<const u32x4_t*>(&wsh[b][ec[c]][8 * i]);
                float a = acc[c];
                a = fmaf(x0, __uint_as_float(w.x << 16), a);
                a = fmaf(x1, __uint_as_float(w.x & 0xffff0000u), a);
                a = fmaf(x2, __uint_as_float(w.y << 16), a);
                a = fmaf(x3, __uint_as_float(w.y & 0xffff0000u), a);
                a = fmaf(x4, __uint_as_float(w.z << 16), a);
                a = fmaf(x5, __uint_as_float(w.z & 0xffff0000u), a);
                a = fmaf(x6, __uint_as_float(w.w << 16), a);
                a = fmaf(x7, __uint_as_float(w.w & 0xffff0000u), a);
                acc[c] = a;
            }
            // Keep the compiler from hoisting every fragment read of the chunk
            // (registers, not latency, bound this kernel's occupancy).
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int nmax = 0;  // chains any lane of this wave runs (uniform)
#pragma unroll
    for (int c = 0; c < CPL; ++c) nmax += __ballot(on[c]) != 0 ? 1 : 0;

    u32x4_t xn[XQ];
    fetch(0);
    stash(0);
    __syncthreads();
    int buf = 0;
    const int nch = d / DC;
    for (int ch = 0; ch < nch; ++ch) {
        // Next chunk in flight during this one: its x into xn, its weights
        // into registers (stored to the other buffer after the chains).
        if (ch + 1 < nch) {
            const int k1 = (ch + 1) * DC;
#pragma unroll
            for (int i = 0; i < XQ; ++i) xn[i] = *reinterpret_cast<const u32x4_t*>(xt + k1 + 8 * i);
#pragma unroll
            for (int i = 0; i < WQ; ++i) {
                const int q = (tid + NT * i) * 8;
                const int e = q / DC, c = q % DC;
                wrg[i] = (u32x4_t){0u, 0u, 0u, 0u};
                if (tid + NT * i < WP && e < E) wrg[i] = *reinterpret_cast<const u32x4_t*>(wr + (size_t)e * d + k1 + c);
            }
        }
        // The wave's chain count (uniform) picks an unrolled chunk.
        static_for<CPL>([&](auto IC) {
            constexpr int n = decltype(IC)::value + 1;
            if (nmax == n) chunk(std::integral_constant<int, n>{}, buf);
        });
        if (ch + 1 < nch) {
            stash(buf ^ 1);
#pragma unroll
            for (int i = 0; i < XQ; ++i) xr[i] = xn[i];
        }
        __syncthreads();
        buf ^= 1;
    }

    // Selection (the ring is free after the last barrier).
    chain_select<TPB, LPT, CPL>(lds, tl, g, t, T, nc, K, on, ec, acc, bc, bias != nullptr, topk_idx, topk_gate);
}

// Exact logits for small batches, where streaming every expert's weights
// through LDS per block of tokens costs more than the candidates need: one
// 64-lane wave per TPB = 64 / LPT tokens, one candidate chain per lane (LPT =
// the candidate slots). The block's x rows are staged in LDS widened to fp32;
// each lane reads its candidate's router-weight row, widened to fp32 by the
// norm kernel (wr32), straight from global memory in groups of 32 columns,
// two groups ahead of the multiply-adds. A multiply-add then costs one FMA
// plus a quarter of an LDS and of a global read, against three VALU
// operations with bf16 operands (both widenings); at a few waves per CU the
// kernel is bound by each wave's issue and latency, not by bandwidth. The
// chain is the same fused multiply-add sequence over i = 0..d-1, from +0, on
// the same (exactly widened) values as in k_router_chain.
//
// Blocks from chain_blocks on route the tokens of the overflow queue instead
// (exact_list_run), so that no separate launch is needed; the chain blocks
// skip queued tokens and write nothing for them. Dynamic LDS: max(TPB d fp32,
// the selection's arrays). d is a multiple of 64.
template <int LPT>
__global__ __launch_bounds__(kWave) void k_router_chain_direct(const bf16_t* __restrict__ x,
                                                             const float* __restrict__ wr32,
                                                             const bf16_t* __restrict__ wr,
                                                             const float* __restrict__ bias,
                                                             const uint16_t* __restrict__ cand,
                                                             const int32_t* __restrict__ ncand, int T, int d, int E,
                                                             int K, int32_t* __restrict__ topk_idx,
                                                             float* __restrict__ topk_gate, int chain_blocks,
                                                             const int32_t* __restrict__ ovf_count,
                                                             const int32_t* __restrict__ ovf_list) {
    if ((int)blockIdx.x >= chain_blocks) {
        exact_list_run(x, wr, bias, d, E, K, ovf_count, ovf_list, topk_idx, topk_gate,
                       (int)blockIdx.x - chain_blocks, (int)gridDim.x - chain_blocks);
        return;
    }
    constexpr int TPB = kWave / LPT;
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_dyn[];
    const int tid = threadIdx.x;
    const int g = tid % LPT;
    const int tl = tid / LPT;
    const int t = blockIdx.x * TPB + tl;
    int nc = t < T ? ncand[t] : 0;
    nc = nc < 0 ? 0 : nc;  // queued tokens are routed by the queue blocks
    const bool on[1] = {g < nc};
    const int ec[1] = {on[0] ? (int)cand[(size_t)t * LPT + g] : 0};
    const float bc[1] = {(bias && on[0]) ? bias[ec[0]] : 0.0f};

    // x rows of the block's tokens, widened to fp32 (tokens past T copy row
    // T - 1; their chains are off).
    float* xs = reinterpret_cast<float*>(lds_dyn);
    // Four 16-byte pieces per lane and round, all loaded before the writes.
    const bf16_t* xt = x + (size_t)(t < T ? t : T - 1) * d;
    for (int i0 = g * 8; i0 < d; i0 += 4 * LPT * 8) {
        u32x4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i0 + u * LPT * 8 < d) v[u] = *reinterpret_cast<const u32x4_t*>(xt + i0 + u * LPT * 8);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * LPT * 8;
            if (i < d) {
                *reinterpret_cast<float4*>(xs + tl * d + i) =
                    make_float4(__uint_as_float(v[u].x << 16), __uint_as_float(v[u].x & 0xffff0000u),
                                __uint_as_float(v[u].y << 16), __uint_as_float(v[u].y & 0xffff0000u));
                *reinterpret_cast<float4*>(xs + tl * d + i + 4) =
                    make_float4(__uint_as_float(v[u].z << 16), __uint_as_float(v[u].z & 0xffff0000u),
                                __uint_as_float(v[u].w << 16), __uint_as_float(v[u].w & 0xffff0000u));
            }
        }
    }
    __syncthreads();

    float acc[1] = {0.0f};
    if (__ballot(on[0]) != 0) {
        const float* we = wr32 + (size_t)ec[0] * d;
        const float* xr = xs + tl * d;
        const int ng = d / 32;  // even, >= 2
        // Ring of RB groups of 32 columns of weights in registers, RB - 1
        // groups ahead of the multiply-adds, and the x values of the next
        // group read from LDS while the current group's multiply-adds run: at
        // a wave or two per SIMD nothing else hides either latency.
        constexpr int RB = 4;
        float4 w[RB][8], xv[2][8];
        auto load = [&](int b, int grp) {
#pragma unroll
            for (int u = 0; u < 8; ++u) w[b][u] = *reinterpret_cast<const float4*>(we + grp * 32 + 4 * u);
        };
        auto read_x = [&](int b, int grp) {
#pragma unroll
            for (int u = 0; u < 8; ++u) xv[b][u] = *reinterpret_cast<const float4*>(xr + grp * 32 + 4 * u);
        };
        float a = 0.0f;
#pragma unroll
        for (int b = 0; b < RB - 1; ++b)
            if (b < ng) load(b, b);
        read_x(0, 0);
        for (int n = 0; n < ng; n += RB) {
            static_for<RB>([&](auto BC) {
                constexpr int b = decltype(BC)::value;
                if (n + b < ng) {
                    if (n + b + RB - 1 < ng) load((b + RB - 1) % RB, n + b + RB - 1);
                    if (n + b + 1 < ng) read_x((b + 1) & 1, n + b + 1);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        a = fmaf(xv[b & 1][u].x, w[b][u].x, a);
                        a = fmaf(xv[b & 1][u].y, w[b][u].y, a);
                        a = fmaf(xv[b & 1][u].z, w[b][u].z, a);
                        a = fmaf(xv[b & 1][u].w, w[b][u].w, a);
                    }
                }
            });
        }
        acc[0] = a;
    }
    __syncthreads();  // the selection reuses the x rows' LDS
    chain_select<TPB, LPT, 1>(lds_dyn, tl, g, t, T, nc, K, on, ec, acc, bc, bias != nullptr, topk_idx, topk_gate);
}

}  // namespace

namespace {

template <typename TIn>
hipError_t launch_logits(const moe_desc_t& d, const void* x, const void* w_router, float* logits, int ld,
                         hipStream_t s) {
    auto go = [&](auto kern, int tr, int er) -> hipError_t {
        const long long total = ((long long)d.T + tr - 1) / tr * ((d.E + er - 1) / er);
        hipLaunchKernelGGL(kern, dim3((unsigned)((total + kNumXcd - 1) / kNumXcd * kNumXcd)), dim3(256), 0, s,
                           static_cast<const TIn*>(x), static_cast<const TIn*>(w_router), logits, d.T, d.d, d.E, ld);
        return hipGetLastError();
    };
    // 32 x 32 wave tiles read a quarter of the LDS bytes and permute half as
    // much per multiply-add, but a chain step takes 32 cycles instead of 8 to
    // 12 and there are a quarter of the waves: they pay once the 16 x 16 tiles
    // give each SIMD three or more waves (T E / 1024; 459k: 18.5 us against
    // 24.6, 918k: 36 against 33, 1.05M: 29 against 27, 16.8M: 566 against 452).
    const int64_t work = (int64_t)d.T * ((d.E + 31) / 32 * 32);
    if (work < 800000) {
        // Two slabs of 256-byte row pieces, or four of 128 bytes (d an odd
        // multiple of 64 in bf16).
        if ((size_t)d.d * sizeof(TIn) % 256 == 0) return go(k_router_logits<TIn, 16, 2, 2, 8, 2>, 32, 32);
        return go(k_router_logits<TIn, 16, 2, 2, 4, 4>, 32, 32);
    }
    if (d.E <= 32) return go(k_router_logits<TIn, 32, 4, 1, 4, 2>, 128, 32);
    return go(k_router_logits<TIn, 32, 2, 2, 4, 2>, 64, 64);
}

}  // namespace

hipError_t launch_router_exact(const moe_desc_t& d, const void* x, const void* w_router, const float* bias,
                               float* logits, int ld, int32_t* topk_idx, float* topk_gate, hipStream_t s) {
    const hipError_t e = d.dtype == MOE_BF16 ? launch_logits<bf16_t>(d, x, w_router, logits, ld, s)
                                             : launch_logits<float>(d, x, w_router, logits, ld, s);
    if (e != hipSuccess) return e;
    if (d.E > 256) {
        hipLaunchKernelGGL(k_topk, dim3((d.T + 3) / 4), dim3(256), 0, s, logits, ld, bias, d.T, d.E, d.K, topk_idx,
                           topk_gate);
        return hipGetLastError();
    }
    auto go = [&](auto kern) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3((d.T + 15) / 16), dim3(256), 0, s, logits, ld, bias, d.T, d.E, d.K, topk_idx,
                           topk_gate);
        return hipGetLastError();
    };
    if (d.E <= 64) return go(k_topk16<4>);
    if (d.E <= 128) return go(k_topk16<8>);
    return go(k_topk16<16>);
}

}  // namespace moe

namespace moe {

int router_cand_slots(int K) { return K <= 8 ? 16 : 32; }

float router_fast_bound_constant(int d) {
    const double u = 1.0 / 16777216.0;
    const double gamma = d * u / (1.0 - d * u);
    return (float)((gamma + 4.0 * d * u) * 1.01);
}

bool router_small_batch(const moe_desc_t& d) { return d.T < 256 * 64; }

// Every logit by the matrix-core chain, or only the candidates of a bf16
// pre-pass? The chain costs 2 T E d flop at 100 to 115 TFLOP/s; the pre-pass
// runs at the bf16 rate and its repair costs about eight chains per token plus
// three more launches. Measured (us, exact against repair): E = 64 wins at every
// T (768 wide: 13 / 17 at 5 tokens, 42 / 59 at 32768, 73 / 89 at 65536); with
// 64 < E <= 256 up to the large-batch chain kernel (E = 128, d = 1024: 52 / 138
// at 16383 tokens, but 68 / 68 at 18432 and 163 / 113 at 65536; E = 256, d =
// 1536: 125 / 187 at 16383, 151 / 116 at 18432); else only where the interval
// test fails. Its width grows with d |x| |w|: past some d most experts become
// candidates and most tokens go through the overflow queue, which costs up to
// 130 times the chain. Where that begins depends on the data, which is not known
// here; the lines are those of normal weights of deviation 0.02 and unit x. Large
// batches, E = 256: 384 / 261 at d = 2112 and 40000 tokens, 2560 0.77, 2688 1.0,
// 3072 582 / 1526; E = 512: 860 / 558 at 2112, 2432 0.97 to 1.18, 2688 2.3; E =
// 1024: 1656 / 1261 at 2112, 2240 1.2. Small ones (more than 256 experts): 2000
// tokens, E = 1024, d = 2112 118 / 424 (K = 4: 102 / 64), 300 tokens, E = 300, d =
// 4096 49 / 638; E = 300, d = 1024, 1025 tokens 34 / 31. Smaller weights would
// carry the repair further (deviation 0.002, 40000 tokens, d = 3072, E = 256 548 /
// 370, E = 1024 2311 / 1069): the bounded cost is preferred.
bool router_exact(const moe_desc_t& d) {
    if (d.dtype != MOE_BF16 || (d.flags & MOE_FLAG_EXACT_ROUTER) || d.E <= 64) return true;
    if (router_small_batch(d)) return d.E <= 256 || d.d > 2048;
    return d.d > (d.E <= 256 ? 2624 : (d.E <= 512 ? 2368 : 2176));
}

hipError_t launch_router_fast_finish(const moe_desc_t& d, const float* s_fast, int ld, int nsplit, const void* x,
                                     const float* xnorm2, const void* w_router, const float* bias, float* wnorm,
                                     float* wr32, uint16_t* cand, int32_t* ncand, int32_t* ovf_count, int32_t* ovf_list,
                                     int32_t* topk_idx, float* topk_gate, hipStream_t s) {
    const bf16_t* xb = static_cast<const bf16_t*>(x);
    const bf16_t* wb = static_cast<const bf16_t*>(w_router);
    // The candidate kernels add at most 8 parts, those of up to 256 experts none.
    if (nsplit < 1 || nsplit > 8 || (d.E <= 256 && nsplit > 1)) return hipErrorInvalidValue;
    const bool small = router_small_batch(d);
    // Weight-row norms (the token norms are formed in the candidate kernel);
    // for small batches also the fp32 copy of the weights the chains read.
    hipLaunchKernelGGL(k_row_norms, dim3((d.E + 3) / 4), dim3(256), 0, s, wb, d.E, wnorm, d.d, ovf_count,
                       small ? wr32 : nullptr);
    const size_t sstride = (size_t)d.T * ld;
    const float cst = router_fast_bound_constant(d.d);
    const int ns = router_cand_slots(d.K);
    // Candidates: 16 lanes per token, or 64 for more than 256 experts; there
    // blocks of one wave for small batches, so that every CU gets work (with
    // fewer experts only large batches come here, with unsplit logits).
    auto cands = [&](auto kern, int lpa, int threads) {
        const int tpb = threads / lpa;
        hipLaunchKernelGGL(kern, dim3((d.T + tpb - 1) / tpb), dim3(threads), 0, s, s_fast, xb, xnorm2, d.d, wnorm, bias,
                           d.T, d.E, ld, d.K, cst, cand, ncand, ovf_count, ovf_list, nsplit, sstride);
    };
    // E / LPA experts per lane (8 or 16), so that every lane of a token holds
    // experts and L is taken over all of them.
    auto wide = [&](auto split, auto whole) { nsplit > 1 ? cands(split, 64, kWave) : cands(whole, 64, small ? kWave : 256); };
    if (d.E <= 128) ns == 16 ? cands(k_router_cand<16, 8, 16, false>, 16, 256) : cands(k_router_cand<16, 8, 32, false>, 16, 256);
    else if (d.E <= 256) ns == 16 ? cands(k_router_cand<16, 16, 16, false>, 16, 256) : cands(k_router_cand<16, 16, 32, false>, 16, 256);
    else if (d.E <= 512) ns == 16 ? wide(k_router_cand<64, 8, 16, true>, k_router_cand<64, 8, 16, false>)
                                  : wide(k_router_cand<64, 8, 32, true>, k_router_cand<64, 8, 32, false>);
    else ns == 16 ? wide(k_router_cand<64, 16, 16, true>, k_router_cand<64, 16, 16, false>)
                  : wide(k_router_cand<64, 16, 32, true>, k_router_cand<64, 16, 32, false>);
    // Exact chains: 256 (or 128) tokens per block of 1024 threads while that
    // still gives a block per CU, then 64 tokens per block, then (small
    // batches) one wave per 4 (or 2) tokens reading weights directly.
#define MOE_CHAIN(TPBv, LPTv, CPLv, EMv, DCv)                                                               \
    hipLaunchKernelGGL((k_router_chain<TPBv, LPTv, CPLv, EMv, DCv>), dim3((d.T + TPBv - 1) / TPBv + 64),     \
                       dim3(TPBv * LPTv), 0, s, xb, wb, bias, cand, ncand, d.T, d.d, d.E, d.K, topk_idx, topk_gate, \
                       (d.T + TPBv - 1) / TPBv, ovf_count, ovf_list)
#define MOE_CHAIN_E(TPBv, LPTv, CPLv, DCv)                                                                     \
    do {                                                                                                    \
        if (d.E <= 256) MOE_CHAIN(TPBv, LPTv, CPLv, 256, DCv);                                         \
        else MOE_CHAIN(TPBv, LPTv, CPLv, 1024, 16);                                                         \
    } while (0)
    const int big_tpb = ns == 16 ? 256 : 128;
    if (d.T >= 256 * big_tpb) {
        if (ns == 16) MOE_CHAIN_E(256, 4, 4, 64); else MOE_CHAIN_E(128, 8, 4, 64);
    } else if (d.T >= 256 * 64) {
        if (ns == 16) MOE_CHAIN_E(64, 4, 4, 64); else MOE_CHAIN_E(64, 8, 4, 64);
    } else {
        // One wave per 64 / ns tokens, fp32 weights straight from global
        // memory; 64 more one-wave blocks route the overflow queue.
        const int tpb = kWave / ns;
        const size_t sel = (size_t)tpb * (ns * 12 + kMaxK * 8);
        const size_t xs = (size_t)tpb * d.d * 4;
        const size_t shm = xs > sel ? xs : sel;
        const int chain_blocks = (d.T + tpb - 1) / tpb;
        const dim3 grid(chain_blocks + 64);
        auto launch = [&](auto kern) -> hipError_t {
            hipLaunchKernelGGL(kern, grid, dim3(kWave), shm, s, xb, wr32, wb, bias, cand, ncand, d.T, d.d, d.E, d.K,
                               topk_idx, topk_gate, chain_blocks, ovf_count, ovf_list);
            return hipGetLastError();
        };
        return ns == 16 ? launch(k_router_chain_direct<16>) : launch(k_router_chain_direct<32>);
    }
#undef MOE_CHAIN_E
#undef MOE_CHAIN
    return hipGetLastError();
}

}  // namespace moe
