// Grouped expert GEMMs (paper App. "MoE Kernel", Algorithm 1 Phases 2-3,
// with fc1 -> GELU -> fc2 experts; Sec. 3.3 "Optimized Kernel": all experts
// in one launch, activation fused into the GEMM epilogue).
//
// One launch covers every expert: a device-side tile list (TileDesc, built
// from the expert offsets) gives each M-tile's expert and rows, so the host
// never learns the per-expert loads. The grid is an upper bound; tiles past
// the device-side count exit at once.
//
// Block-to-tile order is XCD aware: MI355X dispatches consecutive workgroups
// round-robin over its 8 XCDs, each with its own L2, so workgroup b is mapped
// to logical tile (b % 8) * ceil(total / 8) + b / 8. Each XCD then walks a
// contiguous run of tiles, and the N-tiles of one M-tile (which share the
// gathered A rows) and the M-tiles of one expert (which share its weights)
// meet in the same L2.
//
// bf16: v_mfma_f32_32x32x16_bf16 with fp32 accumulators. Both operands are
// K-contiguous (token rows and nn.Linear weight rows; the backward's dA and dx
// contract along the weight rows and read their fragments with the transposing
// LDS reads, as wgrad.hip does) and stream global -> LDS
// in 64-wide K slabs through rings of a few slabs (buffer_load ... lds), with
// 16-byte chunks XOR-swizzled by row so that the rows a fragment read touches
// spread over the LDS banks. The kernels:
//   k_gemm_bf16  tiled, one tile per workgroup (256-, 128- or 64-row tiles, 64- to
//                256-column tiles); every epilogue, including the backward's
//   k_gemm_sp    256 x 256 tiles, four waves of 128 x 128, copies paced by
//                hand against the MFMAs (used where K is one slab)
//   k_gemm_pp    the persistent form of k_gemm_sp: one workgroup per CU walks
//                its tiles with the slab pipeline running across them; the
//                large-batch forward and backward products
//   k_gemm_f32   fp32 layers (v_mfma_f32_32x32x2_f32)
// Epilogues (EPI_*): GELU or SwiGLU to bf16 (first layer), scatter to slot
// order (second layer), fp32 store, the gate-weighted combine, and the
// backward's recompute (with fp32 pre-activations), dA through GELU' or
// SwiGLU' and fp32 slot gradients.
#include "gemm_device.h"
#include "moe_internal.h"

#include <math.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

namespace moe {
// Workgroups of a persistent kernel: per_cu per CU (a multiple of the XCD
// count), fewer when the grid-sizing bound on the tiles is smaller.
int persistent_grid(long long tile_bound, int per_cu) {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < kNumXcd)
            n = 256;
        cus[dev] = n / kNumXcd * kNumXcd;
    }
    const long long bound = (tile_bound + kNumXcd - 1) / kNumXcd * kNumXcd;
    const long long most = (long long)per_cu * cus[dev];
    return (int)(bound < most ? bound : most);
}

namespace {

__device__ __forceinline__ float gelu_erf(float v) {
    return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
}

struct TileCoord {
    int e, row0, rows, n0;
    bool valid;
};

// Logical tile of workgroup `b`: XCD-aware order, N-tiles of one M-tile adjacent.
// GROUPED: M-tiles come from the device-side tile table; otherwise one dense
// group of a.dense_rows rows.
template <bool GROUPED>
__device__ __forceinline__ TileCoord locate_tile(const GemmArgs& a, int bm, int bn) {
    TileCoord tc;
    tc.valid = false;
    const int n_n = a.N / bn;
    const int total_m = GROUPED ? *a.n_tiles : (a.dense_rows + bm - 1) / bm;
    const int total = total_m * n_n;
    const int per = (total + kNumXcd - 1) / kNumXcd;
    const int b = blockIdx.x;
    const int j = b / kNumXcd;
    if (j >= per) return tc;
    const int lid = (b % kNumXcd) * per + j;
    if (lid >= total) return tc;
    const int mt = lid / n_n;
    tc.n0 = (lid - mt * n_n) * bn;
    if (GROUPED) {
        const TileDesc t = a.tiles[mt];
        tc.e = t.e;
        tc.row0 = t.row0;
        tc.rows = t.rows;
    } else {
        tc.e = 0;
        tc.row0 = mt * bm;
        tc.rows = min(bm, a.dense_rows - tc.row0);
    }
    tc.valid = true;
    return tc;
}

// Gradients of SiLU(g) * u from the gradient da of the product: (dg, du) =
// (da u SiLU'(g), da SiLU(g)), SiLU'(g) = s (1 + g (1 - s)), s = Sigmoid(g).
__device__ __forceinline__ void swiglu_grad(float g, float u, float da, float& dg, float& du) {
    const float sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.44269504f));
    dg = da * u * (sg * fmaf(g, 1.0f - sg, 1.0f));
    du = da * (g * sg);
}

// SwiGLU activation of one column: SiLU(gate) * up, or 0 past the valid width.
__device__ __forceinline__ float swiglu_col(float g, float u, bool valid) {
    return valid ? silu_as(g) * u : 0.0f;
}

// Weight rows a tile may read: the group's rows (B rows past b_rows, when
// set, read as zeros through the buffer-resource bound).
__device__ __forceinline__ int weight_rows(const GemmArgs& a) { return a.b_rows > 0 ? a.b_rows : a.N; }

// Epilogues of a first expert layer: their token rows are gathered from x.
__host__ __device__ constexpr bool fc1_epi(int epi) {
    return epi == EPI_GELU_STORE || epi == EPI_SWIGLU_STORE || epi == EPI_SWIGLU_BWD;
}

// Backward products whose weights the bf16 kernels read as they lie in
// memory, the contraction along their rows.
__host__ __device__ constexpr bool kmajor_epi(int epi) {
    return epi == EPI_DGELU || epi == EPI_DSWIGLU || epi == EPI_SCATTER_SLOT_F32;
}

// Derivative of gelu_sig, so that the backward differentiates the function
// the forward evaluated: with sg = Sigmoid(s), e = exp(-s), 1 - sg = e sg and
// d/dx [x sg] = sg (1 + x e sg s'(x)), s'(x) = a0 + 3 a1 x^2 + 5 a2 x^4 (past
// the clamp e sg is below 1e-11 and the term vanishes). Its largest absolute
// difference from Phi(x) + x phi(x) is 1.1e-4.
__device__ __forceinline__ float gelu_sig_grad(float x) {
    const float xc = __builtin_amdgcn_fmed3f(x, -8.0f, 8.0f);
    const float x2 = xc * xc;
    const float e = __builtin_amdgcn_exp2f(xc * fmaf(fmaf(kGeluB2, x2, kGeluB1), x2, kGeluB0));
    const float sg = __builtin_amdgcn_rcpf(1.0f + e);
    const float ds = fmaf(fmaf(5.0f * kGeluA2, x2, 3.0f * kGeluA1), x2, kGeluA0);
    return sg * fmaf(x * e * sg, ds, 1.0f);
}

// bf16 grouped / dense GEMM, C[m, n] = sum_k X[m, k] W[n, k], fp32 accumulation.
//
// Tiles of BM token rows x BN output columns; WAVES_M x WAVES_N waves, each
// owning a (BM / WAVES_M) x (BN / WAVES_N) sub-tile of 32x32 MFMA blocks.
// The weight fragment is the MFMA's first operand and the token fragment the
// second, so each lane's accumulators hold ONE token row and, per block,
// four runs of four consecutive output columns: the epilogue writes 8- or
// 16-byte row-contiguous pieces with one row address per lane.
//
// K slabs of BK (32 or 64) stream global -> LDS through a ring of STAGES
// buffers with buffer_load ... lds (the K offset is a scalar, so issuing a
// copy costs no vector instructions), STAGES - 1 slabs ahead of the MFMAs. A
// wave fills whole 1 KB pieces: lane l of piece q lands in slot q*64 + l =
// (row, physical chunk) and loads logical chunk physical ^ swizzle(row); the
// swizzle puts the 16 rows read together by a quarter-wave of a fragment read
// on 16 distinct 16-byte bank groups of the 64-bank LDS. Fragments for the
// next 16-wide K step are read while the MFMAs of the current one run.
template <int BM, int BN, int WAVES_M, int WAVES_N, int BK, int STAGES, int EPI, bool GROUPED, int WPE>
__global__ __launch_bounds__(WAVES_M* WAVES_N* kWave) __attribute__((amdgpu_waves_per_eu(WPE, 8)))
void k_gemm_bf16(const GemmArgs a) {
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int NT = NW * kWave;
    constexpr int CPR = BK / 8;  // 16-byte chunks per LDS row
    constexpr int ROWB = BK * 2;
    constexpr int KS = BK / 16;  // MFMA K steps per slab
    constexpr int WTM = BM / WAVES_M;
    constexpr int WTN = BN / WAVES_N;
    constexpr int FM = WTM / 32;
    constexpr int FN = WTN / 32;
    static_assert(FM >= 1 && FN >= 1, "wave tile must hold at least one 32x32 block");
    constexpr int A_PIECES = BM * CPR / kWave;
    constexpr int B_PIECES = BN * CPR / kWave;
    static_assert(A_PIECES % NW == 0 && B_PIECES % NW == 0, "pieces must split evenly over waves");
    constexpr int AP = A_PIECES / NW;
    constexpr int BP = B_PIECES / NW;
    constexpr int STAGE = (BM + BN) * ROWB;
    static_assert(CPR == 4 || CPR == 8, "BK must be 32 or 64");
    static_assert(STAGES >= 2 && STAGES <= 5, "2 to 5 stages");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES * STAGE];
    __shared__ int32_t srow[BM];
    // A rows gathered through the row map (first layers, the backward's dA).
    constexpr bool A_GATHER = fc1_epi(EPI) || EPI == EPI_GELU_BWD || EPI == EPI_DGELU || EPI == EPI_DSWIGLU;
    // Output rows scattered to slot order (second layer, the backward's dx).
    constexpr bool O_SCATTER = EPI == EPI_SCATTER_SLOT || EPI == EPI_SCATTER_SLOT_F32;
    const TileCoord tc = locate_tile<GROUPED>(a, BM, BN);
    if (!tc.valid) return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // Row ids: gathered operand rows, or output slots.
    for (int r = tid; r < BM; r += NT) {
        const int rr = r < tc.rows ? r : tc.rows - 1;  // pad rows repeat the last valid row
        const int p = tc.row0 + rr;
        int v = p;
        if (A_GATHER && a.row_mode == ROWS_GATHER_TOKENS) v = a.row_map[p] / a.route_k;
        if (A_GATHER && a.row_mode == ROWS_GATHER_SLOTS) v = a.row_map[p];
        if (O_SCATTER) v = a.row_map[p];
        srow[r] = v;
    }
    __syncthreads();

    constexpr bool SWIGLU = EPI == EPI_SWIGLU_STORE || EPI == EPI_SWIGLU_BWD;
    constexpr bool DSW = EPI == EPI_DSWIGLU;  // two bf16 outputs per element (dG, dU)
    constexpr int HW = WTN / 2;  // SwiGLU: activation columns per wave
    static_assert(!SWIGLU || FN % 2 == 0, "SwiGLU waves hold gate and up blocks in pairs");
    const int Kd = a.Kdim;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.A, a.a_bytes);
    // K-major weights ([Kdim][N]): a slab is 64 rows of WROWB bytes, whose chunks
    // are swizzled so that a transposing read's 4 rows x 32 columns per half wave
    // (16 chunks) fall in distinct banks.
    constexpr bool KM = kmajor_epi(EPI);
    constexpr int WROWB = BN * 2, WCPR = BN / 8;
    static_assert(!KM || (BK == 64 && (BN == 64 || BN == 128)), "K-major weight slabs are 64 rows of 64 or 128 columns");
    auto wswz = [](int r) { return BN == 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; };
    const uint32_t krow = (uint32_t)a.N * 2;
    // SwiGLU: the group's 2 act_n weight rows; reads past them return zeros.
    const __amdgpu_buffer_rsrc_t wres =
        KM ? make_rsrc(static_cast<const bf16_t*>(a.B) + (size_t)tc.e * a.b_group_stride + tc.n0,
                       (uint32_t)a.b_group_stride * 2u - (uint32_t)tc.n0 * 2u)
           : make_rsrc(static_cast<const bf16_t*>(a.B) + (size_t)tc.e * a.b_group_stride,
                       (uint32_t)(SWIGLU ? 2 * a.act_n : weight_rows(a)) * Kd * 2);

    constexpr int SWZ_SHIFT = CPR == 8 ? 1 : 2;
    constexpr int SWZ_MASK = CPR - 1;
    const uint32_t rstride = (uint32_t)(Kd * 2);

    uint32_t xv[AP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int sl = (wave + NW * i) * kWave + lane;
        const int r = sl / CPR, pch = sl % CPR;
        const int c = pch ^ ((r >> SWZ_SHIFT) & SWZ_MASK);
        int xrow;
        if (A_GATHER) xrow = srow[r];
        else xrow = tc.row0 + (r < tc.rows ? r : tc.rows - 1);
        xv[i] = (uint32_t)xrow * rstride + c * 16;
    }
    uint32_t wv[BP];
#pragma unroll
    for (int i = 0; i < BP; ++i) {
        const int sl = (wave + NW * i) * kWave + lane;
        const int r = sl / CPR, pch = sl % CPR;
        const int c = pch ^ ((r >> SWZ_SHIFT) & SWZ_MASK);
        // SwiGLU: tile column r is wave block r / WTN; its first HW columns
        // are the gate rows and the last HW the up rows of the same HW
        // activation columns. Gate rows past act_n read (finite) up rows,
        // whose activations the epilogue zeroes.
        int wrow = tc.n0 + r;
        if (SWIGLU) {
            const int w = r % WTN;
            wrow = tc.n0 / 2 + (r / WTN) * HW + w % HW + (w >= HW ? a.act_n : 0);
        }
        wv[i] = (uint32_t)wrow * rstride + c * 16;
        if (KM) wv[i] = (uint32_t)(sl / WCPR) * krow + (uint32_t)((sl % WCPR) ^ wswz(sl / WCPR)) * 16u;
    }

    f32x16_t acc[FN][FM];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    // Per-lane fragment offsets: row fr of a 32-row block, chunk (ks*2 + fk)
    // swizzled; the swizzle depends only on fr because blocks start at
    // multiples of 32 rows.
    const int fr = lane & 31;
    const int fk = lane >> 5;
    const int lane_sw = (fr >> SWZ_SHIFT) & SWZ_MASK;
    uint32_t xoff[KS], woff[KS], wkoff[FN];
    const uint32_t base = lds_address(smem);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint32_t k = fr * ROWB + (((ks * 2 + fk) ^ lane_sw) << 4);
        xoff[ks] = base + (wm * WTM) * ROWB + k;
        woff[ks] = base + BM * ROWB + (wn * WTN) * ROWB + k;
    }
    const int r4 = (lane & 15) >> 2;
#pragma unroll
    for (int j = 0; j < FN; ++j) {  // K-major weights: by 32-column block
        const int c = wn * (WTN / 8) + j * 4 + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
        wkoff[j] = base + BM * ROWB + (uint32_t)(fk * 8 + r4) * WROWB + (uint32_t)(c ^ wswz(r4)) * 16u + (lane & 1) * 8u;
    }
    // K range: the whole row, or (split K, dense fp32 output) part blockIdx.y of
    // gridDim.y equal parts.
    int nk = Kd / BK;
    uint32_t kbase = 0;
    if constexpr (!GROUPED && EPI == EPI_STORE_F32) {
        nk /= (int)gridDim.y;
        kbase = (uint32_t)blockIdx.y * (uint32_t)nk * BK * 2;
    }

    auto issue = [&](int stage, int kslab) {
        uint8_t* buf = smem + stage * STAGE;
        const uint32_t soff = kbase + (uint32_t)kslab * BK * 2;
#pragma unroll
        for (int i = 0; i < AP; ++i) copy16_to_lds(xres, xv[i], soff, buf + (wave + NW * i) * 1024);
#pragma unroll
        for (int i = 0; i < BP; ++i) {
            if constexpr (KM) {
                // Stacked weights (a.b_half > 0), as in k_gemm_pp.
                const int half = EPI == EPI_SCATTER_SLOT_F32 ? a.b_half : 0;
                const int up = half > 0 && kslab * BK >= half ? 1 : 0;
                const int kk = kslab * BK - up * half;
                uint32_t v = wv[i] + (uint32_t)(kk + (up ? a.act_n : 0)) * krow;
                if (half > 0 && ((wave + NW * i) * kWave + lane) / WCPR + kk >= a.act_n) v = kWgradNoRow;
                uint8_t* const dst = buf + BM * ROWB + (wave + NW * i) * 1024;
                if (a.b_nt) copy16_to_lds_nt(wres, v, 0, dst);
                else copy16_to_lds(wres, v, 0, dst);
                continue;
            }
            // Weights read once in this launch (a.b_nt: one M-tile per expert
            // on average) stream past the caches.
            if (a.b_nt)
                copy16_to_lds_nt(wres, wv[i], soff, buf + BM * ROWB + (wave + NW * i) * 1024);
            else
                copy16_to_lds(wres, wv[i], soff, buf + BM * ROWB + (wave + NW * i) * 1024);
        }
    };
    auto read_frags = [&](uint32_t sbase, auto KSC, bf16x8_t* xf, bf16x8_t* wf, u32x2_t (*wh)[2]) {
        constexpr int ks = decltype(KSC)::value;
        const uint32_t xa = xoff[ks] + sbase, wa = woff[ks] + sbase;
        if constexpr (FM >= 1) xf[0] = lds_read16<0 * 32 * ROWB>(xa);
        if constexpr (FM >= 2) xf[1] = lds_read16<1 * 32 * ROWB>(xa);
        if constexpr (FM >= 3) xf[2] = lds_read16<2 * 32 * ROWB>(xa);
        if constexpr (FM >= 4) xf[3] = lds_read16<3 * 32 * ROWB>(xa);
        if constexpr (KM) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                lds_read_tr8_asm<ks * 16 * WROWB>(wh[j][0], wkoff[j] + sbase);
                lds_read_tr8_asm<ks * 16 * WROWB + 4 * WROWB>(wh[j][1], wkoff[j] + sbase);
            }
            return;
        }
        if constexpr (FN >= 1) wf[0] = lds_read16<0 * 32 * ROWB>(wa);
        if constexpr (FN >= 2) wf[1] = lds_read16<1 * 32 * ROWB>(wa);
        if constexpr (FN >= 3) wf[2] = lds_read16<2 * 32 * ROWB>(wa);
        if constexpr (FN >= 4) wf[3] = lds_read16<3 * 32 * ROWB>(wa);
        static_assert(FM <= 4 && FN <= 4, "at most 4x4 blocks per wave");
    };
    auto settle = [&](bf16x8_t* xf, bf16x8_t* wf, u32x2_t (*wh)[2]) {
        wait_lgkmcnt0();
#pragma unroll
        for (int i = 0; i < FM; ++i) tie(xf[i]);
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            if constexpr (KM) {
                tie(wh[j][0]);
                tie(wh[j][1]);
                wf[j] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(wh[j][0], wh[j][1], 0, 1, 2, 3));
            } else {
                tie(wf[j]);
            }
        }
    };

#pragma unroll
    for (int sl = 0; sl < STAGES - 1; ++sl)
        if (sl < nk) issue(sl, sl);

    int cur_stage = 0;
    for (int kt = 0; kt < nk; ++kt) {
        // Slab kt must have landed; later prefetched slabs stay in flight.
        const int ahead = min(nk - 1 - kt, STAGES - 2);
        if constexpr (STAGES >= 5) { if (ahead >= 3) { wait_vmcnt<3 * (AP + BP)>(); goto waited; } }
        if constexpr (STAGES >= 4) { if (ahead >= 2) { wait_vmcnt<2 * (AP + BP)>(); goto waited; } }
        if constexpr (STAGES >= 3) { if (ahead >= 1) { wait_vmcnt<AP + BP>(); goto waited; } }
        wait_vmcnt<0>();
    waited:
        barrier_no_fence();
        if (kt + STAGES - 1 < nk) {
            int st = cur_stage + STAGES - 1;
            if (st >= STAGES) st -= STAGES;
            issue(st, kt + STAGES - 1);
        }
        const uint32_t sbase = cur_stage * STAGE;
        bf16x8_t xf[2][FM], wf[2][FN];
        u32x2_t wh[2][FN][2];  // K-major weights: the two row halves of each fragment
        read_frags(sbase, std::integral_constant<int, 0>{}, xf[0], wf[0], wh[0]);
        settle(xf[0], wf[0], wh[0]);
        static_for<KS>([&](auto KSC) {
            constexpr int ks = decltype(KSC)::value, c = ks & 1;
            if constexpr (ks + 1 < KS)
                read_frags(sbase, std::integral_constant<int, ks + 1>{}, xf[c ^ 1], wf[c ^ 1], wh[c ^ 1]);
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[c][j], xf[c][i], acc[j][i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (ks + 1 < KS) settle(xf[c ^ 1], wf[c ^ 1], wh[c ^ 1]);
        });
        if (++cur_stage == STAGES) cur_stage = 0;
    }

    // Epilogue, one 32-row block of the wave tile at a time. Block (j, i):
    // this lane's token row is i*32 + (lane & 31); accumulator 4g + q is column
    // j*32 + 8g + 4*(lane >> 5) + q. The block is activated / converted and
    // written to the wave's own LDS area row by row (rows padded by 16 bytes
    // so the 32 rows of one write spread over the banks), then read back as
    // 16-byte row pieces so that consecutive lanes store whole 128-byte lines.
    // The fused combine (dense, K <= 8) stages the shared expert's fp32 output.
    constexpr bool COMB = EPI == EPI_COMBINE;
    static_assert(!(COMB && GROUPED), "the fused combine is a dense (shared expert) epilogue");
    constexpr bool OUT_F32 = EPI == EPI_STORE_F32 || EPI == EPI_SCATTER_SLOT_F32 || COMB;
    constexpr int OES = OUT_F32 ? 4 : 2;           // staged element size
    constexpr int SEG = (SWIGLU ? HW : WTN) * OES * (DSW ? 2 : 1);  // bytes of one wave-tile row
    constexpr int RSTR = SEG + 16;                 // padded LDS row stride
    constexpr int CPRO = SEG / 16;                 // 16-byte pieces per row
    constexpr int PIECES = 32 * CPRO / kWave;      // pieces per lane per block
    static_assert(NW * 32 * RSTR <= STAGES * STAGE, "epilogue staging must fit in the stage buffers");
    static_assert((32 * CPRO) % kWave == 0, "row pieces must split evenly over the wave");
    __syncthreads();  // every wave is done with the stage buffers
    uint8_t* stg = smem + wave * 32 * RSTR;
    // First output column of this wave's rows (SwiGLU: activation column,
    // rows act_ld apart).
    const int ocol0 = SWIGLU ? tc.n0 / 2 + wn * HW : tc.n0 + wn * WTN;
    const size_t ostride = SWIGLU ? (size_t)a.act_ld : (DSW ? 2 * (size_t)a.act_ld : (size_t)a.N);
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        if constexpr (DSW) {
            // dG in the first half of the staging row, dU in the second.
            const int r = wm * WTM + i * 32 + fr;
            const float* grow = static_cast<const float*>(a.aux) +
                                (size_t)(tc.row0 + (r < tc.rows ? r : tc.rows - 1)) * 2 * a.act_ld + ocol0;
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = j * 32 + 8 * g + 4 * fk;
                    const float4 gv = *reinterpret_cast<const float4*>(grow + c);
                    const float4 uv = *reinterpret_cast<const float4*>(grow + a.act_ld + c);
                    const float gg[4] = {gv.x, gv.y, gv.z, gv.w}, uu[4] = {uv.x, uv.y, uv.z, uv.w};
                    float dg[4], du[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        swiglu_grad(gg[q], uu[q], acc[j][i][4 * g + q], dg[q], du[q]);
                        if (ocol0 + c + q >= a.act_n) dg[q] = du[q] = 0.0f;
                    }
                    *reinterpret_cast<uint2*>(stg + fr * RSTR + c * 2) = pack4_bf16(dg[0], dg[1], dg[2], dg[3]);
                    *reinterpret_cast<uint2*>(stg + fr * RSTR + (WTN + c) * 2) =
                        pack4_bf16(du[0], du[1], du[2], du[3]);
                }
        } else if constexpr (SWIGLU) {
#pragma unroll
            for (int j = 0; j < FN / 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = j * 32 + 8 * g + 4 * fk;
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[q] = swiglu_col(acc[j][i][4 * g + q], acc[j + FN / 2][i][4 * g + q],
                                          ocol0 + c + q < a.act_n);
                    *reinterpret_cast<uint2*>(stg + fr * RSTR + c * 2) = pack4_bf16(v[0], v[1], v[2], v[3]);
                }
        } else {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v0 = acc[j][i][4 * g + 0], v1 = acc[j][i][4 * g + 1];
                    float v2 = acc[j][i][4 * g + 2], v3 = acc[j][i][4 * g + 3];
                    uint8_t* dst = stg + fr * RSTR + (j * 32 + 8 * g + 4 * fk) * OES;
                    if (OUT_F32) {
                        *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
                    } else {
                        if (EPI == EPI_GELU_STORE || EPI == EPI_GELU_BWD) {
                            v0 = gelu_sig(v0); v1 = gelu_sig(v1); v2 = gelu_sig(v2); v3 = gelu_sig(v3);
                        }
                        if (EPI == EPI_DGELU) {  // times GELU' of the stored pre-activation
                            const int r = wm * WTM + i * 32 + fr;
                            const size_t p = (size_t)(tc.row0 + (r < tc.rows ? r : tc.rows - 1));
                            const float4 f = *reinterpret_cast<const float4*>(
                                static_cast<const float*>(a.aux) + p * a.N + ocol0 + j * 32 + 8 * g + 4 * fk);
                            v0 *= gelu_sig_grad(f.x); v1 *= gelu_sig_grad(f.y);
                            v2 *= gelu_sig_grad(f.z); v3 *= gelu_sig_grad(f.w);
                        }
                        *reinterpret_cast<uint2*>(dst) = pack4_bf16(v0, v1, v2, v3);
                    }
                }
        }
        // Each wave reads back only its own area: a wave-level sync suffices.
        wave_sync_lds();
#pragma unroll
        for (int k = 0; k < PIECES; ++k) {
            const int q = lane + kWave * k;
            const int rr = q / CPRO, pc = q % CPRO;
            const int r = wm * WTM + i * 32 + rr;
            const uint4 v = *reinterpret_cast<const uint4*>(stg + rr * RSTR + pc * 16);
            if constexpr (COMB) {
                // y for the piece's four columns, in the separate combine's
                // order: acc = 0, acc = fma(g_j, O_j, acc) for j = 0..K-1 over
                // the token's expert-output rows (slot order), then
                // fma(lambda, S, acc) and one rounding to bf16. Slots past K
                // re-read slot K - 1 and are not added.
                if (r < tc.rows) {
                    const int tok = tc.row0 + r;
                    const int col = ocol0 + pc * 4;
                    const int K = a.route_k;
                    const bf16_t* eo = static_cast<const bf16_t*>(a.eo);
                    float gj[kMaxCombineK];
                    uint2 o[kMaxCombineK];
#pragma unroll
                    for (int j = 0; j < kMaxCombineK; ++j) {
                        const int jj = j < K ? j : K - 1;
                        gj[j] = a.gate[(size_t)tok * K + jj];
                        o[j] = *reinterpret_cast<const uint2*>(eo + ((size_t)tok * K + jj) * a.N + col);
                    }
                    float c4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int j = 0; j < kMaxCombineK; ++j)
                        if (j < K) {
                            c4[0] = fmaf(gj[j], __uint_as_float(o[j].x << 16), c4[0]);
                            c4[1] = fmaf(gj[j], __uint_as_float(o[j].x & 0xffff0000u), c4[1]);
                            c4[2] = fmaf(gj[j], __uint_as_float(o[j].y << 16), c4[2]);
                            c4[3] = fmaf(gj[j], __uint_as_float(o[j].y & 0xffff0000u), c4[3]);
                        }
                    const float sv[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                                         __uint_as_float(v.w)};
                    uint32_t h[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        uint32_t u = __float_as_uint(fmaf(a.lambda, sv[q], c4[q]));
                        u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even (finite values)
                        h[q] = u >> 16;
                    }
                    *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.C) + (size_t)tok * a.N + col) =
                        make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
                }
                continue;
            }
            if (r < tc.rows && (!SWIGLU || ocol0 < a.act_ld)) {
                size_t orow = O_SCATTER ? (size_t)srow[r] : (size_t)(tc.row0 + r);
                void* obase = a.C;
                if constexpr (!GROUPED && EPI == EPI_STORE_F32)  // split K: this part's partial sums
                    obase = static_cast<float*>(a.C) + (size_t)blockIdx.y * a.dense_rows * a.N;
                size_t ocol = (size_t)ocol0;
                int pcc = pc;
                if (DSW && pc >= CPRO / 2) {  // the dU half goes act_ld columns further on
                    ocol += a.act_ld;
                    pcc -= CPRO / 2;
                }
                uint8_t* out = static_cast<uint8_t*>(obase) + (orow * ostride + ocol) * OES + pcc * 16;
                *reinterpret_cast<uint4*>(out) = v;
            }
        }
        wave_sync_lds();
    }
    if constexpr (EPI == EPI_SWIGLU_BWD) {
        // Second output: the fp32 gate and up pre-activations, G at column c and
        // U at act_ld + c of C2's rows (2 act_ld), staged as [G | U] per row.
        constexpr int SEG2 = 2 * HW * 4, RSTR2 = SEG2 + 16, CPRO2 = SEG2 / 16, PIECES2 = 32 * CPRO2 / kWave;
        static_assert(NW * 32 * RSTR2 <= STAGES * STAGE, "epilogue staging must fit in the stage buffers");
        __syncthreads();  // the wider rows overlap other waves' first-pass areas
        uint8_t* stg2 = smem + wave * 32 * RSTR2;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int j = 0; j < FN / 2; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = j * 32 + 8 * g + 4 * fk;
                    *reinterpret_cast<float4*>(stg2 + fr * RSTR2 + c * 4) =
                        make_float4(acc[j][i][4 * g + 0], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2],
                                    acc[j][i][4 * g + 3]);
                    const int ju = j + FN / 2;
                    *reinterpret_cast<float4*>(stg2 + fr * RSTR2 + (HW + c) * 4) =
                        make_float4(acc[ju][i][4 * g + 0], acc[ju][i][4 * g + 1], acc[ju][i][4 * g + 2],
                                    acc[ju][i][4 * g + 3]);
                }
            wave_sync_lds();
#pragma unroll
            for (int k = 0; k < PIECES2; ++k) {
                const int q = lane + kWave * k;
                const int rr = q / CPRO2, pc = q % CPRO2;
                const int r = wm * WTM + i * 32 + rr;
                const uint4 v = *reinterpret_cast<const uint4*>(stg2 + rr * RSTR2 + pc * 16);
                if (r < tc.rows && ocol0 < a.act_ld) {
                    const bool up = pc >= CPRO2 / 2;
                    const size_t col = (size_t)ocol0 + (up ? a.act_ld : 0);
                    uint8_t* out = static_cast<uint8_t*>(a.C2) +
                                   ((size_t)(tc.row0 + r) * 2 * a.act_ld + col) * 4 + (pc - (up ? CPRO2 / 2 : 0)) * 16;
                    *reinterpret_cast<uint4*>(out) = v;
                }
            }
            wave_sync_lds();
        }
    }
    if constexpr (EPI == EPI_GELU_BWD) {
        // Second output: the pre-activation (acc) in fp32 (rows of N), the same staging.
        constexpr int SEG2 = WTN * 4, RSTR2 = SEG2 + 16, CPRO2 = SEG2 / 16, PIECES2 = 32 * CPRO2 / kWave;
        static_assert(NW * 32 * RSTR2 <= STAGES * STAGE, "epilogue staging must fit in the stage buffers");
        __syncthreads();  // the wider rows overlap other waves' first-pass areas
        uint8_t* stg2 = smem + wave * 32 * RSTR2;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<float4*>(stg2 + fr * RSTR2 + (j * 32 + 8 * g + 4 * fk) * 4) =
                        make_float4(acc[j][i][4 * g + 0], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2],
                                    acc[j][i][4 * g + 3]);
            wave_sync_lds();
#pragma unroll
            for (int k = 0; k < PIECES2; ++k) {
                const int q = lane + kWave * k;
                const int rr = q / CPRO2, pc = q % CPRO2;
                const int r = wm * WTM + i * 32 + rr;
                const uint4 v = *reinterpret_cast<const uint4*>(stg2 + rr * RSTR2 + pc * 16);
                if (r < tc.rows) {
                    uint8_t* out = static_cast<uint8_t*>(a.C2) + ((size_t)(tc.row0 + r) * a.N + ocol0) * 4 + pc * 16;
                    *reinterpret_cast<uint4*>(out) = v;
                }
            }
            wave_sync_lds();
        }
    }
}

// bf16 grouped / dense GEMM, 256 x 256 tiles, four waves of 128 x 128 (one
// wave per SIMD, accumulators in the 256 accumulation registers), 64-wide K
// slabs (whole 128-byte row pieces per copy).
//
// A CU's global -> LDS copy path takes about as long to move a slab as the
// MFMAs take to consume it, so copies must leave at an even pace: every K
// step of 16 MFMAs carries exactly four copies (one after every fourth MFMA)
// and eight fragment reads for the next K step, in an order fixed by hand.
// The token operand has a ring of three slabs and the weight operand a ring
// of two (together the whole 160 KB of LDS), so token copies get more than a
// slab of lead and weight copies, mostly L2 hits, half a slab. One barrier per
// slab sits before its last K step: every wave has read the whole slab by
// then (its buffers can be refilled from that last step on) and has seen its
// own copies of the next slab land (its first fragments are read during that
// last step). Row ids come from the global row map, so no LDS is spent on them.
template <int EPI, bool GROUPED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_gemm_sp(const GemmArgs a) {
    constexpr int BM = 256, BN = 256, NW = 4, WT = 128, FB = WT / 32;
    constexpr int BK = 64, CPR = 8, ROWB = 128, KS = 4;
    constexpr int SLAB = BM * ROWB;           // 32 KB per operand and slab
    constexpr int AST = 3, WST = 2;           // ring depths
    constexpr int WBASE = AST * SLAB;         // weight ring after the token ring
    constexpr int AP = BM * CPR / kWave / NW;  // 8 token copy pieces per wave and slab
    constexpr int BP = BN * CPR / kWave / NW;  // 8 weight copy pieces
    static_assert(AP == 8 && BP == 8, "copy schedule is written for 8 + 8 pieces");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[AST * SLAB + WST * SLAB];

    const TileCoord tc = locate_tile<GROUPED>(a, BM, BN);
    if (!tc.valid) return;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    const int Kd = a.Kdim;
    const int nk = Kd / BK;

    auto row_id = [&](int r) {  // operand / output row id of tile row r (pad rows repeat the last)
        const int p = tc.row0 + (r < tc.rows ? r : tc.rows - 1);
        if (EPI == EPI_GELU_STORE && a.row_mode == ROWS_GATHER_TOKENS) return a.row_map[p] / a.route_k;
        if (EPI == EPI_SCATTER_SLOT) return a.row_map[p];
        return p;
    };

    const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.A, a.a_bytes);
    const __amdgpu_buffer_rsrc_t wres =
        make_rsrc(static_cast<const bf16_t*>(a.B) + (size_t)tc.e * a.b_group_stride, (uint32_t)weight_rows(a) * Kd * 2);
    const __amdgpu_buffer_rsrc_t xnull = make_rsrc(a.A, 0);
    const __amdgpu_buffer_rsrc_t wnull =
        make_rsrc(static_cast<const bf16_t*>(a.B) + (size_t)tc.e * a.b_group_stride, 0);
    uint32_t xv[AP], wv[BP];
#pragma unroll
    for (int i = 0; i < AP; ++i) {
        const int sl = (wave + NW * i) * kWave + lane;
        const int r = sl / CPR, pch = sl % CPR;
        const int c = pch ^ ((r >> 1) & 7);
        const int xrow = EPI == EPI_GELU_STORE ? row_id(r) : tc.row0 + (r < tc.rows ? r : tc.rows - 1);
        xv[i] = (uint32_t)xrow * (uint32_t)(Kd * 2) + c * 16;
    }
#pragma unroll
    for (int i = 0; i < BP; ++i) {
        const int sl = (wave + NW * i) * kWave + lane;
        const int r = sl / CPR, pch = sl % CPR;
        const int c = pch ^ ((r >> 1) & 7);
        wv[i] = (uint32_t)(tc.n0 + r) * (uint32_t)(Kd * 2) + c * 16;
    }

    f32x16_t acc[FB][FB];
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    const int fr = lane & 31;
    const int fk = lane >> 5;
    const int lane_sw = (fr >> 1) & 7;
    uint32_t xoff[KS], woff[KS];
    const uint32_t base = lds_address(smem);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint32_t k = fr * ROWB + (((ks * 2 + fk) ^ lane_sw) << 4);
        xoff[ks] = base + (wm * WT) * ROWB + k;
        woff[ks] = base + WBASE + (wn * WT) * ROWB + k;
    }

    // Slab m's copy source: real slabs through the sized resources, slabs
    // past the last through the zero-size ones at an in-range offset.
    auto slab_src = [&](int m, uint32_t& soff, __amdgpu_buffer_rsrc_t& xr, __amdgpu_buffer_rsrc_t& wr) {
        const bool real = m < nk;
        soff = (uint32_t)(real ? m : nk - 1) * BK * 2;
        xr = real ? xres : xnull;
        wr = real ? wres : wnull;
    };
    // Copy piece L (constant) of this wave: token operand (IS_A) or weights.
    auto copy_a = [&](auto LC, int stage, uint32_t soff, __amdgpu_buffer_rsrc_t xr) {
        constexpr int L = decltype(LC)::value;
        copy16_to_lds(xr, xv[L], soff, smem + stage * SLAB + (wave + NW * L) * 1024);
    };
    auto copy_w = [&](auto LC, int stage, uint32_t soff, __amdgpu_buffer_rsrc_t wr) {
        constexpr int L = decltype(LC)::value;
        copy16_to_lds(wr, wv[L], soff, smem + WBASE + stage * SLAB + (wave + NW * L) * 1024);
    };

    bf16x8_t xf[2][FB], wf[2][FB];
    auto read_frag = [&](auto NBC, auto QC, uint32_t abase, uint32_t wbase, int ks) {
        constexpr int nb = decltype(NBC)::value, q = decltype(QC)::value;
        if constexpr (q < FB) xf[nb][q] = lds_read16<q * 32 * ROWB>(xoff[ks] + abase);
        else wf[nb][q - FB] = lds_read16<(q - FB) * 32 * ROWB>(woff[ks] + wbase);
    };
    auto settle = [&](auto CBC) {
        constexpr int cb = decltype(CBC)::value;
        wait_lgkmcnt0();
#pragma unroll
        for (int i = 0; i < FB; ++i) tie(xf[cb][i]);
#pragma unroll
        for (int j = 0; j < FB; ++j) tie(wf[cb][j]);
    };
    // One K step: 16 MFMAs on buffer CB, fragment q of the next K step after
    // MFMA q (q < 8), copy number q / 4 of the step's four after MFMA q when
    // q % 4 == 1. COPY(c) issues the step's c-th copy.
    auto kstep = [&](auto CBC, uint32_t rabase, uint32_t rwbase, int rks, auto&& copy) {
        constexpr int cb = decltype(CBC)::value;
        static_for<FB * FB>([&](auto QC) {
            constexpr int q = decltype(QC)::value;
            constexpr int j = q / FB, i = q % FB;
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[cb][j], xf[cb][i], acc[j][i], 0, 0, 0);
            if constexpr (q < 2 * FB)
                read_frag(std::integral_constant<int, cb ^ 1>{}, QC, rabase, rwbase, rks);
            if constexpr (q % 4 == 1) copy(std::integral_constant<int, q / 4>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // Prologue: token slab 0, weight slab 0, token slab 1, the first half of
    // weight slab 1 (what the loop would have issued before step 0); wait for
    // slab 0 of both operands; read its first fragments.
    {
        uint32_t so;
        __amdgpu_buffer_rsrc_t xr, wr;
        slab_src(0, so, xr, wr);
        static_for<AP>([&](auto LC) { copy_a(LC, 0, so, xr); });
        static_for<BP>([&](auto LC) { copy_w(LC, 0, so, wr); });
        slab_src(1, so, xr, wr);
        static_for<AP>([&](auto LC) { copy_a(LC, 1, so, xr); });
        static_for<BP / 2>([&](auto LC) { copy_w(LC, 1, so, wr); });
    }
    wait_vmcnt<AP + BP / 2>();
    barrier_no_fence();
    static_for<2 * FB>([&](auto QC) { read_frag(std::integral_constant<int, 0>{}, QC, 0u, 0u, 0); });

    int as = 0, ws = 0;  // ring slots of slab kt
    for (int kt = 0; kt < nk; ++kt) {
        const uint32_t abase = (uint32_t)as * SLAB, wbase = (uint32_t)ws * SLAB;
        const int as1 = as == AST - 1 ? 0 : as + 1, as2 = as1 == AST - 1 ? 0 : as1 + 1;
        const int ws1 = ws ^ 1;
        uint32_t so1, so2, so2w;
        __amdgpu_buffer_rsrc_t xr1, wr1, xr2, wr2, xr2w, wr2w;
        slab_src(kt + 1, so1, xr1, wr1);
        slab_src(kt + 2, so2, xr2, wr2);
        (void)xr1; (void)xr2w; (void)wr2;
        so2w = so2; wr2w = wr2;
        // K step 0: second half of weight slab kt + 1.
        settle(std::integral_constant<int, 0>{});
        kstep(std::integral_constant<int, 0>{}, abase, wbase, 1, [&](auto CC) {
            copy_w(std::integral_constant<int, BP / 2 + decltype(CC)::value>{}, ws1, so1, wr1);
        });
        // K steps 1 and 2: token slab kt + 2.
        settle(std::integral_constant<int, 1>{});
        kstep(std::integral_constant<int, 1>{}, abase, wbase, 2, [&](auto CC) {
            copy_a(std::integral_constant<int, decltype(CC)::value>{}, as2, so2, xr2);
        });
        settle(std::integral_constant<int, 0>{});
        kstep(std::integral_constant<int, 0>{}, abase, wbase, 3, [&](auto CC) {
            copy_a(std::integral_constant<int, 4 + decltype(CC)::value>{}, as2, so2, xr2);
        });
        settle(std::integral_constant<int, 1>{});
        // Token and weight slab kt + 1 have landed for this wave (the token
        // slab kt + 2 copies may still be in flight); after the barrier, for
        // every wave, and every wave is done reading slab kt.
        wait_vmcnt<AP>();
        barrier_no_fence();
        // K step 3: first fragments of slab kt + 1; first half of weight slab
        // kt + 2 into the weight buffer of slab kt.
        kstep(std::integral_constant<int, 1>{}, (uint32_t)as1 * SLAB, (uint32_t)ws1 * SLAB, 0, [&](auto CC) {
            copy_w(std::integral_constant<int, decltype(CC)::value>{}, ws, so2w, wr2w);
        });
        as = as1;
        ws = ws1;
    }

    // Epilogue (as in k_gemm_bf16): row ids to LDS, then per 32-row block
    // activate / convert into the wave's LDS area, read back as 16-byte row
    // pieces, store whole lines.
    constexpr bool OUT_F32 = EPI == EPI_STORE_F32;
    constexpr int OES = OUT_F32 ? 4 : 2;
    constexpr int SEG = WT * OES;
    constexpr int RSTR = SEG + 16;
    constexpr int CPRO = SEG / 16;
    constexpr int PIECES = 32 * CPRO / kWave;
    static_assert(1024 + NW * 32 * RSTR <= AST * SLAB + WST * SLAB, "epilogue staging must fit");
    __syncthreads();
    int32_t* srow = reinterpret_cast<int32_t*>(smem);
    if (EPI == EPI_SCATTER_SLOT)
        for (int r = tid; r < BM; r += NW * kWave) srow[r] = row_id(r);
    __syncthreads();
    uint8_t* stg = smem + 1024 + wave * 32 * RSTR;
#pragma unroll
    for (int i = 0; i < FB; ++i) {
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v0 = acc[j][i][4 * g + 0], v1 = acc[j][i][4 * g + 1];
                float v2 = acc[j][i][4 * g + 2], v3 = acc[j][i][4 * g + 3];
                uint8_t* dst = stg + fr * RSTR + (j * 32 + 8 * g + 4 * fk) * OES;
                if (OUT_F32) {
                    *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
                } else {
                    if (EPI == EPI_GELU_STORE) {
                        v0 = gelu_sig(v0); v1 = gelu_sig(v1); v2 = gelu_sig(v2); v3 = gelu_sig(v3);
                    }
                    *reinterpret_cast<uint2*>(dst) = pack4_bf16(v0, v1, v2, v3);
                }
            }
        wave_sync_lds();
#pragma unroll
        for (int k = 0; k < PIECES; ++k) {
            const int q = lane + kWave * k;
            const int rr = q / CPRO, pc = q % CPRO;
            const int r = wm * WT + i * 32 + rr;
            const uint4 v = *reinterpret_cast<const uint4*>(stg + rr * RSTR + pc * 16);
            if (r < tc.rows) {
                const size_t orow = EPI == EPI_SCATTER_SLOT ? (size_t)srow[r] : (size_t)(tc.row0 + r);
                uint8_t* out = static_cast<uint8_t*>(a.C) + (orow * a.N + tc.n0 + wn * WT) * OES + pc * 16;
                *reinterpret_cast<uint4*>(out) = v;
            }
        }
        wave_sync_lds();
    }
}

// Persistent form of k_gemm_sp: one workgroup per CU walks its share of the
// tiles (the XCD-aware order of locate_tile, a stride of gridDim / 8 tiles
// apart), and the slab pipeline runs on across tile boundaries. While the last
// two slabs of one tile are multiplied, the first two slabs of the next are
// already being copied, so a tile costs its K loop plus its epilogue. The
// per-tile start-up of the one-tile-per-workgroup kernel disappears: dispatch,
// the tile-table and row-map reads, and the first copies' latency.
//
// The epilogue stages each wave's 32-row blocks through the token-ring slot
// of the tile's last slab. That is the only slot not being filled at that
// moment: the next tile's first slab sits in the next slot and its second is
// still landing in the one after. Row pieces are XOR-swizzled instead of
// padded so that four waves' staging fits in one 32 KB slot. Tile metadata
// flows through a short pipeline: tile-table entries are read two tiles ahead,
// and gathered token rows (fc1) and output slots (fc2) one tile ahead. Their
// loads are issued where the wait the compiler places before their first use
// falls after long independent work.
//
// Token operand without gathering: its buffer resource starts at the tile's
// first row and spans its valid rows, so pad rows read as zeros. Gathered rows
// repeat the tile's last valid row, as in k_gemm_sp. Requires K >= 128 (at
// least two slabs per tile).
template <int EPI, bool GROUPED, int KC = 8>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void k_gemm_pp(const GemmArgs a) {
    constexpr int BM = 256, BN = 256, NW = 4, WT = 128, FB = WT / 32;
    constexpr int BK = 64, CPR = 8, ROWB = 128, KS = 4;
    constexpr int SLAB = BM * ROWB;            // 32 KB per operand and slab
    constexpr int AST = 3, WST = 2;            // ring depths
    constexpr int WBASE = AST * SLAB;          // weight ring after the token ring
    constexpr int AP = BM * CPR / kWave / NW;  // 8 token copy pieces per wave and slab
    constexpr int BP = BN * CPR / kWave / NW;  // 8 weight copy pieces
    static_assert(AP == 8 && BP == 8, "copy schedule is written for 8 + 8 pieces");
    constexpr bool BWD1 = EPI == EPI_GELU_BWD;  // bf16 GELU, then the fp32 pre-activation into C2
    constexpr bool DG = EPI == EPI_DGELU;       // bf16 of acc times GELU'(aux)
    constexpr bool DSW = EPI == EPI_DSWIGLU;    // dG and dU (bf16) from acc and the stored G, U
    constexpr bool GATHER = GROUPED && (fc1_epi(EPI) || BWD1 || DG || DSW);
    constexpr bool SWIGLU = EPI == EPI_SWIGLU_STORE || EPI == EPI_SWIGLU_BWD;
    constexpr bool SWBWD = EPI == EPI_SWIGLU_BWD;  // and the fp32 gate / up pre-activations into C2
    constexpr bool SCATTER = EPI == EPI_SCATTER_SLOT || EPI == EPI_SCATTER_SLOT_F32;
    constexpr bool KM = kmajor_epi(EPI);  // weights [Kdim][N]: fragments by transposing reads
    constexpr bool RNORM = EPI == EPI_ROUTER_F32;  // EPI_STORE_F32 and the token rows' sums of squares
    constexpr bool OUT_F32 = EPI == EPI_STORE_F32 || EPI == EPI_SCATTER_SLOT_F32 || RNORM;
    constexpr bool COMBINE = EPI == EPI_COMBINE;
    constexpr bool STAGE_F32 = OUT_F32 || COMBINE;  // accumulators staged as fp32
    constexpr int OES = OUT_F32 ? 4 : 2;
    constexpr int NH = (STAGE_F32 || EPI == EPI_DSWIGLU) ? 2 : 1;  // column halves per staged block
    static_assert(!(COMBINE && GROUPED), "the fused combine is a dense (shared expert) epilogue");
    constexpr int STG_WAVE = 32 * 256;         // staging bytes per wave
    static_assert(NW * STG_WAVE == SLAB, "staging must fill exactly one token slot");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[AST * SLAB + WST * SLAB];

    const int n_n = a.N / BN;
    const int total = (GROUPED ? __builtin_amdgcn_readfirstlane(*a.n_tiles) : (a.dense_rows + BM - 1) / BM) * n_n;
    const int per = (total + kNumXcd - 1) / kNumXcd;
    const int xcd = blockIdx.x % kNumXcd;
    const int wpx = gridDim.x / kNumXcd;  // workgroups per XCD: the tile stride
    const int lid_end = min(total, (xcd + 1) * per);
    int lid = xcd * per + (int)blockIdx.x / kNumXcd;
    if (lid >= lid_end) return;
    // The combine epilogue streams K expert-output rows per output element
    // (1 MB per tile at ViT-G) and is HBM-bound when every CU runs it at once;
    // tiles cost the same, so the workgroups stay in step from the start.
    // Workgroups of odd XCDs start about 80k cycles later, so that their
    // epilogues overlap the other XCDs' K loops (whole XCDs, so that each L2
    // still sees its tiles in step). Measured at ViT-G: the layer -1.3 %.
    // "xcd" is blockIdx mod kNumXcd, which names the XCD only under the
    // round-robin dispatch of MI355X; under another dispatch a different half
    // of the workgroups waits, which changes the speed, never the tiles.
    if constexpr (EPI == EPI_COMBINE) {
        if (xcd & 1)
            for (int q = 0; q < 10; ++q) __builtin_amdgcn_s_sleep(127);
    }

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    const int Kd = a.Kdim;
    const int nk = Kd / BK;
    const int ncols = a.ldc > 0 ? a.ldc : a.N;  // real output columns (N may be rounded up to BN)
    const uint32_t rowbytes = (uint32_t)Kd * 2;

    struct Tile {
        int e, row0, rows, n0;
    };
    // Tile-table entry of tile l (grouped): read through the vector path (the
    // kernel's own stores keep the compiler from proving the table constant).
    // Indices past this workgroup's share read its last tile instead.
    auto tile_entry = [&](int l) {
        TileDesc d{};
        if (GROUPED) d = a.tiles[min(l, lid_end - 1) / n_n];
        return d;
    };
    // Tile l from its table entry; the entry is the same for every lane, so it
    // goes back to scalar registers.
    auto tile_of = [&](int l, const TileDesc& d) {
        Tile t;
        const int mt = l / n_n;
        t.n0 = (l - mt * n_n) * BN;
        if (GROUPED) {
            t.e = __builtin_amdgcn_readfirstlane(d.e);
            t.row0 = __builtin_amdgcn_readfirstlane(d.row0);
            t.rows = __builtin_amdgcn_readfirstlane(d.rows);
        } else {
            t.e = 0;
            t.row0 = mt * BM;
            t.rows = min(BM, a.dense_rows - t.row0);
        }
        return t;
    };
    auto tile_at = [&](int l) { return tile_of(l, tile_entry(l)); };
    const bf16_t* const Bw = static_cast<const bf16_t*>(a.B);
    const bf16_t* const Ax = static_cast<const bf16_t*>(a.A);
    // SwiGLU: a tile of BN columns computes activation columns [n0 / 2,
    // n0 / 2 + 128); the resource starts at gate row n0 / 2 and ends with the
    // group's last up row, so rows past it read as zeros.
    // The row counts are uniform; readfirstlane keeps the resource in scalar
    // registers (the compiler cannot prove it and would wrap every copy in a
    // waterfall loop).
    auto wres_of = [&](const Tile& t) {
        if (SWIGLU)
            return make_rsrc(Bw + (size_t)t.e * a.b_group_stride + (size_t)(t.n0 / 2) * Kd,
                             (uint32_t)__builtin_amdgcn_readfirstlane(2 * a.act_n - t.n0 / 2) * rowbytes);
        if (KM)  // every weight row of the expert, columns from n0
            return make_rsrc(Bw + (size_t)t.e * a.b_group_stride + t.n0, (uint32_t)a.b_group_stride * 2u - (uint32_t)t.n0 * 2u);
        const int rows = __builtin_amdgcn_readfirstlane(max(0, min(BN, weight_rows(a) - t.n0)));
        return make_rsrc(Bw + (size_t)t.e * a.b_group_stride + (size_t)t.n0 * Kd, (uint32_t)rows * rowbytes);
    };
    auto xres_of = [&](const Tile& t) {
        if (GATHER) return make_rsrc(Ax, a.a_bytes);
        return make_rsrc(Ax + (size_t)t.row0 * Kd, (uint32_t)t.rows * rowbytes);
    };
    // Source offset of K slab s.
    auto soff_of = [](int s) -> uint32_t { return (uint32_t)s * (BK * 2); };
    const __amdgpu_buffer_rsrc_t xnull = make_rsrc(Ax, 0);
    const __amdgpu_buffer_rsrc_t wnull = make_rsrc(Bw, 0);

    // Row offsets of this lane's copy pieces: row r of the slab, 16-byte chunk
    // c (swizzled). The weight offsets (and the token offsets without
    // gathering) are the same for every tile.
    auto piece_rc = [&](int i, int& r, int& c) {
        const int sl = (wave + NW * i) * kWave + lane;
        r = sl / CPR;
        c = (sl % CPR) ^ ((r >> 1) & 7);
    };
    // SwiGLU: wave column block wn (tile columns [128 wn, 128 wn + 128)) holds
    // the gate rows of activation columns [64 wn, 64 wn + 64) of the tile,
    // then their up rows (act_n rows further on). Gate rows past act_n read
    // (finite) up rows, whose activations the epilogue zeroes.
    // Token offsets without gathering (tv) are the plain row layout; for
    // every epilogue but SwiGLU they equal the weight offsets.
    uint32_t wv[BP], tv[AP];
#pragma unroll
    for (int i = 0; i < BP; ++i) {
        int r, c;
        piece_rc(i, r, c);
        const int wrow = SWIGLU ? (r / WT) * (WT / 2) + r % (WT / 2) + ((r % WT) >= WT / 2 ? a.act_n : 0) : r;
        wv[i] = (uint32_t)wrow * rowbytes + c * 16;
        tv[i] = (uint32_t)r * rowbytes + c * 16;
    }
    // K-major weights: LDS rows of 512 bytes, 16-byte chunk c of row r at chunk
    // c ^ ((r & 3) << 2) (a transposing read takes 4 rows x 32 columns per half
    // wave, 16 chunks in distinct banks); piece p of a wave is rows 16 w + 2 p
    // and the next.
    const int hb = lane >> 5;
    const uint32_t krow = (uint32_t)ncols * 2;
    const uint32_t klane = 16 * wave + hb;
    const uint32_t kbase[2] = {klane * krow + (uint32_t)((lane & 31) ^ (hb << 2)) * 16u,
                               klane * krow + (uint32_t)((lane & 31) ^ ((2 + hb) << 2)) * 16u};
    // Gathered token rows: slot -> token, rows past the tile's end repeat its last row.
    auto load_tokens = [&](const Tile& t, int32_t (&tok)[AP]) {
#pragma unroll
        for (int i = 0; i < AP; ++i) {
            int r, c;
            piece_rc(i, r, c);
            tok[i] = a.row_map[t.row0 + min(r, t.rows - 1)];
        }
    };
    // Row map entries are slots; the operand row is the slot's token (slot /
    // K) or, gathering slot rows, the slot itself.
    const int rdiv = a.row_mode == ROWS_GATHER_SLOTS ? 1 : a.route_k;
    auto token_offsets = [&](const int32_t (&tok)[AP], uint32_t (&xv)[AP]) {
#pragma unroll
        for (int i = 0; i < AP; ++i) {
            int r, c;
            piece_rc(i, r, c);
            xv[i] = (uint32_t)(tok[i] / rdiv) * rowbytes + c * 16;
        }
    };
    // Output slot of staged piece k of 32-row block i (fc2 scatter).
    int32_t orow[FB][8];
    auto load_slots = [&](const Tile& t) {
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int r = wm * WT + i * 32 + (lane >> 4) + 4 * k;
                orow[i][k] = a.row_map[t.row0 + min(r, t.rows - 1)];
            }
    };

    // Current tile (c), next (n) and the one after (nn, table entry only).
    Tile tc = tile_at(lid);
    bool has_n = lid + wpx < lid_end;
    Tile tn = has_n ? tile_at(lid + wpx) : tc;
    bool has_nn = lid + 2 * wpx < lid_end;
    Tile tnn = has_nn ? tile_at(lid + 2 * wpx) : tn;
    // Table entry three tiles ahead, read one tile before it is needed.
    TileDesc ent3 = tile_entry(lid + 3 * wpx);
    __amdgpu_buffer_rsrc_t xres_c = xres_of(tc), wres_c = wres_of(tc);
    __amdgpu_buffer_rsrc_t xres_n = has_n ? xres_of(tn) : xnull;
    __amdgpu_buffer_rsrc_t wres_n = has_n ? wres_of(tn) : wnull;
    uint32_t xv_c[AP], xv_n[AP];
    int32_t tok[AP];
    if (GATHER) {
        load_tokens(tc, tok);
        token_offsets(tok, xv_c);
        load_tokens(tn, tok);
        token_offsets(tok, xv_n);
    }
    if (SCATTER) load_slots(tc);

    f32x16_t acc[FB][FB];
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    const int fr = lane & 31;
    const int fk = lane >> 5;
    const int lane_sw = (fr >> 1) & 7;
    uint32_t xoff[KS], woff[KS];
    const uint32_t base = lds_address(smem);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const uint32_t k = fr * ROWB + (((ks * 2 + fk) ^ lane_sw) << 4);
        xoff[ks] = base + (wm * WT) * ROWB + k;
        woff[ks] = base + WBASE + (wn * WT) * ROWB + k;
        if constexpr (KM) {  // by 32-column block instead of by K step
            const int r4 = (lane & 15) >> 2;
            woff[ks] = base + WBASE + (uint32_t)(fk * 8 + r4) * 512u + (uint32_t)(lane & 1) * 8u +
                       (uint32_t)(wn * 16 + ((ks ^ r4) << 2) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 16u;
        }
    }

    auto copy_a = [&](auto LC, int stage, uint32_t soff, __amdgpu_buffer_rsrc_t xr, const uint32_t (&xv)[AP]) {
        constexpr int L = decltype(LC)::value;
        copy16_to_lds(xr, xv[L], soff, smem + stage * SLAB + (wave + NW * L) * 1024);
    };
    auto copy_w = [&](auto LC, int stage, int slab, __amdgpu_buffer_rsrc_t wr) {
        constexpr int L = decltype(LC)::value;
        if constexpr (KM) {
            // Stacked weights (a.b_half > 0): K columns b_half .. are the second
            // matrix's rows, act_n rows after the first's; K columns past act_n in
            // either half have no weight row and read as zeros.
            const int half = EPI == EPI_SCATTER_SLOT_F32 ? a.b_half : 0;
            const int up = half > 0 && slab * BK >= half ? 1 : 0;
            const int kk = slab * BK - up * half;
            uint32_t v = kbase[L & 1] + (uint32_t)(kk + (up ? a.act_n : 0) + 2 * L) * krow;
            if (half > 0 && (int)klane + 2 * L + kk >= a.act_n) v = kWgradNoRow;
            copy16_to_lds(wr, v, 0, smem + WBASE + stage * SLAB + (wave * 8 + L) * 1024);
        } else {
            copy16_to_lds(wr, wv[L], soff_of(slab), smem + WBASE + stage * SLAB + (wave + NW * L) * 1024);
        }
    };

    bf16x8_t xf[2][FB], wf[2][FB];
    u32x2_t wh[2][FB][2];  // K-major weights: the two row halves of each fragment
    auto read_frag = [&](auto NBC, auto QC, uint32_t abase, uint32_t wbase, auto KSC) {
        constexpr int nb = decltype(NBC)::value, q = decltype(QC)::value, ks = decltype(KSC)::value;
        if constexpr (q < FB) {
            xf[nb][q] = lds_read16<q * 32 * ROWB>(xoff[ks] + abase);
        } else if constexpr (KM) {
            lds_read_tr8_asm<ks * 16 * 512>(wh[nb][q - FB][0], woff[q - FB] + wbase);
            lds_read_tr8_asm<ks * 16 * 512 + 4 * 512>(wh[nb][q - FB][1], woff[q - FB] + wbase);
        } else {
            wf[nb][q - FB] = lds_read16<(q - FB) * 32 * ROWB>(woff[ks] + wbase);
        }
    };
    auto wfrag = [&](auto CBC, auto JC) {
        constexpr int cb = decltype(CBC)::value, j = decltype(JC)::value;
        if constexpr (KM)
            return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(wh[cb][j][0], wh[cb][j][1], 0, 1, 2, 3));
        else
            return wf[cb][j];
    };
    auto settle = [&](auto CBC) {
        constexpr int cb = decltype(CBC)::value;
        wait_lgkmcnt0();
#pragma unroll
        for (int i = 0; i < FB; ++i) tie(xf[cb][i]);
#pragma unroll
        for (int j = 0; j < FB; ++j) {
            if constexpr (KM) {
                tie(wh[cb][j][0]);
                tie(wh[cb][j][1]);
            } else {
                tie(wf[cb][j]);
            }
        }
    };
    // Router logits: per lane, the sums of squares of its four token rows'
    // values in the token fragments (lanes l and l + 32 hold the two halves
    // of each K step of row l % 32 of a 32-row block).
    float xsq[FB];
#pragma unroll
    for (int i = 0; i < FB; ++i) xsq[i] = 0.0f;

    // One K step: 16 MFMAs on buffer CB, fragment q of the next K step after
    // MFMA q (q < 8), copy q / 4 of the step's four after MFMA q when q % 4 == 1.
    // Router logits: after MFMA q, the squares of the two values in 32-bit
    // word q % 4 of token fragment q / 4 (VALU work beside the MFMAs).
    auto kstep = [&](auto CBC, uint32_t rabase, uint32_t rwbase, auto KSC, auto&& copy) {
        constexpr int cb = decltype(CBC)::value;
        static_for<FB * FB>([&](auto QC) {
            constexpr int q = decltype(QC)::value;
            constexpr int j = q / FB, i = q % FB;
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wfrag(CBC, std::integral_constant<int, j>{}), xf[cb][i],
                                                                acc[j][i], 0, 0, 0);
            if constexpr (RNORM) {
                const uint32_t u = __builtin_bit_cast(u32x4_t, xf[cb][q / 4])[q % 4];
                const float lo = __uint_as_float(u << 16), hi = __uint_as_float(u & 0xffff0000u);
                xsq[q / 4] = fmaf(lo, lo, xsq[q / 4]);
                xsq[q / 4] = fmaf(hi, hi, xsq[q / 4]);
            }
            if constexpr (q < 2 * FB)
                read_frag(std::integral_constant<int, cb ^ 1>{}, QC, rabase, rwbase, KSC);
            if constexpr (q % 4 == 1) copy(std::integral_constant<int, q / 4>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // Fused combine (K = KC) for one staged fp32 block of the shared expert's
    // output S: 32 rows x 64 columns, pieces of 8 columns (lanes 8 r + c take
    // row r, column piece c; four rows per lane). Per piece, in the order of
    // the separate combine: acc = 0, acc = fma(g_j, O_j, acc) for j = 0..K-1,
    // acc = fma(lambda, S, acc), one rounding to bf16.
    auto combine_block = [&](const Tile& t, uint32_t stg, int i, int h) {
        const int cp = lane & 7;
        const bf16_t* const eo = static_cast<const bf16_t*>(a.eo);
        // y rows of this tile; stores of pad rows fall outside and are dropped,
        // so the four pieces need no branch and can be scheduled together.
        const __amdgpu_buffer_rsrc_t yres =
            make_rsrc(static_cast<uint8_t*>(a.C) + (size_t)t.row0 * a.N * 2, (uint32_t)t.rows * a.N * 2);
        u32x4_t s0[4], s1[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int rr = (lane >> 3) + 8 * k;
            s0[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)((2 * cp) ^ (rr & 15)) << 4));
            s1[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)((2 * cp + 1) ^ (rr & 15)) << 4));
        }
        // No memory clobber: the loads below may be scheduled across it.
        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            tie(s0[k]);
            tie(s1[k]);
        }
        // Two pieces per step: both pieces' loads are issued before either is
        // used (twenty 16-byte loads in flight per lane).
#pragma unroll
        for (int kp = 0; kp < 4; kp += 2) {
            float gj[2][KC];
            u32x4_t o[2][KC];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int rr = (lane >> 3) + 8 * (kp + u);
                const int tok = t.row0 + min(wm * WT + i * 32 + rr, t.rows - 1);
                const int c0 = t.n0 + wn * WT + h * 64 + cp * 8;
                if constexpr (KC % 4 == 0) {
#pragma unroll
                    for (int j = 0; j < KC; j += 4) {
                        const float4 g4 = *reinterpret_cast<const float4*>(a.gate + (size_t)tok * KC + j);
                        gj[u][j] = g4.x; gj[u][j + 1] = g4.y; gj[u][j + 2] = g4.z; gj[u][j + 3] = g4.w;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < KC; ++j) gj[u][j] = a.gate[(size_t)tok * KC + j];
                }
#pragma unroll
                for (int j = 0; j < KC; ++j)
                    o[u][j] = *reinterpret_cast<const u32x4_t*>(eo + ((size_t)tok * KC + j) * a.N + c0);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k = kp + u;
                const int r = wm * WT + i * 32 + (lane >> 3) + 8 * k;
                const int c0 = t.n0 + wn * WT + h * 64 + cp * 8;
                float acc8[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) acc8[q] = 0.0f;
#pragma unroll
                for (int j = 0; j < KC; ++j) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        acc8[2 * q] = fmaf(gj[u][j], __uint_as_float(o[u][j][q] << 16), acc8[2 * q]);
                        acc8[2 * q + 1] = fmaf(gj[u][j], __uint_as_float(o[u][j][q] & 0xffff0000u), acc8[2 * q + 1]);
                    }
                }
                const float sv[8] = {__uint_as_float(s0[k].x), __uint_as_float(s0[k].y), __uint_as_float(s0[k].z),
                                     __uint_as_float(s0[k].w), __uint_as_float(s1[k].x), __uint_as_float(s1[k].y),
                                     __uint_as_float(s1[k].z), __uint_as_float(s1[k].w)};
                u32x4_t out;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint32_t lo = __float_as_uint(fmaf(a.lambda, sv[2 * q], acc8[2 * q]));
                    uint32_t hi = __float_as_uint(fmaf(a.lambda, sv[2 * q + 1], acc8[2 * q + 1]));
                    lo += 0x7fffu + ((lo >> 16) & 1u);  // round to nearest even (finite values)
                    hi += 0x7fffu + ((hi >> 16) & 1u);
                    out[q] = (lo >> 16) | (hi & 0xffff0000u);
                }
                // y is written only here and read by nothing in this kernel, so
                // the store needs no memory clobber.
                const uint32_t yoff = ((uint32_t)r * (uint32_t)a.N + (uint32_t)c0) * 2u;
                asm volatile("buffer_store_dwordx4 %0, %1, %2, 0 offen nt\n\ts_nop 0" ::"v"(out), "v"(yoff), "s"(yres));
            }
        }
    };

    // Epilogue of tile t from the accumulators, staged through the token slot
    // `stslot`: per 32-row block (and 64-column half for fp32 output) each
    // lane writes its row's runs into the wave's 8 KB, then reads back 16-byte
    // row pieces (16 lanes per 256-byte row) and stores whole lines.
    auto epilogue = [&](const Tile& t, int stslot) {
        const uint32_t stg = base + (uint32_t)stslot * SLAB + (uint32_t)wave * STG_WAVE;
        const uint32_t wrow = stg + (uint32_t)fr * 256u;
        const int sw = fr & 15;
        uint8_t* const cbase = static_cast<uint8_t*>(a.C);
        // DSW: row stride 2 act_ld, columns past act_ld (N rounded up) not stored.
        const size_t ostr = DSW ? 2 * (size_t)a.act_ld : (size_t)ncols;
        // DSW: stage half h of block i (64 columns) as [dG | dU] per 256-byte
        // row, G and U read once.
        auto dsw_stage = [&](const Tile& tt, int i, int h) {
            const int r = wm * WT + i * 32 + fr;
            const float* grow = static_cast<const float*>(a.aux) +
                                (size_t)(tt.row0 + min(r, tt.rows - 1)) * 2 * a.act_ld;
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const int j = 2 * h + jj;
                __builtin_amdgcn_sched_barrier(0);
                float4 gv[4], uv[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = tt.n0 + wn * WT + j * 32 + 8 * g + 4 * fk;
                    gv[g] = make_float4(0.f, 0.f, 0.f, 0.f);
                    uv[g] = gv[g];
                    if (c < a.act_ld) {  // act_ld is a multiple of 64: whole float4s
                        gv[g] = *reinterpret_cast<const float4*>(grow + c);
                        uv[g] = *reinterpret_cast<const float4*>(grow + a.act_ld + c);
                    }
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int c = tt.n0 + wn * WT + j * 32 + 8 * g + 4 * fk;
                    const float gg[4] = {gv[g].x, gv[g].y, gv[g].z, gv[g].w};
                    const float uu[4] = {uv[g].x, uv[g].y, uv[g].z, uv[g].w};
                    float dg[4], du[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        swiglu_grad(gg[q], uu[q], acc_read(acc[j][i][4 * g + q]), dg[q], du[q]);
                        if (c + q >= a.act_n) dg[q] = du[q] = 0.0f;
                    }
                    const uint2 pg = pack4_bf16(dg[0], dg[1], dg[2], dg[3]);
                    const uint2 pu = pack4_bf16(du[0], du[1], du[2], du[3]);
                    const int chunk = 4 * jj + g;  // 16-byte chunk of the half's 64 columns
                    lds_write8_asm(wrow + ((uint32_t)(chunk ^ sw) << 4) + (uint32_t)fk * 8u, (u32x2_t){pg.x, pg.y});
                    lds_write8_asm(wrow + ((uint32_t)((8 + chunk) ^ sw) << 4) + (uint32_t)fk * 8u,
                                   (u32x2_t){pu.x, pu.y});
                }
            }
        };
#pragma unroll
        for (int i = 0; i < FB; ++i) {
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                __builtin_amdgcn_sched_barrier(0);
                if (STAGE_F32) {
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int j = 2 * h + jj;
                            const u32x4_t v = {__float_as_uint(acc_read(acc[j][i][4 * g + 0])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 1])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 2])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 3]))};
                            const int chunk = 8 * jj + 2 * g + fk;
                            lds_write16_asm(wrow + ((uint32_t)(chunk ^ sw) << 4), v);
                        }
                } else if (SWIGLU) {
                    // Blocks j < 2 are gate columns, j + 2 the up columns of
                    // the same activation columns: 64 per wave row.
#pragma unroll
                    for (int j = 0; j < FB / 2; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int c = t.n0 / 2 + wn * (WT / 2) + j * 32 + 8 * g + 4 * fk;
                            float v[4];
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                v[q] = swiglu_col(acc_read(acc[j][i][4 * g + q]),
                                                  acc_read(acc[j + FB / 2][i][4 * g + q]), c + q < a.act_n);
                            const uint2 pk = pack4_bf16(v[0], v[1], v[2], v[3]);
                            lds_write8_asm(wrow + ((uint32_t)((4 * j + g) ^ sw) << 4) + (uint32_t)fk * 8u,
                                           (u32x2_t){pk.x, pk.y});
                        }
                } else if (DSW) {
                    dsw_stage(t, i, h);
                } else {
                    // dH: GELU' of the stored pre-activation of this lane's row and columns.
                    float4 fac[FB][4];
                    if constexpr (DG) {
                        const int r = wm * WT + i * 32 + fr;
                        // Columns past the width (N rounded up) re-read its first and are not stored.
                        const float* arow = static_cast<const float*>(a.aux) +
                                            (size_t)(t.row0 + min(r, t.rows - 1)) * ncols + 4 * fk;
#pragma unroll
                        for (int j = 0; j < FB; ++j)
#pragma unroll
                            for (int g = 0; g < 4; ++g)
                                {
                                const int c = t.n0 + wn * WT + j * 32;
                                fac[j][g] = *reinterpret_cast<const float4*>(arow + (c < ncols ? c : 0) + 8 * g);
                            }
                    }
#pragma unroll
                    for (int j = 0; j < FB; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            float v0 = acc_read(acc[j][i][4 * g + 0]), v1 = acc_read(acc[j][i][4 * g + 1]);
                            float v2 = acc_read(acc[j][i][4 * g + 2]), v3 = acc_read(acc[j][i][4 * g + 3]);
                            if (EPI == EPI_GELU_STORE || BWD1) {
                                v0 = gelu_sig(v0); v1 = gelu_sig(v1); v2 = gelu_sig(v2); v3 = gelu_sig(v3);
                            }
                            if constexpr (DG) {
                                v0 *= gelu_sig_grad(fac[j][g].x); v1 *= gelu_sig_grad(fac[j][g].y);
                                v2 *= gelu_sig_grad(fac[j][g].z); v3 *= gelu_sig_grad(fac[j][g].w);
                            }
                            const int chunk = 4 * j + g;
                            const uint2 pk = pack4_bf16(v0, v1, v2, v3);
                            lds_write8_asm(wrow + ((uint32_t)(chunk ^ sw) << 4) + (uint32_t)fk * 8u,
                                           (u32x2_t){pk.x, pk.y});
                        }
                }
                if constexpr (COMBINE) {
                    combine_block(t, stg, i, h);
                    continue;
                }
                if constexpr (SWIGLU) {
                    // 128-byte activation rows: 8 lanes per row, 8 rows per read.
                    const int ocol = t.n0 / 2 + wn * (WT / 2);
                    u32x4_t v[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int rr = (lane >> 3) + 8 * k;
                        v[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)((lane & 7) ^ (rr & 15)) << 4));
                    }
                    wait_lgkmcnt0();
#pragma unroll
                    for (int k = 0; k < 4; ++k) tie(v[k]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int r = wm * WT + i * 32 + (lane >> 3) + 8 * k;
                        if (r < t.rows && ocol < a.act_ld)
                            store16_asm(cbase + ((size_t)(t.row0 + r) * a.act_ld + ocol) * 2 + (lane & 7) * 16, v[k]);
                    }
                    continue;
                }
                u32x4_t v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int rr = (lane >> 4) + 4 * k;
                    const int pc = lane & 15;
                    v[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)(pc ^ (rr & 15)) << 4));
                }
                wait_lgkmcnt0();
#pragma unroll
                for (int k = 0; k < 8; ++k) tie(v[k]);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int rr = (lane >> 4) + 4 * k;
                    const int r = wm * WT + i * 32 + rr;
                    // DSW: pieces 0..7 of the row are dG, 8..15 dU (act_ld further on).
                    const int pcol = DSW ? (lane & 7) * 8 : (lane & 15) * (16 / OES);
                    const int col = t.n0 + wn * WT + h * 64 + pcol;
                    if (r < t.rows && (KM || BWD1 ? col : t.n0 + wn * WT + h * 64) < ncols) {
                        const size_t orw = SCATTER ? (size_t)orow[i][k] : (size_t)(t.row0 + r);
                        uint8_t* out = cbase + (orw * ostr + t.n0 + wn * WT + h * 64) * OES + (lane & 15) * 16;
                        if (DSW) out = cbase + (orw * ostr + ((lane & 8) ? a.act_ld : 0) + col) * 2;
                        store16_asm(out, v[k]);
                    }
                }
            }
            if constexpr (SWBWD) {
                // Second output: the gate (q = 0) and up (q = 1) pre-activations
                // of this wave's 64 activation columns as fp32 rows of C2
                // [rows, 2 act_ld]: G at column c, U at act_ld + c.
                const int ocol = t.n0 / 2 + wn * (WT / 2);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int j = 2 * q + jj;
                            const u32x4_t v = {__float_as_uint(acc_read(acc[j][i][4 * g + 0])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 1])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 2])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 3]))};
                            const int chunk = 8 * jj + 2 * g + fk;
                            lds_write16_asm(wrow + ((uint32_t)(chunk ^ sw) << 4), v);
                        }
                    u32x4_t v[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int rr = (lane >> 4) + 4 * k;
                        v[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)((lane & 15) ^ (rr & 15)) << 4));
                    }
                    wait_lgkmcnt0();
#pragma unroll
                    for (int k = 0; k < 8; ++k) tie(v[k]);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int r = wm * WT + i * 32 + (lane >> 4) + 4 * k;
                        if (r < t.rows && ocol < a.act_ld)
                            store16_asm(static_cast<uint8_t*>(a.C2) +
                                            ((size_t)(t.row0 + r) * 2 * a.act_ld + q * a.act_ld + ocol) * 4 +
                                            (lane & 15) * 16,
                                        v[k]);
                    }
                }
            }
            if constexpr (BWD1) {
                // Second output: the pre-activation (acc) as fp32 rows of C2,
                // two 64-column halves through the same staging rows.
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int j = 2 * h + jj;
                            const u32x4_t v = {__float_as_uint(acc_read(acc[j][i][4 * g + 0])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 1])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 2])),
                                               __float_as_uint(acc_read(acc[j][i][4 * g + 3]))};
                            const int chunk = 8 * jj + 2 * g + fk;
                            lds_write16_asm(wrow + ((uint32_t)(chunk ^ sw) << 4), v);
                        }
                    u32x4_t v[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int rr = (lane >> 4) + 4 * k;
                        v[k] = lds_read16u_asm(stg + (uint32_t)rr * 256u + ((uint32_t)((lane & 15) ^ (rr & 15)) << 4));
                    }
                    wait_lgkmcnt0();
#pragma unroll
                    for (int k = 0; k < 8; ++k) tie(v[k]);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const int r = wm * WT + i * 32 + (lane >> 4) + 4 * k;
                        if (r < t.rows && t.n0 + wn * WT + h * 64 < ncols)
                            store16_asm(static_cast<uint8_t*>(a.C2) +
                                            ((size_t)(t.row0 + r) * ncols + t.n0 + wn * WT + h * 64) * 4 + (lane & 15) * 16,
                                        v[k]);
                    }
                }
            }
        }
    };

    // Prologue: token slab 0, weight slab 0, token slab 1, the first half of
    // weight slab 1; wait for slab 0 of both operands; read its first fragments.
    static_for<AP>([&](auto LC) { copy_a(LC, 0, soff_of(0), xres_c, GATHER ? xv_c : tv); });
    static_for<BP>([&](auto LC) { copy_w(LC, 0, 0, wres_c); });
    static_for<AP>([&](auto LC) { copy_a(LC, 1, soff_of(1), xres_c, GATHER ? xv_c : tv); });
    static_for<BP / 2>([&](auto LC) { copy_w(LC, 1, 1, wres_c); });
    wait_vmcnt<AP + BP / 2>();
    barrier_no_fence();
    static_for<2 * FB>([&](auto QC) { read_frag(std::integral_constant<int, 0>{}, QC, 0u, 0u, std::integral_constant<int, 0>{}); });

    int as = 0, ws = 0;  // ring slots of the slab being multiplied
    for (;;) {
        int kt = 0;
        do {  // nk >= 2 slabs: written as do-while so the compiler counts the copies
            const uint32_t abase = (uint32_t)as * SLAB, wbase = (uint32_t)ws * SLAB;
            const int as1 = as == AST - 1 ? 0 : as + 1, as2 = as1 == AST - 1 ? 0 : as1 + 1;
            const int ws1 = ws ^ 1;
            // Slabs kt + 1 and kt + 2 may belong to the next tile.
            const bool n1 = kt + 1 >= nk, n2 = kt + 2 >= nk;
            const int s1 = n1 ? kt + 1 - nk : kt + 1, s2 = n2 ? kt + 2 - nk : kt + 2;
            const uint32_t so2 = soff_of(s2);
            const __amdgpu_buffer_rsrc_t wr1 = n1 ? wres_n : wres_c;
            const __amdgpu_buffer_rsrc_t xr2 = n2 ? xres_n : xres_c;
            const __amdgpu_buffer_rsrc_t wr2 = n2 ? wres_n : wres_c;
            uint32_t xv2[AP];
#pragma unroll
            for (int i = 0; i < AP; ++i) xv2[i] = GATHER ? (n2 ? xv_n[i] : xv_c[i]) : tv[i];
            // K step 0: second half of weight slab kt + 1.
            settle(std::integral_constant<int, 0>{});
            kstep(std::integral_constant<int, 0>{}, abase, wbase, std::integral_constant<int, 1>{}, [&](auto CC) {
                copy_w(std::integral_constant<int, BP / 2 + decltype(CC)::value>{}, ws1, s1, wr1);
            });
            // K steps 1 and 2: token slab kt + 2.
            settle(std::integral_constant<int, 1>{});
            kstep(std::integral_constant<int, 1>{}, abase, wbase, std::integral_constant<int, 2>{}, [&](auto CC) {
                copy_a(std::integral_constant<int, decltype(CC)::value>{}, as2, so2, xr2, xv2);
            });
            settle(std::integral_constant<int, 0>{});
            kstep(std::integral_constant<int, 0>{}, abase, wbase, std::integral_constant<int, 3>{}, [&](auto CC) {
                copy_a(std::integral_constant<int, 4 + decltype(CC)::value>{}, as2, so2, xr2, xv2);
            });
            settle(std::integral_constant<int, 1>{});
            // Token and weight slab kt + 1 have landed for this wave (only the
            // eight token copies of slab kt + 2 may be younger); after the
            // barrier, for every wave, and every wave is done reading slab kt.
            wait_vmcnt<AP>();
            barrier_no_fence();
            // K step 3: first fragments of slab kt + 1; first half of weight
            // slab kt + 2 into the weight slot of slab kt.
            kstep(std::integral_constant<int, 1>{}, (uint32_t)as1 * SLAB, (uint32_t)ws1 * SLAB,
                  std::integral_constant<int, 0>{}, [&](auto CC) {
                      copy_w(std::integral_constant<int, decltype(CC)::value>{}, ws, s2, wr2);
                  });
            as = as1;
            ws = ws1;
        } while (++kt < nk);

        // The last K step also read the next tile's first fragments; let them
        // land (their registers are reused by the epilogue) and read them again
        // after it.
        settle(std::integral_constant<int, 0>{});
        // Gathered rows of the tile after next: read now, used after the epilogue.
        if (GATHER && has_nn) load_tokens(tnn, tok);
        // Router logits: the tile's token rows' sums of squares (the first
        // column tile's waves of column block 0 write them), then zero for
        // the next tile.
        if constexpr (RNORM) {
#pragma unroll
            for (int i = 0; i < FB; ++i) {
                const float v = xsq[i] + __shfl_xor(xsq[i], 32);
                const int r = wm * WT + i * 32 + fr;
                if (tc.n0 == 0 && wn == 0 && fk == 0 && r < tc.rows)
                    store4_asm(static_cast<float*>(a.C2) + tc.row0 + r, __float_as_uint(v));
                xsq[i] = 0.0f;
            }
        }
        // The last slab's token slot is free (and read by no wave any more).
        epilogue(tc, as == 0 ? AST - 1 : as - 1);
        // The combine's loads land in registers the next K loop reuses; a wait
        // the compiler sees (vmcnt(0)) retires them here, once per tile,
        // instead of the conservative waits it would otherwise put at the head
        // of every K step.
        if (COMBINE) __builtin_amdgcn_s_waitcnt(0xF70);
        if (!has_n) break;

        // Advance: n -> c, nn -> n, and the table entry of the tile after that.
        lid += wpx;
        tc = tn;
        xres_c = xres_n;
        wres_c = wres_n;
        has_n = has_nn;
        tn = tnn;
        xres_n = has_n ? xres_of(tn) : xnull;
        wres_n = has_n ? wres_of(tn) : wnull;
        if (GATHER) {
#pragma unroll
            for (int i = 0; i < AP; ++i) xv_c[i] = xv_n[i];
            if (has_n) token_offsets(tok, xv_n);
        }
        has_nn = lid + 2 * wpx < lid_end;
        if (has_nn) tnn = tile_of(lid + 2 * wpx, ent3);
        ent3 = tile_entry(lid + 3 * wpx);
        if (SCATTER) load_slots(tc);
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int i = 0; i < FB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;
        // Every wave has read its staged rows before the next tile's token
        // copies refill that slot.
        barrier_no_fence();
        static_for<2 * FB>([&](auto QC) {
            read_frag(std::integral_constant<int, 0>{}, QC, (uint32_t)as * SLAB, (uint32_t)ws * SLAB,
                      std::integral_constant<int, 0>{});
        });
    }
    wait_vmcnt<0>();
}

// fp32 layers: 64 x 64 tiles on v_mfma_f32_32x32x2_f32 (141 TFLOP/s sustained,
// twice the vector ALUs' rate; every product is added with one fused
// multiply-add, so the error is that of an fp32 fma chain).
//
// Four waves, 2 x 2, each 32 rows x 32 columns; the weights are the MFMA's
// rows, so a lane holds runs of four columns of one token row. 128-byte row
// pieces (32 columns) of both operands stream into a ring of three slabs (48
// KB: three workgroups per CU, whose MFMAs fill each other's barriers and
// epilogues), chunks swizzled by row. A lane reads 16-byte chunk 2 c + lane / 32 of its
// row for the four MFMAs of 8 columns (which so take them in the order 0 4 1 5
// 2 6 3 7). Vector operations and fp32 MFMAs slow each other down (two between
// dependent MFMAs: 64 -> 84 cycles each), so the loop has none: the read
// addresses are constants per lane and the slots compile-time offsets.
//
// Measured on ViT-B widths, 2304 tokens (64 experts, 288 rows each; 64 x 64
// VALU tiles before): grouped fc1 242 -> 122 us (90 TFLOP/s, 100 with the pad
// rows), fc2 222 -> 116 us, shared layers 72 -> 34 us each (432 workgroups for
// 256 CUs); 64 x 128 tiles take 122, 124 and 35 us and double the tiny layer's.
template <int EPI, bool GROUPED>
__global__ __launch_bounds__(256) void k_gemm_f32(const GemmArgs a) {
    constexpr int BM = 64, BN = 64, ST = 3, ROWB = 128;
    constexpr int SLAB = (BM + BN) * ROWB;
    constexpr int P = (BM + BN) / 8 / 4;  // 1 KB copy pieces (8 rows) per wave and slab
    constexpr bool GATHER = EPI == EPI_GELU_STORE && GROUPED;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[ST * SLAB];
    const TileCoord tc = locate_tile<GROUPED>(a, BM, BN);
    if (!tc.valid) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t rowb = (uint32_t)a.Kdim * 4u;
    const __amdgpu_buffer_rsrc_t xres = make_rsrc(a.A, a.a_bytes);
    const __amdgpu_buffer_rsrc_t wres =
        make_rsrc(static_cast<const float*>(a.B) + (size_t)tc.e * a.b_group_stride, (uint32_t)a.N * rowb);
    uint32_t off[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int r = (wave + 4 * i) * 8 + lane / 8;
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        uint32_t row;
        if (r < BM) {  // pad rows repeat the last valid row
            const int p = tc.row0 + min(r, tc.rows - 1);
            row = GATHER && a.row_mode == ROWS_GATHER_TOKENS ? (uint32_t)(a.row_map[p] / a.route_k) : (uint32_t)p;
        } else {
            row = (uint32_t)(tc.n0 + r - BM);
        }
        off[i] = row * rowb + c * 16;
    }
    auto issue = [&](int slot, int kt) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const bool tok = (wave + 4 * i) * 8 < BM;  // uniform per wave
            copy16_to_lds(tok ? xres : wres, off[i], (uint32_t)kt * ROWB, smem + slot * SLAB + (wave + 4 * i) * 1024);
        }
    };
    const int fr = lane & 31, q = lane >> 5;
    uint32_t xa[4], wa[4];  // this lane's chunk of column group c
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t o = lds_address(smem) + (uint32_t)(fr * ROWB) + (uint32_t)(((2 * c + q) ^ ((fr >> 1) & 7)) << 4);
        xa[c] = o + (uint32_t)(wm * 32 * ROWB);
        wa[c] = o + (uint32_t)((BM + wn * 32) * ROWB);
    }
    bf16x8_t xf[4], wf[4];  // 16 bytes each: four fp32 values
    auto read_group = [&](auto SC, auto CC) {
        constexpr int S = decltype(SC)::value, c = decltype(CC)::value;
        xf[c] = lds_read16<S * SLAB>(xa[c]);
        wf[c] = lds_read16<S * SLAB>(wa[c]);
    };
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    // The MFMAs of column groups 2 h and 2 h + 1, whose fragments are awaited
    // here; the fragments of the other two groups (slab slot RS) are read
    // between them.
    auto mul_half = [&](auto HC, auto RSC) {
        constexpr int h = decltype(HC)::value;
        wait_lgkmcnt0();
#pragma unroll
        for (int c = 2 * h; c < 2 * h + 2; ++c) {
            tie(xf[c]);
            tie(wf[c]);
        }
        static_for<2>([&](auto CC) {
            constexpr int c = 2 * h + decltype(CC)::value;
            const u32x4_t xv = __builtin_bit_cast(u32x4_t, xf[c]), wv = __builtin_bit_cast(u32x4_t, wf[c]);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(wv[m]), __uint_as_float(xv[m]), acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (m == 0) {
                    read_group(RSC, std::integral_constant<int, (c + 2) % 4>{});
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        });
    };
    const int nk = a.Kdim / 32;
    // Slab kt's copies have landed for this wave; `ahead` younger slabs in flight.
    auto wait_slab = [&](int ahead) {
        static_for<ST - 1>([&](auto AC) {
            constexpr int A = decltype(AC)::value;
            if (ahead == A) wait_vmcnt<A * P>();
        });
    };
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
        if (s < nk) issue(s, s);
    wait_slab(min(nk, ST - 1) - 1);
    barrier_no_fence();
    static_for<2>([&](auto CC) { read_group(std::integral_constant<int, 0>{}, CC); });
    // Slab kt in slot S; returns whether it was the last.
    int kt = 0;
    auto step = [&](auto SC) {
        constexpr int S = decltype(SC)::value, N = (S + 1) % ST;
        // Slab kt + ST - 1 goes to the slot of slab kt - 1, which every wave
        // finished reading before the last barrier.
        if (kt + ST - 1 < nk) issue((S + ST - 1) % ST, kt + ST - 1);
        mul_half(std::integral_constant<int, 0>{}, SC);
        // Group 2 and 3's fragments are awaited before the barrier: past it
        // this slot may be refilled.
        wait_lgkmcnt0();
        if (++kt < nk) {
            wait_slab(min(nk - 1, kt + ST - 2) - kt);
            barrier_no_fence();
        }
        // The last slab reads the next slot's old bytes, which nothing uses.
        mul_half(std::integral_constant<int, 1>{}, std::integral_constant<int, N>{});
        return kt == nk;
    };
    for (;;) {
        if (step(std::integral_constant<int, 0>{})) break;
        if (step(std::integral_constant<int, 1>{})) break;
        if (step(std::integral_constant<int, 2>{})) break;
    }
    wait_lgkmcnt0();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        tie(xf[c]);
        tie(wf[c]);
    }
    const int r = wm * 32 + fr;
    if (r >= tc.rows) return;
    const size_t orow = EPI == EPI_SCATTER_SLOT ? (size_t)a.row_map[tc.row0 + r] : (size_t)(tc.row0 + r);
    float* const out = static_cast<float*>(a.C) + orow * a.N + tc.n0 + wn * 32 + 4 * q;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = acc[4 * g + u];
            if (EPI == EPI_GELU_STORE) v[u] = gelu_erf(v[u]);
        }
        *reinterpret_cast<float4*>(out + 8 * g) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

template <int BM, int BN, int WM, int WN, int BK, int ST, int WPE, int EPI, bool GROUPED>
hipError_t launch_bf16(const GemmArgs& a, hipStream_t s) {
    const int n_n = a.N / BN;
    const long long total = (long long)a.max_tiles * n_n;
    const long long grid = (total + kNumXcd - 1) / kNumXcd * kNumXcd;
    // Split K (dense fp32 output only): the parts along the grid's y.
    const int splits = (!GROUPED && EPI == EPI_STORE_F32 && a.k_splits > 1) ? a.k_splits : 1;
    if (splits > 1 && (a.Kdim / BK) % splits) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_bf16<BM, BN, WM, WN, BK, ST, EPI, GROUPED, WPE>), dim3((unsigned)grid, splits),
                       dim3(WM * WN * kWave), 0, s, a);
    return hipGetLastError();
}

template <int EPI, bool GROUPED, int KC = 8>
hipError_t launch_pp(const GemmArgs& a, hipStream_t s) {
    const int grid = persistent_grid((long long)a.max_tiles * (a.N / 256));
    hipLaunchKernelGGL((k_gemm_pp<EPI, GROUPED, KC>), dim3((unsigned)grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

// The fused combine is compiled for each K (its gate and expert-row loads are
// unrolled over the K slots).
hipError_t launch_pp_combine(const GemmArgs& a, hipStream_t s) {
    switch (a.route_k) {
        case 1: return launch_pp<EPI_COMBINE, false, 1>(a, s);
        case 2: return launch_pp<EPI_COMBINE, false, 2>(a, s);
        case 3: return launch_pp<EPI_COMBINE, false, 3>(a, s);
        case 4: return launch_pp<EPI_COMBINE, false, 4>(a, s);
        case 5: return launch_pp<EPI_COMBINE, false, 5>(a, s);
        case 6: return launch_pp<EPI_COMBINE, false, 6>(a, s);
        case 7: return launch_pp<EPI_COMBINE, false, 7>(a, s);
        case 8: return launch_pp<EPI_COMBINE, false, 8>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int EPI, bool GROUPED>
hipError_t launch_sp(const GemmArgs& a, hipStream_t s) {
    const int n_n = a.N / 256;
    const long long total = (long long)a.max_tiles * n_n;
    const long long grid = (total + kNumXcd - 1) / kNumXcd * kNumXcd;
    hipLaunchKernelGGL((k_gemm_sp<EPI, GROUPED>), dim3((unsigned)grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int EPI, bool GROUPED>
hipError_t launch_f32(const GemmArgs& a, hipStream_t s) {
    const long long total = (long long)a.max_tiles * (a.N / 64);
    const long long grid = (total + kNumXcd - 1) / kNumXcd * kNumXcd;
    hipLaunchKernelGGL((k_gemm_f32<EPI, GROUPED>), dim3((unsigned)grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Small launches, where every 64 x 64 tile is resident at once and a workgroup's
// chain of K slabs, a memory latency apart, is the time: 64 x 64 tiles (more
// workgroups) with a ring as deep as the residency allows, five slabs at one
// workgroup per CU, four at two. 0 for larger launches. ViT-L widths, 5 tokens:
// routed first layer 11.8 -> 9.8 us, shared layers 10.8 -> 8.8 and 9.9 -> 8.2 us
// against 64 x 128 tiles with three slabs; the layer 61.0 -> 56.6 us.
int small_ring(const GemmArgs& a) {
    const long long wgs = (long long)a.max_tiles * (a.N / 64), cus = persistent_grid(1 << 20);
    if (a.k_splits > 1 || wgs > 2 * cus) return 0;
    return wgs <= cus ? 5 : 4;
}
template <int EPI, bool GROUPED>
hipError_t launch_64(const GemmArgs& a, hipStream_t s) {
    const int ring = small_ring(a);
    if (ring == 5) return launch_bf16<64, 64, 2, 2, 64, 5, 1, EPI, GROUPED>(a, s);
    if (ring == 4) return launch_bf16<64, 64, 2, 2, 64, 4, 2, EPI, GROUPED>(a, s);
    if (a.N % 128 == 0) return launch_bf16<64, 128, 1, 4, 64, 3, 2, EPI, GROUPED>(a, s);
    return launch_bf16<64, 64, 2, 2, 64, 3, 2, EPI, GROUPED>(a, s);
}

// 128-row tiles: 128 x 128 (four waves of 64 x 64, two slabs in the ring, two
// workgroups per CU) or 128 x 64.
template <int EPI, bool GROUPED>
hipError_t launch_128(const GemmArgs& a, hipStream_t s) {
    if (a.N % 128 == 0) return launch_bf16<128, 128, 2, 2, 64, 2, 2, EPI, GROUPED>(a, s);
    return launch_bf16<128, 64, 2, 2, 64, 3, 2, EPI, GROUPED>(a, s);
}

// Tile shapes. Large groups (M-tiles of 256 token rows): 256 x 256 on the
// persistent kernel when N allows and K spans at least two slabs (the paced
// one-tile kernel for one slab), else 256 x 128 or 256 x 64 tiled. Between
// (gemm_tile_bm, gemm_dense_bm) 128 x 128 or 128 x 64. Small
// groups (M-tiles of 64 rows, the weight-read-bound regime where an expert
// sees a few dozen tokens): 64 x 128 or 64 x 64 with three slabs in the ring
// and several workgroups per CU, to keep many weight loads in flight.
template <int EPI, bool GROUPED>
hipError_t dispatch_bf16(int bm, const GemmArgs& a, hipStream_t s) {
    if (bm == 256) {
        if (a.N % 256 == 0) {
            const bool gather_ok = !(GROUPED && EPI == EPI_GELU_STORE) || a.row_mode == ROWS_GATHER_TOKENS;
            if (a.Kdim >= 128 && gather_ok) return launch_pp<EPI, GROUPED>(a, s);
            return launch_sp<EPI, GROUPED>(a, s);
        }
        // The grouped layers with N an odd multiple of 128 (ViT-B's h = 384):
        // N rounded up to the persistent kernel's 256-column tile, weight rows
        // past N read as zeros and columns past N not stored. A third more
        // MFMA work than the 256 x 128 tiles, but on the persistent kernel.
        if constexpr (GROUPED && (EPI == EPI_GELU_STORE || EPI == EPI_SCATTER_SLOT))
            if (a.N % 128 == 0 && a.Kdim >= 128 &&
                (EPI == EPI_SCATTER_SLOT || a.row_mode == ROWS_GATHER_TOKENS)) {
                GemmArgs p = a;
                p.b_rows = a.N;
                p.ldc = a.N;
                p.N = (a.N + 255) / 256 * 256;
                return launch_pp<EPI, GROUPED>(p, s);
            }
        if (a.N % 128 == 0) return launch_bf16<256, 128, 2, 2, 64, 2, 1, EPI, GROUPED>(a, s);
        return launch_bf16<256, 64, 4, 1, 64, 2, 1, EPI, GROUPED>(a, s);
    }
    if (bm == 128) return launch_128<EPI, GROUPED>(a, s);
    if (bm == 64) return launch_64<EPI, GROUPED>(a, s);
    return hipErrorInvalidValue;
}

// Whether a backward product runs on the persistent kernel: SwiGLU dA at any
// width, as the recompute before it; the others at multiples of its 256-column
// tile, and at widths that it pads by at most a third where it still gains over
// the 256 x 128 and 256 x 64 tiles: launches of 700 tiles (nearly three passes
// over the CUs) or more, or, with contractions of 384 and up, passes whose tiles
// hold 0.65 of all CUs' columns in real work (0.55 against the slower 256 x 64
// tiles, at odd multiples of 64). Whole backward over 282 shapes, persistent
// against tiled: from 700 tiles 1.00 to 1.62 times as fast at every width (192 to
// 1216); with fewer, above the lines 0.97 to 1.28, below them 0.63 at the least
// (4 experts of 600 rows).
bool gemm_backward_pp(int bm, int epilogue, const GemmArgs& a) {
    if (bm != 256 || a.Kdim < 128) return false;
    const int cols = (a.N + 255) / 256;
    if (epilogue == EPI_DSWIGLU || a.N % 256 == 0) return true;
    if (cols * 256 * 3 > a.N * 4) return false;
    const long long tiles = (long long)a.mean_tiles * cols, passes = (tiles + 255) / 256;
    const double fill = (double)a.mean_tiles * a.N / (256.0 * 256 * passes);
    return tiles >= 700 || (a.Kdim >= 384 && fill >= (a.N % 128 == 0 ? 0.65 : 0.55));
}

// Backward products: the persistent kernel where gemm_backward_pp says so, N
// rounded up to the tile (weights past N read as zeros or as other weights and
// feed columns that are not stored), else the tiled kernel with 256-, 128- or
// 64-row tiles.
template <int EPI, bool GROUPED>
hipError_t dispatch_tiled(int bm, const GemmArgs& a, hipStream_t s) {
    if (gemm_backward_pp(bm, EPI, a)) {
        GemmArgs p = a;
        p.b_rows = a.N;
        p.ldc = a.N;
        p.N = (a.N + 255) / 256 * 256;
        return launch_pp<EPI, GROUPED>(p, s);
    }
    if (bm == 256) {
        if (a.N % 128 == 0) return launch_bf16<256, 128, 2, 2, 64, 2, 1, EPI, GROUPED>(a, s);
        return launch_bf16<256, 64, 4, 1, 64, 2, 1, EPI, GROUPED>(a, s);
    }
    if (bm == 128) return launch_128<EPI, GROUPED>(a, s);
    if (bm == 64) {
        if (a.N % 128 == 0) return launch_bf16<64, 128, 1, 4, 64, 3, 2, EPI, GROUPED>(a, s);
        return launch_bf16<64, 64, 2, 2, 64, 3, 2, EPI, GROUPED>(a, s);
    }
    return hipErrorInvalidValue;
}

// SwiGLU first layer: the virtual column count N follows from the tile shape
// (each tile of BN columns computes BN / 2 activation columns).
template <bool GROUPED>
hipError_t dispatch_swiglu(int bm, GemmArgs a, hipStream_t s) {
    if (a.act_n < 1 || a.act_ld < a.act_n || a.act_ld % 64) return hipErrorInvalidValue;
    if (bm == 256) {
        if (a.Kdim < 128 || (GROUPED && a.row_mode != ROWS_GATHER_TOKENS)) return hipErrorInvalidValue;
        a.N = 2 * ((a.act_ld + 127) / 128 * 128);
        return launch_pp<EPI_SWIGLU_STORE, GROUPED>(a, s);
    }
    if (bm == 128) {
        a.N = 2 * a.act_ld;
        return launch_bf16<128, 128, 2, 2, 64, 2, 2, EPI_SWIGLU_STORE, GROUPED>(a, s);
    }
    if (bm == 64) {
        a.N = 2 * a.act_ld;
        if ((long long)a.max_tiles * (a.N / 128) <= persistent_grid(1 << 20))  // as small_ring, one workgroup per CU
            return launch_bf16<64, 128, 2, 2, 64, 5, 1, EPI_SWIGLU_STORE, GROUPED>(a, s);
        return launch_bf16<64, 128, 2, 2, 64, 3, 2, EPI_SWIGLU_STORE, GROUPED>(a, s);
    }
    return hipErrorInvalidValue;
}

// Backward's first-layer recompute for SwiGLU experts: the persistent kernel
// (as the forward), else the tiled kernel with 2 x 2 waves (each wave 32 gate
// + 32 up columns), N = 2 act_ld.
hipError_t dispatch_swiglu_bwd(int bm, GemmArgs a, hipStream_t s) {
    if (a.act_n < 1 || a.act_ld < a.act_n || a.act_ld % 64) return hipErrorInvalidValue;
    if (bm == 256 && a.Kdim >= 128) {
        a.N = 2 * ((a.act_ld + 127) / 128 * 128);
        return launch_pp<EPI_SWIGLU_BWD, true>(a, s);
    }
    a.N = 2 * a.act_ld;
    if (bm == 256) return launch_bf16<256, 128, 2, 2, 64, 2, 1, EPI_SWIGLU_BWD, true>(a, s);
    if (bm == 128) return launch_bf16<128, 128, 2, 2, 64, 2, 2, EPI_SWIGLU_BWD, true>(a, s);
    if (bm == 64) return launch_bf16<64, 128, 2, 2, 64, 3, 2, EPI_SWIGLU_BWD, true>(a, s);
    return hipErrorInvalidValue;
}

template <bool GROUPED>
hipError_t dispatch(const moe_desc_t& d, int epilogue, int bm, const GemmArgs& a, hipStream_t s) {
    if (d.dtype == MOE_BF16) {
        switch (epilogue) {
            case EPI_GELU_STORE: return dispatch_bf16<EPI_GELU_STORE, GROUPED>(bm, a, s);
            case EPI_SWIGLU_STORE: return dispatch_swiglu<GROUPED>(bm, a, s);
            case EPI_GELU_BWD:
                if (GROUPED) return dispatch_tiled<EPI_GELU_BWD, true>(bm, a, s);
                break;
            case EPI_DGELU:
                if (GROUPED) return dispatch_tiled<EPI_DGELU, true>(bm, a, s);
                break;
            case EPI_SCATTER_SLOT_F32:
                if (GROUPED) return dispatch_tiled<EPI_SCATTER_SLOT_F32, true>(bm, a, s);
                break;
            case EPI_SWIGLU_BWD:
                if (GROUPED) return dispatch_swiglu_bwd(bm, a, s);
                break;
            case EPI_DSWIGLU:
                if (GROUPED) return dispatch_tiled<EPI_DSWIGLU, true>(bm, a, s);
                break;
            case EPI_SCATTER_SLOT:
                if (GROUPED) return dispatch_bf16<EPI_SCATTER_SLOT, true>(bm, a, s);
                break;
            case EPI_STORE_F32:
                if (!GROUPED) return dispatch_bf16<EPI_STORE_F32, false>(bm, a, s);
                break;
            case EPI_ROUTER_F32:
                if (!GROUPED && bm == 256 && a.N % 256 == 0 && a.Kdim >= 128 && a.k_splits <= 1 && a.C2)
                    return launch_pp<EPI_ROUTER_F32, false>(a, s);
                break;
            case EPI_COMBINE:
                if (!GROUPED && gemm_combine_fusable(d, bm, a.N, a.Kdim) && a.route_k == d.K)
                {
                    if (bm == 256) return launch_pp_combine(a, s);
                    if (bm == 128) return launch_128<EPI_COMBINE, false>(a, s);
                    return launch_64<EPI_COMBINE, false>(a, s);
                }
                break;
        }
    } else {
        if (bm != 64) return hipErrorInvalidValue;
        switch (epilogue) {
            case EPI_GELU_STORE: return launch_f32<EPI_GELU_STORE, GROUPED>(a, s);
            case EPI_SCATTER_SLOT:
                if (GROUPED) return launch_f32<EPI_SCATTER_SLOT, true>(a, s);
                break;
            case EPI_STORE_F32:
                if (!GROUPED) return launch_f32<EPI_STORE_F32, false>(a, s);
                break;
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

// What the persistent kernel's 256 x 256 tiles would do for the two grouped
// layers on 256 CUs, for loads known by their mean alone: `share`, the part of
// the time spent on real rows and columns, where a pass over the CUs costs its
// slabs and about nine more (pipeline fill and epilogue) whether every CU has a
// tile or not, and `tiles` of the narrower layer. M-tiles: half a ragged tile per
// expert and a standard deviation of it, or, for loads close to the mean, those
// of experts with Poisson counts.
struct Fill256 {
    double share, tiles;
};
static Fill256 fill256(const moe_desc_t& d) {
    constexpr int kCus = 256, kTail = 9;
    const bool swiglu = d.flags & MOE_FLAG_SWIGLU;
    const int hh = act_stride(d, d.h);
    const double slots = (double)d.T * d.K, rows = slots / d.E, full = slots / 256;
    auto above = [&](int n) { return 0.5 * std::erfc((n - rows) / std::sqrt(2 * rows)); };  // P(count > n)
    const double tiles = std::max(full + 0.5 * (d.E + std::sqrt((double)d.E)), d.E * (1 + above(256) + above(512)));
    double work = 0, time = 0;
    auto layer = [&](int n, int cols, int k) {
        work += full * n / 256 * (k / 64);
        time += std::ceil(tiles * cols / kCus) * kCus * (k / 64 + kTail);
    };
    layer(swiglu ? 2 * hh : hh, swiglu ? (hh + 127) / 128 : (hh + 255) / 256, d.d);
    layer(d.d, (d.d + 255) / 256, hh);
    return {work / time, tiles * ((std::min(d.d, hh) + 255) / 256)};
}

// The least share with which the 256-row tiles are taken, by what else makes
// them slower than 64-row tiles: few tiles (a pass that some XCD or expert
// overfills weighs more), narrow layers (short contractions beside the
// epilogue) and the backward's longer epilogues. Each line lies where, of 1800
// forward pairs and 1630 backward calls of 4 to 256 experts, 128 to 511 rows,
// widths 256 to 1536, balanced and skewed, none (backward: next to none) above it
// was slower than with 64-row tiles: forward 0.99 to 1.50 times as fast above the
// lines (1.07 over all shapes, 1.09 with the better of the two everywhere) and
// 0.73 at the least below them, backward 0.94 to 1.24 (1.03 over all) and 0.70.
static double least_share(double tiles, int width, bool swiglu, bool backward) {
    if (backward) {
        if (tiles >= 640) return width >= 700 ? (swiglu ? 0.28 : 0.25) : (swiglu ? 0.30 : 0.26);
        return tiles >= 400 ? 0.295 : (tiles >= 200 ? 0.32 : 1.0);
    }
    if (tiles >= 640) return width >= 700 ? 0.18 : (width >= 512 ? 0.28 : 0.31);
    if (tiles >= 400) return width >= 700 ? 0.26 : (width >= 512 ? 0.29 : 0.31);
    if (tiles >= 200 && swiglu && width >= 700) return 0.28;
    return tiles >= 170 ? 0.30 : 0.32;
}

int gemm_tile_bm(const moe_desc_t& d, int64_t avg_rows, bool backward) {
    if (d.dtype != MOE_BF16) return 64;
    if (avg_rows >= 512) return 256;
    const bool swiglu = d.flags & MOE_FLAG_SWIGLU;
    const int hh = act_stride(d, d.h), width = hh < d.d ? hh : d.d;
    // With fewer rows the 256-row tiles (widths the persistent kernel takes, from
    // 128 rows) only where they fill enough of the chip, whatever the loads: a
    // few experts or narrow layers leave most CUs without a tile, and ragged or
    // skewed loads pad (8 experts, d = h = 768, 130 rows: 64-row tiles 17 us for
    // the two products, 256-row tiles 46; 128 experts, d = h = 512, 130 rows,
    // skewed: 54 and 76). ViT-H, 260 rows (share 0.32): 166 and 155 us a layer;
    // ViT-L, 448 rows (0.35): 335 and 311; ViT-G, 160 rows (0.32): 609 and 556.
    if (d.d % 128 == 0 && (swiglu || d.h % 128 == 0) && avg_rows >= 128) {
        const Fill256 f = fill256(d);
        if (f.share >= least_share(f.tiles, width, swiglu, backward)) return 256;
    }
    // 128-row tiles from 192 rows where those fill the CUs' two places about
    // twice (896 tiles in the narrower layer) and no layer is only 256 columns
    // wide (200 experts, d = h = 256, 330 rows: 64-row tiles 55 us, 128-row tiles
    // 57). ViT-L, 64- and 128-row tiles: 131 rows 158 and 163, 200 rows (800
    // tiles) 188 and 190, 250 rows (1000) 212 and 201.
    const int64_t tiles = (int64_t)d.T * d.K / 128 * (width / 128);
    return avg_rows >= 192 && width >= 320 && tiles >= 896 ? 128 : 64;
}

int gemm_dense_bm(const moe_desc_t& d) {
    if (d.dtype != MOE_BF16) return 64;
    const int ldh = act_stride(d, d.h_shared), n = ldh < d.d ? ldh : d.d, wide = ldh < d.d ? d.d : ldh;
    // 256-row tiles only when they still give a few workgroups per CU.
    const int64_t tiles = ((int64_t)d.T + 255) / 256 * (n / 256 > 0 ? n / 256 : 1);
    if (tiles >= 512) return 256;
    // 128-row tiles where those of the narrower layer give most CUs two
    // workgroups, but not up to 128 tiles past the 512 places, where a second
    // pass is nearly empty (GELU layers of like widths; SwiGLU's longer first
    // layer hides it), and not for layers under 384 columns. Shared layers, 64-
    // against 128-row tiles, 384 to 510 tiles 1.04 to 1.13, 513 to 640 0.82 to
    // 0.98 (SwiGLU 0.99 to 1.12), more 0.99 to 1.15; widths 256 and 320 0.94 to 1.03.
    const int64_t half = ((int64_t)d.T + 127) / 128 * (n / 128);
    const bool spill = half > 512 && half <= 640 && !(d.flags & MOE_FLAG_SWIGLU) && wide < 3 * n;
    return n >= 384 && half >= 384 && !spill ? 128 : 64;
}

bool gemm_combine_fusable(const moe_desc_t& d, int bm, int n, int kdim) {
    // The persistent 256 x 256 kernel with its combine epilogue, or the tiled
    // kernel's 128- or 64-row tiles with theirs (K <= 8 either way).
    if (d.dtype != MOE_BF16 || d.K > kMaxCombineK) return false;
    return (bm == 256 && n % 256 == 0 && kdim >= 128) || (bm <= 128 && n % 64 == 0);
}

hipError_t launch_gemm(const moe_desc_t& d, int epilogue, int bm, const GemmArgs& a, hipStream_t s) {
    // Grouped (routed experts, tile table) and dense (shared expert) launches
    // are separate kernel instances.
    if (a.tiles) return dispatch<true>(d, epilogue, bm, a, s);
    return dispatch<false>(d, epilogue, bm, a, s);
}

}  // namespace moe
