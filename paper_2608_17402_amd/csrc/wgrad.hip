// Weight gradients of the expert-MLP backward: dW[e] = sum over the rows p of
// expert e of A[p, :]^T B[p, :] (fp32), straight from the row-major tensors.
// One operand is in sorted order (the activation, or dH), the other is
// gathered (output gradients by slot, or x by token).
//
// MFMA fragments of both operands run along the contraction, which is the row
// index here, so the K slabs (64 rows x 256 columns) are read from LDS with
// CDNA4's transposing 8-byte reads (ds_read_b64_tr_b16): two of them give a
// lane the 8 rows of its column. No transposed copy of any tensor is made.
#include "gemm_device.h"
#include "moe_internal.h"

namespace moe {
namespace {

// Persistent 256 x 256 tiles, as k_gemm_pp: four waves of 128 x 128, a ring of
// three slabs for A and of two for B (160 KB), copies paced against the MFMAs,
// the slab pipeline running on across tiles. TS = 128: tiles of 128 x 128, waves
// of 64 x 64, 80 KB and so two workgroups per CU, for launches that have few
// tiles or widths that 256-column tiles pad badly.
//
// LDS layout of a slab: 64 rows of 2 TS bytes, the 16-byte chunk c of row r at
// chunk c ^ ((r & 3) << 2). A transposing read of half a wave touches 4
// consecutive rows x 32 columns: 16 chunks, all in distinct banks. A 1 KB copy
// moves RP = 2 (4) rows; LDS row 16 w + RP p + b (wave w, piece p of NP = 8 (4),
// b = lane * RP / 64) holds position 16 w + NP b + p of the slab, so that a lane's
// NP gathered rows are consecutive table entries (16 or 8 bytes per half slab).
// The order of the positions inside a K step is the same for both operands and
// changes nothing.
//
// Gathered rows come from a table of byte offsets per window position; the
// padding positions hold kWgradNoRow, past every buffer's end, and read as
// zeros. The sorted operand's buffer resource ends with the item's last row,
// so its padding rows read as zeros too. Widths need not be multiples of 256:
// columns past the width read other finite or non-finite data of the tensor
// (or zeros past its end), which reaches only outputs that are not stored.
//
// Bound by the MFMAs and the slab copies together, as k_gemm_pp; against slab-major
// transposed operands (gathered and transposed by kernels of their own, or written
// twice by the epilogues before) a K step issues 16 8-byte fragment
// reads instead of 8 16-byte ones (the same LDS bytes), and about 7 GB of copies
// per ViT-G call are gone. Whole backward: ViT-G widths, 65536 tokens skewed
// 9.23 -> 7.82 ms; H layer (SwiGLU), 4100 tokens 1111 -> 913 us; ViT-B training
// step, 18432 tokens 1739 -> 1477 us.
//
// GA: A is the gathered operand (dW2 = Gout^T act), else B (dW1 = dH^T x).
template <bool GA, int TS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TS == 256 ? 1 : 2, TS == 256 ? 1 : 2)))
void k_wgrad(const WgradArgs a) {
    static_assert(TS == 256 || TS == 128, "four waves of 128 x 128 or 64 x 64");
    constexpr int BM = TS, BN = TS, WT = TS / 2, FB = WT / 32;
    constexpr int BK = 64, ROWB = TS * 2;
    constexpr int SLAB = BK * ROWB;  // 32 (16) KB per operand and slab
    constexpr int AST = 3, WST = 2;  // ring depths
    constexpr int WBASE = AST * SLAB;
    constexpr int STG_WAVE = SLAB / 4;  // epilogue staging bytes per wave
    constexpr int NP = SLAB / 4096;     // 1 KB copies per wave, operand and slab
    constexpr int RP = 16 / NP;         // LDS rows per copy
    constexpr int LPR = kWave / RP;     // lanes (16-byte chunks) per row
    __shared__ __attribute__((aligned(1024))) uint8_t smem[AST * SLAB + WST * SLAB];

    const int n_n = (a.N + BN - 1) / BN;
    const int m_per = (a.M + BM - 1) / BM;
    const int total = __builtin_amdgcn_readfirstlane(*a.n_items) * m_per * n_n;
    const int per = (total + kNumXcd - 1) / kNumXcd;
    const int xcd = blockIdx.x % kNumXcd;
    const int wpx = gridDim.x / kNumXcd;  // workgroups per XCD: the tile stride
    const int lid_end = min(total, (xcd + 1) * per);
    int lid = xcd * per + (int)blockIdx.x / kNumXcd;
    if (lid >= lid_end) return;

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wm = wave >> 1, wn = wave & 1;
    const uint32_t arow = (uint32_t)a.M * 2, brow = (uint32_t)a.N * 2;  // row bytes

    struct Tile {
        int e, dest, m0, n0;
        int q0, nk;      // first window position, K slabs
        int row0, rows;  // first sorted row, rows that exist
    };
    // Item of tile l; indices past this workgroup's share read its last tile.
    auto tile_entry = [&](int l) { return a.items[min(l, lid_end - 1) / n_n / m_per]; };
    auto tile_of = [&](int l, const WgradItem& d) {
        Tile t;
        const int mt = l / n_n;
        t.n0 = (l - mt * n_n) * BN;
        t.m0 = (mt - (mt / m_per) * m_per) * BM;
        t.e = __builtin_amdgcn_readfirstlane(d.e);
        t.dest = __builtin_amdgcn_readfirstlane(d.dest);
        t.q0 = __builtin_amdgcn_readfirstlane(d.q0);
        t.nk = __builtin_amdgcn_readfirstlane(d.klen) / BK;
        t.row0 = __builtin_amdgcn_readfirstlane(d.row0);
        t.rows = __builtin_amdgcn_readfirstlane(d.rows);
        return t;
    };
    auto tile_at = [&](int l) { return tile_of(l, tile_entry(l)); };
    const bf16_t* const Ap = static_cast<const bf16_t*>(a.A);
    const bf16_t* const Bp = static_cast<const bf16_t*>(a.B);
    auto sorted_res = [&](const bf16_t* p, const Tile& t, int cols, int c0) {
        const uint32_t bytes = t.rows > 0 ? (uint32_t)t.rows * (uint32_t)cols * 2u - (uint32_t)c0 * 2u : 0u;
        return make_rsrc(p + (size_t)t.row0 * cols + c0, bytes);
    };
    auto ares_of = [&](const Tile& t) {
        return GA ? make_rsrc(Ap + t.m0, a.gather_bytes - (uint32_t)t.m0 * 2u) : sorted_res(Ap, t, a.M, t.m0);
    };
    auto bres_of = [&](const Tile& t) {
        return GA ? sorted_res(Bp, t, a.N, t.n0) : make_rsrc(Bp + t.n0, a.gather_bytes - (uint32_t)t.n0 * 2u);
    };
    const __amdgpu_buffer_rsrc_t anull = make_rsrc(Ap, 0);
    const __amdgpu_buffer_rsrc_t bnull = make_rsrc(Bp, 0);

    // This lane's pieces: source position lpos + p, source chunk by the parity
    // of p (LDS row 16 w + 2 p + hb).
    const int hb = lane / LPR;
    const uint32_t lpos = 16 * wave + NP * hb;
    const uint32_t cofs[2] = {(uint32_t)(lane % LPR ^ (hb << 2)) * 16u, (uint32_t)(lane % LPR ^ ((RP + hb) % 4 << 2)) * 16u};
    const uint32_t srow = GA ? brow : arow;  // row bytes of the sorted operand
    const uint32_t sbase[2] = {lpos * srow + cofs[0], lpos * srow + cofs[1]};
    typedef uint32_t half_t __attribute__((ext_vector_type(NP / 2)));
    half_t glo, ghi;  // byte offsets of the first and second half of the next gathered slab's pieces

    Tile tc = tile_at(lid);
    bool has_n = lid + wpx < lid_end;
    Tile tn = has_n ? tile_at(lid + wpx) : tc;
    bool has_nn = lid + 2 * wpx < lid_end;
    Tile tnn = has_nn ? tile_at(lid + 2 * wpx) : tn;
    WgradItem ent3 = tile_entry(lid + 3 * wpx);
    __amdgpu_buffer_rsrc_t ares_c = ares_of(tc), bres_c = bres_of(tc);
    __amdgpu_buffer_rsrc_t ares_n = has_n ? ares_of(tn) : anull;
    __amdgpu_buffer_rsrc_t bres_n = has_n ? bres_of(tn) : bnull;

    // Table entries of slab s, counted from the current tile's first slab and
    // running on into the next two tiles (s <= nk + 2, and a tile has at least
    // two slabs, so the tile after next is reached with its first slab only).
    auto table_at = [&](int s) {
        int q;
        if (s < tc.nk) q = tc.q0 + s * BK;
        else if (s - tc.nk < tn.nk) q = tn.q0 + (s - tc.nk) * BK;
        else q = tnn.q0;
        return reinterpret_cast<const half_t*>(a.tab + q + lpos);
    };

    f32x16_t acc[FB][FB];
#pragma unroll
    for (int j = 0; j < FB; ++j)
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;

    const int fr = lane & 31;
    const int fk = lane >> 5;
    const uint32_t base = lds_address(smem);
    // Read addresses of the four 32-column blocks: lane 16 g + r of a quarter
    // wave names row r / 4 and columns 4 (r % 4) .. of columns 16 (g % 2) ..;
    // K step ks and the row half are offsets.
    const int r4 = (lane & 15) >> 2;
    uint32_t xoff[FB], woff[FB];
#pragma unroll
    for (int i = 0; i < FB; ++i) {
        const uint32_t row = (uint32_t)(fk * 8 + r4) * ROWB + (uint32_t)(lane & 1) * 8u;
        const uint32_t c = (uint32_t)(2 * ((lane >> 4) & 1) + ((lane & 3) >> 1));
        xoff[i] = base + row + ((uint32_t)((wm * FB + i) ^ r4) * 4u + c) * 16u;
        woff[i] = base + WBASE + row + ((uint32_t)((wn * FB + i) ^ r4) * 4u + c) * 16u;
    }

    // Piece L of an operand's slab: gathered from the table word, sorted at row
    // lpos + L of slab s.
    auto word = [&](auto LC) -> uint32_t {
        constexpr int L = decltype(LC)::value;
        return L < NP / 2 ? glo[L % (NP / 2)] : ghi[L % (NP / 2)];
    };
    auto copy_a = [&](auto LC, int stage, int s, __amdgpu_buffer_rsrc_t r) {
        constexpr int L = decltype(LC)::value;
        const uint32_t v = GA ? word(LC) + cofs[L & 1] : sbase[L & 1] + (uint32_t)(s * BK + L) * srow;
        copy16_to_lds(r, v, 0, smem + stage * SLAB + (wave * NP + L) * 1024);
    };
    auto copy_b = [&](auto LC, int stage, int s, __amdgpu_buffer_rsrc_t r) {
        constexpr int L = decltype(LC)::value;
        const uint32_t v = GA ? sbase[L & 1] + (uint32_t)(s * BK + L) * srow : word(LC) + cofs[L & 1];
        copy16_to_lds(r, v, 0, smem + WBASE + stage * SLAB + (wave * NP + L) * 1024);
    };

    u32x2_t xf[2][FB][2], wf[2][FB][2];  // the two row halves of each fragment
    auto read_frag = [&](auto NBC, auto QC, auto KSC, uint32_t abase, uint32_t wbase) {
        constexpr int nb = decltype(NBC)::value, q = decltype(QC)::value, ks = decltype(KSC)::value;
        if constexpr (q < FB) {
            lds_read_tr8_asm<ks * 16 * ROWB>(xf[nb][q][0], xoff[q] + abase);
            lds_read_tr8_asm<ks * 16 * ROWB + 4 * ROWB>(xf[nb][q][1], xoff[q] + abase);
        } else {
            lds_read_tr8_asm<ks * 16 * ROWB>(wf[nb][q - FB][0], woff[q - FB] + wbase);
            lds_read_tr8_asm<ks * 16 * ROWB + 4 * ROWB>(wf[nb][q - FB][1], woff[q - FB] + wbase);
        }
    };
    auto settle = [&](auto CBC) {
        constexpr int cb = decltype(CBC)::value;
        wait_lgkmcnt0();
#pragma unroll
        for (int i = 0; i < FB; ++i) {
            tie(xf[cb][i][0]);
            tie(xf[cb][i][1]);
        }
#pragma unroll
        for (int j = 0; j < FB; ++j) {
            tie(wf[cb][j][0]);
            tie(wf[cb][j][1]);
        }
    };
    auto frag = [](const u32x2_t(&h)[2]) {
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3));
    };
    // One K step: 16 (4) MFMAs on buffer CB, fragment q of the next K step after
    // MFMA q (q < 8 or 4), copy q / 4 (q / 2) of the step's four (two) after MFMA q
    // when q % 4 (q % 2) == 1.
    constexpr int CE = FB * FB / (NP / 2);  // MFMAs per copy
    auto kstep = [&](auto CBC, auto KSC, uint32_t rabase, uint32_t rwbase, auto&& copy) {
        constexpr int cb = decltype(CBC)::value;
        static_for<FB * FB>([&](auto QC) {
            constexpr int q = decltype(QC)::value;
            constexpr int j = q / FB, i = q % FB;
            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(wf[cb][j]), frag(xf[cb][i]), acc[j][i], 0, 0, 0);
            if constexpr (q < 2 * FB) read_frag(std::integral_constant<int, cb ^ 1>{}, QC, KSC, rabase, rwbase);
            if constexpr (q % CE == 1) copy(std::integral_constant<int, q / CE>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    // Stores tile t, staged through A's ring slot `stslot` as k_gemm_pp does:
    // 32 rows x 64 (32) columns at a time, whole 256-byte (128-byte) row pieces
    // out. Stacked gate and up gradients (a.h > 0: M = 2 ld rows, gate row r at r,
    // up row r at ld + r) leave out the padding rows.
    const int Mout = a.h > 0 ? 2 * a.h : a.M;
    auto epilogue = [&](const Tile& t, int stslot) {
        constexpr int JB = TS == 256 ? 2 : 1;  // 32-column blocks per staged piece
        constexpr int SROW = JB * 128, SCH = SROW / 16;  // bytes and 16-byte chunks of a staged row
        constexpr int RPR = kWave / SCH, NR = 32 / RPR;  // rows per read, reads per piece
        const uint32_t stg = base + (uint32_t)stslot * SLAB + (uint32_t)wave * STG_WAVE;
        const uint32_t wrow = stg + (uint32_t)(fr * SROW);
        const int sw = fr & (SCH - 1);
        float* const ob = t.dest < 0 ? a.out + (size_t)t.e * Mout * a.N : a.partials + (size_t)t.dest * Mout * a.N;
#pragma unroll
        for (int i = 0; i < FB; ++i)
#pragma unroll
            for (int h = 0; h < FB / JB; ++h) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int j = JB * h + jj;
                        const u32x4_t v = {__float_as_uint(acc_read(acc[j][i][4 * g + 0])),
                                           __float_as_uint(acc_read(acc[j][i][4 * g + 1])),
                                           __float_as_uint(acc_read(acc[j][i][4 * g + 2])),
                                           __float_as_uint(acc_read(acc[j][i][4 * g + 3]))};
                        lds_write16_asm(wrow + ((uint32_t)((8 * jj + 2 * g + fk) ^ sw) << 4), v);
                    }
                u32x4_t v[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    const int rr = lane / SCH + RPR * k;
                    v[k] = lds_read16u_asm(stg + (uint32_t)(rr * SROW) + ((uint32_t)(lane % SCH ^ (rr & (SCH - 1))) << 4));
                }
                wait_lgkmcnt0();
#pragma unroll
                for (int k = 0; k < NR; ++k) tie(v[k]);
                const int col = t.n0 + wn * WT + h * JB * 32;  // N is a multiple of 64
#pragma unroll
                for (int k = 0; k < NR; ++k) {
                    int m = t.m0 + wm * WT + i * 32 + lane / SCH + RPR * k;
                    bool keep = m < a.M && col < a.N;
                    if (a.h > 0) {
                        const int ld = a.M / 2, up = m >= ld ? 1 : 0;
                        const int r = m - up * ld;
                        keep = keep && r < a.h;
                        m = r + up * a.h;
                    }
                    if (keep) store16_asm(ob + (size_t)m * a.N + col + lane % SCH * 4, v[k]);
                }
            }
    };

    // Prologue: A slab 0, B slab 0, A slab 1, the first half of B slab 1.
    using std::integral_constant;
    auto first = [&](auto&& get) {
        const half_t* const p = get;
        glo = p[0];
        ghi = p[1];
    };
    first(table_at(0));
    static_for<NP>([&](auto LC) { copy_a(LC, 0, 0, ares_c); });
    static_for<NP>([&](auto LC) { copy_b(LC, 0, 0, bres_c); });
    first(table_at(1));
    static_for<NP>([&](auto LC) { copy_a(LC, 1, 1, ares_c); });
    static_for<NP / 2>([&](auto LC) { copy_b(LC, 1, 1, bres_c); });
    // GA: the next copies of A are slab 2's. Else B's: the second half of slab
    // 1's pieces, then the first half of slab 2's.
    glo = table_at(2)[0];
    if (GA) ghi = table_at(2)[1];
    // vmcnt(0) the compiler sees: it would otherwise count the table loads as
    // fresh at the first pass and wait in every pass for copies not yet needed.
    __builtin_amdgcn_s_waitcnt(0xF70);
    wait_vmcnt<0>();
    barrier_no_fence();
    static_for<2 * FB>([&](auto QC) { read_frag(integral_constant<int, 0>{}, QC, integral_constant<int, 0>{}, 0u, 0u); });

    int as = 0, ws = 0;  // ring slots of the slab being multiplied
    for (;;) {
        int kt = 0;
        do {
            const uint32_t abase = (uint32_t)as * SLAB, wbase = (uint32_t)ws * SLAB;
            const int as1 = as == AST - 1 ? 0 : as + 1, as2 = as1 == AST - 1 ? 0 : as1 + 1;
            const int ws1 = ws ^ 1;
            // Slabs kt + 1 and kt + 2 may belong to the next tile.
            const int nkc = tc.nk;
            const bool n1 = kt + 1 >= nkc, n2 = kt + 2 >= nkc;
            const int s1 = n1 ? kt + 1 - nkc : kt + 1, s2 = n2 ? kt + 2 - nkc : kt + 2;
            const __amdgpu_buffer_rsrc_t br1 = n1 ? bres_n : bres_c;
            const __amdgpu_buffer_rsrc_t ar2 = n2 ? ares_n : ares_c;
            const __amdgpu_buffer_rsrc_t br2 = n2 ? bres_n : bres_c;
            // K step 0: second half of B slab kt + 1.
            settle(integral_constant<int, 0>{});
            kstep(integral_constant<int, 0>{}, integral_constant<int, 1>{}, abase, wbase,
                  [&](auto CC) { copy_b(integral_constant<int, NP / 2 + decltype(CC)::value>{}, ws1, s1, br1); });
            if (!GA) {
                ghi = table_at(kt + 2)[1];
                __builtin_amdgcn_sched_barrier(0);
            }
            // K steps 1 and 2: A slab kt + 2.
            settle(integral_constant<int, 1>{});
            kstep(integral_constant<int, 1>{}, integral_constant<int, 2>{}, abase, wbase,
                  [&](auto CC) { copy_a(integral_constant<int, decltype(CC)::value>{}, as2, s2, ar2); });
            settle(integral_constant<int, 0>{});
            kstep(integral_constant<int, 0>{}, integral_constant<int, 3>{}, abase, wbase,
                  [&](auto CC) { copy_a(integral_constant<int, NP / 2 + decltype(CC)::value>{}, as2, s2, ar2); });
            settle(integral_constant<int, 1>{});
            // Slab kt + 1 of both operands has landed for this wave: of the
            // operations after its last copy at least the NP copies of A
            // slab kt + 2 may still be in flight. After the barrier it has for
            // every wave, and every wave is done reading slab kt.
            wait_vmcnt<NP>();
            barrier_no_fence();
            if (GA) {
                const half_t* const p = table_at(kt + 3);
                glo = p[0];
                ghi = p[1];
                __builtin_amdgcn_sched_barrier(0);
            }
            // K step 3: first fragments of slab kt + 1; first half of B slab
            // kt + 2 into the slot of slab kt.
            kstep(integral_constant<int, 1>{}, integral_constant<int, 0>{}, (uint32_t)as1 * SLAB, (uint32_t)ws1 * SLAB,
                  [&](auto CC) { copy_b(integral_constant<int, decltype(CC)::value>{}, ws, s2, br2); });
            if (!GA) {
                glo = table_at(kt + 3)[0];
                __builtin_amdgcn_sched_barrier(0);
            }
            as = as1;
            ws = ws1;
        } while (++kt < tc.nk);

        // The last K step also read the next tile's first fragments; let them
        // land (the epilogue reuses their registers) and read them again after it.
        settle(integral_constant<int, 0>{});
        epilogue(tc, as == 0 ? AST - 1 : as - 1);
        if (!has_n) break;

        lid += wpx;
        tc = tn;
        ares_c = ares_n;
        bres_c = bres_n;
        has_n = has_nn;
        tn = tnn;
        ares_n = has_n ? ares_of(tn) : anull;
        bres_n = has_n ? bres_of(tn) : bnull;
        has_nn = lid + 2 * wpx < lid_end;
        if (has_nn) tnn = tile_of(lid + 2 * wpx, ent3);
        ent3 = tile_entry(lid + 3 * wpx);
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int i = 0; i < FB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;
        // Every wave has read its staged rows before the next tile's copies
        // refill that slot.
        barrier_no_fence();
        static_for<2 * FB>([&](auto QC) {
            read_frag(integral_constant<int, 0>{}, QC, integral_constant<int, 0>{}, (uint32_t)as * SLAB,
                      (uint32_t)ws * SLAB);
        });
    }
    wait_vmcnt<0>();
}

}  // namespace

// Tile: 256 x 256 (one workgroup per CU), or 128 x 128 (two per CU) where fewer
// than 128 tiles of 256 x 256 would run, half of the CUs or more idle, or where
// those would pad the widths by 1.6 times or more of what 128 x 128 tiles do
// (320 columns: 512 against 384 both ways). Whole backward, 256 against 128
// over 856 shapes: under 64 tiles 1.13 to 1.68 times as long, 64 to 127 1.01 to
// 1.33, 128 to 191 0.91 to 1.16, more 0.91 to 1.23; padding ratios of 1.6 or
// more 1.02 to 1.68 at any count. 8 experts of 2048 rows, d = 320, h = 448: each
// product 76 -> 40 us; 8 of 8192 rows, d = h = 320: 139 -> 98 us (with one item
// per expert; BackwardPlan::slabs shortens them).
hipError_t launch_wgrad(const WgradArgs& a, bool gather_a, hipStream_t s) {
    auto tiles = [&](long long items, int ts) { return items * ((a.M + ts - 1) / ts) * ((a.N + ts - 1) / ts); };
    auto go = [&](auto kern, int ts, int per_cu) -> hipError_t {
        hipLaunchKernelGGL(kern, dim3((unsigned)persistent_grid(tiles(a.items_max, ts), per_cu)), dim3(256), 0, s, a);
        return hipGetLastError();
    };
    // tiles(5, 256) * 4 >= tiles(8, 128): an area ratio of 1.6.
    if (tiles(a.items_mean, 256) < 128 || tiles(5, 256) * 4 >= tiles(8, 128))
        return gather_a ? go(k_wgrad<true, 128>, 128, 2) : go(k_wgrad<false, 128>, 128, 2);
    return gather_a ? go(k_wgrad<true, 256>, 256, 1) : go(k_wgrad<false, 256>, 256, 1);
}

}  // namespace moe
