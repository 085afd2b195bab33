// Data-movement kernels of the expert-MLP backward: the plan of the
// weight-gradient products (per-expert K windows cut into work items), its row
// tables and the sum of their partial blocks, and the per-token sum of the slot
// gradients. The products themselves run on the MFMA kernels
// of gemm.hip and wgrad.hip.
#include "moe_internal.h"

namespace moe {
namespace {

// Plan of the weight-gradient products, one workgroup:
//  - K windows: expert e owns positions koff[e] .. koff[e+1], its row count
//    rounded up to a multiple of 64 (the K slab) and to at least two slabs
//    (the persistent kernel's pipeline holds two; an empty expert's positions
//    all read as zeros, so its gradient comes out 0);
//  - work items: each window cut into pieces of at most `slabs` <= kWgradSlabs slabs,
//    split evenly (sizes differ by at most one slab, and every piece keeps
//    at least two slabs, as a window does), so that no tile runs
//    much longer than the others under a skewed load. An expert with one
//    piece writes its gradient directly (dest = -1); the pieces of a longer
//    window write partial blocks dest = first .. first + n - 1, summed
//    afterwards in that order;
//  - rlist: the split experts {e, first partial block, pieces}.
// wcount[0] = items, wcount[1] = split experts.
// One thread per expert (the block is E rounded up to whole waves: 8 experts 7.8
// -> 3.2 us against always 1024 threads).
__global__ __launch_bounds__(1024) void k_wgrad_plan(const int32_t* __restrict__ offsets, int E, int slabs_max,
                                                    int32_t* __restrict__ koff, WgradItem* __restrict__ items,
                                                    TileDesc* __restrict__ rlist, int32_t* __restrict__ wcount) {
    __shared__ int32_t count_of[kWgradSlabs + 1], cursor[kWgradSlabs + 1];  // items, next position per length (slabs)
    __shared__ int4 wave_sum[1024 / kWave];
    static_assert(kMaxE <= 1024, "one expert per thread");
    const int e = threadIdx.x, lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, waves = blockDim.x / kWave;
    const int start = e < E ? offsets[e] : 0, count = e < E ? offsets[e + 1] - start : 0;
    const int len = e < E ? max(128, (count + 63) / 64 * 64) : 0;
    const int n = (len + slabs_max * 64 - 1) / (slabs_max * 64);
    for (int i = threadIdx.x; i <= kWgradSlabs; i += blockDim.x) count_of[i] = 0;
    // Running sums over the experts: window positions, items, partial blocks,
    // split experts. In a wave, then over the waves (256 experts: 19.7 -> 9.6 us
    // for the kernel, against one thread's loop over the experts).
    int4 v = make_int4(len, n, n > 1 ? n : 0, n > 1 ? 1 : 0);
    const int4 own = v;
#pragma unroll
    for (int o = 1; o < kWave; o *= 2) {
        const int4 u = make_int4(__shfl_up(v.x, o), __shfl_up(v.y, o), __shfl_up(v.z, o), __shfl_up(v.w, o));
        if (lane >= o) v = make_int4(v.x + u.x, v.y + u.y, v.z + u.z, v.w + u.w);
    }
    if (lane == kWave - 1) wave_sum[wave] = v;
    __syncthreads();
    int4 before = make_int4(v.x - own.x, v.y - own.y, v.z - own.z, v.w - own.w), all = make_int4(0, 0, 0, 0);
    for (int w = 0; w < waves; ++w) {
        const int4 u = wave_sum[w];
        if (w < wave) before = make_int4(before.x + u.x, before.y + u.y, before.z + u.z, before.w + u.w);
        all = make_int4(all.x + u.x, all.y + u.y, all.z + u.z, all.w + u.w);
    }
    const int first = n > 1 ? before.z : -1;  // first partial block
    if (e < E) {
        koff[e] = before.x;
        if (n > 1) rlist[before.w] = TileDesc{e, first, n, 0};
    }
    if (e == 0) {
        koff[E] = all.x;
        wcount[0] = all.y;
        wcount[1] = all.w;
    }
    // Items in descending order of length (slabs, 2 .. kWgradSlabs), so that
    // the persistent workgroups running neighbouring items stay in step and
    // the row and column tiles of one item meet in L2 slab by slab (and the
    // longest items start first), dealt round-robin over the XCDs: each XCD
    // walks a contiguous range of the list, so rank p goes to range p % 8 as
    // its (p / 8)-th item, and every range gets the same mix of lengths.
    // Placement within one length follows LDS atomics; every item writes
    // fixed outputs, so the order changes no result.
    const int slabs = len / 64, base = e < E ? slabs / n : 0;
    const int extra = slabs - base * n;  // the first `extra` pieces take one more slab
    if (e < E) {
        if (extra) atomicAdd(&count_of[base + 1], extra);
        if (n > extra) atomicAdd(&count_of[base], n - extra);
    }
    __syncthreads();
    // Wave 0: cursor[sz] = items longer than sz, a running sum from the longest.
    if (wave == 0)
        for (int hi = kWgradSlabs, longer = 0; hi >= 0; hi -= kWave) {
            const int sz = hi - lane, own_c = sz >= 0 ? count_of[sz] : 0;
            int c = own_c;
#pragma unroll
            for (int o = 1; o < kWave; o *= 2) {
                const int u = __shfl_up(c, o);
                if (lane >= o) c += u;
            }
            if (sz >= 0) cursor[sz] = longer + c - own_c;
            longer += __shfl(c, kWave - 1);
        }
    __syncthreads();
    if (e >= E) return;
    for (int c = 0, s0 = 0; c < n; ++c) {
        const int sz = base + (c < extra ? 1 : 0);
        WgradItem t{};
        t.e = e;
        t.q0 = before.x + s0 * 64;
        t.klen = sz * 64;
        t.dest = n > 1 ? first + c : -1;
        t.row0 = start + s0 * 64;
        t.rows = max(0, min(sz * 64, count - s0 * 64));
        const int p = atomicAdd(&cursor[sz], 1), b = p % kNumXcd;
        items[b * (all.y / kNumXcd) + min(b, all.y % kNumXcd) + p / kNumXcd] = t;
        s0 += sz;
    }
}

// Gradients of the split experts: out[e] = sum of its partial blocks in
// order (fp32), four elements per thread. The split experts (their number is
// known on the device only) are dealt to the gridDim.y rows of workgroups in
// turn, so that the grid does not hold a row per expert that mostly exits.
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* __restrict__ partials,
                                                     const TileDesc* __restrict__ rlist,
                                                     const int32_t* __restrict__ wcount, size_t mn,
                                                     float* __restrict__ out) {
    const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i >= mn) return;
    const int nsplit = wcount[1];
    for (int y = blockIdx.y; y < nsplit; y += gridDim.y) {
        const TileDesc r = rlist[y];
        float4 acc = *reinterpret_cast<const float4*>(partials + (size_t)r.row0 * mn + i);
        for (int c = 1; c < r.rows; ++c) {
            const float4 v = *reinterpret_cast<const float4*>(partials + ((size_t)r.row0 + c) * mn + i);
            acc.x += v.x;
            acc.y += v.y;
            acc.z += v.z;
            acc.w += v.w;
        }
        *reinterpret_cast<float4*>(out + (size_t)r.e * mn + i) = acc;
    }
}

// Row tables of the weight-gradient products' gathered operands: window
// position q of expert e (q = koff[e] + i) is sorted row offsets[e] + i, the
// padding positions kWgradNoRow. One wave per 64 positions; windows are
// multiples of 64, so they lie in one expert's window.
__global__ __launch_bounds__(256) void k_wgrad_rows(const int32_t* __restrict__ sorted_slots,
                                                   const int32_t* __restrict__ offsets,
                                                   const int32_t* __restrict__ koff, int E, int K, uint32_t row_bytes,
                                                   uint32_t* __restrict__ gtab, uint32_t* __restrict__ xtab) {
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= koff[E]) return;
    int lo = 0, hi = E - 1;  // last expert with koff[e] <= q
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (koff[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    const int i = q - koff[lo], base = offsets[lo];
    uint32_t g = kWgradNoRow, x = kWgradNoRow;
    if (i < offsets[lo + 1] - base) {
        const uint32_t slot = (uint32_t)sorted_slots[base + i];
        g = slot * row_bytes;
        x = slot / (uint32_t)K * row_bytes;
    }
    gtab[q] = g;
    xtab[q] = x;
}

__device__ __forceinline__ uint32_t pack2_bf16_rne(float lo, float hi) {
    uint32_t a = __float_as_uint(lo), b = __float_as_uint(hi);
    a += 0x7fffu + ((a >> 16) & 1u);
    b += 0x7fffu + ((b >> 16) & 1u);
    return (a >> 16) | (b & 0xffff0000u);
}

// dx[t, :] = bf16(sum_j dxs[t K + j, :]) in slot order (fp32 sums), 4 columns
// per thread.
__global__ __launch_bounds__(256) void k_slot_sum(const float* __restrict__ dxs, int T, int K, int d,
                                                 bf16_t* __restrict__ dx) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int q = d / 4;
    if (i >= (size_t)T * q) return;
    const size_t t = i / q;
    const int c = (int)(i % q) * 4;
    float4 acc = *reinterpret_cast<const float4*>(dxs + (t * K) * d + c);
    for (int j = 1; j < K; ++j) {
        const float4 v = *reinterpret_cast<const float4*>(dxs + (t * K + j) * d + c);
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    }
    uint2 o;
    o.x = pack2_bf16_rne(acc.x, acc.y);
    o.y = pack2_bf16_rne(acc.z, acc.w);
    *reinterpret_cast<uint2*>(dx + t * d + c) = o;
}

}  // namespace

hipError_t launch_wgrad_plan(const int32_t* offsets, int E, int slabs, int32_t* koff, WgradItem* items,
                             TileDesc* rlist, int32_t* wcount, hipStream_t s) {
    hipLaunchKernelGGL(k_wgrad_plan, dim3(1), dim3((E + kWave - 1) / kWave * kWave), 0, s, offsets, E, slabs, koff,
                       items, rlist, wcount);
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const float* partials, const TileDesc* rlist, const int32_t* wcount, int E,
                               size_t mn, float* out, hipStream_t s) {
    const size_t blocks = (mn / 4 + 255) / 256;
    hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)blocks, (unsigned)(E < 8 ? E : 8)), dim3(256), 0, s, partials,
                       rlist, wcount, mn, out);
    return hipGetLastError();
}

hipError_t launch_wgrad_rows(const int32_t* sorted_slots, const int32_t* offsets, const int32_t* koff, int E, int K,
                             uint32_t row_bytes, uint32_t* gtab, uint32_t* xtab, int ld, hipStream_t s) {
    hipLaunchKernelGGL(k_wgrad_rows, dim3((unsigned)((ld + 255) / 256)), dim3(256), 0, s, sorted_slots, offsets, koff,
                       E, K, row_bytes, gtab, xtab);
    return hipGetLastError();
}

hipError_t launch_slot_sum(const float* dxs, int T, int K, int d, void* dx, hipStream_t s) {
    const size_t n = (size_t)T * (d / 4);
    hipLaunchKernelGGL(k_slot_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dxs, T, K, d,
                       static_cast<bf16_t*>(dx));
    return hipGetLastError();
}

}  // namespace moe
