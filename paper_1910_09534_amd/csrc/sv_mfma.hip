// Fused dense sweep on the matrix cores (complex64, k = 4..6): single-state
// and batched launches.  The per-tile body (operand layouts, LDS staging of
// the real form of the block) is in sv_device.h.  And the complex128 sweep
// of k = 4, 5 on the FP64 matrix cores.
#include "sv_device.h"

namespace sv {

template <int K, bool FOLD, bool STAGED>
__global__ __launch_bounds__(256) void k_dense_mfma(Sweep a)
{
    __shared__ f4 As[MfmaShape<K>::NA / 4];
    __shared__ float2 Xs[STAGED ? 4 * MfmaShape<K>::XS : 1];
    mfma_stage_matrix<K>(As, (const float2*)a.mat);
    __syncthreads();
    const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const uint64_t nwaves = ((uint64_t)gridDim.x * blockDim.x) >> 6;
    mfma_tiles<K, FOLD, STAGED>(a, As, Xs + (STAGED ? (threadIdx.x >> 6) * MfmaShape<K>::XS : 0), wave,
                                nwaves, a.groups / 16);
}

// Many sweeps (of different states) in one launch: workgroup b belongs to
// the sweep i with items[i].block0 <= b < items[i + 1].block0 (the last
// sweep ends at gridDim.x); its waves stride over that sweep's tiles.
__device__ __forceinline__ int find_item(const Sweep* __restrict__ items, int nitems, uint64_t b)
{
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].block0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int K, bool FOLD, bool STAGED>
__global__ __launch_bounds__(256) void k_dense_mfma_batch(const Sweep* __restrict__ items, int nitems)
{
    __shared__ f4 As[MfmaShape<K>::NA / 4];
    __shared__ float2 Xs[STAGED ? 4 * MfmaShape<K>::XS : 1];
    const int i = find_item(items, nitems, blockIdx.x);
    const Sweep& a = items[i];
    const uint64_t b_end = (i + 1 < nitems) ? items[i + 1].block0 : gridDim.x;
    const uint64_t nb = b_end - a.block0;
    mfma_stage_matrix<K>(As, (const float2*)a.mat);
    __syncthreads();
    const uint64_t wave = (blockIdx.x - a.block0) * (blockDim.x >> 6) + (threadIdx.x >> 6);
    mfma_tiles<K, FOLD, STAGED>(a, As, Xs + (STAGED ? (threadIdx.x >> 6) * MfmaShape<K>::XS : 0), wave,
                                nb * (blockDim.x >> 6), a.groups / 16);
}

template <int K, bool STAGED>
static hipError_t mfma_dispatch(hipStream_t st, const Sweep& a)
{
    const uint64_t tiles = a.groups / 16;
    uint64_t g = (tiles + 3) / 4;
    const uint64_t cap = 256 * (K == 6 ? 2 : 6);
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    if (a.ftab)
        hipLaunchKernelGGL((k_dense_mfma<K, true, STAGED>), dim3((unsigned)g), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_dense_mfma<K, false, STAGED>), dim3((unsigned)g), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_dense_mfma(hipStream_t st, void* psi, int nloc, int k, const int* pos, const void* mat,
                             const DiagSpec* fold, uint64_t idx_offset)
{
    if (k < 4 || k > 6 || nloc < k + 4) return hipErrorInvalidValue;
    const Sweep a = make_sweep(psi, nloc, k, pos, mat, fold, idx_offset);
    switch (k) {
        case 4: return a.staged ? mfma_dispatch<4, true>(st, a) : mfma_dispatch<4, false>(st, a);
        case 5: return a.staged ? mfma_dispatch<5, true>(st, a) : mfma_dispatch<5, false>(st, a);
        case 6: return mfma_dispatch<6, false>(st, a);
    }
    return hipErrorInvalidValue;
}

uint64_t mfma_batch_blocks(uint64_t groups)
{
    // about 8 tiles per wave, 4 waves per workgroup
    const uint64_t tiles = groups / 16;
    const uint64_t b = (tiles + 31) / 32;
    return b < 1 ? 1 : b;
}

hipError_t launch_dense_mfma_batch(hipStream_t st, int k, bool fold, bool staged, const Sweep* d_items,
                                   int nitems, uint64_t total_blocks)
{
    if (nitems <= 0) return hipSuccess;
    if (total_blocks == 0 || total_blocks > 0x7fffffffull) return hipErrorInvalidValue;
    if (staged && k == 6) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total_blocks), block(256);
#define SV_MB(KK, SS)                                                                                 \
    if (fold)                                                                                         \
        hipLaunchKernelGGL((k_dense_mfma_batch<KK, true, SS>), grid, block, 0, st, d_items, nitems);  \
    else                                                                                              \
        hipLaunchKernelGGL((k_dense_mfma_batch<KK, false, SS>), grid, block, 0, st, d_items, nitems);
    switch (k) {
        case 4: if (staged) { SV_MB(4, true) } else { SV_MB(4, false) } break;
        case 5: if (staged) { SV_MB(5, true) } else { SV_MB(5, false) } break;
        case 6: SV_MB(6, false) break;
        default: return hipErrorInvalidValue;
    }
#undef SV_MB
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// complex128, k = 4, 5: v_mfma_f64_16x16x4f64
//
// Sixteen groups per wave and unit.  Lane (j, g) holds group j's amplitudes
// whose two lowest targets are g; the other target bits run over its
// registers (element e = column 4 e + g, the matrix bits taken in ascending
// order of their positions).  The instruction's result item v of lane group g
// is row g + 4 v, so a lane ends with the amplitudes it began with and no
// shuffle or LDS is needed, and one access of a wave spans the four lowest
// free positions and the two lowest targets: whole cache lines also when the
// targets are low.  Four real products in double, the sums of the vector
// form in another order; the matrix stays in registers.
//
// Bound by HBM for k = 4 and 5 (64 products of 64 cycles per 512 amplitudes,
// 16 KiB, at k = 5: 60 % of the time that memory takes).  Measured against
// the vector form (a group per lane): 2^27 amplitudes, k = 4, targets 0-3
// 1,420 -> 836 us (5.1 TB/s), 10-13 806 -> 808; 2^26, k = 5, targets 0-4 767 ->
// 396, 10-14 436 -> 384 (5.6 TB/s); 2^20, k = 5 46 -> 12.6; 2^16, k = 4 (256
// waves where that form had 64 in 16 workgroups) 12.2 -> 6.1 us.  Relative
// error against 80-bit sums: 1.91e-16 and 1.47e-16 (k = 4), 2.70e-16 and
// 1.98e-16 (k = 5).
// ---------------------------------------------------------------------------
typedef double d4 __attribute__((ext_vector_type(4)));

typedef double dd2 __attribute__((ext_vector_type(2)));

template <int K, bool FOLD, bool NT>
__device__ __forceinline__ void dense64_tiles(const Sweep& a, uint64_t t0, uint64_t step, uint64_t t_end)
{
    constexpr int D = 1 << K, RB = D / 16, NE = D / 4;
    double2* __restrict__ psi = (double2*)a.psi;
    const double2* __restrict__ mat = (const double2*)a.mat;
    const int lane = threadIdx.x & 63;
    const int j = lane & 15, g = lane >> 4;
    uint64_t bit[K];
    int own[K];                                          // the matrix's own bit of ascending bit u
#pragma unroll
    for (int u = 0; u < K; ++u) {
        own[u] = a.asc[u];
        bit[u] = 1ull << a.tpos[own[u]];
    }
    const uint64_t lane_off = ((g & 1) ? bit[0] : 0ull) | ((g & 2) ? bit[1] : 0ull);
    uint64_t off[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        off[e] = 0;
#pragma unroll
        for (int u = 2; u < K; ++u)
            if ((e >> (u - 2)) & 1) off[e] |= bit[u];
    }
    auto take = [&](uint64_t i) {
        if (!NT) return psi[i];
        const dd2 w = __builtin_nontemporal_load((const dd2*)(psi + i));
        return double2{w.x, w.y};
    };
    auto base_of = [&](uint64_t t) { return group_base<K>(a, t * 16 + j) | lane_off; };
    double2 xn[NE];
    uint64_t nbase = 0;
    if (t0 < t_end) {
        nbase = base_of(t0);
#pragma unroll
        for (int e = 0; e < NE; ++e) xn[e] = take(nbase + off[e]);
    }
    // A[lane % 16][lane / 16] of each product: row 16 rb + j, column 4 e + g
    double2 A[RB][NE];
    {
        auto index = [&](int c) {
            int i = 0;
#pragma unroll
            for (int u = 0; u < K; ++u) i |= ((c >> u) & 1) << own[u];
            return i;
        };
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int e = 0; e < NE; ++e) A[rb][e] = mat[index(16 * rb + j) * D + index(4 * e + g)];
    }
    for (uint64_t t = t0; t < t_end; t += step) {
        double2 x[NE];
        const uint64_t base = nbase;
#pragma unroll
        for (int e = 0; e < NE; ++e) x[e] = xn[e];
        if (t + step < t_end) {
            nbase = base_of(t + step);
#pragma unroll
            for (int e = 0; e < NE; ++e) xn[e] = take(nbase + off[e]);
        }
        __builtin_amdgcn_sched_barrier(0);               // the next unit's loads stay ahead of the products
        // Ar xr, Ai xi, Ai xr and Ar xi are summed on their own: half as many
        // roundings per sum
        d4 rr[RB], ii[RB], ir[RB], ri[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) rr[rb] = ii[rb] = ir[rb] = ri[rb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                rr[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb][e].x, x[e].x, rr[rb], 0, 0, 0);
                ii[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb][e].y, x[e].y, ii[rb], 0, 0, 0);
                ir[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb][e].y, x[e].x, ir[rb], 0, 0, 0);
                ri[rb] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[rb][e].x, x[e].y, ri[rb], 0, 0, 0);
            }
        uint32_t fb = 0;
        if (FOLD) fb = fold_index(a, base + a.idx_offset);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint64_t o = off[4 * rb + v];
                double yr = rr[rb][v] - ii[rb][v], yi = ir[rb][v] + ri[rb][v];
                if (FOLD) {
                    const double2 p = ((const double2*)a.ftab)[fb | fold_index(a, o)];
                    const double tr = yr * p.x - yi * p.y;
                    yi = yr * p.y + yi * p.x;
                    yr = tr;
                }
                if (NT) __builtin_nontemporal_store(dd2{yr, yi}, (dd2*)(psi + base + o));
                else psi[base + o] = double2{yr, yi};
            }
    }
}

template <int K, bool FOLD, bool NT>
__global__ __launch_bounds__(256, 2) void k_dense64_mfma(Sweep a)
{
    const uint64_t wave = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    dense64_tiles<K, FOLD, NT>(a, wave, (uint64_t)gridDim.x * 4, a.groups / 16);
}

template <int K, bool FOLD>
__global__ __launch_bounds__(256, 2) void k_dense64_mfma_batch(const Sweep* __restrict__ items, int nitems)
{
    const int i = find_item(items, nitems, blockIdx.x);
    const Sweep& a = items[i];
    const uint64_t b_end = (i + 1 < nitems) ? items[i + 1].block0 : gridDim.x;
    const uint64_t nb = b_end - a.block0;
    const uint64_t wave = (blockIdx.x - a.block0) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    dense64_tiles<K, FOLD, false>(a, wave, nb * 4, a.groups / 16);
}

hipError_t launch_dense64_mfma(hipStream_t st, const Sweep& a)
{
    const uint64_t tiles = a.groups / 16;
    if (tiles < 1) return hipErrorInvalidValue;
    // Beyond the 256 MB cache non-temporal accesses and one wave per SIMD; below,
    // plain ones, and two waves at k = 4 (k = 5: 170 registers, 64 products a
    // unit).  Mean of 12 sets of targets (plain, 512 / 256 workgroups at k = 4 / 5
    // -> non-temporal, the same -> non-temporal, 256): 2^27 amplitudes, k = 4 906 ->
    // 838 -> 795 us (k_dense 854), k = 5 836 -> 790 (k_dense 972); 2^24, k = 4 96 ->
    // 109 -> 112 (102), k = 5 112 -> 119 (151); 2^16, k = 4 19.3 a call (25.0).
    uint64_t g = (tiles + 3) / 4;
    const bool nt = (tiles << (a.k + 4)) >= (1ull << 25);
    const uint64_t cap = a.k == 5 || nt ? 256 : 512;
    if (g > cap) g = cap;
    const dim3 grid((unsigned)g), block(256);
#define SV_D64(KK)                                                                                    \
    if (nt) {                                                                                         \
        if (a.ftab) hipLaunchKernelGGL((k_dense64_mfma<KK, true, true>), grid, block, 0, st, a);      \
        else hipLaunchKernelGGL((k_dense64_mfma<KK, false, true>), grid, block, 0, st, a);            \
    } else {                                                                                          \
        if (a.ftab) hipLaunchKernelGGL((k_dense64_mfma<KK, true, false>), grid, block, 0, st, a);     \
        else hipLaunchKernelGGL((k_dense64_mfma<KK, false, false>), grid, block, 0, st, a);           \
    }
    if (a.k == 4) {
        SV_D64(4)
    } else if (a.k == 5) {
        SV_D64(5)
    } else {
        return hipErrorInvalidValue;
    }
#undef SV_D64
    return hipGetLastError();
}

hipError_t launch_dense64_mfma_batch(hipStream_t st, int k, bool fold, const Sweep* d_items, int nitems,
                                     uint64_t total_blocks)
{
    if (nitems <= 0) return hipSuccess;
    if (total_blocks == 0 || total_blocks > 0x7fffffffull || (k != 4 && k != 5)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total_blocks), block(256);
    if (k == 4) {
        if (fold) hipLaunchKernelGGL((k_dense64_mfma_batch<4, true>), grid, block, 0, st, d_items, nitems);
        else hipLaunchKernelGGL((k_dense64_mfma_batch<4, false>), grid, block, 0, st, d_items, nitems);
    } else {
        if (fold) hipLaunchKernelGGL((k_dense64_mfma_batch<5, true>), grid, block, 0, st, d_items, nitems);
        else hipLaunchKernelGGL((k_dense64_mfma_batch<5, false>), grid, block, 0, st, d_items, nitems);
    }
    return hipGetLastError();
}

}  // namespace sv
