// gfx950 kernels of the sliced state-vector path.
//
// Every kernel streams the amplitude array once (read + write) and keeps the
// per-amplitude arithmetic in registers:
//   k_fill    initial state |0...0>                           (8/16 B per amp)
//   k_zero_outside  clear amplitudes outside the reached positions
//   k_dense   fused dense 2^k x 2^k block, optional folded diagonal epilogue
//             (Sec. 5 aggregate gates; Sec. 2 diagonal gates as phases)
//   k_diag    diagonal op on its own                          (Sec. 2 hyperedges)
//   k_bitperm index permutation between layouts               (Sec. 4 reorganisation)
//   k_accum   gather / cross-slice FP64 accumulation          (Sec. 2 slicing)
//   k_norm, k_xeb, k_finish  fixed-order FP64 reductions (deterministic)
//
// Wavefronts are 64 lanes.  Lane l of a dense sweep owns group g = (block
// base + l); the group counter is spread over the non-target bit positions
// in ascending order, so for targets above bit 5 the 64 lanes of one load
// instruction read 64 consecutive amplitudes (512 B for complex64).
#include <algorithm>
#include <cstring>

#include "sv_device.h"

namespace sv {

struct RunsK {
    int count;
    uint64_t mask[kMaxRuns];
    int shift[kMaxRuns];
};

__device__ __forceinline__ uint64_t apply_runs(uint64_t v, const RunsK& r)
{
    uint64_t out = 0;
    for (int i = 0; i < r.count; ++i) {
        const uint64_t b = v & r.mask[i];
        const int s = r.shift[i];
        out |= s >= 0 ? (b << s) : (b >> (-s));
    }
    return out;
}

static uint64_t apply_runs_host(uint64_t v, const BitRuns& r)
{
    uint64_t out = 0;
    for (int i = 0; i < r.count; ++i) {
        const uint64_t b = v & r.mask[i];
        const int s = r.shift[i];
        out |= s >= 0 ? (b << s) : (b >> (-s));
    }
    return out;
}

static RunsK to_k(const BitRuns& b)
{
    RunsK r;
    r.count = b.count;
    for (int i = 0; i < kMaxRuns; ++i) {
        r.mask[i] = b.mask[i];
        r.shift[i] = b.shift[i];
    }
    return r;
}

BitRuns make_runs(int nbits, const int* from, const int* to)
{
    // bit from[p] of the input goes to bit to[p] of the output; group
    // maximal runs of consecutive source bits that keep the same shift.
    int dst_of[64];
    for (int i = 0; i < 64; ++i) dst_of[i] = -1;
    for (int p = 0; p < nbits; ++p) dst_of[from[p]] = to[p];
    BitRuns r;
    int b = 0;
    while (b < 64) {
        if (dst_of[b] < 0) { ++b; continue; }
        const int sh = dst_of[b] - b;
        uint64_t mask = 0;
        while (b < 64 && dst_of[b] >= 0 && dst_of[b] - b == sh) {
            mask |= 1ull << b;
            ++b;
        }
        r.mask[r.count] = mask;
        r.shift[r.count] = sh;
        ++r.count;
    }
    return r;
}

static unsigned grid_for(uint64_t work, unsigned block, unsigned cap = 1u << 20)
{
    uint64_t g = (work + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// ---------------------------------------------------------------------------
// initial state
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fill(uint4* __restrict__ p, uint64_t n16, uint4 first)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        p[i] = (i == 0) ? first : make_uint4(0u, 0u, 0u, 0u);
}

hipError_t launch_init(hipStream_t st, void* psi, int dtype, uint64_t count, bool one_at_zero)
{
    const uint64_t bytes = count * (dtype ? 16u : 8u);
    if (bytes % 16) return hipErrorInvalidValue;
    uint4 first = make_uint4(0u, 0u, 0u, 0u);
    if (one_at_zero) {
        if (dtype) first.y = 0x3FF00000u;   // double 1.0 (high word)
        else first.x = 0x3F800000u;         // float 1.0
    }
    const uint64_t n16 = bytes / 16;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n16, 256)), dim3(256), 0, st, (uint4*)psi, n16, first);
    return hipGetLastError();
}

// amplitudes whose index has a bit outside `support` are zero; memory that
// still holds older values there is cleared (8/16 B written per such amp)
template <typename T>
__global__ __launch_bounds__(256) void k_zero_outside(T* __restrict__ p, uint64_t n, uint64_t outside)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        if (i & outside) p[i] = T{};
}

hipError_t launch_zero_outside(hipStream_t st, void* psi, int dtype, int nloc, uint64_t support)
{
    const uint64_t n = 1ull << nloc;
    const uint64_t outside = (n - 1) & ~support;
    if (!outside) return hipSuccess;
    if (dtype)
        hipLaunchKernelGGL(k_zero_outside<double2>, dim3(grid_for(n, 256)), dim3(256), 0, st, (double2*)psi, n,
                           outside);
    else
        hipLaunchKernelGGL(k_zero_outside<float2>, dim3(grid_for(n, 256)), dim3(256), 0, st, (float2*)psi, n,
                           outside);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// fused dense block (VALU form; the body is dense_group in sv_device.h)
// ---------------------------------------------------------------------------
template <typename R, int K, bool FOLD>
__global__ __launch_bounds__(256) void k_dense(typename Vec2<R>::T* __restrict__ psi,
                                               const typename Vec2<R>::T* __restrict__ mat, Sweep a)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < a.groups; g += stride)
        dense_group<R, K, FOLD>(psi, mat, a, g);
}

// Batched: workgroup b serves sweep i with items[i].block0 <= b < items[i+1].block0,
// one group per lane.  The sweep's matrix is staged in LDS once per
// workgroup and its wave-uniform rows are read from there (the pointers in
// the descriptor table are generic, which rules out scalar global loads).
template <typename R, int K, bool FOLD>
__global__ __launch_bounds__(256) void k_dense_batch(const Sweep* __restrict__ items, int nitems)
{
    using V = typename Vec2<R>::T;
    constexpr int D = 1 << K;
    __shared__ V Ms[D * D];
    int lo = 0, hi = nitems - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].block0 <= blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const Sweep& a = items[lo];
    const V* __restrict__ mat = (const V*)a.mat;
    for (int i = threadIdx.x; i < D * D; i += blockDim.x) Ms[i] = mat[i];
    __syncthreads();
    const uint64_t g = ((uint64_t)blockIdx.x - a.block0) * blockDim.x + threadIdx.x;
    if (g < a.groups) dense_group<R, K, FOLD>((V*)a.psi, (const V*)Ms, a, g);
}

Sweep make_sweep(void* psi, int nloc, int k, const int* pos, const void* mat, const DiagSpec* fold,
                 uint64_t idx_offset)
{
    Sweep a{};
    a.psi = psi;
    a.mat = mat;
    a.k = k;
    a.groups = 1ull << (nloc - k);
    a.idx_offset = idx_offset;
    int sp[kMaxDense];
    for (int j = 0; j < k; ++j) sp[j] = pos[j];
    for (int j = 1; j < k; ++j)
        for (int l = j; l > 0 && sp[l - 1] > sp[l]; --l) {
            const int t = sp[l]; sp[l] = sp[l - 1]; sp[l - 1] = t;
        }
    for (int j = 0; j < k; ++j) a.lowmask[j] = (1ull << sp[j]) - 1;
    for (int j = 0; j < k; ++j) a.tpos[j] = pos[j];
    for (int u = 0; u < k; ++u)
        for (int j = 0; j < k; ++j)
            if (pos[j] == sp[u]) a.asc[u] = j;
    if (fold && fold->m > 0) {
        a.ftab = fold->table;
        a.fold_m = fold->m;
        for (int j = 0; j < fold->m; ++j) a.fold_pos[j] = fold->pos[j];
    }
    // staged matrix-core loads when a target sits in the lowest four positions
    // (k = 4, 5 and at least 16 groups): address order over the tile's
    // involved positions = the four group positions below + the targets
    a.staged = (k >= 4 && k <= 5 && nloc >= k + 4 && sp[0] < 4) ? 1 : 0;
    if (a.staged) {
        int jpos[4], nj = 0;
        for (int p = 0; p < 64 && nj < 4; ++p) {
            bool tgt = false;
            for (int j = 0; j < k; ++j) tgt = tgt || (pos[j] == p);
            if (!tgt) jpos[nj++] = p;
        }
        int inv[kMaxDense + 4], nv = 0;          // involved positions, ascending
        for (int p = 0; p < 64 && nv < k + 4; ++p) {
            bool in = false;
            for (int q = 0; q < 4; ++q) in = in || (jpos[q] == p);
            for (int j = 0; j < k; ++j) in = in || (pos[j] == p);
            if (in) inv[nv++] = p;
        }
        int slot_of[kMaxDense + 4];
        for (int b = 0; b < nv; ++b) {
            slot_of[b] = 0;
            for (int q = 0; q < 4; ++q)
                if (jpos[q] == inv[b]) slot_of[b] = 1 << q;          // group bit q
            for (int j = 0; j < k; ++j)
                if (pos[j] == inv[b]) slot_of[b] = 17 * (1 << j);    // amplitude bit j
        }
        for (int b = 0; b < 6; ++b) {
            a.st_addr_bit[b] = 1ull << inv[b];
            a.st_slot_bit[b] = slot_of[b];
        }
        for (int i = 0; i < (1 << (k - 2)); ++i) {
            uint64_t ad = 0;
            int sl = 0;
            for (int b = 6; b < nv; ++b)
                if ((i >> (b - 6)) & 1) {
                    ad |= 1ull << inv[b];
                    sl += slot_of[b];
                }
            a.st_addr_i[i] = ad;
            a.st_slot_i[i] = sl;
        }
    }
    return a;
}

template <typename R, int K>
static hipError_t dense_dispatch(hipStream_t st, const Sweep& a)
{
    using V = typename Vec2<R>::T;
    const dim3 grid(grid_for(a.groups, 256)), block(256);
    if (a.ftab) hipLaunchKernelGGL((k_dense<R, K, true>), grid, block, 0, st, (V*)a.psi, (const V*)a.mat, a);
    else hipLaunchKernelGGL((k_dense<R, K, false>), grid, block, 0, st, (V*)a.psi, (const V*)a.mat, a);
    return hipGetLastError();
}

hipError_t launch_dense(hipStream_t st, void* psi, int dtype, int nloc, int k, const int* pos,
                        const void* mat, const DiagSpec* fold, uint64_t idx_offset, int mfma_min_k)
{
    if (k < 1 || k > kMaxDense || k > nloc) return hipErrorInvalidValue;
    if (dtype && k > 5) return hipErrorInvalidValue;
    if (dtype == 0 && dense_uses_mfma(k, nloc, mfma_min_k))
        return launch_dense_mfma(st, psi, nloc, k, pos, mat, fold, idx_offset);
    const Sweep a = make_sweep(psi, nloc, k, pos, mat, fold, idx_offset);
    if (dtype && dense64_uses_mfma(k, nloc)) return launch_dense64_mfma(st, a);
    if (dtype == 0) {
        switch (k) {
            case 1: return dense_dispatch<float, 1>(st, a);
            case 2: return dense_dispatch<float, 2>(st, a);
            case 3: return dense_dispatch<float, 3>(st, a);
            case 4: return dense_dispatch<float, 4>(st, a);
            case 5: return dense_dispatch<float, 5>(st, a);
            case 6: return dense_dispatch<float, 6>(st, a);
        }
    } else {
        switch (k) {
            case 1: return dense_dispatch<double, 1>(st, a);
            case 2: return dense_dispatch<double, 2>(st, a);
            case 3: return dense_dispatch<double, 3>(st, a);
            case 4: return dense_dispatch<double, 4>(st, a);
            case 5: return dense_dispatch<double, 5>(st, a);
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_dense_batch(hipStream_t st, int dtype, int k, bool fold, const Sweep* d_items,
                              int nitems, uint64_t total_blocks)
{
    if (nitems <= 0) return hipSuccess;
    if (total_blocks == 0 || total_blocks > 0x7fffffffull) return hipErrorInvalidValue;
    if (k < 1 || k > kMaxDense || (dtype && k > 5)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)total_blocks), block(256);
#define SV_DB(RR, KK)                                                                              if (fold)                                                                                          hipLaunchKernelGGL((k_dense_batch<RR, KK, true>), grid, block, 0, st, d_items, nitems);       else                                                                                               hipLaunchKernelGGL((k_dense_batch<RR, KK, false>), grid, block, 0, st, d_items, nitems);
    if (dtype == 0) {
        switch (k) {
            case 1: SV_DB(float, 1) break;
            case 2: SV_DB(float, 2) break;
            case 3: SV_DB(float, 3) break;
            case 4: SV_DB(float, 4) break;
            case 5: SV_DB(float, 5) break;
            case 6: SV_DB(float, 6) break;
        }
    } else {
        switch (k) {
            case 1: SV_DB(double, 1) break;
            case 2: SV_DB(double, 2) break;
            case 3: SV_DB(double, 3) break;
            case 4: SV_DB(double, 4) break;
            case 5: SV_DB(double, 5) break;
        }
    }
#undef SV_DB
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// diagonal op
// ---------------------------------------------------------------------------
// A workgroup takes one chunk of amplitudes (256 lanes, one 16-byte access
// each).  A lane puts the gate's positions inside a chunk together from its
// lane bits; the positions above are the same for the whole chunk.  Beyond
// 256 MiB of state they choose the part of the table that the workgroup copies
// to a sub-table in LDS, and the lanes read that.  DIRECT: the lanes read the
// table itself, where the sub-table would be as large as the chunk (nothing is
// read twice; 2^27 complex64 amplitudes, m = 12 on the lowest positions 490 ->
// 381 us), and up to 256 MiB, where the copy and its barrier only lengthen the
// chain (with upload and wait, complex64: 2^16, m = 12 36.2 -> 35.9, 2^24, m = 12
// 78 -> 75).  NT: non-temporal accesses, beyond 256 MiB only: the memory-side
// cache holds a state up to there (2^24 complex128, m = 3: 101 us with them, 91
// without; 2^25: 183 both).
//
// Bound by HBM: 2^28 complex64 amplitudes, m = 6 take 680-690 us (6.2-6.3 TB/s)
// against 970-987 with one amplitude per access and its table index put
// together from the whole address, 2^27 complex128 687 against 722.  Chunks of
// 2, 4 and 8 accesses a lane take 690, 726 and 797 us, persistent workgroups
// 810-850.
struct DiagK {
    uint64_t count;                          // amplitudes
    uint64_t idx_offset;
    int nlow, nhigh;
    uint32_t lane_sub[8], pair_sub;          // sub-table index of lane bit b and of position 0 (complex64)
    uint32_t sub_tab[kMaxDiag];              // table index of sub-table bit k
    int high_pos[kMaxDiag];
    uint32_t high_tab[kMaxDiag];
};

template <typename R, bool DIRECT, bool NT>
__global__ __launch_bounds__(256) void k_diag(typename Vec2<R>::T* __restrict__ psi,
                                              const typename Vec2<R>::T* __restrict__ table, DiagK a)
{
    using V = typename Vec2<R>::T;
    constexpr int E = 16 / sizeof(V);        // amplitudes per access
    typedef R A __attribute__((ext_vector_type(2 * E)));
    extern __shared__ double2 diag_lds[];
    V* sub = (V*)diag_lds;
    const int tid = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * (256 * E), at = base + (uint64_t)tid * E;
    const bool in = at < a.count;
    A x{};
    if (in) x = NT ? __builtin_nontemporal_load((const A*)(psi + at)) : *(const A*)(psi + at);
    uint32_t hi = 0;
    // Where latency counts (states that the cache holds), the positions' arguments
    // in one wait (past nhigh they hold no table bit), and no more of them than
    // most gates need: a wait for each position made m = 12 on 2^24 complex128
    // amplitudes 110.7 us, twelve at once make it 105.9, but m = 1 on 2^22
    // complex64 25.7 instead of 24.7.  On larger states, where memory hides the
    // waits, only what set bits need is read (2^28 complex64, m = 6 688 against
    // 694 us, m = 12 711 against 726).
    auto take = [&](int k) { hi |= (((base + a.idx_offset) >> a.high_pos[k]) & 1) ? a.high_tab[k] : 0u; };
    if (!DIRECT) {
        for (int k = 0; k < a.nhigh; ++k)
            if (((base + a.idx_offset) >> a.high_pos[k]) & 1) hi |= a.high_tab[k];
    } else if (a.nhigh <= 4) {
#pragma unroll
        for (int k = 0; k < 4; ++k) take(k);
    } else {
#pragma unroll
        for (int k = 0; k < kMaxDiag; ++k) take(k);
    }
    uint32_t li = DIRECT ? hi : 0;
#pragma unroll
    for (int b = 0; b < 8; ++b)
        if ((tid >> b) & 1) li |= a.lane_sub[b];
    const V* tab = DIRECT ? table : sub;
    if (!DIRECT) {
        for (int s = tid; s < (1 << a.nlow); s += 256) {
            uint32_t t = hi;
            for (int k = 0; k < a.nlow; ++k)
                if ((s >> k) & 1) t |= a.sub_tab[k];
            sub[s] = table[t];
        }
        __syncthreads();
    }
    A y;
#pragma unroll
    for (int q = 0; q < E; ++q) {
        const V p = tab[q ? li | a.pair_sub : li];
        const R vr = x[2 * q], vi = x[2 * q + 1];
        y[2 * q] = vr * p.x - vi * p.y;
        y[2 * q + 1] = vr * p.y + vi * p.x;
    }
    if (in) {
        if (NT) __builtin_nontemporal_store(y, (A*)(psi + at));
        else *(A*)(psi + at) = y;
    }
}

hipError_t launch_diag(hipStream_t st, void* psi, int dtype, int nloc, uint64_t idx_offset,
                       const DiagSpec& d)
{
    if (d.m < 1 || d.m > kMaxDiag) return hipErrorInvalidValue;
    const int pb = dtype ? 0 : 1;            // position 0 is inside an access (complex64)
    const int cb = pb + 8;                   // positions inside a chunk
    int low = 0;                             // gate positions inside a chunk
    for (int j = 0; j < d.m; ++j) low += d.pos[j] < cb && d.pos[j] < nloc;
    // up to 256 MiB the state stays in the memory-side cache between calls
    const bool cached = nloc <= 24 + pb, direct = cached || low == cb;
    DiagK a{};
    int asc[kMaxDiag];                       // the gate's bits by ascending position
    for (int j = 0; j < d.m; ++j) {
        int i = j;
        for (; i > 0 && d.pos[asc[i - 1]] > d.pos[j]; --i) asc[i] = asc[i - 1];
        asc[i] = j;
    }
    for (int i = 0; i < d.m; ++i) {
        const int p = d.pos[asc[i]];
        const uint32_t bit = 1u << asc[i];
        // (positions from nloc on are sliced: their bits are idx_offset's)
        if (p >= cb || p >= nloc) {
            a.high_pos[a.nhigh] = p;
            a.high_tab[a.nhigh++] = bit;
            continue;
        }
        const uint32_t s = direct ? bit : 1u << a.nlow;
        a.sub_tab[a.nlow++] = bit;
        if (p < pb) a.pair_sub = s;
        else a.lane_sub[p - pb] = s;
    }
    const uint64_t grid = nloc > cb ? 1ull << (nloc - cb) : 1;
    const size_t lds = direct ? 0 : ((size_t)1 << a.nlow) * (dtype ? 16 : 8);
    const auto f32 = cached ? k_diag<float, true, false> : direct ? k_diag<float, true, true> : k_diag<float, false, true>;
    const auto f64 = cached ? k_diag<double, true, false> : direct ? k_diag<double, true, true> : k_diag<double, false, true>;
    // a launch takes fewer than 2^32 work items: 32 GiB of state each, whose
    // offset adds to the slice's
    const uint64_t part = std::min<uint64_t>(grid, 1ull << 23);
    for (uint64_t g = 0; g < grid; g += part) {
        const uint64_t at = g << cb;
        a.idx_offset = idx_offset + at;
        a.count = std::min<uint64_t>(1ull << nloc, part << cb);
        if (dtype == 0)
            hipLaunchKernelGGL(f32, dim3((unsigned)part), dim3(256), lds, st, (float2*)psi + at, (const float2*)d.table, a);
        else
            hipLaunchKernelGGL(f64, dim3((unsigned)part), dim3(256), lds, st, (double2*)psi + at, (const double2*)d.table, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// bit permutation (out-of-place gather form)
// ---------------------------------------------------------------------------
template <typename V>
__global__ __launch_bounds__(256) void k_bitperm(const V* __restrict__ in, V* __restrict__ out,
                                                 uint64_t count, RunsK dst_to_src)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t o = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; o < count; o += stride)
        out[o] = in[apply_runs(o, dst_to_src)];
}

// Tiled bit permutation.  A tile is the 2^t elements whose source bits
// outside T are fixed, where T holds the lowest source bits and the source
// bits of the lowest destination bits: the tile is read in source order
// (runs of 2^a consecutive elements), parked in LDS, and written in
// destination order (again runs of 2^a consecutive elements), so both the
// reads and the writes are whole cache lines whichever bits move where.
// Element e of the tile (bit j <-> source bit T_j, ascending) goes to LDS
// slot e + e / 32; write-order element f (bit j <-> destination bit U_j,
// ascending) reads slot of e(f).  Every map is linear over disjoint bits, so
// each splits into a per-lane part (bits 0..7) and a per-iteration part.
constexpr int kPermT = 12;                 // widest tile (2^12 elements)
struct PermK {
    int t;                                 // tile bits
    int nfree;                             // source bits outside the tile
    uint64_t free_src[64];                 // source offset of tile-id bit i
    uint64_t free_dst[64];                 // destination offset of the same bit
    uint64_t lane_src[8], lane_dst[8];     // offsets of lane bit b (read order / write order)
    uint32_t lane_e[8];                    // tile-local source index of write-order lane bit b
    uint64_t it_src[1 << (kPermT - 8)], it_dst[1 << (kPermT - 8)];
    uint32_t it_e[1 << (kPermT - 8)];
};

__device__ __forceinline__ uint32_t pslot(uint32_t e) { return e + (e >> 5); }

typedef float pf2 __attribute__((ext_vector_type(2)));
typedef double pd2 __attribute__((ext_vector_type(2)));

template <typename V>
__global__ __launch_bounds__(256) void k_bitperm_tiled(const V* __restrict__ in, V* __restrict__ out, PermK p)
{
    extern __shared__ unsigned char permlds[];
    V* T = (V*)permlds;
    const uint64_t tile = blockIdx.x;
    uint64_t sb = 0, db = 0;
    for (int i = 0; i < p.nfree; ++i)
        if ((tile >> i) & 1) {
            sb |= p.free_src[i];
            db |= p.free_dst[i];
        }
    const int tid = threadIdx.x;
    uint64_t ls = 0, ld = 0;
    uint32_t le = 0;
#pragma unroll
    for (int b = 0; b < 8; ++b)
        if ((tid >> b) & 1) {
            ls |= p.lane_src[b];
            ld |= p.lane_dst[b];
            le |= p.lane_e[b];
        }
    const int iters = 1 << (p.t - 8);
    for (int k = 0; k < iters; ++k) {
        const uint32_t e = (uint32_t)tid + 256u * k;
        T[pslot(e)] = __builtin_nontemporal_load(in + (sb + ls + p.it_src[k]));
    }
    __syncthreads();
    const uint32_t sle = pslot(le);
    for (int k = 0; k < iters; ++k)
        __builtin_nontemporal_store(T[sle + pslot(p.it_e[k])], out + (db + ld + p.it_dst[k]));
}

hipError_t launch_bitperm(hipStream_t st, const void* in, void* out, int dtype, int nbits,
                          const BitRuns& dst_to_src)
{
    const uint64_t count = 1ull << nbits;
    const RunsK r = to_k(dst_to_src);
    // source bit of each destination bit, and the reverse
    int src_of[64], dst_of[64];
    for (int d = 0; d < nbits; ++d) {
        const uint64_t sv = apply_runs_host(1ull << d, dst_to_src);
        src_of[d] = sv ? __builtin_ctzll(sv) : -1;
    }
    bool ok = nbits >= 9 && nbits <= 63;
    for (int d = 0; d < nbits && ok; ++d) ok = src_of[d] >= 0 && src_of[d] < nbits;
    if (ok) {
        for (int d = 0; d < nbits; ++d) dst_of[src_of[d]] = d;
        const int esz = dtype == 0 ? 8 : 16;
        const int tmax = esz == 8 ? kPermT : kPermT - 1;
        const int t = nbits < tmax ? nbits : tmax;
        const int a = t / 2 < 6 ? t / 2 : 6;                   // contiguous run bits
        bool inT[64] = {};
        int cnt = 0;
        auto add = [&](int b) { if (!inT[b]) { inT[b] = true; ++cnt; } };
        for (int b = 0; b < a; ++b) add(b);
        for (int d = 0; d < a; ++d) add(src_of[d]);
        for (int b = 0; b < nbits && cnt < t; ++b) add(b);
        PermK p{};
        p.t = cnt;
        int T[64], U[64], nt = 0;
        for (int b = 0; b < nbits; ++b)
            if (inT[b]) T[nt++] = b;
        int nu = 0;
        for (int d = 0; d < nbits; ++d)
            if (inT[src_of[d]]) U[nu++] = d;
        int tpos_of_src[64];
        for (int j = 0; j < nt; ++j) tpos_of_src[T[j]] = j;
        p.nfree = 0;
        for (int b = 0; b < nbits; ++b)
            if (!inT[b]) {
                p.free_src[p.nfree] = 1ull << b;
                p.free_dst[p.nfree] = 1ull << dst_of[b];
                ++p.nfree;
            }
        for (int b = 0; b < 8; ++b) {
            p.lane_src[b] = 1ull << T[b];
            p.lane_dst[b] = 1ull << U[b];
            p.lane_e[b] = 1u << tpos_of_src[src_of[U[b]]];
        }
        for (int k = 0; k < (1 << (p.t - 8)); ++k) {
            uint64_t s_ = 0, d_ = 0;
            uint32_t e_ = 0;
            for (int c = 0; 8 + c < p.t; ++c)
                if ((k >> c) & 1) {
                    s_ |= 1ull << T[8 + c];
                    d_ |= 1ull << U[8 + c];
                    e_ |= 1u << tpos_of_src[src_of[U[8 + c]]];
                }
            p.it_src[k] = s_;
            p.it_dst[k] = d_;
            p.it_e[k] = e_;
        }
        const uint64_t tiles = count >> p.t;
        const size_t lds = (size_t)((1u << p.t) + ((1u << p.t) >> 5)) * esz;
        if (tiles <= 0x7fffffffull) {
            if (dtype == 0)
                hipLaunchKernelGGL(k_bitperm_tiled<pf2>, dim3((unsigned)tiles), dim3(256), lds, st,
                                   (const pf2*)in, (pf2*)out, p);
            else
                hipLaunchKernelGGL(k_bitperm_tiled<pd2>, dim3((unsigned)tiles), dim3(256), lds, st,
                                   (const pd2*)in, (pd2*)out, p);
            return hipGetLastError();
        }
    }
    const dim3 grid(grid_for(count, 256)), block(256);
    if (dtype == 0)
        hipLaunchKernelGGL(k_bitperm<float2>, grid, block, 0, st, (const float2*)in, (float2*)out, count, r);
    else
        hipLaunchKernelGGL(k_bitperm<double2>, grid, block, 0, st, (const double2*)in, (double2*)out, count, r);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// gather / cross-slice accumulation in FP64
// ---------------------------------------------------------------------------
template <typename R>
__global__ __launch_bounds__(256) void k_accum(const typename Vec2<R>::T* __restrict__ psi, int nloc,
                                               uint64_t slice, RunsK l2p, int64_t count,
                                               const uint64_t* __restrict__ bits,
                                               const double2* __restrict__ tcol,
                                               const int* __restrict__ rowmap,
                                               double2* __restrict__ acc)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= count) return;
    const uint64_t ph = apply_runs(bits[j], l2p);
    const uint64_t t = nloc >= 64 ? 0 : (ph >> nloc);
    const uint64_t li = ph & ((nloc >= 64) ? ~0ull : ((1ull << nloc) - 1));
    if (tcol == nullptr) {
        if (t == slice) {
            const auto a = psi[li];
            double2 s = acc[j];
            s.x += (double)a.x;
            s.y += (double)a.y;
            acc[j] = s;
        }
    } else {
        const auto a = psi[li];
        const double2 w = tcol[rowmap[t]];
        const double ar = (double)a.x, ai = (double)a.y;
        double2 s = acc[j];
        s.x += w.x * ar - w.y * ai;
        s.y += w.x * ai + w.y * ar;
        acc[j] = s;
    }
}

hipError_t launch_accumulate(hipStream_t st, const void* psi_slice, int dtype, int nloc,
                             uint64_t slice, const BitRuns& log_to_phys, int64_t count,
                             const uint64_t* bits, const void* tcol, const int* rowmap,
                             double* acc)
{
    if (count <= 0) return hipSuccess;
    const RunsK r = to_k(log_to_phys);
    const dim3 grid((unsigned)((count + 255) / 256)), block(256);
    if (dtype == 0)
        hipLaunchKernelGGL(k_accum<float>, grid, block, 0, st, (const float2*)psi_slice, nloc, slice, r,
                           count, bits, (const double2*)tcol, rowmap, (double2*)acc);
    else
        hipLaunchKernelGGL(k_accum<double>, grid, block, 0, st, (const double2*)psi_slice, nloc, slice,
                           r, count, bits, (const double2*)tcol, rowmap, (double2*)acc);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// deterministic FP64 reductions
// ---------------------------------------------------------------------------
// Block-level tree in LDS with a fixed shape: the result depends only on the
// input and the launch geometry, which depends only on the size.
template <int W>
__device__ __forceinline__ void block_tree(double (*sh)[256], double* v)
{
    const int t = threadIdx.x;
#pragma unroll
    for (int w = 0; w < W; ++w) sh[w][t] = v[w];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) {
#pragma unroll
            for (int w = 0; w < W; ++w) sh[w][t] += sh[w][t + h];
        }
        __syncthreads();
    }
#pragma unroll
    for (int w = 0; w < W; ++w) v[w] = sh[w][0];
}

// Four 16-byte accesses per lane in flight: with one amplitude at a time a
// state of 2^20 to 2^24 amplitudes waits for memory (15.5 us a state; here 5).
template <typename R>
__global__ __launch_bounds__(256) void k_norm(const typename Vec2<R>::T* __restrict__ psi,
                                              uint64_t per_block, double* __restrict__ partial)
{
    using V = typename Vec2<R>::T;
    constexpr int E = 16 / sizeof(V);                    // amplitudes per access
    typedef R A __attribute__((ext_vector_type(2 * E)));
    __shared__ double sh[1][256];
    const A* p = (const A*)(psi + (uint64_t)blockIdx.x * per_block);
    const uint64_t count = per_block / E;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint64_t i = threadIdx.x; i < count; i += 4 * 256) {
        A x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            x[u] = i + 256 * u < count ? p[i + 256 * u] : A{};
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 2 * E; ++c) s[u] = fma((double)x[u][c], (double)x[u][c], s[u]);
    }
    double v[1] = {(s[0] + s[1]) + (s[2] + s[3])};
    block_tree<1>(sh, v);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

hipError_t launch_norm_partials(hipStream_t st, const void* psi, int dtype, int nloc,
                                double* partial, int* nblocks)
{
    const int lb = nloc > 20 ? 12 : (nloc > 8 ? nloc - 8 : 0);
    const int nb = 1 << lb;
    const uint64_t per = 1ull << (nloc - lb);
    if (dtype == 0)
        hipLaunchKernelGGL(k_norm<float>, dim3(nb), dim3(256), 0, st, (const float2*)psi, per, partial);
    else
        hipLaunchKernelGGL(k_norm<double>, dim3(nb), dim3(256), 0, st, (const double2*)psi, per, partial);
    *nblocks = nb;
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_xeb(const double2* __restrict__ amps, int64_t count,
                                             int64_t per_block, double logN,
                                             double* __restrict__ partial)
{
    __shared__ double sh[2][256];
    const int64_t b0 = (int64_t)blockIdx.x * per_block;
    const double N = exp2(logN);
    double v[2] = {0.0, 0.0};
    for (int64_t i = threadIdx.x; i < per_block; i += 256) {
        const int64_t j = b0 + i;
        if (j >= count) break;
        const double2 a = amps[j];
        const double p = N * (a.x * a.x + a.y * a.y);
        v[0] += p;
        v[1] += log(p);
    }
    block_tree<2>(sh, v);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = v[0];
        partial[2 * blockIdx.x + 1] = v[1];
    }
}

hipError_t launch_xeb_partials(hipStream_t st, const double* amps, int64_t count, double logN,
                               double* partial, int* nblocks)
{
    int nb = (int)((count + 4095) / 4096);
    if (nb < 1) nb = 1;
    if (nb > 4096) nb = 4096;
    const int64_t per = (count + nb - 1) / nb;
    hipLaunchKernelGGL(k_xeb, dim3(nb), dim3(256), 0, st, (const double2*)amps, count, per, logN, partial);
    *nblocks = nb;
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_finish(const double* __restrict__ partial, int count, int width,
                                                double* __restrict__ out)
{
    __shared__ double sh[2][256];
    double v[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < count; b += 256)
        for (int w = 0; w < width && w < 2; ++w) v[w] += partial[(int64_t)b * width + w];
    block_tree<2>(sh, v);
    if (threadIdx.x == 0)
        for (int w = 0; w < width && w < 2; ++w) out[w] = v[w];
}

hipError_t launch_finish_sum(hipStream_t st, const double* partial, int count, int width, double* out)
{
    if (width < 1 || width > 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(256), 0, st, partial, count, width, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// gather, cross-slice sum, cross-entropy sums and norm of a resident state
// ---------------------------------------------------------------------------
// One launch where there were six and four copies (k_accum per slice, k_xeb,
// two k_finish, the cleared accumulators, the row map): on small states a
// reduction is launches: 16 qubits, depth 8, complex128, 2^16 bitstrings take
// 183 us with this and k_upload against 278, and a diagonal gate on 18 qubits with
// k_upload alone 20.0 against 23.8.  The last workgroup to finish (a ticket that it resets) adds
// the workgroups' partial sums, each in a fixed order.
template <typename R>
__global__ __launch_bounds__(256) void k_reduce(const typename Vec2<R>::T* __restrict__ psi, int nloc, int ns,
                                                RunsK l2p, int64_t count, int64_t per,
                                                const uint64_t* __restrict__ bits,
                                                const double2* __restrict__ tcols, const int* __restrict__ rowmap,
                                                double2* __restrict__ out, double logn, double* part,
                                                int norm_count, unsigned* ticket, double* stats)
{
    __shared__ double sh[2][256];
    __shared__ bool last;
    const double N = exp2(logn);
    const int64_t j0 = (int64_t)blockIdx.x * per;
    const uint64_t low = (1ull << nloc) - 1;
    double v[2] = {0.0, 0.0};
    for (int64_t i = threadIdx.x; i < per && j0 + i < count; i += 256) {
        const int64_t j = j0 + i;
        const uint64_t ph = apply_runs(bits[j], l2p);
        double2 s = {0.0, 0.0};
        if (tcols == nullptr) {
            const auto a = psi[ph];
            s.x = (double)a.x;
            s.y = (double)a.y;
        } else {
            const int r = rowmap[ph >> nloc];
            for (int t = 0; t < ns; ++t) {
                const auto a = psi[((uint64_t)t << nloc) | (ph & low)];
                const double2 w = tcols[(int64_t)t * ns + r];
                const double ar = (double)a.x, ai = (double)a.y;
                s.x += w.x * ar - w.y * ai;
                s.y += w.x * ai + w.y * ar;
            }
        }
        out[j] = s;
        if (stats) {
            const double p = N * (s.x * s.x + s.y * s.y);
            v[0] += p;
            v[1] += log(p);
        }
    }
    if (!stats) return;
    double* mine = part + ((int)kPartDoubles - kReducePart);
    block_tree<2>(sh, v);
    if (threadIdx.x == 0) {
        mine[2 * blockIdx.x] = v[0];
        mine[2 * blockIdx.x + 1] = v[1];
        __threadfence();
        last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    v[0] = v[1] = 0.0;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += 256) {
        v[0] += mine[2 * b];
        v[1] += mine[2 * b + 1];
    }
    block_tree<2>(sh, v);
    double w[1] = {0.0};
    for (int b = threadIdx.x; b < norm_count; b += 256) w[0] += part[b];
    __syncthreads();
    block_tree<1>(*(double(*)[1][256])sh, w);
    if (threadIdx.x == 0) {
        stats[0] = w[0];
        stats[1] = v[0];
        stats[2] = v[1];
        *ticket = 0;
    }
}

hipError_t launch_reduce(hipStream_t st, const void* psi, int dtype, int nloc, int ns, const BitRuns& log_to_phys,
                         int64_t count, const uint64_t* bits, const void* tcols, const int* rowmap, double* out,
                         double logn, double* part, int norm_count, unsigned* ticket, double* stats)
{
    if (count < 1 && !stats) return hipSuccess;
    if (norm_count > (int)kPartDoubles - kReducePart) return hipErrorInvalidValue;
    const RunsK r = to_k(log_to_phys);
    int64_t nb = (count + 255) / 256;
    if (nb < 1) nb = 1;
    if (nb > kReduceBlocks) nb = kReduceBlocks;
    const int64_t per = (count + nb - 1) / nb;
    if (dtype == 0)
        hipLaunchKernelGGL(k_reduce<float>, dim3((unsigned)nb), dim3(256), 0, st, (const float2*)psi, nloc, ns, r, count,
                           per, bits, (const double2*)tcols, rowmap, (double2*)out, logn, part, norm_count, ticket,
                           stats);
    else
        hipLaunchKernelGGL(k_reduce<double>, dim3((unsigned)nb), dim3(256), 0, st, (const double2*)psi, nloc, ns, r,
                           count, per, bits, (const double2*)tcols, rowmap, (double2*)out, logn, part, norm_count,
                           ticket, stats);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// small uploads
// ---------------------------------------------------------------------------
struct UploadK {
    uint4 d[kUploadMax / 16];
};

__global__ __launch_bounds__(256) void k_upload(uint4* __restrict__ dst, int n16, UploadK u)
{
    if ((int)threadIdx.x < n16) dst[threadIdx.x] = u.d[threadIdx.x];
}

hipError_t launch_upload(hipStream_t st, void* dst, const void* src, size_t bytes)
{
    static_assert(kUploadMax % 16 == 0 && kUploadMax / 16 <= 256, "one access a lane");
    if (bytes > kUploadMax || bytes % 16) return hipErrorInvalidValue;
    UploadK u;
    std::memcpy(u.d, src, bytes);
    hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, st, (uint4*)dst, (int)(bytes / 16), u);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a slice of the pinned tier to or from a device slot, over the host link
// ---------------------------------------------------------------------------
template <bool IN>
__global__ __launch_bounds__(256) void k_files(uint4* __restrict__ slot, FilesK a)
{
    const uint64_t n16 = 1ull << (a.s + a.lg), stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) {
        int64_t at = (int64_t)(i & ((1ull << a.lg) - 1)) * 16;
        for (int b = 0; b < a.s; ++b)
            if ((i >> (a.lg + b)) & 1) at += a.off[b];
        uint4* host = (uint4*)((char*)a.host + at);
        if (IN) slot[i] = *host;
        else *host = slot[i];
    }
}

hipError_t launch_files(hipStream_t st, void* slot, const FilesK& a, bool in)
{
    if (a.s < 0 || a.s > kMaxFileBits || a.lg < 0 || a.s + a.lg > 32) return hipErrorInvalidValue;
    const uint64_t n16 = 1ull << (a.s + a.lg);
    const dim3 grid((unsigned)std::min<uint64_t>((n16 + 255) / 256, 1024));
    if (in) hipLaunchKernelGGL(k_files<true>, grid, dim3(256), 0, st, (uint4*)slot, a);
    else hipLaunchKernelGGL(k_files<false>, grid, dim3(256), 0, st, (uint4*)slot, a);
    return hipGetLastError();
}

}  // namespace sv
