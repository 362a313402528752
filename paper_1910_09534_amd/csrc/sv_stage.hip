// Staged sweep: several dense blocks applied in one pass over HBM.  The
// appendix uses cache blocking to form the 5-qubit aggregate gates
// themselves (each "cache" line of its listing is one aggregate); here a
// second level of blocking applies a run of aggregates to an LDS-resident
// tile, so the run costs one HBM round trip instead of one per aggregate.
// This file chooses the tiles and holds the fp32 form; the split-fp16 form
// (unitary complex64 blocks, the default) is in sv_split.hip, the FP64 form
// (complex128) in sv_stage64.hip.
//
// A stage is a run of consecutive dense blocks (k = 4 or 5) whose target
// positions, together with positions 0..3, fit in t <= 14 tile positions
// (complex128: 13) P[0] < ... < P[t-1] (P[0..3] = 0..3; free low positions widen
// the tile as far as its limit and the LDS budget allow).  A tile is the 2^t
// amplitudes whose other bits equal the tile id.  In the fp32 form a persistent
// workgroup (256 lanes, 512 at t = 14) loops over tiles:
//   1. the next tile's loads are issued (into registers; each lane holds
//      pairs of adjacent amplitudes, 16 bytes per access: position 0 is
//      always a tile position);
//   2. each block runs on the LDS tile: pairs of 16-group units per wave
//      through the three real products of the matrix-core form
//      (v_mfma_f32_16x16x4f32, same operand layout as the single sweep),
//      reading and writing LDS, with a workgroup barrier between blocks;
//   3. the tile is written back, then the next tile is parked in LDS.
// The next tile's loads precede this tile's stores, so parking never waits
// for stores.  Re M and Im M of every block are staged in LDS once per
// workgroup.  Every workgroup runs the same number of tile iterations, so
// the barriers are reached uniformly.
#include <algorithm>
#include <atomic>
#include <cmath>

#include "sv_device.h"

#include <type_traits>

namespace sv {

constexpr int kStageMaxOps = 8;
constexpr int kStageMaxT = 14;
constexpr int kStageMaxLds = 80 * 1024;     // tiles of up to 13 positions: two 256-lane workgroups per CU
constexpr int kStageMaxLds14 = 160 * 1024;  // 14 positions: one workgroup per CU

// LDS a tile of t positions may use, and its workgroup size
static inline int stage_lds_limit_t(int t) { return t >= 14 ? kStageMaxLds14 : kStageMaxLds; }
// lanes of an fp32-form workgroup: 256 for tiles of up to 13 positions; 14
// positions take the whole LDS, one workgroup per CU, of 512 lanes
static inline int stage_threads(int t) { return t >= 14 ? 512 : 256; }

struct StageK {
    uint64_t tiles;                          // 2^(nloc - t)
    // tile id bits go, in ascending order, to the set bits of tmask (the
    // positions outside the tile that can be non-zero); consecutive tiles of
    // a workgroup are gridDim.x apart, their bases tstep = that stride
    // spread onto tmask apart (added in the masked number system)
    uint64_t tmask;
    uint64_t tstep;
    // amplitudes on tile positions no earlier operation has reached are
    // zero but their memory may hold older values: tile-local index bits
    // (bit b = position P[b]) of such elements, parked in LDS as zeros
    uint32_t newmask_t;
    uint64_t dep_lane[10];                   // global offset of lane bit b (8 lane bits; 9 at t = 14)
    uint64_t dep_i[32];                      // global offset of the pair index bits above the lane bits
    int t;
    int nops;
    int from_e0;                             // 1: input is |0...0>, not read
    double* norm_out;                        // non-null: per-workgroup FP64 sum of |psi|^2 of the result
    int op_k[kStageMaxOps];
    int op_bits[kStageMaxOps][kMaxDense];    // tile-local bit of matrix bit j
    int op_lowmask_bits[kStageMaxOps][kMaxDense];  // the same bits, ascending
    int op_aoff[kStageMaxOps];               // float offset of the op's operand matrices in LDS
    const float2* op_mat[kStageMaxOps];      // row-major complex matrices (device)
};

// tile-local index -> LDS slot (one pad element per 16)
__device__ __forceinline__ int lslot(int i) { return i + (i >> 4); }

// Group index -> tile-local index: zero bits inserted at the block's target
// bits (low[u] = (1 << target_u) - 1, ascending).  The map acts bit by bit,
// so spread(a | b) = spread(a) | spread(b) for disjoint a, b; likewise
// lslot(a | b) = lslot(a) + lslot(b), which splits every LDS address into a
// wave-uniform part (the unit) and per-lane constants of the block.
template <int K>
__device__ __forceinline__ int spread(int g, const int (&low)[K])
{
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const int lw = g & low[u];
        g = ((g ^ lw) << 1) | lw;
    }
    return g;
}

// NU (1 or 2) 16-group units of one block on the LDS tile, processed together
// by the calling wave: their loads are issued together and their 6 NU
// accumulator chains interleave on the matrix core.  The LDS slot of operand
// element m (matrix column 4 m + h) of unit q is su[q] + sx[m] + cx and that
// of result r = 16 rb + 4 h + v is su[q] + sy[4 rb + v] + cy: su, sx, sy are
// wave-uniform, cx, cy per lane.
template <int K, int NU>
__device__ __forceinline__ void stage_units(const f4 (&av)[3][MfmaShape<K>::RB][MfmaShape<K>::KQ],
                                            const int (&sx)[MfmaShape<K>::D / 4],
                                            const int (&sy)[MfmaShape<K>::D / 4], int cx, int cy,
                                            const int (&su)[2], float2* __restrict__ T)
{
    using S = MfmaShape<K>;
    constexpr int RB = S::RB, KQ = S::KQ, NE = S::D / 4;
    float2 x[NU][NE];
#pragma unroll
    for (int m = 0; m < NE; ++m)
#pragma unroll
        for (int q = 0; q < NU; ++q) x[q][m] = T[(su[q] + sx[m]) + cx];
    f4 acc[NU][3][RB];
#pragma unroll
    for (int q = 0; q < NU; ++q)
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) acc[q][p][rb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sq = 0; sq < KQ; ++sq) {
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
            for (int q = 0; q < NU; ++q) {
                const float2 xv = x[q][4 * sq + s4];
                const float bs = xv.x + xv.y;
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    acc[q][0][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[0][rb][sq][s4], xv.x, acc[q][0][rb], 0, 0, 0);
                    acc[q][1][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[1][rb][sq][s4], xv.y, acc[q][1][rb], 0, 0, 0);
                    acc[q][2][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[2][rb][sq][s4], bs, acc[q][2][rb], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int q = 0; q < NU; ++q) {
                const float p1 = acc[q][0][rb][v], p2 = acc[q][1][rb][v], p3 = acc[q][2][rb][v];
                T[(su[q] + sy[4 * rb + v]) + cy] = float2{p1 - p2, p3 - p1 - p2};
            }
}

template <int K, int NT>
__device__ __forceinline__ void stage_block(const StageK& a, int o, const f4* __restrict__ As,
                                            float2* __restrict__ T, int wave)
{
    using S = MfmaShape<K>;
    constexpr int RB = S::RB, KQ = S::KQ, NE = S::D / 4;
    const int lane = threadIdx.x & 63;
    constexpr int nw = NT / 64;
    const int j = lane & 15, h = lane >> 4;
    int bit[K], low[K];
#pragma unroll
    for (int u = 0; u < K; ++u) {
        bit[u] = 1 << a.op_bits[o][u];
        low[u] = (1 << a.op_lowmask_bits[o][u]) - 1;
    }
    // this wave's operand fragments of Re M and Im M, read from LDS once per
    // block and tile; the third operand Re M + Im M is formed here
    f4 av[3][RB][KQ];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int sq = 0; sq < KQ; ++sq) av[p][rb][sq] = As[((p * RB + rb) * KQ + sq) * 64 + lane];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int sq = 0; sq < KQ; ++sq) av[2][rb][sq] = av[0][rb][sq] + av[1][rb][sq];
    // slot offsets: per lane, the unit's group j with the lane's h bits (h
    // selects matrix bits 0, 1 of an operand and bits 2, 3 of a result);
    // uniform, the remaining matrix bits of element m / result (rb, v)
    const int lj = lslot(spread<K>(j, low));
    const int cx = lj + lslot(((h & 1) ? bit[0] : 0) | ((h & 2) ? bit[1] : 0));
    const int cy = lj + lslot(((h & 1) ? bit[2] : 0) | ((h & 2) ? bit[3] : 0));
    int sx[NE], sy[NE];
#pragma unroll
    for (int m = 0; m < NE; ++m) {
        int off = 0;
#pragma unroll
        for (int u = 2; u < K; ++u)
            if ((m >> (u - 2)) & 1) off |= bit[u];
        sx[m] = lslot(off);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int off = (v & 1) ? bit[0] : 0;
            off |= (v & 2) ? bit[1] : 0;
#pragma unroll
            for (int u = 4; u < K; ++u)
                if ((rb >> (u - 4)) & 1) off |= bit[u];
            sy[4 * rb + v] = lslot(off);
        }
    // units wave, wave + nw, ... in pairs (the wave's trip count is uniform)
    const int units = 1 << (a.t - K - 4);
    for (int unit = wave; unit < units; unit += 2 * nw) {
        const int su[2] = {lslot(spread<K>(unit * 16, low)), lslot(spread<K>((unit + nw) * 16, low))};
        if (unit + nw < units) stage_units<K, 2>(av, sx, sy, cx, cy, su, T);
        else stage_units<K, 1>(av, sx, sy, cx, cy, su, T);
    }
}

// TW: tile width t (9..14), PER = 2^t / lanes elements per lane.  WIDE: the
// lane part of an element's address needs more than 32 bits of byte offset
// (otherwise element addresses are a wave-uniform 64-bit base plus a 32-bit
// per-lane offset, so loads and stores take the scalar-base form).
template <int TW, bool WIDE, bool ZERO>
__global__ __launch_bounds__(TW >= 14 ? 512 : 256) void k_stage(float2* __restrict__ psi, StageK a)
{
    // lanes NT (2^LB), PER amplitudes per lane in PER / 2 adjacent pairs
    constexpr int NT = TW >= 14 ? 512 : 256, LB = TW >= 14 ? 9 : 8;
    constexpr int PER = 1 << (TW - LB);
    extern __shared__ f4 smem[];
    float2* T = (float2*)smem;                                   // tile, padded
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    f4* Abase = smem + ((lslot(1 << TW) * 8 + 15) / 16);          // operand matrices
    // stage every block's operand matrices in operand order
    for (int o = 0; o < a.nops; ++o) {
        const int k = a.op_k[o];
        const int D = 1 << k, RB = D / 16, KQ = D / 16, NA = 2 * RB * KQ * 256;
        float* dst = (float*)(Abase) + a.op_aoff[o];
        const float2* mat = a.op_mat[o];
        for (int i = threadIdx.x; i < NA; i += NT) {
            const int s4 = i & 3, l = (i >> 2) & 63, blk = i >> 8;
            const int sq = blk % KQ, rb = (blk / KQ) % RB, p = blk / (KQ * RB);
            const int R = 16 * rb + (l & 15);
            const int C = 4 * (4 * sq + s4) + (l >> 4);
            const float2 m = mat[R * D + C];
            dst[i] = p == 0 ? m.x : m.y;
        }
    }
    // element pair m of lane l: tile-local indices (l << 1) + 2 NT m + {0, 1}
    // (tile bit 0 is position 0: the pair is two adjacent amplitudes, one
    // 16-byte access); their LDS slots are lslot(2 l) + ES2 m + {0, 1}
    constexpr int PP = PER / 2, ES2 = 2 * NT + (2 * NT) / 16;
    uint64_t dl = 0;
    for (int b = 0; b < LB; ++b)
        if ((threadIdx.x >> b) & 1) dl |= a.dep_lane[b];
    const uint32_t dlb = (uint32_t)(dl * sizeof(float2));       // used when !WIDE
    auto elem = [&](uint64_t tb, int m) -> float4* {
        if (WIDE) return (float4*)(psi + (tb + dl + a.dep_i[m]));
        return (float4*)((char*)(psi + (tb + a.dep_i[m])) + dlb);
    };
    const int ls = lslot(2 * threadIdx.x);
    float4 xr[PP];
    auto load_tile = [&](uint64_t tile, uint64_t tb) {
        if (a.from_e0) {
#pragma unroll
            for (int m = 0; m < PP; ++m) xr[m] = float4{0.f, 0.f, 0.f, 0.f};
            if (tile == 0 && threadIdx.x == 0) xr[0].x = 1.f;
        } else {
#pragma unroll
            for (int m = 0; m < PP; ++m) {
                const f4 v = __builtin_nontemporal_load((const f4*)elem(tb, m));
                xr[m] = float4{v.x, v.y, v.z, v.w};
            }
        }
    };
    // pair m as parked: with ZERO, elements on positions no operation has
    // reached are zero (memory there may hold older values)
    auto parked = [&](int m, float2& e0, float2& e1) {
        e0 = float2{xr[m].x, xr[m].y};
        e1 = float2{xr[m].z, xr[m].w};
        if (ZERO) {
            const uint32_t pi = (uint32_t)((threadIdx.x << 1) + 2 * NT * m);
            if (pi & a.newmask_t) e0 = float2{0.f, 0.f};
            if ((pi | 1u) & a.newmask_t) e1 = float2{0.f, 0.f};
        }
    };
    auto park = [&]() {
#pragma unroll
        for (int m = 0; m < PP; ++m) {
            float2 e0, e1;
            parked(m, e0, e1);
            T[ls + ES2 * m] = e0;
            T[ls + ES2 * m + 1] = e1;
        }
    };
    double nacc = 0.0;                                           // this lane's sum of |psi|^2
    uint64_t tile = blockIdx.x;
    uint64_t tb = spread_bits(tile, a.tmask);
    if (tile < a.tiles) {
        load_tile(tile, tb);
        park();
    }
    __syncthreads();
    // Per tile: issue the next tile's loads, run the blocks on the LDS tile,
    // then store it while parking the next tile in its place.
    // The state streams through once per pass: its loads and stores are
    // non-temporal, and the waves raise their issue priority while they
    // issue them, so that the memory requests of one workgroup go out ahead
    // of the matrix-core work of the other on the same CU.
    for (; tile < a.tiles; tile += gridDim.x) {
        const uint64_t nt = tile + gridDim.x;
        const uint64_t nb = ((tb | ~a.tmask) + a.tstep) & a.tmask;
        const bool next = nt < a.tiles;
        __builtin_amdgcn_s_setprio(1);
        if (next) load_tile(nt, nb);
        __builtin_amdgcn_s_setprio(0);
        for (int o = 0; o < a.nops; ++o) {
            const f4* As = (const f4*)((const float*)Abase + a.op_aoff[o]);
            if (a.op_k[o] == 5) stage_block<5, NT>(a, o, As, T, wave);
            else stage_block<4, NT>(a, o, As, T, wave);
            __syncthreads();
        }
        // Each lane parks the next tile's pairs in the very slots it has just
        // read for its stores (no other lane touches them), pair by pair, so
        // the wait for a pair's load never covers the stores issued before it.
        __builtin_amdgcn_s_setprio(1);
        auto store_park = [&](auto park_next, auto sum_norm) {
#pragma unroll
            for (int m = 0; m < PP; ++m) {
                const float2 v0 = T[ls + ES2 * m], v1 = T[ls + ES2 * m + 1];
                if constexpr (decltype(park_next)::value) {
                    float2 e0, e1;
                    parked(m, e0, e1);
                    T[ls + ES2 * m] = e0;
                    T[ls + ES2 * m + 1] = e1;
                }
                __builtin_nontemporal_store(f4{v0.x, v0.y, v1.x, v1.y}, (f4*)elem(tb, m));
                if constexpr (decltype(sum_norm)::value) {
                    nacc = fma((double)v0.x, (double)v0.x, nacc);
                    nacc = fma((double)v0.y, (double)v0.y, nacc);
                    nacc = fma((double)v1.x, (double)v1.x, nacc);
                    nacc = fma((double)v1.y, (double)v1.y, nacc);
                }
            }
        };
        using yes = std::true_type;
        using no = std::false_type;
        if (next) {
            if (a.norm_out) store_park(yes{}, yes{});
            else store_park(yes{}, no{});
        } else {
            if (a.norm_out) store_park(no{}, yes{});
            else store_park(no{}, no{});
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        tb = nb;
    }
    if (a.norm_out) {
        // fixed-order tree over the workgroup's lanes (the tile buffer is free)
        double* sh = (double*)smem;
        sh[threadIdx.x] = nacc;
        __syncthreads();
        for (int h = NT / 2; h > 0; h >>= 1) {
            if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) a.norm_out[blockIdx.x] = sh[0];
    }
}

int stage_lds_bytes(int t, int nops, const int* ks, int dtype)
{
    int scalars = 0;
    for (int o = 0; o < nops; ++o) scalars += 2 * (1 << (2 * ks[o]));
    if (dtype) {
        // complex128: tile in 32-byte units, then the matrices in double
        const int tile_d4 = (((1 << t) + ((1 << t) >> 4)) * 16 + 31) / 32;
        return tile_d4 * 32 + scalars * 8;
    }
    // complex64: the padded tile (slots lslot(0 .. 2^t - 1), where the
    // operand matrices start: see k_stage), then the matrices in float
    const int tile_f4 = ((1 << t) + ((1 << t) >> 4)) * 8 / 16;
    return tile_f4 * 16 + scalars * 4;
}

// LDS a tile of t positions may use: complex64 as above; complex128 up to the
// whole CU (one workgroup of 512 lanes at t = 13; narrower tiles share it)
static inline int stage_lds_limit_dt(int t, int dtype) { return dtype ? kStageMaxLds14 : stage_lds_limit_t(t); }

// the variant for a tile of t positions (9..14), 64-bit lane offsets, and
// zeroing of stale elements
static void (*stage_kernel(int t, bool wide, bool zero))(float2*, StageK)
{
#define SV_STAGE_CASE(T) \
    case T:              \
        return wide ? (zero ? k_stage<T, true, true> : k_stage<T, true, false>) \
                    : (zero ? k_stage<T, false, true> : k_stage<T, false, false>);
    switch (t) {
        SV_STAGE_CASE(9)
        SV_STAGE_CASE(10)
        SV_STAGE_CASE(11)
        SV_STAGE_CASE(12)
        SV_STAGE_CASE(13)
        SV_STAGE_CASE(14)
    }
#undef SV_STAGE_CASE
    return nullptr;
}

// LDS limit of one variant of the fp32 form (v: 64-bit lane offsets, zeroing)
static hipError_t stage32_prepare(int t, int v)
{
    static std::atomic<bool> done[6][4];
    if (done[t - 9][v]) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute((const void*)stage_kernel(t, v & 1, v & 2),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, stage_lds_limit_t(t));
    if (e == hipSuccess) done[t - 9][v] = true;
    return e;
}

// Launches set their own kernel's LDS limit on its first use; all of them at
// once (some 170 variants, 4 ms) only ahead of a capture.
hipError_t stage_prepare()
{
    static std::atomic<bool> done{false};
    if (done) return hipSuccess;
    for (int t = 9; t <= stage_max_t(0); ++t) {
        for (int v = 0; v < 4; ++v) {
            const hipError_t e = stage32_prepare(t, v);
            if (e != hipSuccess) return e;
        }
        for (int v = 0; v < kSplitForms; ++v) {
            const hipError_t e = split_prepare(t, v);
            if (e != hipSuccess) return e;
        }
    }
    for (int t = 9; t <= stage_max_t(1); ++t)
        for (int v = 0; v < kStage64Forms; ++v) {
            const hipError_t e = stage64_prepare(t, v);
            if (e != hipSuccess) return e;
        }
    done = true;
    return hipSuccess;
}

int split_exponent(double bound)
{
    if (!(bound >= 0.0) || !std::isfinite(bound)) return kNoSplit;
    if (bound < 0x1p-85) return 100;
    int e = 15 - (int)std::ceil(std::log2(bound));
    while (std::ldexp(bound, e) > 32768.0) --e;
    while (e < 100 && std::ldexp(bound, e + 1) <= 32768.0) ++e;
    return e < -100 ? kNoSplit : (e > 100 ? 100 : e);
}

// 14-position tiles need the whole LDS of a CU for one workgroup; where the
// device refuses that, tiles stop at 13 positions (and complex128 states
// take no staged passes)
int stage_max_t(int dtype)
{
    static std::atomic<int> found[2];                     // 0: not asked yet
    const int d = dtype ? 1 : 0;
    int t = found[d];
    if (t == 0) {
        const bool ok = (d ? stage64_prepare(13, 0) : split_prepare(kStageMaxT, 0)) == hipSuccess;
        t = d ? (ok ? 13 : -1) : (ok ? kStageMaxT : 13);
        // (refused, if a narrow tile is not: else asked again)
        if (ok || split_prepare(9, 0) == hipSuccess) found[d] = t;
        if (!ok) (void)hipGetLastError();
    }
    return t < 0 ? 0 : t;
}

int stage_lds_limit(int t, int dtype)
{
    return stage_lds_limit_dt(t, dtype);
}

// Tile positions of a staged pass, ascending, into P (returns t, or -1 when
// the run does not fit): 0..3 plus every target, widened with the lowest
// free positions to the widest tile within t_max that the LDS holds (a
// 14-position tile: one workgroup per CU; 13 and less: two or more).  Wider
// tiles mean longer contiguous runs in memory: with every block of a pass on
// the LDS tile, before the form of sv_split.hip, widening to 14 wherever it
// fits took the 30-qubit depth-14 circuit from 36.4 to 35.2-35.5 ms.  Only positions inside the support widen it: one
// outside would double the amplitudes visited (beyond the 9 the kernel
// needs).
static int stage_positions(int nloc, int nops, const int* ks, const int* const* pos, int t_max,
                           uint64_t support, int* P, int dtype)
{
    if (t_max > stage_max_t(dtype)) t_max = stage_max_t(dtype);
    if (nops < 1 || nops > kStageMaxOps) return -1;
    bool in[64] = {};
    for (int p = 0; p < 4; ++p) in[p] = true;
    for (int o = 0; o < nops; ++o) {
        if (ks[o] < 4 || ks[o] > 5) return -1;
        for (int j = 0; j < ks[o]; ++j) in[pos[o][j]] = true;
    }
    int cnt = 0;
    for (int p = 0; p < 64; ++p) cnt += in[p];
    // support positions free to widen with, lowest first
    int cand[64], nc = 0;
    for (int p = 0; p < nloc; ++p)
        if (!in[p] && ((support >> p) & 1)) cand[nc++] = p;
    auto fits = [&](int tt) { return stage_lds_bytes(tt, nops, ks, dtype) <= stage_lds_limit_dt(tt, dtype); };
    // the widest tile within t_max whose LDS fits (up to 13 positions the
    // limit is the same, so past the first width that fails no narrower
    // one fits; 14 has a limit of its own)
    int want = cnt;
    for (int tt = t_max; tt > cnt; --tt)
        if (tt - cnt <= nc && fits(tt)) {
            want = tt;
            break;
        }
    for (int i = 0; i < want - cnt; ++i) in[cand[i]] = true;
    cnt = want;
    // at least 9 positions, from outside the support if need be
    for (int p = 0; p < nloc && cnt < 9; ++p) {
        if (in[p]) continue;
        if (!fits(cnt + 1)) break;
        in[p] = true;
        ++cnt;
    }
    int t = 0;
    for (int p = 0; p < 64; ++p)
        if (in[p]) P[t++] = p;
    if (t > t_max || t < 9 || nloc < t || !fits(t))
        return -1;
    return t;
}

uint64_t stage_visits(int nloc, int nops, const int* ks, const int* const* pos, int t_max, uint64_t support,
                      int dtype)
{
    int P[64];
    const int t = stage_positions(nloc, nops, ks, pos, t_max, support, P, dtype);
    if (t < 0) return 0;
    uint64_t pmask = 0;
    for (int b = 0; b < t; ++b) pmask |= 1ull << P[b];
    const uint64_t full = nloc >= 64 ? ~0ull : ((1ull << nloc) - 1);
    return (1ull << t) << __builtin_popcountll(full & ~pmask & support);
}

hipError_t launch_stage(hipStream_t st, void* psi, int nloc, int nops, const int* ks, const int* const* pos,
                        const void* const* mats, int t_max, bool from_e0, double* norm_out, int* norm_blocks,
                        int* t_out, uint64_t support, bool garbage, uint64_t* tile_mask_out,
                        uint64_t* amps_out, int split_exp, int dtype, int lone_t)
{
    int P[64];
    bool park = false;
    if (nops == 1 && split_exp != kNoSplit && ks[0] >= 4 && ks[0] <= 5) {
        const uint64_t seen = support & (nloc >= 64 ? ~0ull : (1ull << nloc) - 1);
        const int dev_t = stage_max_t(dtype);
        const SplitLone lone = split_lone(ks[0], pos[0], __builtin_popcountll(seen), std::min(t_max, dev_t),
                                          std::min(lone_t ? lone_t : t_max, dev_t));
        t_max = lone.t_max;
        park = lone.park;
    }
    const int t = stage_positions(nloc, nops, ks, pos, t_max, support, P, dtype);
    if (t < 0) return hipErrorInvalidValue;
    if (dtype && split_exp != kNoSplit) return hipErrorInvalidValue;
    StageK a{};
    a.t = t;
    a.nops = nops;
    a.from_e0 = from_e0 ? 1 : 0;
    a.norm_out = norm_out;
    const bool split = split_exp != kNoSplit;
    if (split && (split_exp < -100 || split_exp > 100)) return hipErrorInvalidValue;
    // tiles: only those whose id bits lie on positions that may be non-zero
    // (support); the other tiles hold zeros and stay zero
    uint64_t pmask = 0;
    for (int b = 0; b < t; ++b) pmask |= 1ull << P[b];
    const uint64_t full = nloc >= 64 ? ~0ull : ((1ull << nloc) - 1);
    support &= full;
    a.tmask = full & ~pmask & support;
    a.tiles = 1ull << __builtin_popcountll(a.tmask);
    const uint64_t newmask = (garbage && !from_e0) ? (pmask & ~support) : 0;
    a.newmask_t = 0;
    for (int b = 0; b < t; ++b)
        if ((newmask >> P[b]) & 1) a.newmask_t |= 1u << b;
    if (split) {
        const hipError_t e = launch_split(st, psi, t, P, nops, ks, pos, mats, a.tiles, a.tmask, newmask, from_e0,
                                          norm_out, norm_blocks, split_exp, park);
        if (t_out) *t_out = t;
        if (tile_mask_out) *tile_mask_out = pmask;
        if (amps_out) *amps_out = a.tiles << t;
        return e;
    }
    if (dtype) {
        const hipError_t e = launch_stage64(st, psi, t, P, nops, ks, pos, mats, a.tiles, a.tmask, newmask, from_e0,
                                            norm_out, norm_blocks);
        if (t_out) *t_out = t;
        if (tile_mask_out) *tile_mask_out = pmask;
        if (amps_out) *amps_out = a.tiles << t;
        return e;
    }
    const int lb = t >= 14 ? 9 : 8;                       // lane bits of the tile index
    // tile bit 0 (position 0) pairs adjacent amplitudes; lane bit b is tile
    // bit b + 1; pair index bit c is tile bit lb + 1 + c
    for (int b = 0; b < lb; ++b) a.dep_lane[b] = 1ull << P[b + 1];
    for (int i = 0; i < (1 << (t - lb - 1)); ++i) {
        uint64_t d = 0;
        for (int b = lb + 1; b < t; ++b)
            if ((i >> (b - lb - 1)) & 1) d |= 1ull << P[b];
        a.dep_i[i] = d;
    }
    int aoff = 0;
    for (int o = 0; o < nops; ++o) {
        a.op_k[o] = ks[o];
        a.op_mat[o] = (const float2*)mats[o];
        a.op_aoff[o] = aoff;
        aoff += 2 * (1 << (2 * ks[o]));
        int tbit[kMaxDense];
        for (int j = 0; j < ks[o]; ++j) {
            int b = 0;
            while (P[b] != pos[o][j]) ++b;
            a.op_bits[o][j] = b;
            tbit[j] = b;
        }
        for (int j = 1; j < ks[o]; ++j)
            for (int l = j; l > 0 && tbit[l - 1] > tbit[l]; --l) {
                const int tmp = tbit[l]; tbit[l] = tbit[l - 1]; tbit[l - 1] = tmp;
            }
        for (int j = 0; j < ks[o]; ++j) a.op_lowmask_bits[o][j] = tbit[j];
    }
    const int lds = stage_lds_bytes(t, nops, ks, 0);
    if (lds > stage_lds_limit_t(t)) return hipErrorInvalidValue;
    // byte offset of the lane part of an element address
    uint64_t dl_max = 0;
    for (int b = 0; b < lb; ++b) dl_max |= a.dep_lane[b];
    const bool wide = dl_max * sizeof(float2) >= (1ull << 32);
    void (*kern)(float2*, StageK) = stage_kernel(t, wide, a.newmask_t != 0);
    if (!kern) return hipErrorInvalidValue;
    {
        const hipError_t e = stage32_prepare(t, (wide ? 1 : 0) | (a.newmask_t ? 2 : 0));
        if (e != hipSuccess) return e;
    }
    // persistent: as many workgroups as are resident (LDS-limited, at most 4
    // per CU)
    int per_cu = (160 * 1024) / lds;
    if (per_cu > 4) per_cu = 4;
    if (per_cu < 1) per_cu = 1;
    uint64_t grid = a.tiles;
    const uint64_t cap = 256ull * per_cu;
    if (grid > cap) grid = cap;
    a.tstep = spread_bits(grid, a.tmask);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(stage_threads(t)), lds, st, (float2*)psi, a);
    if (t_out) *t_out = t;
    if (norm_blocks) *norm_blocks = norm_out ? (int)grid : 0;
    if (tile_mask_out) *tile_mask_out = pmask;
    if (amps_out) *amps_out = a.tiles << t;
    return hipGetLastError();
}

}  // namespace sv
