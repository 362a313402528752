// Staged sweep of complex64 blocks in the split-fp16 form: a run of dense
// 4/5-qubit unitary blocks applied to LDS-resident tiles in one pass over HBM
// (see sv_stage.hip for tiles and supports), every product on the fp16 matrix
// cores at single-precision accuracy.
//
// Precision.  Every real product of a block runs on the fp16 matrix cores:
// each fp32 operand x is split into x_hi = f16(x) and x_lo = f16(x - x_hi)
// (both rounded to nearest), so x_hi + x_lo carries 22 significant bits, and
// A x = A_hi x_hi + A_hi x_lo + A_lo x_hi up to a term of relative size
// 2^-22; the fp16 products are exact and accumulate in fp32 (the
// split-precision scheme of Markidis et al. 2018 and Ootomo & Yokota 2022,
// without their rescaling of the low parts: the tile is scaled by a power of
// two chosen from a bound on the state's norm, so that every amplitude stays
// below 2^15 and typical ones lie far above the fp16 subnormal range; the
// blocks are unitary, so their entries are at most 1).  Complex products use
// four real ones: Re y = Ar xr - Ai xi and Im y = Ai xr + Ar xi.
//
// Work split.  A tile of 2^t amplitudes has 2^(t-4) lanes: each lane owns 16
// amplitudes of every block, as eight 16-byte accesses of two amplitudes that
// differ in position 0.  The operand layout of v_mfma_f32_16x16x32_f16 and
// its result layout are made the same by the order in which the matrix's
// columns are laid along K: lane (j, h) supplies and receives the amplitudes
// of group j whose matrix bits b2, b3 are h; b0, b1 (and b4) run over its
// registers.  So a lane writes a block's results where it read the operands
// (one address computation, no hazard between waves), and the first block of
// a run can take its operands straight from HBM and the last one can store
// its results straight to HBM: a run of n blocks makes n - 1 trips through
// LDS instead of n + 1, and a lone block none.  Where a block's own layout is a
// poor order for the memory, a parking step takes its side of the pass
// (linear_layout, split_lone).
//
// The two amplitudes of an access are two groups when position 0 is no
// target of the block, and two matrix columns (bit b0) when it is.
//
// LDS.  A tile is 2^(t-1) chunks of 16 bytes; chunk c sits at
// c ^ (c >> 3 & 7) ^ (c >> 6 & 7) ^ (c >> 9 & 7) ^ (c >> 12 & 7): linear
// over GF(2), so an address is the XOR of a per-lane, a per-wave and a
// per-access part, with no padding, and eight lanes whose three group bits
// fall into different classes modulo 3 read eight different bank groups.
//
// What bounds it: memory.  On the 30-qubit depth-14 circuit the full passes
// (16 GiB, 2 to 4 blocks) take 3.3-3.9 ms, 4.4-5.2 TB/s, with the matrix cores
// busy 19-42 %, VALU issue 21-43 % and the LDS 9-22 % of the time (0-0.12
// conflict cycles an access); a kernel that only reads and writes tiles of the
// same kind takes 3.1-4.0 ms, by where the tile's positions lie.  The
// circuit takes 26.1 ms against 29.3 ms with every block on the LDS tile
// (park, n blocks, store: 3.6-4.1 ms a pass, padded tile, 0.2-0.3 conflict
// cycles an access); sixteen circuits of 20 to 24 qubits 5.2 against 5.8 ms.
#include <atomic>
#include <cmath>

#include "sv_device.h"

namespace sv {

namespace {

constexpr int kSplitMaxOps = 8 + 2;   // blocks, and a parking step on either side

struct SplitOp {
    const float2* mat;            // row-major complex matrix (device)
    int k;                        // 0: a parking step
    int pair;                     // 1: position 0 is a target (canonical bit b0)
    int perm[5];                  // the matrix's own bit of canonical bit b_u
    int image;                    // byte offset of the operand image in LDS
    uint32_t lds_lane[6];         // LDS byte offset (XOR) of lane bit b
    uint32_t lds_m[3];            // ... of access bit b
    uint32_t lds_wave[4];         // ... of wave bit b
};

struct SplitK {
    uint64_t tiles, tmask, tstep;             // as StageK
    // amplitude offsets of the first block's loads and the last one's
    // stores: lane bits, access index, wave bits.  Loads leave out positions
    // that no operation has reached (their elements are zero and read the
    // reached one's line instead).
    uint64_t ld_lane[6], ld_m[8], ld_wave[4];
    uint64_t st_lane[6], st_m[8], st_wave[4];
    uint32_t z_lane, z_m, z_wave, z_pair;     // unreached bits of the first block's layout
    uint32_t dup;                             // lane bits without a tile bit (9-position tiles)
    int nops;
    int from_e0;                              // 1: input is |0...0>, not read
    int table;                                // byte offset of the per-lane LDS offsets
    float scale, unscale;                     // the tile's scale (a power of two) and its inverse
    double* norm_out;                         // non-null: per-workgroup FP64 sum of |psi|^2 of the result
    SplitOp op[kSplitMaxOps];
};

// register index of element e (canonical bits b0, b1 and, for k = 5, b4) of
// unit q: access m, half (the position-0 bit) of the access
template <int K, bool PAIR>
struct Lay {
    static constexpr int NU = K == 5 ? 2 : 4;           // 16-group units per wave
    static constexpr int NE = K == 5 ? 8 : 4;           // elements per lane and unit
    static constexpr int m(int e, int q)
    {
        return K == 5 ? (PAIR ? (e >> 1) | (q << 2) : e) : (PAIR ? (e >> 1) | (q << 1) : e | ((q >> 1) << 2));
    }
    static constexpr int half(int e, int q) { return PAIR ? e & 1 : q & 1; }
};

__device__ __forceinline__ f4 mma(h8 a, h8 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ h8 as_h8(u4 v) { return __builtin_bit_cast(h8, v); }
__device__ __forceinline__ h8 neg8(h8 v) { return as_h8(__builtin_bit_cast(u4, v) ^ 0x80008000u); }

// hi and lo parts of two values, packed
template <bool SCALED>
__device__ __forceinline__ void split2(float a, float b, float s, uint32_t& hi, uint32_t& lo)
{
    if (SCALED) {
        hi = cpk_hi(a, b, s);
        lo = cpk_lo(a, b, s, hi);
    } else {
        hi = pk_hi(a, b);
        lo = pk_lo(a, b, hi);
    }
}

// A lane's 16 amplitudes as MFMA operands.  k = 5: hi / lo of Re x (c = 0) and
// Im x (c = 1) of each of two units (element e = K index of a 32-deep
// product); k = 4: Re x and Im x of a unit share one product (elements 0..3,
// 4..7), four units.
struct Operands {
    u4 h[4], l[4];                           // k = 5: [2 q + c]; k = 4: [q]
};

template <int K, bool PAIR, bool SCALED>
__device__ __forceinline__ void convert(Operands& x, const f4 (&v)[8], float scale)
{
    using L = Lay<K, PAIR>;
    auto re_of = [&](int e, int q) { return v[L::m(e, q)][2 * L::half(e, q)]; };
    auto im_of = [&](int e, int q) { return v[L::m(e, q)][2 * L::half(e, q) + 1]; };
    // in the order of the accesses, so that the converted values take over
    // their registers
#pragma unroll
    for (int p = 0; p < L::NU / 2; ++p)
#pragma unroll
        for (int w = 0; w < L::NE / 2; ++w) {
#pragma unroll
            for (int q = 2 * p; q < 2 * p + 2; ++q) {
                const int ir = K == 5 ? 2 * q : q, ii = K == 5 ? 2 * q + 1 : q, wi = K == 5 ? w : 2 + w;
                uint32_t h, l;
                split2<SCALED>(re_of(2 * w, q), re_of(2 * w + 1, q), scale, h, l);
                x.h[ir][w] = h, x.l[ir][w] = l;
                split2<SCALED>(im_of(2 * w, q), im_of(2 * w + 1, q), scale, h, l);
                x.h[ii][wi] = h, x.l[ii][wi] = l;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
}

// One block on the lane's operands; out(m, y) takes access m's results.
template <int K, bool PAIR, class Out>
__device__ __forceinline__ void apply(const char* lds, int image, int lane, const Operands& x, Out out)
{
    const f4 z = {0.f, 0.f, 0.f, 0.f};
    if constexpr (K == 5) {
        const h8* a8 = (const h8*)(lds + image);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) {
            // a quarter of the operands at a time (row block, low or high
            // parts): hoisting the others' reads would exceed the 128
            // registers.  Small terms first; four independent chains
            // interleave.
            f4 re[2], im[2];
            if (rb) __builtin_amdgcn_sched_barrier(0);
            {
                const h8 rl = a8[(rb * 4 + 1) * 64 + lane], il = a8[(rb * 4 + 3) * 64 + lane];
                const h8 nl = neg8(il);
#pragma unroll
                for (int q = 0; q < 2; ++q) re[q] = mma(rl, as_h8(x.h[2 * q]), z), im[q] = mma(il, as_h8(x.h[2 * q]), z);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    re[q] = mma(nl, as_h8(x.h[2 * q + 1]), re[q]), im[q] = mma(rl, as_h8(x.h[2 * q + 1]), im[q]);
            }
            __builtin_amdgcn_sched_barrier(0);
            {
                const h8 rh = a8[(rb * 4 + 0) * 64 + lane], ih = a8[(rb * 4 + 2) * 64 + lane];
                const h8 nh = neg8(ih);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    re[q] = mma(rh, as_h8(x.l[2 * q]), re[q]), im[q] = mma(ih, as_h8(x.l[2 * q]), im[q]);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    re[q] = mma(nh, as_h8(x.l[2 * q + 1]), re[q]), im[q] = mma(rh, as_h8(x.l[2 * q + 1]), im[q]);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    re[q] = mma(rh, as_h8(x.h[2 * q]), re[q]), im[q] = mma(ih, as_h8(x.h[2 * q]), im[q]);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    re[q] = mma(nh, as_h8(x.h[2 * q + 1]), re[q]), im[q] = mma(rh, as_h8(x.h[2 * q + 1]), im[q]);
            }
            if (PAIR) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        out(u | (rb << 1) | (q << 2),
                            f4{re[q][2 * u], im[q][2 * u], re[q][2 * u + 1], im[q][2 * u + 1]});
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) out(u | (rb << 2), f4{re[0][u], im[0][u], re[1][u], im[1][u]});
            }
        }
    } else {
        const u2* a4 = (const u2*)(lds + image);
        const u2 rh = a4[0 * 64 + lane], rl = a4[1 * 64 + lane], ih = a4[2 * 64 + lane], il = a4[3 * 64 + lane];
        const uint32_t sg = 0x80008000u;
        const h8 reh = as_h8(u4{rh.x, rh.y, ih.x ^ sg, ih.y ^ sg}), rel = as_h8(u4{rl.x, rl.y, il.x ^ sg, il.y ^ sg});
        const h8 imh = as_h8(u4{ih.x, ih.y, rh.x, rh.y}), iml = as_h8(u4{il.x, il.y, rl.x, rl.y});
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            f4 re[2], im[2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
                re[q] = mma(rel, as_h8(x.h[2 * p + q]), z), im[q] = mma(iml, as_h8(x.h[2 * p + q]), z);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                re[q] = mma(reh, as_h8(x.l[2 * p + q]), re[q]), im[q] = mma(imh, as_h8(x.l[2 * p + q]), im[q]);
#pragma unroll
            for (int q = 0; q < 2; ++q)
                re[q] = mma(reh, as_h8(x.h[2 * p + q]), re[q]), im[q] = mma(imh, as_h8(x.h[2 * p + q]), im[q]);
            if (PAIR) {
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        out(u | ((2 * p + q) << 1),
                            f4{re[q][2 * u], im[q][2 * u], re[q][2 * u + 1], im[q][2 * u + 1]});
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) out(u | (p << 2), f4{re[0][u], im[0][u], re[1][u], im[1][u]});
            }
        }
    }
}

// s_waitcnt operands: at most 0 / 8 vector memory operations outstanding
constexpr int kWaitLoads0 = 0x0f70, kWaitLoads8 = 0x0f78;

// The kernel's LDS is one dynamic block starting at offset 0 (it declares no
// other), so LDS addresses are plain 32-bit offsets.
typedef __attribute__((address_space(3))) f4 lds_f4;
__device__ __forceinline__ f4 lds_get(uint32_t at) { return *(const lds_f4*)(uintptr_t)at; }
__device__ __forceinline__ void lds_put(uint32_t at, f4 x) { *(lds_f4*)(uintptr_t)at = x; }

// keeps a block form's reads inside its own branch: merged with the other
// forms' they would be converted piecemeal, in more registers
template <int K, bool PAIR>
__device__ __forceinline__ uint32_t own(uint32_t at)
{
    asm volatile("; block form %1 %2" : "+v"(at) : "i"(K), "i"((int)PAIR));
    return at;
}

// lanes of a workgroup for a tile of t positions
constexpr int split_lanes(int t) { return t <= 10 ? 64 : 1 << (t - 4); }

// Sixteen waves per CU (four per SIMD, 128 VGPRs each): one workgroup of 1024
// lanes at t = 14, two of 512 at 13, and so on, as far as their matrices leave
// the LDS room; eight waves at most at t = 9 and 10, of one wave each.
// K0, P0: the first block's width and whether position 0 is one of its
// targets; ONE: it is the only one.  (Compile-time choices: the prefetched
// operands then stay in one set of registers round the tile loop, where
// several variants of that block in one kernel had copied them, and waited
// for the loads to do so, or spilled.)
template <int TW, bool ZERO, int K0, bool P0, bool ONE>
__global__ __launch_bounds__(split_lanes(TW), 4) void k_split(float2* __restrict__ psi, SplitK a)
{
    constexpr int NT = split_lanes(TW);
    extern __shared__ f4 split_smem[];
    char* lds = (char*)split_smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    uint64_t ldl = 0, stl = 0, ldw = 0, stw = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) ldl |= a.ld_lane[b], stl |= a.st_lane[b];
#pragma unroll
    for (int b = 0; b < 4; ++b)
        if ((wave >> b) & 1) ldw |= a.ld_wave[b], stw |= a.st_wave[b];
    // elements of this lane on positions no operation has reached are zero
    const bool zl = ZERO && ((lane & a.z_lane) | (wave & a.z_wave)) != 0;
    f4 raw[8];
    auto load_tile = [&](uint64_t base_index, bool read) {
        if (read) {
            const float2* base = psi + (base_index | ldw);
#pragma unroll
            for (int m = 0; m < 8; ++m) raw[m] = __builtin_nontemporal_load((const f4*)(base + a.ld_m[m] + ldl));
        } else {
#pragma unroll
            for (int m = 0; m < 8; ++m) raw[m] = f4{0.f, 0.f, 0.f, 0.f};
        }
    };
    uint64_t tile = blockIdx.x;
    uint64_t tb = spread_bits(tile, a.tmask);
    load_tile(tb, !a.from_e0);                           // (the grid has no more workgroups than tiles)
    if (a.from_e0 && tile == 0 && (threadIdx.x & ~a.dup) == 0) raw[0][0] = 1.f;
    // every block's operands, split and in operand order, and the lanes' LDS
    // offsets: once per workgroup
    for (int o = 0; o < a.nops; ++o) {
        const SplitOp& op = a.op[o];
        const int k = op.k, D = 1 << k;
        const float2* mat = op.mat;
        for (int i = threadIdx.x; k && i < 4 * D; i += NT) {
            const int R = i & (D - 1), g = i >> k;
            int row = 0;
#pragma unroll
            for (int u = 0; u < 5; ++u) row |= ((R >> u) & 1) << op.perm[u];
            const float2* src = mat + row * D + (((g & 1) << op.perm[2]) | ((g >> 1) << op.perm[3]));
            u4 rh, rl, ih, il;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                rh[w] = rl[w] = ih[w] = il[w] = 0;
                if (k == 5 || w < 2) {
                    const int c = ((w & 1) << op.perm[1]) | ((w >> 1) << op.perm[4]);
                    const float2 m0 = src[c], m1 = src[c | (1 << op.perm[0])];
                    uint32_t h, l;
                    split2<false>(m0.x, m1.x, 1.f, h, l);
                    rh[w] = h, rl[w] = l;
                    split2<false>(m0.y, m1.y, 1.f, h, l);
                    ih[w] = h, il[w] = l;
                }
            }
            if (k == 5) {
                u4* dst = (u4*)(lds + op.image) + (R >> 4) * 256 + (R & 15) + 16 * g;
                dst[0] = rh, dst[64] = rl, dst[128] = ih, dst[192] = il;
            } else {
                u2* dst = (u2*)(lds + op.image) + R + 16 * g;
                dst[0] = u2{rh.x, rh.y}, dst[64] = u2{rl.x, rl.y};
                dst[128] = u2{ih.x, ih.y}, dst[192] = u2{il.x, il.y};
            }
        }
        if (threadIdx.x < 64) {
            uint32_t x = 0;
#pragma unroll
            for (int b = 0; b < 6; ++b)
                if ((lane >> b) & 1) x ^= op.lds_lane[b];
            ((uint32_t*)(lds + a.table))[o * 64 + lane] = x;
        }
    }
    __syncthreads();
    auto address = [&](int o) {
        const SplitOp& op = a.op[o];
        uint32_t w = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) w ^= op.lds_wave[b] & (0u - (uint32_t)((wave >> b) & 1));
        return ((const uint32_t*)(lds + a.table))[o * 64 + lane] ^ w;
    };
    auto offset = [&](int o, int m) {
        const SplitOp& op = a.op[o];
        return ((m & 1) ? op.lds_m[0] : 0u) ^ ((m & 2) ? op.lds_m[1] : 0u) ^ ((m & 4) ? op.lds_m[2] : 0u);
    };
    auto read = [&](int o, uint32_t at, f4(&v)[8]) {
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = lds_get(at ^ offset(o, m));
    };
    double nacc = 0.0;                                   // this lane's sum of |psi|^2
    auto store = [&](int m, f4 x) {
        const float r = a.unscale;
        const f4 y = {x[0] * r, x[1] * r, x[2] * r, x[3] * r};
        __builtin_nontemporal_store(y, (f4*)(psi + (tb | stw) + a.st_m[m] + stl));
        if (a.norm_out) {
#pragma unroll
            for (int c = 0; c < 4; ++c) nacc = fma((double)y[c], (double)y[c], nacc);
        }
    };
    using c0 = std::integral_constant<int, 0>;
    using c4 = std::integral_constant<int, 4>;
    using c5 = std::integral_constant<int, 5>;
    auto form = [&](int o, auto&& f) {
        const int ty = (a.op[o].k == 5 ? 2 : 0) | a.op[o].pair;
        switch (ty) {
            case 0: f(c4{}, std::false_type{}); break;
            case 1: f(c4{}, std::true_type{}); break;
            case 2: f(c5{}, std::false_type{}); break;
            case 3: f(c5{}, std::true_type{}); break;
            default: __builtin_unreachable();
        }
    };
    uint64_t nb = tb;                                    // the tile in the registers, then in flight
    bool next = true;
    // the loaded tile's operands (elements never reached as zeros), the next
    // tile's loads, and every block but the last one
    auto head = [&](auto out0) {
        if (ZERO) {
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const bool zm = zl || (m & a.z_m);
                if (zm) raw[m][0] = raw[m][1] = 0.f;
                if (zm || a.z_pair) raw[m][2] = raw[m][3] = 0.f;
            }
        }
        Operands x0;
        if constexpr (K0 == 0) {
            const float r = a.scale;
#pragma unroll
            for (int m = 0; m < 8; ++m) out0(m, f4{raw[m][0] * r, raw[m][1] * r, raw[m][2] * r, raw[m][3] * r});
            __builtin_amdgcn_sched_barrier(0);
        } else {
            convert<K0, P0, true>(x0, raw, a.scale);
        }
        nb = ((tb | ~a.tmask) + a.tstep) & a.tmask;
        tile += gridDim.x;
        next = tile < a.tiles;
        __builtin_amdgcn_s_setprio(1);
        load_tile(nb, next && !a.from_e0);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (K0 != 0) apply<K0, P0>(lds, a.op[0].image, lane, x0, out0);
    };
    // the first tile's loads end here, as every later tile's do at the loop's
    // end: waits inside the loop then never cover the stores
    __builtin_amdgcn_s_waitcnt(kWaitLoads0);
    for (;;) {
        if constexpr (ONE) {
            head(store);
        } else {
            const uint32_t at0 = address(0);
            head([&](int m, f4 y) { lds_put(at0 ^ offset(0, m), y); });
            __syncthreads();
            for (int o = 1; o + 1 < a.nops; ++o) {
                form(o, [&](auto kk, auto pp) {
                    const uint32_t at = own<decltype(kk)::value, decltype(pp)::value>(address(o));
                    f4 v[8];
                    Operands x;
                    read(o, at, v);
                    convert<decltype(kk)::value, decltype(pp)::value, false>(x, v, 1.f);
                    apply<decltype(kk)::value, decltype(pp)::value>(
                        lds, a.op[o].image, lane, x, [&](int m, f4 y) { lds_put(at ^ offset(o, m), y); });
                });
                __syncthreads();
            }
            const int o = a.nops - 1;
            auto tail = [&](auto kk, auto pp) {
                constexpr int K = decltype(kk)::value;
                f4 v[8];
                read(o, own<K, decltype(pp)::value>(address(o)), v);
                __syncthreads();                         // the tile may be overwritten
                if constexpr (K == 0) {
#pragma unroll
                    for (int m = 0; m < 8; ++m) store(m, v[m]);
                } else {
                    Operands x;
                    convert<K, decltype(pp)::value, false>(x, v, 1.f);
                    apply<K, decltype(pp)::value>(lds, a.op[o].image, lane, x, store);
                }
            };
            if (a.op[o].k == 0) tail(c0{}, std::false_type{});
            else form(o, tail);
        }
        if (!next) break;
        tb = nb;
        // the next tile's loads are older than this tile's eight stores
        __builtin_amdgcn_s_waitcnt(kWaitLoads8);
    }
    if (a.norm_out) {
        // fixed-order tree over the workgroup's lanes (lanes whose bits are not
        // all tile bits repeat others)
        if (lane & a.dup) nacc = 0.0;
        __syncthreads();
        double* sh = (double*)lds;
        sh[threadIdx.x] = nacc;
        __syncthreads();
        for (int h = NT / 2; h > 0; h >>= 1) {
            if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) a.norm_out[blockIdx.x] = sh[0];
    }
}

using SplitKernel = void (*)(float2*, SplitK);

template <int TW, bool ZERO, bool ONE>
SplitKernel split_kernel_t(int k, int pair)
{
    if constexpr (!ONE)
        if (k == 0) return k_split<TW, ZERO, 0, false, false>;
    if (k == 5) return pair ? k_split<TW, ZERO, 5, true, ONE> : k_split<TW, ZERO, 5, false, ONE>;
    return pair ? k_split<TW, ZERO, 4, true, ONE> : k_split<TW, ZERO, 4, false, ONE>;
}

SplitKernel split_kernel(int t, bool zero, int k, int pair, bool one)
{
    switch (t) {
#define SV_SPLIT_CASE(T)                                                                                \
    case T:                                                                                             \
        if (one) return zero ? split_kernel_t<T, true, true>(k, pair) : split_kernel_t<T, false, true>(k, pair); \
        return zero ? split_kernel_t<T, true, false>(k, pair) : split_kernel_t<T, false, false>(k, pair);
        SV_SPLIT_CASE(9)
        SV_SPLIT_CASE(10)
        SV_SPLIT_CASE(11)
        SV_SPLIT_CASE(12)
        SV_SPLIT_CASE(13)
        SV_SPLIT_CASE(14)
#undef SV_SPLIT_CASE
    }
    return nullptr;
}

// Where the t tile bits of one block go: lane bits (j0..j3, then canonical
// b2, b3), access bits, wave bits; -1 = none.
struct SplitLayout {
    int lane[6], m[3], wave[4];
    int perm[5];
    int pair;
};

// A parking step (the tile copied to or from LDS before the first or after the
// last block): lanes, then waves, then accesses by ascending tile bits, so that
// at any time the workgroup reads or writes one contiguous stretch.  For blocks
// whose own layout makes half-line accesses (split_narrow): alone on 2^30
// amplitudes 4.0-4.1 ms without, 3.3 with it after the block, 2.94 with both;
// for other first and last blocks the trips through LDS cost more than the
// order gives (30 qubits, depth 14: 25.96 ms without, 27.1 with it in front,
// 26.9 behind, 28.3 both).
SplitLayout linear_layout(int t)
{
    SplitLayout L;
    for (int& x : L.lane) x = -1;
    for (int& x : L.m) x = -1;
    for (int& x : L.wave) x = -1;
    for (int u = 0; u < 5; ++u) L.perm[u] = 0;
    L.pair = 0;
    int b = 1;
    for (int i = 0; i < 6; ++i)
        if (t > 9 || i != 3) L.lane[i] = b++;            // (9 positions: lane bit 3 is spare, as for blocks)
    for (int i = 0; b < t - 3; ++i) L.wave[i] = b++;
    for (int i = 0; i < 3; ++i) L.m[i] = b++;
    return L;
}

// targets: tile bit of each matrix bit.  Matrix bits: the target at tile bit
// 0 is b0; of the others the two lowest are b2, b3 (lane bits, so that an
// access spans as much contiguous memory as it can), the rest b0, b1, b4.
// Group bits: blocks that touch HBM take the lowest free tile bits, again
// for contiguous accesses; blocks inside a run take three free bits of
// different classes modulo 3 (see the chunk order above).
SplitLayout split_layout(int t, int k, const int* tbit, bool hbm)
{
    SplitLayout L;
    for (int& x : L.lane) x = -1;
    for (int& x : L.m) x = -1;
    for (int& x : L.wave) x = -1;
    for (int u = 0; u < 5; ++u) L.perm[u] = 0;
    bool target[64] = {};
    int rest[5], nr = 0;
    L.pair = 0;
    int b0 = -1;
    for (int b = 0; b < t; ++b)
        for (int j = 0; j < k; ++j)
            if (tbit[j] == b) {
                target[b] = true;
                if (b == 0) L.pair = 1, b0 = j;
                else rest[nr++] = j;
            }
    int canon[5];
    canon[2] = rest[0], canon[3] = rest[1];
    if (L.pair) {
        canon[0] = b0, canon[1] = rest[2], canon[4] = k == 5 ? rest[3] : 0;
    } else {
        canon[0] = rest[2], canon[1] = rest[3], canon[4] = k == 5 ? rest[4] : 0;
    }
    for (int u = 0; u < k; ++u) L.perm[u] = canon[u];
    L.lane[4] = tbit[canon[2]], L.lane[5] = tbit[canon[3]];
    int nm = 0;
    if (!L.pair) L.m[nm++] = tbit[canon[0]];
    L.m[nm++] = tbit[canon[1]];
    if (k == 5) L.m[nm++] = tbit[canon[4]];
    int fr[64], nf = 0;                       // free tile bits but 0, ascending
    for (int b = 1; b < t; ++b)
        if (!target[b]) fr[nf++] = b;
    const int nu = 3 - nm, nj = nf - nu < 4 ? nf - nu : 4;
    // the group bits' pool: all free bits, or the lowest nj
    const int pool = hbm ? nj : nf;
    bool used[64] = {};
    int got = 0;
    for (int cls = 0; cls < 3 && got < nj; ++cls)
        for (int i = 0; i < pool; ++i)
            if (!used[fr[i]] && (fr[i] - 1) % 3 == cls) {
                used[fr[i]] = true;
                L.lane[got++] = fr[i];
                break;
            }
    for (int i = 0; i < pool && got < nj; ++i)
        if (!used[fr[i]]) {
            used[fr[i]] = true;
            L.lane[got++] = fr[i];
        }
    int nw = 0;
    for (int i = 0; i < nf; ++i) {
        if (used[fr[i]]) continue;
        if (nm < 3) L.m[nm++] = fr[i];
        else L.wave[nw++] = fr[i];
    }
    return L;
}

// LDS byte offset of tile bit b (b >= 1; bit 0 is inside a 16-byte chunk)
uint32_t split_chunk(int b)
{
    if (b < 1) return 0;
    const int c = b - 1;
    return ((1u << c) | (c >= 3 ? 1u << (c % 3) : 0u)) * 16u;
}

// A block on all of positions 1, 2, 3: an access of a wave then reads or writes
// 64 contiguous bytes at a time (the two lowest targets are lane bits, the
// third is not), half a cache line.
bool split_narrow(int k, const int* pos)
{
    int low = 0;
    for (int j = 0; j < k; ++j)
        if (pos[j] >= 1 && pos[j] <= 3) low |= 1 << pos[j];
    return low == 14;
}

// amplitudes (as bits) from which a lone block's pass is parked, narrowed, or
// wider than the default limit
constexpr int kLoneBits = 27, kLoneNarrowBits = 24, kLoneWideBits = 28;

}  // namespace

// A pass of one block.  What it costs is the order in which it touches memory:
// on the block's own layout the waves of a wide tile hold accesses whose
// addresses agree in the bits that choose the memory channel.  Parked on both
// sides, a 14-position tile is read and written as one stretch of 128 KiB;
// without that width, short tiles spread over more workgroups do better.  Mean
// over 12 sets of targets (direct, 13 positions -> direct, 12 -> parked, 13 ->
// parked, 14): 2^30 amplitudes, 5 qubits 3,482 -> 3,355 -> 3,352 -> 3,178 us, 4
// qubits 3,472 -> 3,447 -> 3,332 -> 3,176; 2^25, 5 qubits 124 -> 119 -> 121 ->
// 122, 4 qubits 116 -> 110 -> 111 -> 114; 2^22 32.1 and 25.4 direct against 35
// and 27 parked.
//
// Where the caller left the tile limit at its default of 13, a block of 5 qubits
// on a large state takes 14 positions all the same: direct, 12, is as fast as
// parked, 13, on average, but up to a fifth slower for single sets of targets.
// 32 sets each, mean and slowest set against parked 13-position tiles with the
// block on LDS (direct, 12 -> parked, 14): 2^27 437 us: 417, 0.93 -> 428, 0.94;
// 2^28 853: 859, 0.83 -> 831, 0.91; 2^29 1,758: 1,683, 0.85 -> 1,637, 0.91; 2^30
// 3,465: 3,435, 0.83 -> 3,267, 0.93.  4 qubits (parked, 13 -> parked, 14): 2^29
// 1,668: 1,612, 0.92 -> 1,591, 0.89; 2^30 3,449: 3,317, 1.00 -> 3,239, 0.95.
SplitLone split_lone(int k, const int* pos, int bits, int t_max, int wide_max)
{
    if (bits < kLoneNarrowBits || split_narrow(k, pos)) return {t_max, false};
    if (bits >= kLoneBits && t_max >= 14) return {14, true};
    if (bits >= kLoneWideBits && k == 5 && wide_max >= 14) return {14, true};
    if (bits >= kLoneBits && k == 4 && t_max >= 13) return {13, true};
    return {t_max < 12 ? t_max : 12, false};
}

hipError_t split_prepare(int t, int v)
{
    static std::atomic<bool> done[6][kSplitForms];
    if (done[t - 9][v]) return hipSuccess;
    const SplitKernel kern = v < 16 ? split_kernel(t, v & 1, v & 2 ? 5 : 4, (v >> 2) & 1, v & 8)
                                    : split_kernel(t, v & 1, 0, 0, false);
    const hipError_t e =
        hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, stage_lds_limit(t));
    if (e == hipSuccess) done[t - 9][v] = true;
    return e;
}

hipError_t launch_split(hipStream_t st, void* psi, int t, const int* P, int nops, const int* ks,
                        const int* const* pos, const void* const* mats, uint64_t tiles, uint64_t tmask,
                        uint64_t newmask, bool from_e0, double* norm_out, int* norm_blocks, int split_exp, bool park)
{
    if (t < 9 || t > 14 || nops < 1 || nops > kSplitMaxOps - 2) return hipErrorInvalidValue;
    // sides that go through a parking step
    bool in = park || split_narrow(ks[0], pos[0]), out = park || split_narrow(ks[nops - 1], pos[nops - 1]);
    {
        int need = (8 << t) + (nops + 2) * 256;
        for (int o = 0; o < nops; ++o) need += 8 << (2 * ks[o]);
        if (need > (t >= 14 ? 160 : 80) * 1024) in = out = false;
    }
    SplitK a{};
    a.tiles = tiles;
    a.tmask = tmask;
    const int steps = nops + in + out;
    a.nops = steps;
    a.from_e0 = from_e0 ? 1 : 0;
    a.norm_out = norm_out;
    a.scale = std::ldexp(1.0f, split_exp);
    a.unscale = std::ldexp(1.0f, -split_exp);
    int at = 8 << t;
    for (int o = 0; o < steps; ++o) {
        const int blk = o - in;
        const bool park = blk < 0 || blk >= nops;
        int tbit[kMaxDense];
        for (int j = 0; !park && j < ks[blk]; ++j) {
            int b = 0;
            while (b < t && P[b] != pos[blk][j]) ++b;
            if (b == t) return hipErrorInvalidValue;
            tbit[j] = b;
        }
        const bool hbm = o == 0 || o == steps - 1;
        const SplitLayout L = park ? linear_layout(t) : split_layout(t, ks[blk], tbit, hbm);
        SplitOp& op = a.op[o];
        op.mat = park ? nullptr : (const float2*)mats[blk];
        op.k = park ? 0 : ks[blk];
        op.pair = L.pair;
        for (int u = 0; u < 5; ++u) op.perm[u] = L.perm[u];
        op.image = at;
        if (!park) at += 8 << (2 * ks[blk]);
        for (int b = 0; b < 6; ++b) op.lds_lane[b] = split_chunk(L.lane[b]);
        for (int b = 0; b < 3; ++b) op.lds_m[b] = split_chunk(L.m[b]);
        for (int b = 0; b < 4; ++b) op.lds_wave[b] = split_chunk(L.wave[b]);
        auto where = [&](int b) { return b < 0 ? 0ull : 1ull << P[b]; };
        if (o == 0) {
            auto reached = [&](int b) { return where(b) & ~newmask; };
            auto fresh = [&](int b) { return (where(b) & newmask) != 0; };
            for (int b = 0; b < 6; ++b) {
                a.ld_lane[b] = reached(L.lane[b]);
                if (fresh(L.lane[b])) a.z_lane |= 1u << b;
                if (L.lane[b] < 0) a.dup |= 1u << b;
            }
            for (int b = 0; b < 4; ++b) {
                a.ld_wave[b] = reached(L.wave[b]);
                if (fresh(L.wave[b])) a.z_wave |= 1u << b;
            }
            for (int b = 0; b < 3; ++b)
                if (fresh(L.m[b])) a.z_m |= 1u << b;
            for (int m = 0; m < 8; ++m)
                for (int b = 0; b < 3; ++b)
                    if ((m >> b) & 1) a.ld_m[m] |= reached(L.m[b]);
            a.z_pair = (newmask >> P[0]) & 1;
        }
        if (o == steps - 1) {
            for (int b = 0; b < 6; ++b) a.st_lane[b] = where(L.lane[b]);
            for (int b = 0; b < 4; ++b) a.st_wave[b] = where(L.wave[b]);
            for (int m = 0; m < 8; ++m)
                for (int b = 0; b < 3; ++b)
                    if ((m >> b) & 1) a.st_m[m] |= where(L.m[b]);
        }
    }
    a.table = at;
    const int lds = at + steps * 256;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const int nt = split_lanes(t);
    // persistent: as many workgroups as are resident (sixteen waves per CU,
    // or what the LDS holds)
    int per_cu = (160 * 1024) / lds;
    if (per_cu > 1024 / nt) per_cu = 1024 / nt;
    if (per_cu > 8) per_cu = 8;
    uint64_t grid = a.tiles;
    const uint64_t cap = 256ull * per_cu;
    if (grid > cap) grid = cap;
    a.tstep = spread_bits(grid, a.tmask);
    const bool zero = newmask != 0, one = steps == 1;
    const int k0 = a.op[0].k, pair0 = a.op[0].pair;
    const hipError_t e = split_prepare(t, (k0 ? (k0 == 5 ? 2 : 0) | pair0 << 2 | (one ? 8 : 0) : 16) | (zero ? 1 : 0));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(split_kernel(t, zero, k0, pair0, one), dim3((unsigned)grid), dim3(nt), lds, st, (float2*)psi, a);
    if (norm_blocks) *norm_blocks = norm_out ? (int)grid : 0;
    return hipGetLastError();
}

}  // namespace sv
