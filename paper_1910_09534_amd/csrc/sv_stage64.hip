// Staged sweep of complex128 blocks (Sec. 5 computes in double): a run of
// dense 4/5-qubit blocks applied to LDS-resident tiles in one pass over HBM
// (see sv_stage.hip for tiles and supports), every product on the FP64 matrix
// cores as three real ones (3M: P1 = Ar xr, P2 = Ai xi, P3 = (Ar + Ai)(xr + xi);
// Re y = P1 - P2, Im y = P3 - P1 - P2).
//
// Work split.  A tile of 2^t amplitudes has 2^(t-4) lanes; each lane owns 16
// amplitudes of every block, one per 16-byte access.
// v_mfma_f64_16x16x4f64 takes operand (k = h) and gives result row h + 4 v in
// lane (j, h), so lane (j, h) supplies and receives the amplitudes of group j
// whose matrix bits b0, b1 are h; b2, b3 (and b4) run over its registers.  So a
// lane writes a block's results where it read the operands, the first block of
// a run takes its operands straight from HBM and the last one stores its
// results straight to HBM: a run of n blocks makes n - 1 trips through LDS
// instead of n + 1.  b0, b1 are the two lowest targets and the group bits of
// these two blocks the lowest free tile bits, for contiguous accesses.
//
// The first block's operands stay in their registers until its products have
// read them; the next tile's loads then go into the same registers, a unit
// (16 groups) at a time, and are in flight during all the other blocks.
//
// What bounds it: two blocks of 5 and 4 qubits, memory (450 us for 2 x 1 GiB,
// 4.8 TB/s; a lone 5-qubit sweep takes 424); four blocks of 4 qubits, the time
// round the barriers: a block takes 8,700 cycles, of them 6,144 of matrix-core
// work (64 cycles an instruction, eight 16-group units a SIMD), the rest the
// first operands after a barrier and the last results before it, which both
// waves of a SIMD meet together (540-570 us a pass).  26 qubits, depth 14:
// 4,917 us with every block on the LDS tile (park, n blocks, store), 4,265 us
// here.  Four real products instead of three take 10,460 cycles a block; the
// results of a unit formed beside the next one's products, 8,660 and spills,
// whose reloads wait for all loads in flight (640 us a pass).
//
// LDS.  Amplitude i of the tile sits at i ^ (i >> 3 & 7) ^ (i >> 6 & 7) ^
// (i >> 9 & 7) ^ (i >> 12 & 7): linear over GF(2) and without padding, as in
// the split-fp16 form.
#include <atomic>
#include <type_traits>

#include "sv_device.h"

namespace sv {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double dd2 __attribute__((ext_vector_type(2)));

constexpr int kMaxOps64 = 8;

struct Op64 {
    const double2* mat;           // row-major complex matrix (device)
    int k;
    int perm[5];                  // the matrix's own bit of canonical bit b_u
    int image;                    // byte offset of the operand image in LDS
    uint32_t lds_lane[6];         // LDS byte offset (XOR) of lane bit b
    uint32_t lds_m[4];            // ... of access bit b
    uint32_t lds_wave[3];         // ... of wave bit b
};

struct Stage64K {
    uint64_t tiles, tmask, tstep;             // as StageK
    // amplitude offsets of the first block's loads and the last one's stores:
    // lane bits, access index, wave bits.  Loads leave out positions that no
    // operation has reached (their elements are zero and read the reached
    // one's line instead).
    uint64_t ld_lane[6], ld_m[16], ld_wave[3];
    uint64_t st_lane[6], st_m[16], st_wave[3];
    uint32_t z_lane, z_m, z_wave;             // unreached bits of the first block's layout
    uint32_t dup;                             // lane bits without a tile bit (9-position tiles)
    int nops;
    int from_e0;                              // 1: input is |0...0>, not read
    int table;                                // byte offset of the per-lane LDS offsets
    double* norm_out;                         // non-null: per-workgroup sum of |psi|^2 of the result
    Op64 op[kMaxOps64];
};

// LDS addresses are plain 32-bit offsets: one dynamic block, starting at 0
typedef __attribute__((address_space(3))) dd2 lds_dd2;
__device__ __forceinline__ dd2 lds_get(uint32_t at) { return *(const lds_dd2*)(uintptr_t)at; }
__device__ __forceinline__ void lds_put(uint32_t at, dd2 x) { *(lds_dd2*)(uintptr_t)at = x; }

// s_waitcnt operands: at most 0 / 16 vector memory operations outstanding
constexpr int kWait64Loads0 = 0x0f70, kWait64Loads16 = 0x4f70;

// keeps a block form's reads inside its own branch
template <int K>
__device__ __forceinline__ uint32_t own(uint32_t at)
{
    asm volatile("; block form %1" : "+v"(at) : "i"(K));
    return at;
}

// One block on the lane's 16 amplitudes (access m = element | unit << (K - 2)):
// get(m) gives access m's operand, out(m, y) takes its result, done(q) follows
// when unit q's operands have been used for the last time.  A unit's operands
// are fetched during the products of the one before.
template <int K, class Get, class Out, class Done>
__device__ __forceinline__ void apply64(uint32_t image, int lane, Get get, Out out, Done done)
{
    constexpr int D = 1 << K, RB = D / 16, KQ = D / 16, NE = D / 4, NU = 16 / NE;
    // operand image: [part][row block][step pair][lane] of two doubles
    const uint32_t at = image + 16 * lane;
    dd2 x[16];
    auto fetch = [&](int q) {
#pragma unroll
        for (int s = 0; s < NE; ++s) x[s | (q << (K - 2))] = get(s | (q << (K - 2)));
    };
    fetch(0);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        double ar[NE], ai[NE], as[NE];
#pragma unroll
        for (int s2 = 0; s2 < 2 * KQ; ++s2) {
            const dd2 r = lds_get(at + ((0 * RB + rb) * 2 * KQ + s2) * 1024);
            const dd2 i = lds_get(at + ((1 * RB + rb) * 2 * KQ + s2) * 1024);
            ar[2 * s2] = r.x, ar[2 * s2 + 1] = r.y;
            ai[2 * s2] = i.x, ai[2 * s2 + 1] = i.y;
            as[2 * s2] = r.x + i.x, as[2 * s2 + 1] = r.y + i.y;
        }
#pragma unroll
        for (int q = 0; q < NU; ++q) {
            if (rb == 0 && q + 1 < NU) {
                fetch(q + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            d4 p1 = {0.0, 0.0, 0.0, 0.0}, p2 = p1, p3 = p1;
#pragma unroll
            for (int s = 0; s < NE; ++s) {
                const dd2 v = x[s | (q << (K - 2))];
                p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[s], v.x, p1, 0, 0, 0);
                p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[s], v.y, p2, 0, 0, 0);
                p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(as[s], v.x + v.y, p3, 0, 0, 0);
            }
            if (rb == RB - 1) done(q);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                out((v + 4 * rb) | (q << (K - 2)), dd2{p1[v] - p2[v], p3[v] - p1[v] - p2[v]});
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// lanes of a workgroup for a tile of t positions
constexpr int stage64_lanes(int t) { return t <= 10 ? 64 : 1 << (t - 4); }

// Up to eight waves per CU (two per SIMD, 256 VGPRs each): one workgroup of 512
// lanes at t = 13, two of 256 at 12 where two tiles and their matrices fit the
// LDS (four 4-qubit blocks do not: four waves), and so on.  K0:
// the first block's width; ONE: it is the only one.  (Compile-time choices, so
// that the operands in flight stay in one set of registers round the loop.)
template <int TW, bool ZERO, int K0, bool ONE>
__global__ __launch_bounds__(stage64_lanes(TW), 2) void k_stage64(double2* __restrict__ psi, Stage64K a)
{
    constexpr int NT = stage64_lanes(TW);
    extern __shared__ dd2 smem64[];
    char* lds = (char*)smem64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    uint64_t ldl = 0, stl = 0, ldw = 0, stw = 0;
#pragma unroll
    for (int b = 0; b < 6; ++b)
        if ((lane >> b) & 1) ldl |= a.ld_lane[b], stl |= a.st_lane[b];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        if ((wave >> b) & 1) ldw |= a.ld_wave[b], stw |= a.st_wave[b];
    // elements of this lane on positions no operation has reached are zero
    const bool zl = ZERO && ((lane & a.z_lane) | (wave & a.z_wave)) != 0;
    constexpr int NE0 = 1 << (K0 - 2);                   // elements per unit of the first block
    dd2 raw[16];
    auto load_unit = [&](int q, uint64_t base_index, bool read) {
        if (read) {
            const double2* base = psi + (base_index | ldw);
#pragma unroll
            for (int m = q * NE0; m < (q + 1) * NE0; ++m)
                raw[m] = __builtin_nontemporal_load((const dd2*)(base + a.ld_m[m] + ldl));
        } else {
#pragma unroll
            for (int m = q * NE0; m < (q + 1) * NE0; ++m) raw[m] = dd2{0.0, 0.0};
        }
    };
    uint64_t tile = blockIdx.x;
    uint64_t tb = spread_bits(tile, a.tmask);
#pragma unroll
    for (int q = 0; q < 16 / NE0; ++q) load_unit(q, tb, !a.from_e0);   // (no more workgroups than tiles)
    if (a.from_e0 && tile == 0 && (threadIdx.x & ~a.dup) == 0) raw[0].x = 1.0;
    // every block's operand image and the lanes' LDS offsets: once per workgroup
    for (int o = 0; o < a.nops; ++o) {
        const Op64& op = a.op[o];
        const int k = op.k, RB = 1 << (k - 4);
        for (int i = threadIdx.x; i < 1 << (2 * k); i += NT) {
            // i = [row block][step pair][lane][step of the pair]
            const int l = (i >> 1) & 63, s = ((i >> 7) & (2 * RB - 1)) * 2 + (i & 1), rb = i >> (7 + 1 + (k - 4));
            const int R = 16 * rb + (l & 15), C = 4 * s + (l >> 4);
            int row = 0, col = 0;
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                row |= ((R >> u) & 1) << op.perm[u];
                col |= ((C >> u) & 1) << op.perm[u];
            }
            const double2 v = op.mat[(row << k) + col];
            double* dst = (double*)(lds + op.image) + i;
            dst[0] = v.x;
            dst[1 << (2 * k)] = v.y;
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
    // a block's place in LDS: looked up before the barrier in front of it (the
    // asm keeps it there)
    struct Place {
        uint32_t at, image, m[4];
        int k;
    };
    auto place = [&](int o) {
        const Op64& op = a.op[o];
        uint32_t w = 0;
#pragma unroll
        for (int b = 0; b < 3; ++b) w ^= op.lds_wave[b] & (0u - (uint32_t)((wave >> b) & 1));
        Place p;
        p.at = ((const uint32_t*)(lds + a.table))[o * 64 + lane] ^ w;
        p.image = op.image;
        p.k = op.k;
#pragma unroll
        for (int b = 0; b < 4; ++b) p.m[b] = op.lds_m[b];
        asm volatile("" : "+v"(p.at), "+s"(p.image), "+s"(p.k), "+s"(p.m[0]), "+s"(p.m[1]), "+s"(p.m[2]), "+s"(p.m[3]));
        return p;
    };
    auto slot = [&](const Place& p, int m) {
        return p.at ^ ((m & 1) ? p.m[0] : 0u) ^ ((m & 2) ? p.m[1] : 0u) ^ ((m & 4) ? p.m[2] : 0u) ^
               ((m & 8) ? p.m[3] : 0u);
    };
    double nacc = 0.0;                                   // this lane's sum of |psi|^2
    auto store = [&](int m, dd2 y) {
        __builtin_nontemporal_store(y, (dd2*)(psi + (tb | stw) + a.st_m[m] + stl));
        if (a.norm_out) nacc = fma(y.x, y.x, fma(y.y, y.y, nacc));
    };
    auto form = [&](const Place& p, auto&& f) {
        if (p.k == 5) f(std::integral_constant<int, 5>{});
        else f(std::integral_constant<int, 4>{});
    };
    uint64_t nb = tb;                                    // the tile in the registers, then in flight
    bool next = true;
    // the first block: the loaded tile's operands (elements never reached as
    // zeros), its products, the next tile's loads
    auto head = [&](auto out0) {
        if (ZERO) {
#pragma unroll
            for (int m = 0; m < 16; ++m)
                if (zl || (m & a.z_m)) raw[m] = dd2{0.0, 0.0};
        }
        nb = ((tb | ~a.tmask) + a.tstep) & a.tmask;
        tile += gridDim.x;
        next = tile < a.tiles;
        apply64<K0>(a.op[0].image, lane, [&](int m) { return raw[m]; }, out0,
                    [&](int q) { load_unit(q, nb, next && !a.from_e0); });
    };
    // waits for loads stand here and at the loop's end: inside the loop they
    // would cover the stores
    __builtin_amdgcn_s_waitcnt(kWait64Loads0);
    for (;;) {
        if constexpr (ONE) {
            head(store);
        } else {
            const Place p0 = place(0);
            head([&](int m, dd2 y) { lds_put(slot(p0, m), y); });
            Place p = place(1);
            __syncthreads();
            for (int o = 1; o + 1 < a.nops; ++o) {
                form(p, [&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    Place c = p;
                    c.at = own<K>(p.at);
                    apply64<K>(c.image, lane, [&](int m) { return lds_get(slot(c, m)); },
                               [&](int m, dd2 y) { lds_put(slot(c, m), y); }, [](int) {});
                });
                p = place(o + 1);
                __syncthreads();
            }
            form(p, [&](auto kk) {
                constexpr int K = decltype(kk)::value;
                Place c = p;
                c.at = own<K>(p.at);
                dd2 x[16];
#pragma unroll
                for (int m = 0; m < 16; ++m) x[m] = lds_get(slot(c, m));
                __syncthreads();                         // the tile may be overwritten
                apply64<K>(c.image, lane, [&](int m) { return x[m]; }, store, [](int) {});
            });
        }
        if (!next) break;
        tb = nb;
        if constexpr (!ONE) __builtin_amdgcn_s_waitcnt(kWait64Loads16);   // older than this tile's 16 stores
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

using Stage64Kernel = void (*)(double2*, Stage64K);

template <int TW>
Stage64Kernel stage64_kernel_t(bool zero, int k, bool one)
{
    if (zero) {
        if (k == 5) return one ? k_stage64<TW, true, 5, true> : k_stage64<TW, true, 5, false>;
        return one ? k_stage64<TW, true, 4, true> : k_stage64<TW, true, 4, false>;
    }
    if (k == 5) return one ? k_stage64<TW, false, 5, true> : k_stage64<TW, false, 5, false>;
    return one ? k_stage64<TW, false, 4, true> : k_stage64<TW, false, 4, false>;
}

Stage64Kernel stage64_kernel(int t, bool zero, int k, bool one)
{
    switch (t) {
        case 9: return stage64_kernel_t<9>(zero, k, one);
        case 10: return stage64_kernel_t<10>(zero, k, one);
        case 11: return stage64_kernel_t<11>(zero, k, one);
        case 12: return stage64_kernel_t<12>(zero, k, one);
        case 13: return stage64_kernel_t<13>(zero, k, one);
    }
    return nullptr;
}

// Where the t tile bits of one block go: lane bits (j0..j3, then canonical
// b0, b1), access bits, wave bits; -1 = none.
struct Layout64 {
    int lane[6], m[4], wave[3];
    int perm[5];
};

// targets: tile bit of each matrix bit.  Group bits: blocks that touch HBM take
// the lowest free tile bits, for contiguous accesses; blocks inside a run take
// three free bits of different classes modulo 3 (see the LDS order above).
Layout64 layout64(int t, int k, const int* tbit, bool hbm)
{
    Layout64 L;
    for (int& x : L.lane) x = -1;
    for (int& x : L.m) x = -1;
    for (int& x : L.wave) x = -1;
    for (int u = 0; u < 5; ++u) L.perm[u] = 0;
    bool target[64] = {};
    int canon = 0;
    for (int b = 0; b < t; ++b)
        for (int j = 0; j < k; ++j)
            if (tbit[j] == b) {
                target[b] = true;
                L.perm[canon++] = j;
            }
    L.lane[4] = tbit[L.perm[0]], L.lane[5] = tbit[L.perm[1]];
    int nm = 0;
    for (int u = 2; u < k; ++u) L.m[nm++] = tbit[L.perm[u]];
    int fr[64], nf = 0;                       // free tile bits, ascending
    for (int b = 0; b < t; ++b)
        if (!target[b]) fr[nf++] = b;
    const int nu = 4 - nm, nj = nf - nu < 4 ? nf - nu : 4;
    const int pool = hbm ? nj : nf;
    bool used[64] = {};
    int got = 0;
    for (int cls = 0; cls < 3 && got < nj; ++cls)
        for (int i = 0; i < pool; ++i)
            if (!used[i] && fr[i] % 3 == cls) {
                used[i] = true;
                L.lane[got++] = fr[i];
                break;
            }
    for (int i = 0; i < pool && got < nj; ++i)
        if (!used[i]) {
            used[i] = true;
            L.lane[got++] = fr[i];
        }
    int nw = 0;
    for (int i = 0; i < nf; ++i) {
        if (used[i]) continue;
        if (nm < 4) L.m[nm++] = fr[i];
        else L.wave[nw++] = fr[i];
    }
    return L;
}

// LDS byte offset of tile bit b
uint32_t slot64(int b)
{
    return b < 0 ? 0u : ((1u << b) | (b >= 3 ? 1u << (b % 3) : 0u)) * 16u;
}

}  // namespace

hipError_t stage64_prepare(int t, int v)
{
    static std::atomic<bool> done[5][kStage64Forms];
    if (done[t - 9][v]) return hipSuccess;
    const hipError_t e =
        hipFuncSetAttribute((const void*)stage64_kernel(t, v & 1, v & 2 ? 5 : 4, v & 4),
                            hipFuncAttributeMaxDynamicSharedMemorySize, stage_lds_limit(t, 1));
    if (e == hipSuccess) done[t - 9][v] = true;
    return e;
}

hipError_t launch_stage64(hipStream_t st, void* psi, int t, const int* P, int nops, const int* ks,
                          const int* const* pos, const void* const* mats, uint64_t tiles, uint64_t tmask,
                          uint64_t newmask, bool from_e0, double* norm_out, int* norm_blocks)
{
    if (t < 9 || t > 13 || nops < 1 || nops > kMaxOps64) return hipErrorInvalidValue;
    Stage64K a{};
    a.tiles = tiles;
    a.tmask = tmask;
    a.nops = nops;
    a.from_e0 = from_e0 ? 1 : 0;
    a.norm_out = norm_out;
    int at = 16 << t;
    for (int o = 0; o < nops; ++o) {
        if (ks[o] < 4 || ks[o] > 5) return hipErrorInvalidValue;
        int tbit[kMaxDense];
        for (int j = 0; j < ks[o]; ++j) {
            int b = 0;
            while (b < t && P[b] != pos[o][j]) ++b;
            if (b == t) return hipErrorInvalidValue;
            tbit[j] = b;
        }
        const Layout64 L = layout64(t, ks[o], tbit, o == 0 || o == nops - 1);
        Op64& op = a.op[o];
        op.mat = (const double2*)mats[o];
        op.k = ks[o];
        for (int u = 0; u < 5; ++u) op.perm[u] = L.perm[u];
        op.image = at;
        at += 16 << (2 * ks[o]);
        for (int b = 0; b < 6; ++b) op.lds_lane[b] = slot64(L.lane[b]);
        for (int b = 0; b < 4; ++b) op.lds_m[b] = slot64(L.m[b]);
        for (int b = 0; b < 3; ++b) op.lds_wave[b] = slot64(L.wave[b]);
        auto where = [&](int b) { return b < 0 ? 0ull : 1ull << P[b]; };
        if (o == 0) {
            auto reached = [&](int b) { return where(b) & ~newmask; };
            auto fresh = [&](int b) { return (where(b) & newmask) != 0; };
            for (int b = 0; b < 6; ++b) {
                a.ld_lane[b] = reached(L.lane[b]);
                if (fresh(L.lane[b])) a.z_lane |= 1u << b;
                if (L.lane[b] < 0) a.dup |= 1u << b;
            }
            for (int b = 0; b < 3; ++b) {
                a.ld_wave[b] = reached(L.wave[b]);
                if (fresh(L.wave[b])) a.z_wave |= 1u << b;
            }
            for (int b = 0; b < 4; ++b)
                if (fresh(L.m[b])) a.z_m |= 1u << b;
            for (int m = 0; m < 16; ++m)
                for (int b = 0; b < 4; ++b)
                    if ((m >> b) & 1) a.ld_m[m] |= reached(L.m[b]);
        }
        if (o == nops - 1) {
            for (int b = 0; b < 6; ++b) a.st_lane[b] = where(L.lane[b]);
            for (int b = 0; b < 3; ++b) a.st_wave[b] = where(L.wave[b]);
            for (int m = 0; m < 16; ++m)
                for (int b = 0; b < 4; ++b)
                    if ((m >> b) & 1) a.st_m[m] |= where(L.m[b]);
        }
    }
    a.table = at;
    const int lds = at + nops * 256;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    const int nt = stage64_lanes(t);
    // persistent: as many workgroups as are resident (eight waves per CU, or
    // what the LDS holds)
    int per_cu = (160 * 1024) / lds;
    if (per_cu > 512 / nt) per_cu = 512 / nt;
    uint64_t grid = a.tiles;
    const uint64_t cap = 256ull * per_cu;
    if (grid > cap) grid = cap;
    a.tstep = spread_bits(grid, a.tmask);
    const bool zero = newmask != 0, one = nops == 1;
    const int k0 = a.op[0].k;
    const hipError_t e = stage64_prepare(t, (zero ? 1 : 0) | (k0 == 5 ? 2 : 0) | (one ? 4 : 0));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(stage64_kernel(t, zero, k0, one), dim3((unsigned)grid), dim3(nt), lds, st, (double2*)psi, a);
    if (norm_blocks) *norm_blocks = norm_out ? (int)grid : 0;
    return hipGetLastError();
}

}  // namespace sv
