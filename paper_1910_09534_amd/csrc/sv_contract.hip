// Contraction of two tensors over their entanglement indices (App. A: the
// equation that eliminates the indices introduced by EI and E2Q; Sec. 2:
// contraction deferral sums the shared indices and takes the outer product
// over the others):
//
//     out[x2 * 2^n1 + x1] = sum_e t1[e * 2^n1 + x1] * t2[e * 2^n2 + x2]
//
// With N = 2^n1, M = 2^n2 and K = 2^e this is the complex matrix product
// out (M x N) = t2^T (M x K) * t1 (K x N): dense, bound by the matrix
// cores once K reaches a few tens.
//
//   k_contract_split  complex64, large products: the split-fp16 form, 128 x 128
//                     or 128 x 64 output tiles.
//   k_contract_mfma   the same on the fp32 matrix cores where the caller asks
//                     for it: 128 x 64 output tiles per 256-lane workgroup,
//                     64 x 32 per wave, as three real products per 16 x 16
//                     block (3M form: P1 = Br Ar, P2 = Bi Ai,
//                     P3 = (Br + Bi)(Ar + Ai); re = P1 - P2,
//                     im = P3 - P1 - P2) on v_mfma_f32_16x16x4f32, K in chunks
//                     of 16 through double-buffered LDS, the next chunk's
//                     global loads in flight during the products.
//   k_contract_full   complex128, and small complex64 products, from 16 x 16
//                     outputs and K = 4: four real products in the data's own
//                     precision.
//   k_contract_plain  what is left (an output side below 16, K below 4): one
//                     output per lane, a loop over K.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sv_device.h"

namespace sv {

namespace {

typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kCM = 128;          // output rows (x2) per workgroup
constexpr int kCN = 64;           // output columns (x1) per workgroup
constexpr int kCK = 16;           // K per chunk
constexpr int kCThreads = 256;
constexpr int kBStride = kCM + 4; // LDS row strides in complex elements (padding staggers banks)
constexpr int kAStride = kCN + 4;

// t1 and t2 are not __restrict__: loads through such pointers count as
// invariant and are moved past the scheduling fence that keeps them ahead of
// the products
__global__ __launch_bounds__(kCThreads) void k_contract_mfma(const float2* t1, const float2* t2,
                                                             float2* __restrict__ out, int n1, int n2,
                                                             int e, uint32_t tiles_n, uint32_t group)
{
    __shared__ __attribute__((aligned(16))) float2 Bs[2][kCK * kBStride];
    __shared__ __attribute__((aligned(16))) float2 As[2][kCK * kAStride];
    const uint64_t N = 1ull << n1, M = 1ull << n2;
    const uint32_t K = 1u << e;
    // grouped order: `group` consecutive row blocks sweep the column blocks
    // together, so a t1 panel is read once per group of row blocks (per XCD
    // L2) and the group's t2 panels stay in cache across the sweep.  (Giving
    // each XCD a contiguous range of this order instead measured 2x the L2
    // refills.)
    const uint32_t per = group * tiles_n;
    const uint32_t g = blockIdx.x / per, r = blockIdx.x % per;
    const uint32_t tn = r / group, tm = g * group + r % group;
    const uint64_t m0 = (uint64_t)tm * kCM, n0 = (uint64_t)tn * kCN;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 32;
    const int li = lane & 15, lk = lane >> 4;

    // global -> register staging of one K chunk: 4 float4 of t2, 2 of t1 per
    // lane (plain unrolled loops: the arrays stay in registers)
    const uint32_t nchunks = K / kCK;
    // named values rather than arrays: private arrays get moved to LDS
    float4 gb0, gb1, gb2, gb3, ga0, ga1;
    // this lane's slots: t2 rows k = tid / 64 + 4 i, columns 2 (tid % 64);
    // t1 rows k = tid / 32 + 8 i, columns 2 (tid % 32)
    const int kb = tid >> 6, mb2 = 2 * (tid & 63);
    const int ka = tid >> 5, na2 = 2 * (tid & 31);
    const int bo = kb * kBStride + mb2, ao = ka * kAStride + na2;
    const uint64_t bg = (uint64_t)kb * M + m0 + mb2, ag = (uint64_t)ka * N + n0 + na2;
#define SV_CONTRACT_LOAD(kn)                                              \
    do {                                                                  \
        const float2* pb = t2 + bg + (uint64_t)(kn) * M;                  \
        const float2* pa = t1 + ag + (uint64_t)(kn) * N;                  \
        gb0 = *(const float4*)(pb);                                       \
        gb1 = *(const float4*)(pb + 4 * M);                               \
        gb2 = *(const float4*)(pb + 8 * M);                               \
        gb3 = *(const float4*)(pb + 12 * M);                              \
        ga0 = *(const float4*)(pa);                                       \
        ga1 = *(const float4*)(pa + 8 * N);                               \
    } while (0)
#define SV_CONTRACT_PARK(bf)                                              \
    do {                                                                  \
        *(float4*)(&Bs[bf][bo]) = gb0;                                    \
        *(float4*)(&Bs[bf][bo + 4 * kBStride]) = gb1;                     \
        *(float4*)(&Bs[bf][bo + 8 * kBStride]) = gb2;                     \
        *(float4*)(&Bs[bf][bo + 12 * kBStride]) = gb3;                    \
        *(float4*)(&As[bf][ao]) = ga0;                                    \
        *(float4*)(&As[bf][ao + 8 * kAStride]) = ga1;                     \
    } while (0)

    f4v p1[4][2], p2[4][2], p3[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            p1[a][b] = f4v{0.f, 0.f, 0.f, 0.f};
            p2[a][b] = p1[a][b];
            p3[a][b] = p1[a][b];
        }

    SV_CONTRACT_LOAD(0);
    SV_CONTRACT_PARK(0);
    __syncthreads();
    for (uint32_t c = 0; c < nchunks; ++c) {
        const int buf = c & 1;
        // the next chunk's loads are in flight during this chunk's products
        // (the last iteration loads its own chunk again: in bounds, unused)
        SV_CONTRACT_LOAD((c + 1 < nchunks ? c + 1 : c) * kCK);
        // keep the loads ahead of the products (the scheduler would sink
        // them to their use, after the products)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < kCK / 4; ++s) {
            const int k = 4 * s + lk;
            float br[4], bi[4], bs[4], ar[2], ai[2], as_[2];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float2 v = Bs[buf][k * kBStride + wm + 16 * a + li];
                br[a] = v.x;
                bi[a] = v.y;
                bs[a] = v.x + v.y;
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const float2 v = As[buf][k * kAStride + wn + 16 * b + li];
                ar[b] = v.x;
                ai[b] = v.y;
                as_[b] = v.x + v.y;
            }
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    p1[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(br[a], ar[b], p1[a][b], 0, 0, 0);
                    p2[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(bi[a], ai[b], p2[a][b], 0, 0, 0);
                    p3[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(bs[a], as_[b], p3[a][b], 0, 0, 0);
                }
        }
        // park the next chunk in the other buffer (read by nobody since the
        // previous barrier); after the products, so that only this waits
        // for the loads
        __builtin_amdgcn_sched_barrier(0);
        SV_CONTRACT_PARK(buf ^ 1);
        __syncthreads();
    }
#undef SV_CONTRACT_LOAD
#undef SV_CONTRACT_PARK
    // lane holds rows 4 lk + v of each 16-row block, column li of each 16-column block
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint64_t m = m0 + wm + 16 * a + 4 * lk + v;
                const uint64_t n = n0 + wn + 16 * b + li;
                const float x1 = p1[a][b][v], x2 = p2[a][b][v], x3 = p3[a][b][v];
                out[m * N + n] = float2{x1 - x2, x3 - x1 - x2};
            }
}

// ---- split-fp16 form of the matrix-core contraction -----------------------
// 16-deep K chunks as above, with the products on the fp16 matrix cores at
// single-precision accuracy: every input is scaled
// by a power of two (from the largest |component| of its tensor, so that it
// stays below 2^14) and split into hi = f16(x) and lo = f16(x - hi); the
// three products A_hi B_hi + A_hi B_lo + A_lo B_hi accumulate in fp32 on
// v_mfma_f32_16x16x32_f16.  A K chunk of 16 complex values is one 32-deep
// real product: Re = [Br | Bi] [Ar ; -Ai] and Im = [Br | Bi] [Ai ; Ar]
// (B = t2^T, A = t1): six products per 16 x 16 block per chunk, both
// sharing the B operand.  The chunk
// is parked in LDS already split, each row's 16 values contiguous (hi and
// lo of the real and imaginary parts), so a lane reads its 8 operand
// values with one 16-byte access.
// A wave's tile is 64 x 16 CB.  With 64 x 32 (CB = 2) the LDS is busy for 0.92
// of the time that the products take (16 reads and 12 values split per 48
// products), with 64 x 64 (CB = 4: 24 and 16 per 96) for 0.67; that needs 234
// of the 256 registers that two waves per SIMD have.  The next chunk is split
// and parked in four pieces between the products of this one, and each
// piece's registers are loaded again for the chunk after it.  13, 15, 8: 1,690
// us in 64 x 32 with the split after the products, 1,600 in 64 x 64, 1,567 as
// it is (1.05 PFLOP/s of the 24 MNK issued; the vendor's fp16 product reaches
// 1.38), the clock down to 1.7 GHz under the load; 15, 15, 10: 25.3 -> 23.6 ->
// 22.7 ms (1.16).  These are normally distributed values; the tensors of a
// deferred circuit, three quarters of whose entries are zero, draw less power
// and take 17.2 ms at 15, 15, 10 (random values with 90 % zeros: the same).
typedef _Float16 ch8 __attribute__((ext_vector_type(8)));
typedef _Float16 ch4 __attribute__((ext_vector_type(4)));
typedef uint32_t cu4 __attribute__((ext_vector_type(4)));
typedef uint32_t cu2 __attribute__((ext_vector_type(2)));

constexpr int kSRow = 16;                  // f16 per LDS row: the chunk's 16 k values

// element offset in a part of the LDS chunk of row r, k-octet o (0, 1):
// the two octets of a row swap places on every other group of four rows,
// which spreads the 16-byte reads of sixteen consecutive rows over the banks
__device__ __forceinline__ int srow(int r, int o)
{
    return r * kSRow + ((o ^ ((r >> 2) & 1)) << 3);
}

// largest |component| of t2 (blocks below `split`) and of t1 (the others), as
// float bits, into out[0] and out[1] (atomic max: non-negative floats order as
// their bit patterns); four 16-byte loads in flight per lane
__global__ __launch_bounds__(256) void k_absmax(const float4* __restrict__ t2, uint64_t count2,
                                                const float4* __restrict__ t1, uint64_t count1, uint32_t split,
                                                uint32_t* out)
{
    __shared__ float sh[4];
    const bool first = blockIdx.x < split;
    const float4* x = first ? t2 : t1;
    const uint64_t count = first ? count2 : count1;
    const uint64_t stride = (uint64_t)(first ? split : gridDim.x - split) * 256;
    uint64_t i = (uint64_t)(first ? blockIdx.x : blockIdx.x - split) * 256 + threadIdx.x;
    float m = 0.f;
    auto take = [&](float4 v) { m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w)))); };
    for (; i + 3 * stride < count; i += 4 * stride) {
        const float4 v0 = x[i], v1 = x[i + stride], v2 = x[i + 2 * stride], v3 = x[i + 3 * stride];
        take(v0);
        take(v1);
        take(v2);
        take(v3);
    }
    for (; i < count; i += stride) take(x[i]);
#pragma unroll
    for (int h = 32; h > 0; h >>= 1) m = fmaxf(m, __shfl_xor(m, h));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(out + (first ? 0 : 1), __float_as_uint(fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]))));
}

// exponent s with max 2^s <= 2^14 (0 for an all-zero tensor)
__device__ __forceinline__ int scale_exp(uint32_t maxbits)
{
    const float m = __uint_as_float(maxbits);
    if (!(m > 0.f) || !isfinite(m)) return 0;
    int e = 14 - (int)ceilf(log2f(m));
    while (ldexpf(m, e) > 16384.f) --e;
    return e < -100 ? -100 : (e > 100 ? 100 : e);
}

template <int CB>
__global__ __launch_bounds__(kCThreads, CB == 4 ? 2 : 3) void k_contract_split(const float2* t1, const float2* t2,
                                                                 float2* __restrict__ out, int n1, int n2, int e,
                                                                 uint32_t tiles_n, uint32_t group,
                                                                 const uint32_t* __restrict__ maxbits, bool nt)
{
    constexpr int CN = 32 * CB;                // output columns per workgroup
    constexpr int NK = CB == 4 ? 8 : 4;        // k values of a t1 column a lane stages
    // [buffer][part: re hi, re lo, im hi, im lo][row][k]
    __shared__ __attribute__((aligned(16))) _Float16 Bs[2][4][kCM * kSRow];
    __shared__ __attribute__((aligned(16))) _Float16 As[2][4][CN * kSRow];
    const uint64_t N = 1ull << n1, M = 1ull << n2;
    const uint32_t K = 1u << e;
    const uint32_t per = group * tiles_n;
    const uint32_t gq = blockIdx.x / per, rr = blockIdx.x % per;
    const uint32_t tn = rr / group, tm = gq * group + rr % group;
    const uint64_t m0 = (uint64_t)tm * kCM, n0 = (uint64_t)tn * CN;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 16 * CB;
    const int li = lane & 15, g = lane >> 4;
    // staging: t2 column m = tid % 128, k = 8 (tid / 128) + 0..7; t1 column
    // n = tid % CN, k = NK (tid / CN) + 0..NK-1 (each load row is 64 lanes of
    // consecutive columns)
    const int bm = tid & 127, bo = tid >> 7;
    const int an = tid & (CN - 1), aq = tid / CN;
    const uint32_t nchunks = K / kCK;
    float2 gb[8], ga[NK];
    auto load_b = [&](uint32_t c) {
        const float2* pb = t2 + (uint64_t)(c * kCK + 8 * bo) * M + m0 + bm;
#pragma unroll
        for (int k = 0; k < 8; ++k) gb[k] = pb[(uint64_t)k * M];
    };
    auto load_a = [&](uint32_t c) {
        const float2* pa = t1 + (uint64_t)(c * kCK + NK * aq) * N + n0 + an;
#pragma unroll
        for (int k = 0; k < NK; ++k) ga[k] = pa[(uint64_t)k * N];
    };
    load_b(0);
    load_a(0);
    __builtin_amdgcn_sched_barrier(0);
    const int eb = scale_exp(maxbits[0]), ea = scale_exp(maxbits[1]);
    // (the two factors are applied one after the other on the way out:
    // 2^-(eb + ea) alone can leave the float range)
    const float sb = ldexpf(1.f, eb), sa = ldexpf(1.f, ea), ub = ldexpf(1.f, -eb), ua = ldexpf(1.f, -ea);

    // piece 0, 1: real and imaginary parts of the staged t2 values; 2, 3: of t1
    using au = typename std::conditional<CB == 4, cu4, cu2>::type;
    const int pob = srow(bm, bo);
    const int poa = CB == 4 ? srow(an, aq) : srow(an, aq >> 1) + 4 * (aq & 1);
    auto park = [&](int buf, int piece) {
        const bool im = piece & 1;
        if (piece < 2) {
            cu4 hi, lo;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float x0 = im ? gb[2 * w].y : gb[2 * w].x, x1 = im ? gb[2 * w + 1].y : gb[2 * w + 1].x;
                hi[w] = cpk_hi(x0, x1, sb);
                lo[w] = cpk_lo(x0, x1, sb, hi[w]);
            }
            *(cu4*)&Bs[buf][2 * im][pob] = hi;
            *(cu4*)&Bs[buf][2 * im + 1][pob] = lo;
        } else {
            au hi, lo;
#pragma unroll
            for (int w = 0; w < NK / 2; ++w) {
                const float x0 = im ? ga[2 * w].y : ga[2 * w].x, x1 = im ? ga[2 * w + 1].y : ga[2 * w + 1].x;
                hi[w] = cpk_hi(x0, x1, sa);
                lo[w] = cpk_lo(x0, x1, sa, hi[w]);
            }
            *(au*)&As[buf][2 * im][poa] = hi;
            *(au*)&As[buf][2 * im + 1][poa] = lo;
        }
    };

    f4v re[4][CB], im[4][CB];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            re[a][b] = f4v{0.f, 0.f, 0.f, 0.f};
            im[a][b] = re[a][b];
        }
    // lane (li, g): operand element e is k = 8 (g & 1) + e of the real part
    // (g < 2) or the imaginary part (g >= 2).  Re = [Br | Bi] [Ar ; -Ai] and
    // Im = [Br | Bi] [Ai ; Ar]: both products share the A operand, and the
    // -Ai of the real one is the sign flipped in lanes g >= 2 of its other
    // operand
    const int o = g & 1;
    const int pA = g < 2 ? 0 : 2;                 // A operand rows: Br or Bi
    const int pBr = g < 2 ? 0 : 2;                // [Ar ; Ai], Ai negated below
    const int pBi = g < 2 ? 2 : 0;                // [Ai ; Ar]
    const uint32_t neg = g < 2 ? 0u : 0x80008000u;

    auto chunk = [&](int buf, auto more, uint32_t next) {
        ch8 ah[4], al[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int oa = srow(wm + 16 * a + li, o);
            ah[a] = *(const ch8*)&Bs[buf][pA][oa];
            al[a] = *(const ch8*)&Bs[buf][pA + 1][oa];
        }
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            const int ob = srow(wn + 16 * b + li, o);
            const ch8 rh = __builtin_bit_cast(ch8, *(const cu4*)&As[buf][pBr][ob] ^ neg);
            const ch8 rl = __builtin_bit_cast(ch8, *(const cu4*)&As[buf][pBr + 1][ob] ^ neg);
            const ch8 ih = *(const ch8*)&As[buf][pBi][ob];
            const ch8 il = *(const ch8*)&As[buf][pBi + 1][ob];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                re[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[a], rh, re[a][b], 0, 0, 0);
                im[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al[a], ih, im[a][b], 0, 0, 0);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                re[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], rl, re[a][b], 0, 0, 0);
                im[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], il, im[a][b], 0, 0, 0);
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                re[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], rh, re[a][b], 0, 0, 0);
                im[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah[a], ih, im[a][b], 0, 0, 0);
            }
            if (more) {
#pragma unroll
                for (int p = b * 4 / CB; p < (b + 1) * 4 / CB; ++p) {
                    park(buf ^ 1, p);
                    if (p == 1) load_b(next);
                    if (p == 3) load_a(next);
                }
            }
        }
    };
#pragma unroll
    for (int p = 0; p < 4; ++p) park(0, p);
    const uint32_t last = nchunks - 1;
    load_b(last ? 1 : 0);
    load_a(last ? 1 : 0);
    __syncthreads();
    uint32_t c = 0;
    for (; c < last; ++c) {
        chunk(c & 1, std::true_type{}, c + 2 < last ? c + 2 : last);
        __syncthreads();
    }
    chunk(c & 1, std::false_type{}, 0);
    // lane holds rows 4 g + v of each 16-row block, column li of each 16-column block
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint64_t m = m0 + wm + 16 * a + 4 * g + v;
                const uint64_t n = n0 + wn + 16 * b + li;
                const float2 r = float2{re[a][b][v] * ub * ua, im[a][b][v] * ub * ua};
                if (nt) __builtin_nontemporal_store(f2v{r.x, r.y}, (f2v*)(out + m * N + n));
                else out[m * N + n] = r;
            }
}

// ---- full-precision matrix-core form ----------------------------------------
// complex128 on v_mfma_f64_16x16x4f64 and the complex64 shapes that are too
// small for the tiles above on v_mfma_f32_16x16x4f32: four real products
// (Re = Br Ar - Bi Ai, Im = Br Ai + Bi Ar) in the precision of the data, so
// the sums are those of k_contract_plain in another order.  A wave owns
// 16 RB x 16 CB outputs and takes its operands straight from memory (16 lanes
// read 16 consecutive elements): a step of four k for 2 x 2 blocks is 16
// products, 1,024 matrix-core cycles in FP64, against four loads per lane, so
// LDS would save little.  With one block a step is shorter than a load takes:
// KU = 4 steps are loaded ahead at a time, and the SK waves of a workgroup
// take a part of the sum each, added in LDS in a fixed order.
template <typename T>
struct Full;
template <>
struct Full<double> {
    using V = double2;
    typedef double acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mma(double a, double b, acc c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // row of result item v of lane group g
    static __device__ __forceinline__ int row(int g, int v) { return g + 4 * v; }
};
template <>
struct Full<float> {
    using V = float2;
    typedef float acc __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ acc mma(float a, float b, acc c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int g, int v) { return 4 * g + v; }
};

template <typename T, int RB, int CB, int KU, int SK>
__global__ __launch_bounds__(SK > 1 ? 64 * SK : 256) void k_contract_full(
    const typename Full<T>::V* t1, const typename Full<T>::V* t2, typename Full<T>::V* __restrict__ out, int n1,
    int n2, int e, uint32_t tiles_m, uint32_t tiles_n, uint32_t group)
{
    using F = Full<T>;
    using V = typename F::V;
    using acc = typename F::acc;
    const uint64_t N = 1ull << n1, M = 1ull << n2;
    const uint32_t steps = (1u << (e - 2)) / SK;         // four k each
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lk = lane >> 4;
    // grouped order, as above: the waves of a workgroup share a t1 panel
    const uint32_t wg = blockIdx.y * gridDim.x + blockIdx.x;
    const uint32_t wt = SK > 1 ? wg : wg * 4 + wave;
    if (wt >= tiles_m * tiles_n) return;
    const uint32_t per = group * tiles_n;
    const uint32_t g = wt / per, r = wt % per;
    const uint64_t m0 = (uint64_t)(g * group + r % group) * (16 * RB), n0 = (uint64_t)(r / group) * (16 * CB);
    const uint64_t k0 = SK > 1 ? (uint64_t)wave * steps * 4 : 0;
    const V* pb = t2 + (k0 + lk) * M + m0 + li;
    const V* pa = t1 + (k0 + lk) * N + n0 + li;
    // Br Ar, Bi Ai, Br Ai and Bi Ar are summed on their own: the rounding error
    // of one sum of complex products, where one sum of both parts has 1.4 times it
    acc rr[RB][CB], ii[RB][CB], ri[RB][CB], ir[RB][CB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < CB; ++b) rr[a][b] = ii[a][b] = ri[a][b] = ir[a][b] = acc{0, 0, 0, 0};
    V nb[KU][RB], na[KU][CB];
    auto load = [&](uint32_t s) {
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
            for (int a = 0; a < RB; ++a) nb[u][a] = pb[(uint64_t)(s + u) * 4 * M + 16 * a];
#pragma unroll
            for (int b = 0; b < CB; ++b) na[u][b] = pa[(uint64_t)(s + u) * 4 * N + 16 * b];
        }
    };
    load(0);
    for (uint32_t s = 0; s < steps; s += KU) {
        V xb[KU][RB], xa[KU][CB];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
            for (int a = 0; a < RB; ++a) xb[u][a] = nb[u][a];
#pragma unroll
            for (int b = 0; b < CB; ++b) xa[u][b] = na[u][b];
        }
        if (s + KU < steps) load(s + KU);
        // the next steps' loads stay ahead of these products
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < KU; ++u) {
#pragma unroll
            for (int a = 0; a < RB; ++a)
#pragma unroll
                for (int b = 0; b < CB; ++b) {
                    rr[a][b] = F::mma(xb[u][a].x, xa[u][b].x, rr[a][b]);
                    ii[a][b] = F::mma(xb[u][a].y, xa[u][b].y, ii[a][b]);
                    ri[a][b] = F::mma(xb[u][a].x, xa[u][b].y, ri[a][b]);
                    ir[a][b] = F::mma(xb[u][a].y, xa[u][b].x, ir[a][b]);
                }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (SK > 1) {
        // item c = 2 v + {re, im} of lane l, one row of SK parts: lane l's
        // items are added by threads l + 64 c (all of them in flight at once)
        __shared__ T part[SK][RB * CB * 8 * 64];
#pragma unroll
        for (int q = 0; q < RB * CB; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int a = q / CB, b = q % CB;
                part[wave][64 * (8 * q + 2 * v) + lane] = rr[a][b][v] - ii[a][b][v];
                part[wave][64 * (8 * q + 2 * v + 1) + lane] = ri[a][b][v] + ir[a][b][v];
            }
        __syncthreads();
        for (int i = threadIdx.x; i < RB * CB * 4 * 64; i += 64 * SK) {
            const int l = i & 63, v = (i >> 6) & 3, q = i >> 8;
            T sr = 0, si = 0;
#pragma unroll
            for (int w = 0; w < SK; ++w) {
                sr += part[w][64 * (8 * q + 2 * v) + l];
                si += part[w][64 * (8 * q + 2 * v + 1) + l];
            }
            out[(m0 + 16 * (q / CB) + F::row(l >> 4, v)) * N + n0 + 16 * (q % CB) + (l & 15)] = V{sr, si};
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int b = 0; b < CB; ++b)
                out[(m0 + 16 * a + F::row(lk, v)) * N + n0 + 16 * b + li] =
                    V{rr[a][b][v] - ii[a][b][v], ri[a][b][v] + ir[a][b][v]};
}

template <typename T, int RB, int CB, int KU, int SK>
hipError_t launch_full_tiles(hipStream_t st, const void* t1, const void* t2, void* out, int n1, int n2, int e)
{
    using V = typename Full<T>::V;
    const uint64_t tm = (1ull << n2) / (16 * RB), tn = (1ull << n1) / (16 * CB);
    if (tm * tn > 0xfffffff0ull) return hipErrorInvalidValue;
    const uint32_t group = tm < 16 ? (uint32_t)tm : 16;
    const uint64_t wgs = SK > 1 ? tm * tn : (tm * tn + 3) / 4;
    // a grid dimension takes fewer than 2^32 work items (2^34 outputs with a
    // side of 16 have more); both are powers of two
    const uint64_t gx = std::min<uint64_t>(wgs, 1u << 20);
    hipLaunchKernelGGL((k_contract_full<T, RB, CB, KU, SK>), dim3((unsigned)gx, (unsigned)(wgs / gx)),
                       dim3(SK > 1 ? 64 * SK : 256), 0, st, (const V*)t1, (const V*)t2, (V*)out, n1, n2, e,
                       (uint32_t)tm, (uint32_t)tn, group);
    return hipGetLastError();
}

// At least 16 x 16 outputs and four k.  32 x 32 outputs a wave where that
// gives every SIMD one (1,024); in fp32 with the sum in four parts up to 2^22
// outputs (a quarter of the chain: 9, 9, 8 22.9 us in one part of 16 x 16, 22.0
// here; error 2.9e-7 and 1.5e-7); 16 x 16 below, with the sum in 16 or 4 parts
// while the outputs alone leave SIMDs idle and it is long enough to give each
// wave four steps (2^18 outputs, e = 8: 20.6 us in one part, 22.7 in 16).
// Measured (n1, n2, e; k_contract_plain -> here): complex128 12, 13, 6
// 1,874 -> 280 us one after the other, 316-326 on its own (61 and 54 TFLOP/s of
// 8 MNK), 12, 13, 10 28,852 -> 3,901 us (70, the
// FP64 matrix product of the vendor's library reaches 73), 8, 8, 10 280 -> 19
// us, 4, 4, 10 131 -> 16 us, 12, 12, 2 77 -> 45 us; complex64 12, 13, 3 260 ->
// 56 us (4.8 TB/s, HBM), 6, 6, 8 40 -> 10 us.  64 x 32 outputs a wave need 408
// registers in FP64, and 806 us at 12, 13, 6 when held to 256.  Relative error
// against 80-bit sums: 2.0e-16 and 2.0e-16 (7, 8, 5), 2.8e-16 and 2.8e-16 (10,
// 10, 6), 7.6e-16 and 2.4e-16 (5, 6, 9).
template <typename T>
hipError_t launch_full(hipStream_t st, const void* t1, const void* t2, void* out, int n1, int n2, int e)
{
    if (std::is_same<T, float>::value && n2 >= 5 && n1 >= 5 && n1 + n2 >= 18 && n1 + n2 <= 22 && e >= 5)
        return launch_full_tiles<float, 2, 2, 1, 4>(st, t1, t2, out, n1, n2, e);
    if (n2 >= 5 && n1 >= 5 && n1 + n2 >= 20) return launch_full_tiles<T, 2, 2, 1, 1>(st, t1, t2, out, n1, n2, e);
    if (n1 + n2 <= 16 && e >= 8) return launch_full_tiles<T, 1, 1, 4, 16>(st, t1, t2, out, n1, n2, e);
    if (n1 + n2 <= 17 && e >= 6) return launch_full_tiles<T, 1, 1, 4, 4>(st, t1, t2, out, n1, n2, e);
    if (e >= 4) return launch_full_tiles<T, 1, 1, 4, 1>(st, t1, t2, out, n1, n2, e);
    return launch_full_tiles<T, 1, 1, 1, 1>(st, t1, t2, out, n1, n2, e);
}

template <typename T, typename A>
__global__ __launch_bounds__(256) void k_contract_plain(const T* __restrict__ t1, const T* __restrict__ t2,
                                                        T* __restrict__ out, int n1, int n2, int e)
{
    const uint64_t N = 1ull << n1, M = 1ull << n2, K = 1ull << e;
    const uint64_t total = N * M;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t o = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total; o += stride) {
        const uint64_t n = o & (N - 1), m = o >> n1;
        A re = 0, im = 0;
        for (uint64_t k = 0; k < K; ++k) {
            const T a = t1[k * N + n], b = t2[k * M + m];
            re += (A)a.x * (A)b.x - (A)a.y * (A)b.y;
            im += (A)a.x * (A)b.y + (A)a.y * (A)b.x;
        }
        out[o].x = re;
        out[o].y = im;
    }
}

}  // namespace

// complex64 from one 128 x 64 tile and one chunk on, except small products.
// There the tiles leave CUs idle (2^20 outputs are 128 of them), and the split
// form takes three more launches than one kernel, so k_contract_full in fp32 is
// faster up to here, and its error, summed in more parts, no larger.  Measured
// as calls (n1, n2, e; split / 3M -> full): 8, 8, 8 50 / 47 -> 19 us, 9, 9, 10
// 98 / 134 -> 39, 10, 10, 6 47 / 26 -> 24, 10, 10, 9 69 / 77 -> 59, 11, 11, 4 48
// / 25 -> 27, 11, 11, 6 48 / 34 -> 43; past the limits 10, 10, 10 105 / -> 102,
// 11, 11, 7 54 / 46 -> 63, 12, 12, 4 52 / -> 56.  Relative error against 64
// bits: 8, 8, 8 2.6e-7 / 4.1e-7 -> 1.1e-7, 10, 10, 9 3.6e-7 / 5.7e-7 -> 2.1e-7,
// 10, 10, 4 8.8e-8 / 1.2e-7 -> 7.9e-8.
static bool contract_uses_tiles(int n1, int n2, int e, bool split)
{
    if (n2 < 7 || n1 < 6 || e < 4) return false;
    const int n = n1 + n2;
    return !(n <= 20 && n + e <= 29) && !(split && n <= 22 && n + e <= 28);
}

hipError_t launch_contract(hipStream_t st, const void* t1, const void* t2, void* out, int n1, int n2, int e,
                           int dtype, bool split)
{
    if (dtype == 0 && contract_uses_tiles(n1, n2, e, split)) {
        const uint64_t tiles = (1ull << (n2 - 7)) * (1ull << (n1 - 6));
        if (tiles > 0x7fffffffull) return hipErrorInvalidValue;
        const uint32_t tiles_m = 1u << (n2 - 7);
        const uint32_t group = tiles_m < 16 ? tiles_m : 16;
        if (split) {
            // the two tensors' largest |component|, in stream-ordered memory
            // (concurrent contractions on other streams keep their own)
            uint32_t* mx = nullptr;
            hipError_t err = hipMallocAsync((void**)&mx, 2 * sizeof(uint64_t), st);
            if (err != hipSuccess) return err;
            err = launch_init(st, mx, 1, 1, false);
            if (err != hipSuccess) return err;
            const uint64_t c2 = 1ull << (n2 + e - 1), c1 = 1ull << (n1 + e - 1);     // in 16 bytes
            auto grid_for = [](uint64_t count) { return (uint32_t)std::min<uint64_t>(1024, (count + 1023) / 1024); };
            const uint32_t g2 = grid_for(c2), g1 = grid_for(c1);
            hipLaunchKernelGGL(k_absmax, dim3(g2 + g1), dim3(256), 0, st, (const float4*)t2, c2, (const float4*)t1,
                               c1, g2, mx);
            // 128 x 128 outputs from two workgroups per CU on (n1, n2, e; 128 x 64
            // -> 128 x 128: 10, 10, 8 42 -> 47 us, 11, 11, 10 160 -> 158, 12, 13, 8
            // 247 -> 221, 15, 15, 10 25.8 -> 23.0 ms); non-temporal stores where
            // the outputs exceed the 256 MB cache (plain -> non-temporal: 12, 13,
            // 4 64 -> 75 us, 13, 14, 9 1,505 -> 1,471, 13, 15, 8 1,614 -> 1,567)
            const bool nt = n1 + n2 >= 26;
            if (n1 >= 7 && n1 + n2 >= 23)
                hipLaunchKernelGGL((k_contract_split<4>), dim3((unsigned)(tiles / 2)), dim3(kCThreads), 0, st,
                                   (const float2*)t1, (const float2*)t2, (float2*)out, n1, n2, e,
                                   (uint32_t)(1ull << (n1 - 7)), group, (const uint32_t*)mx, nt);
            else
                hipLaunchKernelGGL((k_contract_split<2>), dim3((unsigned)tiles), dim3(kCThreads), 0, st,
                                   (const float2*)t1, (const float2*)t2, (float2*)out, n1, n2, e,
                                   (uint32_t)(1ull << (n1 - 6)), group, (const uint32_t*)mx, nt);
            err = hipGetLastError();
            const hipError_t e2 = hipFreeAsync(mx, st);
            return err != hipSuccess ? err : e2;
        }
        hipLaunchKernelGGL(k_contract_mfma, dim3((unsigned)tiles), dim3(kCThreads), 0, st, (const float2*)t1,
                           (const float2*)t2, (float2*)out, n1, n2, e, (uint32_t)(1ull << (n1 - 6)), group);
        return hipGetLastError();
    }
    if (n1 >= 4 && n2 >= 4 && e >= 2)
        return dtype ? launch_full<double>(st, t1, t2, out, n1, n2, e)
                     : launch_full<float>(st, t1, t2, out, n1, n2, e);
    const uint64_t total = 1ull << (n1 + n2);
    uint64_t grid = (total + 255) / 256;
    if (grid > (1u << 20)) grid = 1u << 20;
    if (dtype == 0)
        hipLaunchKernelGGL((k_contract_plain<float2, float>), dim3((unsigned)grid), dim3(256), 0, st,
                           (const float2*)t1, (const float2*)t2, (float2*)out, n1, n2, e);
    else
        hipLaunchKernelGGL((k_contract_plain<double2, double>), dim3((unsigned)grid), dim3(256), 0, st,
                           (const double2*)t1, (const double2*)t2, (double2*)out, n1, n2, e);
    return hipGetLastError();
}

}  // namespace sv
