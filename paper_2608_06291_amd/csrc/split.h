// fp32 products on the bf16 matrix cores, at fp32 precision.
//
// Every fp32 operand x is split into three bf16 numbers (the three-way bf16
// splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019),
//     x = h + m + l :  h = x rounded to 8 bits, m = x - h rounded to 8 bits,
//     l = the rest (at most 7 bits, so exact),
// and a product a b is the sum of the six partial products
//     l_a h_b + h_a l_b + m_a m_b + m_a h_b + h_a m_b + h_a h_b ,
// each exact in fp32 (8 x 8 bits) and added into the fp32 accumulator of
// v_mfma_f32_32x32x16_bf16, small ones first.
//
// Precision (u = 2^-24, half an ulp).  What is left out, m l + l m + l l, is of
// either sign and at most u |a b| (operands just above a power of two; rms 2^-26
// to 2^-27.5).  With the matrix core's own rounding a single product is off by
// up to 2.7 u |a b| (measured; one fp32 operation 1 u).  Sixteen k's share one
// rounding per partial product, against two k's per rounding of
// v_mfma_f32_32x32x2f32, so from 3 or 4 terms on a sum is nearer to its 64-bit
// value than with fp32 MFMA: rms against sum |a b| over 1, 2, 4, 16, 2000 terms 0.57,
// 0.47, 0.36, 0.21, 0.10 u here and 0.43, 0.44, 0.45, 0.48, 0.13 u there (normal
// operands).  With h truncated instead of rounded, the same number of operations, the
// part left out is four times as large (single products up to 5.4 u); the launches at
// the power limit are then a little quicker (28672 x 8192 solve 65.8 ms, 66.8 with
// rounding), as the signs of m and l vary less.  Rounding in one operand only, told
// apart by the wave, makes the pushes of 64 x 64 and 128 x 128 blocks slower (one-sided
// 4096 x 4096 2%).
// Range: the split is exact for |x| >= 2^-110; below, l falls under bf16's
// smallest number and x is kept to within 2^-133.  An operand that is not finite,
// or above 2^128 - 2^119 (h rounds to infinity), makes the products it enters NaN.
//
// Why: the dense bf16 rate is 16 times the fp32 MFMA rate, six products leave
// a factor 2.7 for the matrix cores (large products here reach 154 TFLOP/s in
// fp32 and 1313 in bf16, so 219 for six products).  The split costs 5.5 VALU
// operations per operand entry, which wide blocks amortise and which overlap
// the MFMAs of the other wave on the SIMD.
#pragma once
#include "common.h"

namespace bk {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int SPK = 16;      // k's per chunk: one MFMA step
constexpr int SPROW = 24;    // bf16 slots per staged row: 16 k's in 48 bytes, so that the
                             // 16-byte reads of 8 consecutive rows meet 8 different
                             // 16-byte columns of the banks

// bf16 pairs packed low, high
struct SplitPair {
    uint32_t h, m, l;
};
__device__ inline SplitPair split_pair(float a, float b) {
    SplitPair s;
    s.h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
    const float ra = a - __uint_as_float(s.h << 16);
    const float rb = b - __uint_as_float(s.h & 0xffff0000u);
    s.m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{ra, rb}, bf16x2));
    const float ta = ra - __uint_as_float(s.m << 16);
    const float tb = rb - __uint_as_float(s.m & 0xffff0000u);
    s.l = __builtin_amdgcn_perm(__float_as_uint(tb), __float_as_uint(ta), 0x07060302u);
    return s;
}

// Splits four consecutive k's of one row and writes the three planes
// (`plane` bf16 slots apart) at dst.  A non-finite entry has m = l = NaN, so
// every product with it is NaN (in plain fp32 it is infinite or NaN), and finite
// products that overflow can be NaN too (their parts overflow with both signs);
// products without such an entry are not touched.
__device__ inline void split_store4(f32x4 v, uint16_t* dst, int plane) {
    const SplitPair p = split_pair(v[0], v[1]), q = split_pair(v[2], v[3]);
    *reinterpret_cast<u32x2*>(dst) = u32x2{p.h, q.h};
    *reinterpret_cast<u32x2*>(dst + plane) = u32x2{p.m, q.m};
    *reinterpret_cast<u32x2*>(dst + 2 * plane) = u32x2{p.l, q.l};
}

// One chunk of a wave's WX x WY blocks of 32 x 32: acc[x][y] += A_x B_y^T over
// the 16 staged k's.  a, b: plane 0 of the wave's first A and B row; lane l
// reads k's 8 (l >> 5) .. + 7 of row l & 31 of each block.
template <int WX, int WY>
__device__ inline void split_mma(const uint16_t* a, const uint16_t* b, int plane, int l,
                                 f32x16 (&acc)[WX][WY]) {
    const int off = (l & 31) * SPROW + (l >> 5) * 8;
    bf16x8 fb[WY][3];
#pragma unroll
    for (int y = 0; y < WY; ++y)
#pragma unroll
        for (int s = 0; s < 3; ++s)
            fb[y][s] = *reinterpret_cast<const bf16x8*>(b + y * 32 * SPROW + s * plane + off);
    // (plane of A, plane of B), small products first.  The chunk's sum starts
    // from zero and is added to the running sum once: one rounding at the
    // running sum's size per 16 k's.  A block is added while the MFMAs of the
    // next one run.
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    f32x16 t[2];
#pragma unroll
    for (int x = 0; x < WX; ++x) {
        bf16x8 fa[3];
#pragma unroll
        for (int s = 0; s < 3; ++s)
            fa[s] = *reinterpret_cast<const bf16x8*>(a + x * 32 * SPROW + s * plane + off);
#pragma unroll
        for (int y = 0; y < WY; ++y) {
            const int i = x * WY + y;
            t[i & 1] = f32x16{0};
#pragma unroll
            for (int p = 0; p < 6; ++p)
                t[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[p]], fb[y][PB[p]], t[i & 1], 0, 0, 0);
            if (i > 0) {
                f32x16& c = acc[(i - 1) / WY][(i - 1) % WY];
                c += t[(i - 1) & 1];
                asm volatile("" : "+v"(c));   // add here: t must not stay live
            }
            if (WX * WY > 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    acc[WX - 1][WY - 1] += t[(WX * WY - 1) & 1];
    asm volatile("" : "+v"(acc[WX - 1][WY - 1]));
}

// A product of MT x MT solver tiles (MT * 32 rows of A times MT * 32 rows of B,
// both with k contiguous), the whole pipeline of one workgroup:
//   MT = 8: 8 waves of 128 x 64, 144 KiB of LDS, one workgroup per CU;
//   MT = 4: 4 waves of 64 x 64, two workgroups per CU;
//   MT = 2: 4 waves of 32 x 32, two chunks per step, two workgroups per CU (with
//     one chunk per step four fit: pushes of 128 tile anti-diagonals 5% faster,
//     those of 16 to 64, which are most, 15 to 25% slower).
// Half of the threads stage A, half B: per chunk of 16 k's a thread converts
// four k's of NU rows.  LDS is double-buffered and NS chunks are in flight in
// registers behind the one being stored, so a global load has NS chunks of
// MFMA work to hide behind (one is enough at MT = 8, where a chunk takes
// 1.3 us or more).  The chunk sums and their order do not depend on MT: every
// entry gets the same bits from all three sizes (chunks of zeros add nothing).
template <int MT>
struct SplitShape {
    static constexpr int WX = MT == 8 ? 4 : MT == 4 ? 2 : 1, WY = MT >= 4 ? 2 : 1;   // blocks per wave
    static constexpr int WN = MT / WY;                    // waves along B
    static constexpr int TH = 64 * (MT / WX) * WN;        // threads
    static constexpr int RP = TH / 8;                     // rows staged per pass (4 threads per row)
    static constexpr int NU = MT * TS / RP;               // passes
    static constexpr int CB = MT == 2 ? 2 : 1;            // chunks per step (one barrier each)
    static constexpr int NS = MT == 8 ? 1 : MT == 4 ? 4 : 3;   // steps in flight
    static constexpr int PLANE = 2 * MT * TS * SPROW;     // rows of A, then rows of B
    static constexpr int LDS = 2 * CB * 3 * PLANE;             // bf16 slots
};

// load(c, u): the thread's four k's, 16 c + 4 (tid & 3) .. + 3, of row
// ((tid mod TH/2) >> 2) + u RP of A (first half of the threads) or B; past the
// last chunk it may return anything (never stored).
template <int MT, class Load>
__device__ inline void split_gemm(uint16_t* S, int nch, int tid, Load load,
                                  f32x16 (&acc)[SplitShape<MT>::WX][SplitShape<MT>::WY]) {
    using C = SplitShape<MT>;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = wv / C::WN, wn = wv % C::WN;
    const int op = wv >= C::TH / 128, t = tid & (C::TH / 2 - 1);
    uint16_t* const dst = S + (op * MT * TS + (t >> 2)) * SPROW + 4 * (t & 3);
    const uint16_t* const fa = S + wm * C::WX * TS * SPROW;
    const uint16_t* const fb = S + (MT * TS + wn * C::WY * TS) * SPROW;
    f32x4 r[C::NS][C::CB][C::NU];
    auto fetch = [&](int step, int s) {
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
#pragma unroll
            for (int u = 0; u < C::NU; ++u) r[s][j][u] = load(step * C::CB + j, u);
    };
    auto store = [&](int sb, int s) {
#pragma unroll
        for (int j = 0; j < C::CB; ++j)
#pragma unroll
            for (int u = 0; u < C::NU; ++u)
                split_store4(r[s][j][u], dst + (sb * C::CB + j) * (3 * C::PLANE) + u * C::RP * SPROW, C::PLANE);
    };
#pragma unroll
    for (int x = 0; x < C::WX; ++x)
#pragma unroll
        for (int y = 0; y < C::WY; ++y) acc[x][y] = f32x16{0};
    const int ns = (nch + C::CB - 1) / C::CB;
#pragma unroll
    for (int s = 0; s < C::NS; ++s) fetch(s, s);
    store(0, 0);
    fetch(C::NS, 0);
    __syncthreads();
    // a step is multiplied from buffer step & 1; the next one waits in set (step + 1) mod NS
    constexpr int U = C::NS % 2 ? 2 * C::NS : C::NS;
    for (int c0 = 0; c0 < ns; c0 += U) {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int c = c0 + i;
            if (c < ns) {   // uniform
#pragma unroll
                for (int j = 0; j < C::CB; ++j) {
                    const int o = ((i & 1) * C::CB + j) * (3 * C::PLANE);
                    split_mma<C::WX, C::WY>(fa + o, fb + o, C::PLANE, l, acc);
                }
                if (c + 1 < ns) {
                    store((i & 1) ^ 1, (i + 1) % C::NS);
                    fetch(c + 1 + C::NS, (i + 1) % C::NS);
                }
                __syncthreads();
            }
        }
    }
}

}  // namespace bk
