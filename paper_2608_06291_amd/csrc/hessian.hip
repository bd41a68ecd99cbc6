// Kronecker-factor construction from calibration samples (Sec. 4 and App. A).
// Every factor the paper forms is a weighted Gram matrix of per-sample vectors,
// possibly multiplied entrywise by a fixed matrix:
//     C = s * (X^T diag(w) X) (.) M,    C_ij = s * M_ij * sum_k w_k X_ki X_kj,
// X the N x d matrix of samples (one row per sample):
//   K-FAC style (App. A):         A = E[a a^T], B = E[b b^T]                  (w = 1, M = 1)
//   single Shampoo step (App. A): A = E[|b|^2 a a^T], B = E[|a|^2 b b^T]      (w = squared norms)
//   MLP-local (App. A, b = D_g W_down^T): b b^T = (g g^T) (.) W_down^T W_down, so
//                                 B = E[g g^T] (.) D^T D with D^T D itself a Gram over the rows of
//                                 D = W_down, and tr(b^T b) = sum_i (D^T D)_ii g_i^2.
// k_sample_weights forms w_k = sum_i c_i X_ki^2 (c = 1: the squared norm).
// k_gram computes the upper-triangle blocks of X^T diag(w) X on the bf16 matrix
// cores from operands split in three (split.h), over slices of the samples; k_gram_reduce adds the slices in a
// fixed order, applies s and M, writes the upper triangle and mirrors it.
#include <algorithm>
#include <cstdio>
#include <string>

#include "bakron.h"
#include "common.h"
#include "split.h"

namespace bk {

constexpr int GB = 128;        // narrow block edge of the Gram and quadratic-form kernels
constexpr int GBW = 256;       // wide block edge
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // rows at any 4-byte address

// The same block in plain fp32 (v_mfma_f32_32x32x2f32), staged as [row][16 k's].
// k_gram and k_quadform take it
//   * for sums of at most PLAIN_TERMS terms, which the split makes less exact
//     (a single product is off by up to 2.7 u, here 1 u; from 5 terms on the split
//     is the more exact one: split.h);
//   * in a second pass over a block in which a result of the split product is not
//     finite, for those results only: an infinite operand, or finite products
//     that overflow, give NaN in the split where fp32 has an infinity.
// Neither needs speed, so LDS is single-buffered.
constexpr int PLAIN_TERMS = 4;
constexpr int PLROW = SPK + 4;   // floats per staged row: 16-byte rows, no bank conflicts

// One chunk of a wave's WX x WY blocks of 32 x 32: lane half h takes k = 8 h + s at step s.
template <int WX, int WY>
__device__ inline void plain_mma(const float* a, const float* b, int l, f32x16 (&acc)[WX][WY]) {
    const int off = (l & 31) * PLROW + (l >> 5) * 8;
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int x = 0; x < WX; ++x) {
            const f32x4 fa = *reinterpret_cast<const f32x4*>(a + x * 32 * PLROW + off + 4 * v);
#pragma unroll
            for (int y = 0; y < WY; ++y) {
                const f32x4 fb = *reinterpret_cast<const f32x4*>(b + y * 32 * PLROW + off + 4 * v);
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s], fb[s], acc[x][y], 0, 0, 0);
                asm volatile("" ::: "memory");   // few operands live at once
            }
        }
}

__device__ inline bool not_finite(float v) { return !(fabsf(v) <= 3.402823466e38f); }

// ----------------------------------------------------------------------------
// w[k] = sum_i c[i] * X[k][i]^2 (c null: c = 1).  One wave per sample row.
template <bool VEC>
__global__ __launch_bounds__(256) void k_sample_weights(const float* __restrict__ X, int64_t N,
                                                        int64_t d, const float* __restrict__ c,
                                                        float* __restrict__ w) {
    const int64_t k = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (k >= N) return;
    const float* row = X + k * d;
    float acc = 0.0f;
    if (VEC) {
        for (int64_t i = 4 * l; i < d; i += 256) {
            const f32x4 x = *reinterpret_cast<const f32x4*>(row + i);
            const f32x4 cc = c ? *reinterpret_cast<const f32x4*>(c + i) : f32x4{1.f, 1.f, 1.f, 1.f};
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = fmaf(cc[u] * x[u], x[u], acc);
        }
    } else {
        for (int64_t i = l; i < d; i += 64) {
            const float x = row[i];
            acc = fmaf(c ? c[i] * x : x, x, acc);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if (l == 0) w[k] = acc;
}

// dst[i] = src[i * (d + 1)]: the diagonal of a d x d matrix.
__global__ __launch_bounds__(256) void k_diag(const float* __restrict__ src, int64_t d,
                                              float* __restrict__ dst) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < d) dst[i] = src[i * (d + 1)];
}

// ----------------------------------------------------------------------------
// Upper-triangle block (bi, bj), bi <= bj, of X^T diag(w) X over the samples of
// one slice [k_lo, k_hi): part[slice][blk] (GT x GT, row-major), on the bf16
// matrix cores with every fp32 operand split in three (split.h).
// A chunk is 16 samples.  Half of the threads stage the block's row features
// (with the weights), half its column features: thread (fi, kq) reads features
// 4 fi .. + 3 of samples 4 kq .. + 3 as four 16-byte row segments, transposes
// them in registers, splits them and writes four 8-byte pieces per plane,
// [plane][feature][sample].  LDS double-buffered, the next chunk in registers
// while the current one is multiplied.
// GT = 256: 8 waves of 128 x 64, one workgroup per CU (144 KiB of LDS);
// GT = 128: 4 waves of 64 x 64, two workgroups per CU.  What limits it
// (counters, 4096 features): no single unit.  The matrix cores are busy 56% of the
// cycles at the 2.0 GHz that the chip holds under this load, the LDS 24%, HBM delivers
// 0.6 TB/s; the one workgroup of a CU meets at a barrier per chunk.  Measured, 524288
// samples: 4096 features 79.8 -> 48.6 ms (110 -> 181 TFLOP/s) against the
// same product on fp32 MFMA, with a relative error against 64 bits of 5e-7
// instead of 3.8e-6; 400 features 1.58 -> 0.99 ms; rows that are not 16-byte
// aligned (3001 features, 100000 samples) 11.6 -> 5.6 ms, as they were read
// one float at a time.
struct GramArgs {
    const float* X;
    int64_t N, d;
    const float* w;
    int64_t slice_rows;   // samples per slice, a multiple of SPK
    int nb, nblk;         // blocks per side, upper-triangle blocks
    int slices;
    float* part;          // [slices][nblk][GT * GT]
};

// Block t of a slice -> (bi, bj), bi <= bj.  The upper triangle is walked in
// 8 x 8 supertiles (row-major over supertiles, row-major inside each), so that
// consecutive blocks share few column ranges of X.
constexpr int GSUPER = 8;
__device__ inline void gram_block_of(int t, int nb, int& bi, int& bj) {
    const int nS = (nb + GSUPER - 1) / GSUPER;
    for (int SI = 0; SI < nS; ++SI) {
        const int r0 = SI * GSUPER, r1 = min(nb, r0 + GSUPER);
        for (int SJ = SI; SJ < nS; ++SJ) {
            const int c0 = SJ * GSUPER, c1 = min(nb, c0 + GSUPER);
            if (SI == SJ) {
                const int w = r1 - r0;
                if (t < w * (w + 1) / 2) {
                    int i = r0;
                    while (t >= r1 - i) {
                        t -= r1 - i;
                        ++i;
                    }
                    bi = i;
                    bj = i + t;
                    return;
                }
                t -= w * (w + 1) / 2;
            } else {
                const int cnt = (r1 - r0) * (c1 - c0);
                if (t < cnt) {
                    bi = r0 + t / (c1 - c0);
                    bj = c0 + t % (c1 - c0);
                    return;
                }
                t -= cnt;
            }
        }
    }
    bi = bj = 0;   // not reached for t < nb (nb + 1) / 2
}

// Work item of a k_gram workgroup.  Workgroups are dealt to the 8 XCDs in
// turn (workgroup v runs on XCD v mod 8), so XCD x is given the contiguous
// range x * per .. of the work list (slices in order, blocks of a slice in
// supertile order): the workgroups resident on one XCD then stream the same
// samples and few column ranges, which stay in that XCD's L2.
constexpr int GXCD = 8;
__device__ inline int gram_work_of(int v, int total) {
    const int per = (total + GXCD - 1) / GXCD;
    return (v % GXCD) * per + v / GXCD;
}

template <int GT, int WX, int WY, bool PLAIN>
__global__ __launch_bounds__(64 * (GT / (32 * WX)) * (GT / (32 * WY)), 2) void k_gram(GramArgs a) {
    constexpr int WN = GT / (32 * WY);                   // waves along the columns
    constexpr int TH = 64 * (GT / (32 * WX)) * WN;
    static_assert(TH == 2 * GT, "one staging thread per 4 features x 4 samples of both operands");
    constexpr int PLANE = 2 * GT * SPROW;                // rows 0 .. GT - 1: A, GT .. 2 GT - 1: B
    __shared__ __attribute__((aligned(16))) uint16_t S[2][3 * PLANE];
    static_assert(2 * GT * PLROW * 4 <= (int)sizeof(S), "fp32 staging");
    __shared__ int redo;
    const int wk = gram_work_of((int)blockIdx.x, a.nblk * a.slices);
    if (wk >= a.nblk * a.slices) return;   // padding of the last XCD's range
    const int slice = wk / a.nblk;
    const int blk = wk % a.nblk;
    int bi, bj;
    gram_block_of(blk, a.nb, bi, bj);
    const int64_t k_lo = (int64_t)slice * a.slice_rows;
    const int64_t k_hi = min(a.N, k_lo + a.slice_rows);
    const int nch = k_hi > k_lo ? (int)((k_hi - k_lo + SPK - 1) / SPK) : 0;

    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = wv / WN, wn = wv % WN;
    // staging role (the operand is the same for a whole wave)
    const int op = wv >= TH / 128;                       // 0: A (weighted), 1: B
    const int t = tid & (TH / 2 - 1);
    const int kq = 4 * (t & 3), fi = 4 * (t >> 2);
    const int64_t f0 = (int64_t)(op ? bj : bi) * GT;
    const int64_t f = f0 + fi, d = a.d;
    const uint32_t off = (uint32_t)kq * (uint32_t)d + (uint32_t)(f < d ? f : 0);
    const bool full = f0 + GT <= d;                      // no feature of the block is padding
    const float* w = op ? nullptr : a.w;
    f32x4 r[4];
    float rw[4];
    int64_t kbase = 0;
    // Loads come from clamped, always valid addresses, so that they stay in
    // flight across the MFMAs of the current chunk; weights and masks are
    // applied when the registers are written to LDS.  Rows need not be 16-byte
    // aligned (the loads need 4).  A row segment that runs past column d reads
    // on into the next row, which exists except at the very end of X: the
    // chunks that come near it read entry by entry.
    auto load = [&](int64_t k0) {
        kbase = k0;
#pragma unroll
        for (int u = 0; u < 4; ++u) rw[u] = w ? w[min(k0 + kq + u, k_hi - 1)] : 1.0f;
        if (k0 + SPK <= k_hi && k0 + SPK + 4 <= a.N) {   // uniform
            const float* base = a.X + k0 * d;
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = *reinterpret_cast<const f32x4u*>(base + off + u * (uint32_t)d);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float* row = a.X + min(k0 + kq + u, k_hi - 1) * d;
#pragma unroll
                for (int v = 0; v < 4; ++v) r[u][v] = row[f + v < d ? f + v : 0];
            }
        }
    };
    auto weigh = [&]() {
        if (!full || kbase + SPK > k_hi) {   // uniform: padding features or samples
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    r[u][v] = (kbase + kq + u < k_hi && f + v < d) ? r[u][v] : 0.0f;
        }
        if (w) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float x = kbase + kq + u < k_hi ? rw[u] : 0.0f;
#pragma unroll
                for (int v = 0; v < 4; ++v) r[u][v] *= x;
            }
        }
    };
    auto store = [&](int sb) {
        weigh();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            split_store4(f32x4{r[0][v], r[1][v], r[2][v], r[3][v]},
                         &S[sb][(op * GT + fi + v) * SPROW + kq], PLANE);
    };
    f32x16 acc[WX][WY];
#pragma unroll
    for (int x = 0; x < WX; ++x)
#pragma unroll
        for (int y = 0; y < WY; ++y) acc[x][y] = f32x16{0};
    // acc[x][y][q] is entry (row (WX wm + x) * 32 + (q >> 2) * 8 + (l >> 5) * 4 + (q & 3),
    // column (WY wn + y) * 32 + (l & 31)) of the block
    float* const P = a.part + ((int64_t)slice * a.nblk + blk) * (GT * GT) +
                     (WX * wm * TS + (l >> 5) * 4) * GT + WY * wn * TS + (l & 31);
    if (tid == 0) redo = PLAIN;
    if constexpr (!PLAIN) {
        if (nch > 0) {
            load(k_lo);
            store(0);
        }
        __syncthreads();
        for (int c = 0; c < nch; ++c) {
            const int sb = c & 1;
            const bool more = c + 1 < nch;
            if (more) load(k_lo + (int64_t)(c + 1) * SPK);
            split_mma<WX, WY>(&S[sb][wm * WX * 32 * SPROW], &S[sb][(GT + wn * WY * 32) * SPROW], PLANE, l, acc);
            if (more) store(sb ^ 1);
            __syncthreads();
        }
        float z = 0.0f;   // stays 0 over finite entries
#pragma unroll
        for (int x = 0; x < WX; ++x)
#pragma unroll
            for (int y = 0; y < WY; ++y)
#pragma unroll
                for (int q = 0; q < 16; ++q) z = fmaf(acc[x][y][q], 0.0f, z);
        if (z != 0.0f) redo = 1;   // (NaN; the same value from every lane)
    }
    __syncthreads();   // (before the stores, which it would wait for)
    if constexpr (!PLAIN) {
#pragma unroll
        for (int x = 0; x < WX; ++x)
#pragma unroll
            for (int y = 0; y < WY; ++y)
#pragma unroll
                for (int q = 0; q < 16; ++q) P[(x * TS + (q >> 2) * 8 + (q & 3)) * GT + y * TS] = acc[x][y][q];
    }
    if (!redo) return;   // uniform
    float* const F = reinterpret_cast<float*>(&S[0][0]);   // rows 0 .. GT - 1: A, GT .. 2 GT - 1: B
#pragma unroll
    for (int x = 0; x < WX; ++x)
#pragma unroll
        for (int y = 0; y < WY; ++y) acc[x][y] = f32x16{0};
    for (int c = 0; c < nch; ++c) {
        load(k_lo + (int64_t)c * SPK);
        weigh();
#pragma unroll
        for (int v = 0; v < 4; ++v)
            *reinterpret_cast<f32x4*>(F + (op * GT + fi + v) * PLROW + kq) = f32x4{r[0][v], r[1][v], r[2][v], r[3][v]};
        __syncthreads();
        plain_mma<WX, WY>(F + wm * WX * 32 * PLROW, F + (GT + wn * WY * 32) * PLROW, l, acc);
        __syncthreads();
    }
    int again = 0;   // opaque: the addresses of the first pass are not kept over this one
    asm volatile("" : "+v"(again));
#pragma unroll
    for (int x = 0; x < WX; ++x)
#pragma unroll
        for (int y = 0; y < WY; ++y)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                float* const e = &P[again + (x * TS + (q >> 2) * 8 + (q & 3)) * GT + y * TS];
                if (PLAIN || not_finite(*e)) *e = acc[x][y][q];
                asm volatile("" ::: "memory");   // one entry at a time
            }
}

// One 32 x 32 sub-tile of a block: sum the slices in order and scale; write
// the upper-triangle entries, C[i][j] = s * G_ij * M_ij (i <= j), and mirror
// them, C[j][i] = s * G_ij * M_ji (i < j), so that C is exactly symmetric when
// M is (the weighted products of a diagonal block are not bitwise symmetric).
// Sub-tiles below the diagonal of a diagonal block are skipped: their entries
// are the mirror of the sub-tile above.  Every entry of C is read (M) and
// written by one thread, so M may alias C.
template <int GT>
__global__ __launch_bounds__(256) void k_gram_reduce(const float* __restrict__ part, int slices,
                                                     int nblk, int nb, int64_t d, float s,
                                                     const float* M, float* C) {
    constexpr int SB = GT / TS;   // sub-tiles per side
    __shared__ float T[TS][TS + 1];
    const int blk = (int)(blockIdx.x / (SB * SB)), sub = (int)(blockIdx.x % (SB * SB));
    int bi, bj;
    gram_block_of(blk, nb, bi, bj);
    const int sr = sub / SB, sc = sub % SB;
    if (bi == bj && sr > sc) return;
    const bool diag = bi == bj && sr == sc;   // the sub-tile straddles the diagonal
    const int r = threadIdx.x >> 3, c4 = 4 * (threadIdx.x & 7);
    const int64_t bo = (int64_t)blk * (GT * GT) + (sr * TS + r) * GT + sc * TS + c4;
    f32x4 g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int sl = 0; sl < slices; ++sl)   // unrolled: 8 loads in flight, added in order
        g += *reinterpret_cast<const f32x4*>(part + (int64_t)sl * nblk * (GT * GT) + bo);
    g *= s;
    const int64_t i = (int64_t)bi * GT + sr * TS + r;
    const int64_t jb = (int64_t)bj * GT + sc * TS + c4;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (i < d && jb + u < d && (!diag || r <= c4 + u)) {
            const int64_t o = i * d + jb + u;
            C[o] = M ? g[u] * M[o] : g[u];
        }
        T[r][c4 + u] = g[u];
    }
    __syncthreads();
    const int64_t il = (int64_t)bj * GT + sc * TS + r;   // mirrored row
    const int64_t jl = (int64_t)bi * GT + sr * TS + c4;  // mirrored columns
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (il < d && jl + u < d && (!diag || r > c4 + u)) {
            const int64_t o = il * d + jl + u;
            const float v = T[c4 + u][r];
            C[o] = M ? v * M[o] : v;
        }
    }
}

// ----------------------------------------------------------------------------
// Launch geometry of one Gram product.  The blocks of one slice are
// consecutive workgroups (they stream the same samples, which stay in L2).
// Block edge and slice count are chosen together by modelled time: rounds of
// workgroups over the chip times the chunks of a slice, plus writing and
// reading back every partial block at about 5 TB/s, plus 0.15 us per slice for
// the reduction's chain of additions.  A chunk of a wide block
// takes 1.9 us (one workgroup per CU), of a narrow one 1.1 us with two
// workgroups per CU; the wide block halves the operand bytes and LDS reads per
// product, the narrow one pads less.
struct GramGeom {
    int gt;               // block edge
    int nb, nblk, slices;
    int64_t slice_rows;
};

static GramGeom gram_geom(int64_t N, int64_t d, int ncu) {
    const int64_t nch = std::max<int64_t>(1, (N + SPK - 1) / SPK);
    GramGeom best{};
    double best_t = 0.0;
    for (int gt : {GBW, GB}) {
        const int64_t nb = (d + gt - 1) / gt, nblk = nb * (nb + 1) / 2;
        const int64_t slots = (gt == GBW ? 1 : 2) * (int64_t)std::max(ncu, 1);
        const double chunk = gt == GBW ? 1.9 : 1.1;
        for (int64_t S = 1; S <= 64 && S <= nch; ++S) {
            const int64_t per = (nch + S - 1) / S;
            const int64_t S_eff = (nch + per - 1) / per;
            const double t = (double)((nblk * S_eff + slots - 1) / slots) * (double)per * chunk +
                             8.0 * gt * gt / 5e6 * (double)(nblk * S_eff) + 0.15 * (double)S_eff;
            if (best.gt == 0 || t < best_t - 1e-9) {
                best_t = t;
                best.gt = gt;
                best.nb = (int)nb;
                best.nblk = (int)nblk;
                best.slices = (int)S_eff;
                best.slice_rows = per * SPK;
            }
        }
    }
    return best;
}

static size_t gram_part_bytes(const GramGeom& g) {
    return (size_t)g.slices * g.nblk * g.gt * g.gt * sizeof(float);
}

static hipError_t run_sample_weights(hipStream_t st, const float* X, int64_t N, int64_t d,
                                     const float* c, float* w) {
    if (N == 0) return hipSuccess;
    const bool vec = d % 4 == 0 && ((uintptr_t)X & 15) == 0 && (!c || ((uintptr_t)c & 15) == 0);
    const dim3 grid((unsigned)((N + 3) / 4));
    if (vec)
        hipLaunchKernelGGL(k_sample_weights<true>, grid, dim3(256), 0, st, X, N, d, c, w);
    else
        hipLaunchKernelGGL(k_sample_weights<false>, grid, dim3(256), 0, st, X, N, d, c, w);
    return hipGetLastError();
}

static hipError_t run_gram(hipStream_t st, const GramGeom& g, const float* X, int64_t N, int64_t d,
                           const float* w, float s, const float* M, float* C, float* part) {
    if (d == 0) return hipSuccess;
    GramArgs a{X, N, d, w, g.slice_rows, g.nb, g.nblk, g.slices, part};
    const int64_t total = (int64_t)g.nblk * g.slices;
    const dim3 grid((unsigned)(((total + GXCD - 1) / GXCD) * GXCD));
    const unsigned subs = (unsigned)(g.nblk * (g.gt / TS) * (g.gt / TS));
    if (N <= PLAIN_TERMS)
        hipLaunchKernelGGL((g.gt == GBW ? k_gram<GBW, 4, 2, true> : k_gram<GB, 2, 2, true>), grid, dim3(2 * g.gt), 0, st, a);
    else
        hipLaunchKernelGGL((g.gt == GBW ? k_gram<GBW, 4, 2, false> : k_gram<GB, 2, 2, false>), grid, dim3(2 * g.gt), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g.gt == GBW)
        hipLaunchKernelGGL(k_gram_reduce<GBW>, dim3(subs), dim3(256), 0, st, part, g.slices, g.nblk,
                           g.nb, d, s, M, C);
    else
        hipLaunchKernelGGL(k_gram_reduce<GB>, dim3(subs), dim3(256), 0, st, part, g.slices, g.nblk,
                           g.nb, d, s, M, C);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Per-sample quadratic forms w_k = x_k^T M x_k (M symmetric d x d): the
// weights tr(b^T B b) of the later Shampoo power steps (App. A).  Workgroup
// (row block R, column block J) computes the GT x GT tile of Y = X M
// (Y_kj = sum_t X_kt M_jt, M symmetric) on the bf16 matrix cores (split.h),
// then part[J][k] = sum_{j in J} Y_kj X_kj.  Both operands are rows with the
// inner index contiguous: half of the threads stage X, half M, each thread 4
// inner entries of 4 rows per 16-wide chunk.  k_quadform_reduce adds the
// column blocks in order.
struct QuadArgs {
    const float* X;
    int64_t N, d;
    const float* M;
    int nJ;
    float* part;   // [nJ][N]
};

template <int GT, int WX, int WY, bool PLAIN>
__global__ __launch_bounds__(64 * (GT / (32 * WX)) * (GT / (32 * WY)), 2) void k_quadform(QuadArgs a) {
    constexpr int WN = GT / (32 * WY);
    constexpr int TH = 64 * (GT / (32 * WX)) * WN;
    static_assert(TH == 2 * GT, "one staging thread per 4 rows x 4 inner entries of both operands");
    constexpr int PLANE = 2 * GT * SPROW;
    __shared__ __attribute__((aligned(16))) uint16_t S[2][3 * PLANE];
    static_assert(2 * GT * PLROW * 4 <= (int)sizeof(S), "fp32 staging");
    __shared__ float red[WN][GT];
    __shared__ int redo;
    const int J = (int)(blockIdx.x % (unsigned)a.nJ);
    const int64_t R = blockIdx.x / (unsigned)a.nJ;
    const int64_t k0 = R * GT, j0 = (int64_t)J * GT;
    const int64_t d = a.d;
    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = wv / WN, wn = wv % WN;
    const int op = wv >= TH / 128;                       // 0: X, 1: M
    const int t = tid & (TH / 2 - 1);
    const int kq = 4 * (t & 3), row0 = t >> 2;           // rows row0 + u GT / 4
    const int64_t rbase = op ? j0 : k0, rows = op ? d : a.N;
    const float* src = op ? a.M : a.X;
    const float* p[4];
    bool in[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t row = rbase + row0 + u * (GT / 4);
        in[u] = row < rows;
        p[u] = src + (in[u] ? row : 0) * d;
    }
    f32x4 r[4];
    auto load = [&](int64_t t0) {
        if (t0 + SPK <= d) {   // uniform: the chunk lies inside the rows
#pragma unroll
            for (int u = 0; u < 4; ++u) r[u] = *reinterpret_cast<const f32x4u*>(p[u] + t0 + kq);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) r[u][v] = t0 + kq + v < d ? p[u][t0 + kq + v] : 0.0f;
        }
    };
    auto store = [&](int sb) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            split_store4(in[u] ? r[u] : f32x4{0.0f, 0.0f, 0.0f, 0.0f},
                         &S[sb][(op * GT + row0 + u * (GT / 4)) * SPROW + kq], PLANE);
    };
    f32x16 acc[WX][WY];
#pragma unroll
    for (int x = 0; x < WX; ++x)
#pragma unroll
        for (int y = 0; y < WY; ++y) acc[x][y] = f32x16{0};
    const int nch = (int)((d + SPK - 1) / SPK);
    if (tid == 0) redo = PLAIN;
    if constexpr (!PLAIN) {
        load(0);
        store(0);
        __syncthreads();
        for (int c = 0; c < nch; ++c) {
            const int sb = c & 1;
            const bool more = c + 1 < nch;
            if (more) load((int64_t)(c + 1) * SPK);
            split_mma<WX, WY>(&S[sb][wm * WX * 32 * SPROW], &S[sb][(GT + wn * WY * 32) * SPROW], PLANE, l, acc);
            if (more) store(sb ^ 1);
            __syncthreads();
        }
    }
    // acc[x][y][q] = Y(row (WX wm + x) * 32 + (q >> 2) * 8 + (l >> 5) * 4 + (q & 3),
    //                  column (WY wn + y) * 32 + (l & 31)); row sums of Y (.) X over
    // the wave's columns, then over the lanes of a row, then over the waves that
    // share the rows
    auto row_sum = [&](int l) -> float {   // of row tid, for tid < GT
        const int lr = l & 31;
#pragma unroll
        for (int x = 0; x < WX; ++x)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int row = (WX * wm + x) * TS + (q >> 2) * 8 + (l >> 5) * 4 + (q & 3);
                const int64_t k = k0 + row;
                float v = 0.0f;
#pragma unroll
                for (int y = 0; y < WY; ++y) {
                    const int64_t j = j0 + (WY * wn + y) * TS + lr;
                    const bool at = k < a.N && j < d;   // (a padding column of an infinite row holds NaN)
                    v = fmaf(at ? acc[x][y][q] : 0.0f, at ? a.X[k * d + j] : 0.0f, v);
                }
#pragma unroll
                for (int off = 16; off >= 1; off >>= 1) v += __shfl_xor(v, off, 32);
                if (lr == 0) red[wn][row] = v;
            }
        __syncthreads();
        float v = 0.0f;
        if (tid < GT) {
            v = red[0][tid];
#pragma unroll
            for (int i = 1; i < WN; ++i) v += red[i][tid];
        }
        return v;
    };
    float v = 0.0f;
    if constexpr (!PLAIN) {
        v = row_sum(l);
        if (tid < GT && not_finite(v)) redo = 1;   // (the same value from every lane)
    }
    __syncthreads();
    if (redo) {   // uniform
        float* const F = reinterpret_cast<float*>(&S[0][0]);   // rows 0 .. GT - 1: X, GT .. 2 GT - 1: M
#pragma unroll
        for (int x = 0; x < WX; ++x)
#pragma unroll
            for (int y = 0; y < WY; ++y) acc[x][y] = f32x16{0};
        for (int c = 0; c < nch; ++c) {
            load((int64_t)c * SPK);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                *reinterpret_cast<f32x4*>(F + (op * GT + row0 + u * (GT / 4)) * PLROW + kq) =
                    in[u] ? r[u] : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            __syncthreads();
            plain_mma<WX, WY>(F + wm * WX * 32 * PLROW, F + (GT + wn * WY * 32) * PLROW, l, acc);
            __syncthreads();
        }
        int l2 = l;   // opaque: the addresses of the first pass are not kept over this one
        asm volatile("" : "+v"(l2));
        const float p = row_sum(l2);
        if (PLAIN || not_finite(v)) v = p;
    }
    if (tid < GT && k0 + tid < a.N) a.part[(int64_t)J * a.N + k0 + tid] = v;
}

__global__ __launch_bounds__(256) void k_quadform_reduce(const float* __restrict__ part, int nJ,
                                                         int64_t N, float* __restrict__ w) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= N) return;
    float s = 0.0f;
    for (int J = 0; J < nJ; ++J) s += part[(int64_t)J * N + k];
    w[k] = s;
}

// C = A (.) B entrywise (n elements); C may alias A or B.
__global__ __launch_bounds__(256) void k_hadamard(const float* A, const float* B, int64_t n,
                                                  float* C) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < n) C[e] = A[e] * B[e];
}

static int device_cus() {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return ncu;
}

static size_t quadform_part_bytes(int64_t N, int64_t d) {
    return (size_t)((d + GB - 1) / GB) * (size_t)std::max<int64_t>(N, 1) * sizeof(float);
}

static hipError_t run_quadform(hipStream_t st, const float* X, int64_t N, int64_t d, const float* M,
                               float* w, float* part) {
    if (N == 0) return hipSuccess;
    // wide blocks where they fill the chip and do not pad a narrow d
    const bool wide = d > GB && ((N + GBW - 1) / GBW) * ((d + GBW - 1) / GBW) >= device_cus();
    const int64_t gt = wide ? GBW : GB;
    const int nJ = (int)std::max<int64_t>(1, (d + gt - 1) / gt);
    QuadArgs a{X, N, d, M, nJ, part};
    const dim3 grid((unsigned)(((N + gt - 1) / gt) * nJ));
    if (d <= PLAIN_TERMS)   // (never wide)
        hipLaunchKernelGGL((k_quadform<GB, 2, 2, true>), grid, dim3(2 * GB), 0, st, a);
    else if (wide)
        hipLaunchKernelGGL((k_quadform<GBW, 4, 2, false>), grid, dim3(2 * GBW), 0, st, a);
    else
        hipLaunchKernelGGL((k_quadform<GB, 2, 2, false>), grid, dim3(2 * GB), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_quadform_reduce, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, st, part,
                       nJ, N, w);
    return hipGetLastError();
}

}  // namespace bk

// ============================================================================
// C ABI (declared in bakron.h)

using bk::GramGeom;

static bakron_status hess_fail(const char* msg) {
    bk::set_last_error(msg);
    return BAKRON_EINVAL;
}

static bakron_status hess_hip(hipError_t e, const char* what) {
    char buf[256];
    std::snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
    bk::set_last_error(buf);
    return e == hipErrorOutOfMemory ? BAKRON_ENOMEM : BAKRON_EHIP;
}

static inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Dimension limits: blocks per side fit the launch grid comfortably.
static const int64_t HESS_DIM_MAX = (int64_t)1 << 17;
static const int64_t HESS_N_MAX = (int64_t)1 << 40;

// Workspace handshake shared by the factor-construction calls: with work ==
// NULL report the size; otherwise check it.
static bakron_status workspace_check(void* work, size_t* work_bytes, size_t need, bool* query) {
    *query = false;
    if (!work_bytes) return hess_fail("work_bytes is NULL");
    if (!work) {
        *work_bytes = need;
        *query = true;
        return BAKRON_OK;
    }
    if (*work_bytes < need) return hess_fail("workspace too small");
    if (((uintptr_t)work & 255) != 0) return hess_fail("workspace not 256-byte aligned");
    return BAKRON_OK;
}

extern "C" bakron_status bakron_sample_weights(const float* X, int64_t N, int64_t d, const float* c,
                                               float* w, hipStream_t stream) {
    bk::set_last_error("");
    if (N < 0 || d < 0 || N > HESS_N_MAX || d > HESS_DIM_MAX) return hess_fail("bad size");
    if (N > 0 && (!w || (d > 0 && !X))) return hess_fail("null pointer");
    hipError_t e = bk::run_sample_weights(stream, X, N, d, c, w);
    return e == hipSuccess ? BAKRON_OK : hess_hip(e, "bakron_sample_weights: launch");
}

extern "C" bakron_status bakron_gram(const float* X, int64_t N, int64_t d, const float* w, float s,
                                     const float* M, float* C, void* work, size_t* work_bytes,
                                     hipStream_t stream) {
    bk::set_last_error("");
    if (N < 0 || d < 0 || N > HESS_N_MAX || d > HESS_DIM_MAX) return hess_fail("bad size");
    const GramGeom g = bk::gram_geom(N, d, bk::device_cus());
    bool query;
    bakron_status st = workspace_check(work, work_bytes, bk::gram_part_bytes(g), &query);
    if (st != BAKRON_OK || query) return st;
    if (d > 0 && (!C || (N > 0 && !X))) return hess_fail("null pointer");
    hipError_t e = bk::run_gram(stream, g, X, N, d, w, s, M, C, static_cast<float*>(work));
    return e == hipSuccess ? BAKRON_OK : hess_hip(e, "bakron_gram: launch");
}

// Carves the workspace: [partials | weights x2 | extra], 256-byte aligned.
struct HessWork {
    float* part;
    float* w0;
    float* w1;
    float* extra;
};
static HessWork carve(void* work, size_t part, size_t wbytes) {
    char* p = static_cast<char*>(work);
    HessWork h;
    h.part = reinterpret_cast<float*>(p);
    h.w0 = reinterpret_cast<float*>(p + align256(part));
    h.w1 = reinterpret_cast<float*>(p + align256(part) + wbytes);
    h.extra = reinterpret_cast<float*>(p + align256(part) + 2 * wbytes);
    return h;
}

// Global (vector) case, App. A: K-FAC, or `iters` unnormalised power steps
// from (I, I).  Step 1 weighs by |b_k|^2 and |a_k|^2; step i > 1 by
// b_k^T B^(i-1) b_k and a_k^T A^(i-1) a_k, after which A and B are
// overwritten in place (the previous pair is no longer needed).
static bakron_status kron_factors_impl(const char* who, const float* a, const float* b, int64_t N,
                                       int64_t n, int64_t m, bool shampoo, int iters, float* A,
                                       float* B, void* work, size_t* work_bytes,
                                       hipStream_t stream) {
    if (N <= 0 || n <= 0 || m <= 0 || N > HESS_N_MAX || n > HESS_DIM_MAX || m > HESS_DIM_MAX ||
        iters < 1 || iters > 64)
        return hess_fail("bad size or iteration count");
    if (iters > 1 && ((N + bk::GB - 1) / bk::GB) * ((std::max(n, m) + bk::GB - 1) / bk::GB) >
                         ((int64_t)1 << 31) - 1)
        return hess_fail("too many samples for the power steps");
    const int ncu = bk::device_cus();
    const GramGeom ga = bk::gram_geom(N, n, ncu), gb = bk::gram_geom(N, m, ncu);
    size_t part = std::max(bk::gram_part_bytes(ga), bk::gram_part_bytes(gb));
    if (iters > 1)
        part = std::max({part, bk::quadform_part_bytes(N, n), bk::quadform_part_bytes(N, m)});
    const size_t wbytes = shampoo ? align256((size_t)N * sizeof(float)) : 0;
    bool query;
    bakron_status st = workspace_check(work, work_bytes, align256(part) + 2 * wbytes, &query);
    if (st != BAKRON_OK || query) return st;
    if (!a || !b || !A || !B) return hess_fail("null pointer");
    const HessWork h = carve(work, part, wbytes);
    const float inv = (float)(1.0 / (double)N);
    float* wa = shampoo ? h.w0 : nullptr;   // weights of B (from a)
    float* wb = shampoo ? h.w1 : nullptr;   // weights of A (from b)
    hipError_t e = hipSuccess;
    for (int it = 1; it <= (shampoo ? iters : 1); ++it) {
        if (shampoo && it == 1) {
            if ((e = bk::run_sample_weights(stream, a, N, n, nullptr, wa)) != hipSuccess ||
                (e = bk::run_sample_weights(stream, b, N, m, nullptr, wb)) != hipSuccess)
                return hess_hip(e, who);
        } else if (shampoo) {
            if ((e = bk::run_quadform(stream, a, N, n, A, wa, h.part)) != hipSuccess ||
                (e = bk::run_quadform(stream, b, N, m, B, wb, h.part)) != hipSuccess)
                return hess_hip(e, who);
        }
        if ((e = bk::run_gram(stream, ga, a, N, n, wb, inv, nullptr, A, h.part)) != hipSuccess ||
            (e = bk::run_gram(stream, gb, b, N, m, wa, inv, nullptr, B, h.part)) != hipSuccess)
            return hess_hip(e, who);
    }
    return BAKRON_OK;
}

// MLP-local case, App. A, b = D_g W_down^T: b b^T = (g g^T) (.) D^T D and
// tr(b^T X b) = g^T (X (.) D^T D) g.  Step 1 of Shampoo weighs A by
// g^T diag(D^T D) g and B by |x|^2; step i > 1 by g^T (B^(i-1) (.) D^T D) g
// and x^T A^(i-1) x.
static bakron_status mlp_local_impl(const char* who, const float* x, const float* g,
                                    const float* D, int64_t N, int64_t dm, int64_t dff,
                                    bool shampoo, int iters, float* A, float* B, void* work,
                                    size_t* work_bytes, hipStream_t stream) {
    if (N <= 0 || dm <= 0 || dff <= 0 || N > HESS_N_MAX || dm > HESS_DIM_MAX || dff > HESS_DIM_MAX ||
        iters < 1 || iters > 64)
        return hess_fail("bad size or iteration count");
    if (iters > 1 && ((N + bk::GB - 1) / bk::GB) * ((std::max(dm, dff) + bk::GB - 1) / bk::GB) >
                         ((int64_t)1 << 31) - 1)
        return hess_fail("too many samples for the power steps");
    const bool multi = shampoo && iters > 1;
    const int ncu = bk::device_cus();
    const GramGeom gx = bk::gram_geom(N, dm, ncu), gg = bk::gram_geom(N, dff, ncu),
                   gd = bk::gram_geom(dm, dff, ncu);
    size_t part = std::max({bk::gram_part_bytes(gx), bk::gram_part_bytes(gg),
                            bk::gram_part_bytes(gd)});
    if (multi)
        part = std::max({part, bk::quadform_part_bytes(N, dm), bk::quadform_part_bytes(N, dff)});
    const size_t wbytes = shampoo ? align256((size_t)N * sizeof(float)) : 0;
    // extra: the diagonal of D^T D (step 1), and D^T D itself kept apart from B
    // for the later steps
    const size_t cbytes = shampoo ? align256((size_t)dff * sizeof(float)) : 0;
    const size_t dbytes = multi ? (size_t)dff * (size_t)dff * sizeof(float) : 0;
    bool query;
    bakron_status st =
        workspace_check(work, work_bytes, align256(part) + 2 * wbytes + cbytes + dbytes, &query);
    if (st != BAKRON_OK || query) return st;
    if (!x || !g || !D || !A || !B) return hess_fail("null pointer");
    const HessWork h = carve(work, part, wbytes);
    const float inv = (float)(1.0 / (double)N);
    float* wx = shampoo ? h.w0 : nullptr;   // weights of B (from x)
    float* wg = shampoo ? h.w1 : nullptr;   // weights of A (from g)
    float* cdiag = h.extra;
    float* DtD = multi ? reinterpret_cast<float*>(reinterpret_cast<char*>(h.extra) + cbytes) : B;
    hipError_t e;
    // D^T D (rows of D = W_down as samples)
    if ((e = bk::run_gram(stream, gd, D, dm, dff, nullptr, 1.0f, nullptr, DtD, h.part)) != hipSuccess)
        return hess_hip(e, who);
    const int64_t nn = dff * dff;
    for (int it = 1; it <= (shampoo ? iters : 1); ++it) {
        if (shampoo && it == 1) {
            hipLaunchKernelGGL(bk::k_diag, dim3((unsigned)((dff + 255) / 256)), dim3(256), 0, stream,
                               DtD, dff, cdiag);
            if ((e = hipGetLastError()) != hipSuccess ||
                (e = bk::run_sample_weights(stream, g, N, dff, cdiag, wg)) != hipSuccess ||
                (e = bk::run_sample_weights(stream, x, N, dm, nullptr, wx)) != hipSuccess)
                return hess_hip(e, who);
        } else if (shampoo) {
            // B <- B^(i-1) (.) D^T D, the matrix of g's quadratic form
            hipLaunchKernelGGL(bk::k_hadamard, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, stream,
                               B, DtD, nn, B);
            if ((e = hipGetLastError()) != hipSuccess ||
                (e = bk::run_quadform(stream, g, N, dff, B, wg, h.part)) != hipSuccess ||
                (e = bk::run_quadform(stream, x, N, dm, A, wx, h.part)) != hipSuccess)
                return hess_hip(e, who);
        }
        // A = E[w_g x x^T]; B = E[w_x g g^T] (.) D^T D (in place over D^T D in
        // the one-step case)
        if ((e = bk::run_gram(stream, gx, x, N, dm, wg, inv, nullptr, A, h.part)) != hipSuccess ||
            (e = bk::run_gram(stream, gg, g, N, dff, wx, inv, DtD, B, h.part)) != hipSuccess)
            return hess_hip(e, who);
    }
    return BAKRON_OK;
}

extern "C" bakron_status bakron_kron_factors(const float* a, const float* b, int64_t N, int64_t n,
                                             int64_t m, int32_t style, float* A, float* B,
                                             void* work, size_t* work_bytes, hipStream_t stream) {
    bk::set_last_error("");
    if (style != BAKRON_KFAC && style != BAKRON_SHAMPOO) return hess_fail("bad style");
    return kron_factors_impl("bakron_kron_factors", a, b, N, n, m, style == BAKRON_SHAMPOO, 1, A, B,
                             work, work_bytes, stream);
}

extern "C" bakron_status bakron_kron_factors_iter(const float* a, const float* b, int64_t N,
                                                  int64_t n, int64_t m, int32_t iters, float* A,
                                                  float* B, void* work, size_t* work_bytes,
                                                  hipStream_t stream) {
    bk::set_last_error("");
    return kron_factors_impl("bakron_kron_factors_iter", a, b, N, n, m, true, iters, A, B, work,
                             work_bytes, stream);
}

extern "C" bakron_status bakron_mlp_local_factors(const float* x, const float* g, const float* D,
                                                  int64_t N, int64_t dm, int64_t dff, int32_t style,
                                                  float* A, float* B, void* work, size_t* work_bytes,
                                                  hipStream_t stream) {
    bk::set_last_error("");
    if (style != BAKRON_KFAC && style != BAKRON_SHAMPOO) return hess_fail("bad style");
    return mlp_local_impl("bakron_mlp_local_factors", x, g, D, N, dm, dff, style == BAKRON_SHAMPOO, 1,
                          A, B, work, work_bytes, stream);
}

extern "C" bakron_status bakron_mlp_local_factors_iter(const float* x, const float* g,
                                                       const float* D, int64_t N, int64_t dm,
                                                       int64_t dff, int32_t iters, float* A,
                                                       float* B, void* work, size_t* work_bytes,
                                                       hipStream_t stream) {
    bk::set_last_error("");
    return mlp_local_impl("bakron_mlp_local_factors_iter", x, g, D, N, dm, dff, true, iters, A, B,
                          work, work_bytes, stream);
}

extern "C" bakron_status bakron_quadform_weights(const float* X, int64_t N, int64_t d,
                                                 const float* M, float* w, void* work,
                                                 size_t* work_bytes, hipStream_t stream) {
    bk::set_last_error("");
    if (N < 0 || d < 0 || N > HESS_N_MAX || d > HESS_DIM_MAX ||
        ((N + bk::GB - 1) / bk::GB) * ((d + bk::GB - 1) / bk::GB) > ((int64_t)1 << 31) - 1)
        return hess_fail("bad size");
    bool query;
    bakron_status st = workspace_check(work, work_bytes, bk::quadform_part_bytes(N, d), &query);
    if (st != BAKRON_OK || query) return st;
    if (N > 0 && (!w || (d > 0 && (!X || !M)))) return hess_fail("null pointer");
    if (d == 0) {   // empty forms: w = 0 (the weight kernel with no features)
        hipError_t e = bk::run_sample_weights(stream, X, N, 0, nullptr, w);
        return e == hipSuccess ? BAKRON_OK : hess_hip(e, "bakron_quadform_weights");
    }
    hipError_t e = bk::run_quadform(stream, X, N, d, M, w, static_cast<float*>(work));
    return e == hipSuccess ? BAKRON_OK : hess_hip(e, "bakron_quadform_weights: launch");
}
