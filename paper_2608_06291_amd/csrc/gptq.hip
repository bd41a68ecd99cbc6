// One-sided rounding for B = I (GPTQ, Alg. 1 applied to every row of W with
// the Hessian A; Sec. 1 and Table 1: n sequential steps, O(mn^2) work).
//
// With B = I the feedback of Eq. (1) never crosses rows:
//     W~_pq = W0_pq + sum_{j<q} E_pj L^A_qj ,   E = V - W~ ,
// so the rows are independent and each row is a sequential pass over its n
// columns.  Two levels of blocking (GPTQ's lazy batch updates):
//   * ranges of GR column tiles (1024 columns).  Once a range is rounded, its
//     errors are pushed into every later column of a working copy W' of W
//     in one full-chip product (k_gptq_push), so the bulk of
//     the O(mn^2) work does not depend on how many rows there are;
//   * inside a range, blocks of 32 columns (one factor tile), k_gptq:
//     1. lazy feedback: W~[rows, blk] = W'[rows, blk] + E[rows, range start
//        .. blk] L^A[blk, ...]^T, a dense product on fp32 MFMA over the
//        earlier blocks of the range;
//     2. the 32 columns of the block in order: quantise column j of every
//        row, then add E[:, j] L^A[q, j] to the later columns q of the block.
// The sums are the same elementary updates of Eq. (1), in another order.
//
// A k_gptq workgroup owns 16 rows and walks the blocks of one range; the errors
// of the last RT blocks stay in LDS, older ones of the range (if RT is less than
// its length) are read back from memory.  In step 1 each of its 4 waves multiplies a
// quarter of the source tiles with v_mfma_f32_16x16x4f32 (A = the 16 error rows,
// B = the factor tile rows, so D[i][j] = sum_k E[i][k] L^A[j][k]), with the
// factor tiles of the next two in flight; the four partial sums meet in LDS.
// In step 2 each wave owns 4 rows, 16 lanes per row with the block columns c
// and c + 16 in registers; the error of column j is broadcast along its 16
// lanes with a DPP row broadcast, so no barrier is needed inside the block.
// What bounds it: the chain of 32 dependent columns per block and the memory
// latency between two blocks, so all that a block needs besides the errors is
// read ahead of it.  512 x 1500 (47 blocks, one push): 334 us with a lane shuffle
// through LDS per column, the errors re-read from memory and the block's inputs
// read after step 1; 253 us now.
#include <utility>

#include "common.h"
#include "split.h"

namespace bk {

struct GptqArgs {
    int64_t m, n;
    int nt;           // column tiles
    int64_t ldE;      // row stride of the error workspace (nt * 32)
    const float* Wb;  // base values of the range: W (the first range) or W'
    int64_t ldWb;     // their row stride
    const float* LA;  // packed unit-lower factor tiles
    float* E;         // errors, ceil(m/16)*16 x nt*32 row-major (workspace)
    int b_begin, b_end;   // the column tiles of this launch
    QuantArgs q;
    int8_t* codes;
    float* V;
    float* pre;       // may be null
};

constexpr int GR = 32;   // column tiles per range (1024 columns; the default of run_gptq)

__device__ inline f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

__device__ inline void mfma16_8(f32x4 a0, f32x4 a1, f32x4 b0, f32x4 b1, f32x4& acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[t], b0[t], acc, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t], b1[t], acc, 0, 0, 0);
}

constexpr int GW = 4;   // waves per workgroup

// f(0), f(1), .. with the index as a constant
template <class F, int... J>
__device__ __forceinline__ void columns(F& f, std::integer_sequence<int, J...>) {
    (f(std::integral_constant<int, J>{}), ...);
}

// RT: the last RT column tiles of errors are kept in LDS (a ring); OLD: the range
// may be longer, then the errors of the older tiles come from memory.  WG:
// workgroups per CU.
template <int RT, bool OLD, int WG>
__global__ __launch_bounds__(64 * GW, WG) void k_gptq(GptqArgs a) {
    constexpr int ESTR = RT * TS + 4;
    __shared__ float part[GW][16][33];   // per wave: partial 16 x 32 lazy products
    __shared__ __attribute__((aligned(16))) float Es[16][ESTR];   // errors of the last RT tiles
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int64_t row0 = (int64_t)blockIdx.x * 16;
    // step 1 lane roles: A row i16, k chunk [8 s, 8 s + 8) of every source tile
    const int i16 = l & 15, s = l >> 4;
    // step 2 lane roles: row rr of the 16, block columns c16 and c16 + 16
    const int rr = 4 * w + (l >> 4), c16 = l & 15;
    const int64_t row = row0 + rr;
    const float qlo = a.q.qlo, qhi = a.q.qhi;
    const float nan = __builtin_nanf("");

    // the factor tiles of the wave's next two sources; the first two of a block
    // are read while the block before it is rounded
    // (block bn, source tile kt; an old tile's errors were written RT blocks ago)
    f32x4 f[2][4], eo[2][2];
    const float* const erow = a.E + (row0 + i16) * a.ldE + 8 * s;
    auto ldf = [&](const float* p, int bn, int kt, int q) {
        f[q][0] = ld4(p);
        f[q][1] = ld4(p + 4);
        f[q][2] = ld4(p + 16 * TS);
        f[q][3] = ld4(p + 16 * TS + 4);
        if (OLD && kt < bn - RT) {   // uniform
            eo[q][0] = ld4(erow + kt * TS);
            eo[q][1] = ld4(erow + kt * TS + 4);
        }
    };
    for (int b = a.b_begin; b < a.b_end; ++b) {
        // the block's own inputs, in flight during step 1: base values, scales and
        // L^A[col][blk] of the lane's two columns
        const int64_t col0 = (int64_t)b * TS + c16, col1 = col0 + 16;
        const bool in0 = row < a.m && col0 < a.n, in1 = row < a.m && col1 < a.n;
        const float w0 = in0 ? a.Wb[row * a.ldWb + col0] : 0.0f;
        const float w1 = in1 ? a.Wb[row * a.ldWb + col1] : 0.0f;
        const float s0 = entry_scale(a.q, row, col0, a.m, a.n);
        const float s1 = entry_scale(a.q, row, col1, a.m, a.n);
        f32x4 u0[TS / 4], u1[TS / 4];
        {
            const float* d = a.LA + packed_tile_offset(b, b);
#pragma unroll
            for (int j = 0; j < TS / 4; ++j) {
                u0[j] = ld4(d + c16 * TS + 4 * j);
                u1[j] = ld4(d + (16 + c16) * TS + 4 * j);
            }
        }
        // 1. lazy feedback from the range's source tiles kt < b (a quarter per wave),
        // the factor tiles of two in flight: set 0 holds tiles w, w + 2 GW,
        // ..., set 1 tiles w + GW, w + 3 GW, ...; the errors are in LDS
        f32x4 acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = {0.0f, 0.0f, 0.0f, 0.0f};
        {
            const float* lt = a.LA + packed_tile_offset(b, 0) + i16 * TS + 8 * s;
            auto mul = [&](int kt, int q) {
                f32x4 x0 = eo[q][0], x1 = eo[q][1];
                if (!OLD || kt >= b - RT) {   // uniform
                    const float* e = &Es[i16][(OLD ? (kt - a.b_begin) % RT : kt - a.b_begin) * TS + 8 * s];
                    x0 = ld4(e);
                    x1 = ld4(e + 4);
                }
                mfma16_8(x0, x1, f[q][0], f[q][1], acc0);   // output columns 0..15 of the block
                mfma16_8(x0, x1, f[q][2], f[q][3], acc1);   // output columns 16..31
            };
            int kt = a.b_begin + w;
            for (; kt + GW < b; kt += 2 * GW) {
                mul(kt, 0);
                if (kt + 2 * GW < b) ldf(lt + (kt + 2 * GW) * TILE_ELEMS, b, kt + 2 * GW, 0);
                mul(kt + GW, 1);
                if (kt + 3 * GW < b) ldf(lt + (kt + 3 * GW) * TILE_ELEMS, b, kt + 3 * GW, 1);
            }
            if (kt < b) mul(kt, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            part[w][4 * s + r][i16] = acc0[r];
            part[w][4 * s + r][16 + i16] = acc1[r];
        }
        __syncthreads();

        // 2. the block's 32 columns in order, 16 lanes per row
        float h0 = part[0][rr][c16], h1 = part[0][rr][16 + c16];
#pragma unroll
        for (int v = 1; v < GW; ++v) {
            h0 += part[v][rr][c16];
            h1 += part[v][rr][16 + c16];
        }
        if (in0) h0 += w0;
        if (in1) h1 += w1;
        const float is0 = s0 > 0.0f ? 1.0f / s0 : 0.0f;   // zero scale: alphabet {0}
        const float is1 = s1 > 0.0f ? 1.0f / s1 : 0.0f;
        // strictly below the diagonal
        float c0[TS], c1[TS];
#pragma unroll
        for (int j = 0; j < TS; ++j) {
            c0[j] = j < c16 ? u0[j >> 2][j & 3] : 0.0f;
            c1[j] = j < 16 + c16 ? u1[j >> 2][j & 3] : 0.0f;
        }
        if (b + 1 < a.b_end) {
            const float* lt = a.LA + packed_tile_offset(b + 1, 0) + i16 * TS + 8 * s;
            const int kt = a.b_begin + w;
            if (kt <= b) ldf(lt + kt * TILE_ELEMS, b + 1, kt, 0);
            if (kt + GW <= b) ldf(lt + (kt + GW) * TILE_ELEMS, b + 1, kt + GW, 1);
        }
        float e0 = 0.0f, e1 = 0.0f, x0 = 0.0f, x1 = 0.0f;
        auto column = [&](auto C) {
            constexpr int j = C.value;
            constexpr bool hi = j >= 16;                   // column j sits in slot 1
            const float hv = hi ? h1 : h0, iv = hi ? is1 : is0, sv = hi ? s1 : s0;
            const float xv = hv * iv;
            const float cq = __builtin_amdgcn_fmed3f(rintf(xv), qlo, qhi);
            const float ev = fmaf(cq, sv, -hv);
            // the owner of column j is lane (j & 15) of the row's 16 lanes: DPP row
            // broadcast (row_newbcast), one operation instead of a trip through LDS
            const float ej = __int_as_float(
                __builtin_amdgcn_update_dpp(0, __float_as_int(ev), 0x150 + (j & 15), 0xf, 0xf, true));
            if (c16 == (j & 15)) {
                if (hi) { e1 = ev; x1 = xv; } else { e0 = ev; x0 = xv; }
            }
            h0 = fmaf(ej, c0[j], h0);
            h1 = fmaf(ej, c1[j], h1);
        };
        columns(column, std::make_integer_sequence<int, TS>{});
        // errors for the later blocks (every workspace row and column is
        // written, padding included: its errors are 0); outputs
        const int es = (OLD ? (b - a.b_begin) % RT : b - a.b_begin) * TS;
        Es[rr][es + c16] = e0;
        Es[rr][es + 16 + c16] = e1;
        a.E[row * a.ldE + col0] = e0;   // (for the push and for later blocks)
        a.E[row * a.ldE + col1] = e1;
        if (row < a.m) {
            if (col0 < a.n) {
                const int64_t o = row * a.n + col0;
                const float r = __builtin_amdgcn_fmed3f(rintf(x0), qlo, qhi);
                a.codes[o] = (int8_t)(int)r;
                a.V[o] = r * s0;
                if (a.pre) a.pre[o] = s0 > 0.0f ? x0 : nan;
            }
            if (col1 < a.n) {
                const int64_t o = row * a.n + col1;
                const float r = __builtin_amdgcn_fmed3f(rintf(x1), qlo, qhi);
                a.codes[o] = (int8_t)(int)r;
                a.V[o] = r * s1;
                if (a.pre) a.pre[o] = s1 > 0.0f ? x1 : nan;
            }
        }
        __syncthreads();   // the block's errors and the partial sums are reused
    }
}

// The push of a finished range: Wout[p][q] = Win[p][q] + sum_k E[p][k] L^A[q][k]
// over the range's columns k, for every later column q >= qb, on the bf16
// matrix cores with both operands split in three (split.h).  One workgroup per
// MT x MT block of 32 x 32 tiles of W'.  Measured against fp32 MFMA with 128 x 128
// blocks: the whole solve of 4096 x 14336 10.9 -> 9.0 ms, 8192 x 8192 7.0 -> 5.9; the
// 64 x 64 blocks of small pushes take as long as before.
struct PushArgs {
    int64_t m, m16, n;
    int nt;
    int64_t ldE;
    const float* E;
    const float* LA;
    const float* Win;
    int64_t ldIn;
    float* Wout;
    int64_t ldOut;
    int kb, ke;       // the range's column tiles
    int64_t qb;       // first column of the later ranges (a multiple of 32)
};

template <int MT>
__global__ __launch_bounds__(SplitShape<MT>::TH, 2) void k_gptq_push(PushArgs a) {
    using C = SplitShape<MT>;
    __shared__ __attribute__((aligned(16))) uint16_t S[C::LDS];
    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = wv / C::WN, wn = wv % C::WN;
    const int64_t p0 = (int64_t)blockIdx.y * (MT * TS), q0 = a.qb + (int64_t)blockIdx.x * (MT * TS);

    // the thread's rows of its operand (E, or the factor's rows: row r of tile
    // row Q sits at packed_tile_offset(Q, kt) + 32 r); rows past the end are
    // read from the first row (valid memory) and staged as zeros
    const bool opb = wv >= C::TH / 128;
    const int th = tid & (C::TH / 2 - 1), kq = 4 * (th & 3);
    const float* base[C::NU];
    bool in[C::NU];
#pragma unroll
    for (int u = 0; u < C::NU; ++u) {
        const int r = (th >> 2) + u * C::RP;
        if (!opb) {
            in[u] = p0 + r < a.m16;
            base[u] = a.E + (in[u] ? p0 + r : 0) * a.ldE + (int64_t)a.kb * TS + kq;
        } else {
            const int64_t Q = q0 / TS + (r >> 5);
            in[u] = Q < a.nt;
            base[u] = a.LA + packed_tile_offset(in[u] ? Q : q0 / TS, a.kb) + (r & (TS - 1)) * TS + kq;
        }
    }
    const int64_t stride = opb ? TILE_ELEMS : TS;
    const int nch = 2 * (a.ke - a.kb);
    f32x16 acc[C::WX][C::WY];
    split_gemm<MT>(S, nch, tid, [&](int c, int u) {
        const int k = c < nch ? c : nch - 1;   // past the range: not used
        const f32x4 v = *reinterpret_cast<const f32x4*>(base[u] + (k >> 1) * stride + (k & 1) * 16);
        return in[u] ? v : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }, acc);
#pragma unroll
    for (int x = 0; x < C::WX; ++x)
#pragma unroll
        for (int y = 0; y < C::WY; ++y) {
            const int64_t q = q0 + (wn * C::WY + y) * TS + (l & 31);
            if (q >= a.n) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t p = p0 + (wm * C::WX + x) * TS + (r >> 2) * 8 + (l >> 5) * 4 + (r & 3);
                if (p < a.m) a.Wout[p * a.ldOut + q] = a.Win[p * a.ldIn + q] + acc[x][y][r];
            }
        }
}

// errors (ceil(m/16)*16 x nt*32) and the working copy W' (the same shape)
size_t gptq_workspace_floats(int64_t m, int64_t n) {
    return 2 * (size_t)((m + 15) / 16 * 16) * (size_t)((n + TS - 1) / TS * TS);
}

// range_tiles: column tiles per range (0: GR).  Per range one k_gptq launch
// and, unless it is the last, one push: 1024-column ranges measured fastest
// on the paper's Table 3 shapes (128 to 2048 columns tried).
hipError_t run_gptq(hipStream_t st, const float* W, int64_t m, int64_t n, const float* LA, float* E,
                    const QuantArgs& q, int8_t* codes, float* V, float* pre, int range_tiles) {
    const int R = range_tiles > 0 ? range_tiles : GR;
    const int nt = (int)((n + TS - 1) / TS);
    const int64_t ldE = (int64_t)nt * TS, m16 = (m + 15) / 16 * 16;
    float* Wt = E + m16 * ldE;
    // All errors of the range in LDS: two workgroups fit a CU, 512 the chip.  The last
    // half of them: three, 768.  The first is quicker while both take as many rounds of
    // the chip, and where it takes two full rounds against one and a third (us at n =
    // 1024, errors in LDS / in part from memory: 8192 rows 231 / 240, 12288 rows 451 / 331,
    // 16384 rows 458 / 475, 20000 rows 675 / 568, 57344 rows 1657 / 1563).  Same bits.
    const int64_t wg = m16 / 16;
    GptqArgs a;
    a.m = m;
    a.n = n;
    a.nt = nt;
    a.ldE = ldE;
    a.LA = LA;
    a.E = E;
    a.q = q;
    a.codes = codes;
    a.V = V;
    a.pre = pre;
    for (int b0 = 0; b0 < nt; b0 += R) {
        const int b1 = b0 + R < nt ? b0 + R : nt;
        a.b_begin = b0;
        a.b_end = b1;
        a.Wb = b0 == 0 ? W : Wt;
        a.ldWb = b0 == 0 ? n : ldE;
        const dim3 rows((unsigned)wg);
        if (R <= GR && (wg <= 512 || (wg > 768 && wg <= 1024)))
            hipLaunchKernelGGL((k_gptq<GR, false, 2>), rows, dim3(64 * GW), 0, st, a);
        else
            hipLaunchKernelGGL((k_gptq<GR / 2, true, 3>), rows, dim3(64 * GW), 0, st, a);
        if (b1 < nt) {
            PushArgs pa;
            pa.m = m;
            pa.m16 = m16;
            pa.n = n;
            pa.ldE = ldE;
            pa.E = E;
            pa.LA = LA;
            pa.Win = b0 == 0 ? W : Wt;
            pa.ldIn = b0 == 0 ? n : ldE;
            pa.Wout = Wt;
            pa.ldOut = ldE;
            pa.kb = b0;
            pa.ke = b1;
            pa.qb = (int64_t)b1 * TS;
            pa.nt = nt;
            // the widest blocks that give every CU one (256 x 256) or two (128 x
            // 128) workgroups, else 64 x 64
            auto blocks = [&](int64_t e) { return dim3((unsigned)((n - pa.qb + e - 1) / e), (unsigned)((m + e - 1) / e)); };
            const dim3 g8 = blocks(256), g4 = blocks(128), g2 = blocks(64);
            if ((int64_t)g8.x * g8.y >= 256)
                hipLaunchKernelGGL(k_gptq_push<8>, g8, dim3(SplitShape<8>::TH), 0, st, pa);
            else if ((int64_t)g4.x * g4.y >= 256)
                hipLaunchKernelGGL(k_gptq_push<4>, g4, dim3(SplitShape<4>::TH), 0, st, pa);
            else
                hipLaunchKernelGGL(k_gptq_push<2>, g2, dim3(SplitShape<2>::TH), 0, st, pa);
        }
    }
    return hipGetLastError();
}

}  // namespace bk
