// Solver kernels for BaKron (Alg. 6) on gfx950.
//
// Notation.  W~ is the workspace, E = V - W~ the committed errors, L^A / L^B
// the unit-lower normalised factors.  By Eq. (1) the value at which entry
// (p,q) is quantised is
//     W~_pq = W0_pq + sum_{(i,j) < (p,q)} L^B_pi E_ij L^A_qj ,
// the sum running over entries above-left of (p,q).  Split the sum by the
// first column index (App. B, proof of Thm 3.2, and Sec. 3.4's column/row
// splits):
//     W~_pq = W0_pq + sum_{j<q} F_pj L^A_qj + G_pq,
//     G_pq  = sum_{i<p} L^B_pi E_iq,        F_pj = G_pj + E_pj = (L^B E)_pj .
// G carries errors down a column through L^B, F carries them right along a
// row through L^A.  Every elementary update of Alg. 2 is applied exactly once
// this way, with mn(m+n)/2 multiply-adds in total (no band-masking overhead).
//
// Tiling.  TS x TS tiles; tile (I,J) depends only on tiles (I',J') with
// I'<=I, J'<=J, and tiles on one tile anti-diagonal D = I+J are independent.
// Two workspace arrays per tile:
//     X = W0 + (row pushes F L^A^T received so far)  -> after the tile is
//         solved it holds E of the tile;
//     Y = (column pushes L^B E received so far)       -> after the tile is
//         solved it holds F of the tile.
// The divide-and-conquer of Alg. 6 runs over ranges of tile anti-diagonals:
// solve the first half, push all errors of the first half into the second
// half, solve the second half.  The push of a node is two dense products:
//     Y[I,J] += sum_{I'} L^B[I,I'] E[I',J]       (same column, I' in S1)
//     X[I,J] += sum_{J'} F[I,J'] L^A[J,J']^T     (same row,    J' in S1)
// Products between tiles closer than KNEAR + 1 anti-diagonals are pulled by
// the target tile itself just before it is solved (a persistent "segment"
// launch covers a subtree of at most KNEAR + 1 anti-diagonals and orders its
// tiles with per-tile ready flags); node products take only pairs farther
// apart than KNEAR, so each (source, target) tile pair is applied exactly
// once.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "split.h"

#include <vector>

namespace bk {


struct SegArgs {
    int K, L;         // tile anti-diagonals [K, L) of this launch
    int J_lo;         // first tile column (strip) with a tile in [K, L)
    int nstrips;      // strips J_lo .. J_lo + nstrips - 1
    int mt, nt;       // tile grid
    int64_t m, n;     // real sizes
    float* X;         // W0 + node row pushes; E once the tile is solved (column-major tiles)
    float* Y;         // node column pushes; F once the tile is solved (row-major tiles)
    const float* LA;  // packed factor tiles
    const float* LB;
    int b_ident;      // B = I (no column feedback)
    QuantArgs q;
    int8_t* codes;
    float* V;
    float* pre;       // may be null
    int knear;        // pull distances 1..knear (<= KNEAR_MAX)
    int* flags;       // per tile: 1 once rows 0 .. 15 of F are published, 2 once all are
    int* counter;     // strip ticket counter of this launch, 0 at entry
    int* status;      // set to 1 if a wait gave up (never in a correct run); sticky
    int spin_limit;   // polls before a wait gives up
    int late;         // debug (LATE): bit k - 2 set: the poll for F[., J-k] finds it not ready
};

// Bounded wait for a tile's ready flag to reach `level`, executed by a whole
// wave (uniform address).  A strip only ever waits for strips with smaller tickets, and
// tickets are handed out only to running workgroups, so the flag is set by a
// running workgroup; the bound only turns a logic error into a reported
// failure instead of a hang.  Once a wait has given up, the status word stays
// set (until the host reads and clears it) and every later wait returns at
// once, so a failed solve, and every solve after it, ends quickly with its
// output marked invalid.  The data behind the flag is read with
// device-coherent (sc1) loads, so no cache invalidation is needed here.
__device__ inline void wait_ready(const int* flag, int level, int* status, int spin_limit) {
    int it = 0;
    while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < level) {
        __builtin_amdgcn_s_sleep(1);
        if (++it >= spin_limit ||
            __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
    __atomic_signal_fence(__ATOMIC_SEQ_CST);   // keep the data loads after the wait
}

// Raw buffer descriptor over one 32 x 32 fp32 tile (16-byte loads).
__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const float* t) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(t), (short)0, TILE_ELEMS * 4,
                                             0x00020000);
}
constexpr int CPOL_SC1 = 16;   // device-coherent load / store

// Near-field pulls on fp32 MFMA (v_mfma_f32_16x16x4f32).  The pulled sums of
// a tile are two 32 x 32 products per source distance k:
//   row kind    (into X): C[q][p] += sum_j L^A[J, J-k][q][j] F[I, J-k][p][j]
//   column kind (into Y): C[p][q] += sum_i L^B[I, I-k][p][i] E[I-k, J][i][q]
// Every pull wave owns one 16 x 16 block of one of the two, so no partial sums
// have to be combined.  Every
// operand is read as contiguous 16-byte chunks of a row: lane (i, s) of a
// 16 x 16 x 4 step supplies A[i][k] and B[k][i] with k = 8s + 4c + t at step
// (c, t), i.e. chunks 2s and 2s + 1 of row i of both operand tiles.
//
// Factor tiles and the left strips' F tiles are staged in LDS with direct
// global -> LDS loads (no registers in flight), 16-byte chunk c of row r at
// chunk c ^ (r & 7) so that the row-per-lane reads above spread over the banks.
__device__ inline f32x4 lds_chunk(const float* t, int r, int c) {
    return *reinterpret_cast<const f32x4*>(t + r * TS + ((c ^ (r & 7)) << 2));
}
__device__ inline void mfma_8(f32x4 a0, f32x4 a1, f32x4 b0, f32x4 b1, f32x4& acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[t], b0[t], acc, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[t], b1[t], acc, 0, 0, 0);
}
// One wave copies rows 8 rb .. 8 rb + 7 of a row-major tile into a swizzled
// LDS tile: lane l fills physical chunk l & 7 of row 8 rb + (l >> 3).
template <int CPOL>
__device__ inline void stage_rows(const float* src, float* dst, int rb, int l) {
    const int r = 8 * rb + (l >> 3), c = (l & 7) ^ (r & 7);
    __builtin_amdgcn_global_load_lds(src + r * TS + 4 * c,
                                     (__attribute__((address_space(3))) void*)(dst + rb * 256), 16,
                                     0, CPOL);
}

constexpr int RING = KNEAR_MAX;   // E tiles of the strip kept in LDS
constexpr int RSTR = TS + 4;      // LDS row stride: 16-byte rows, conflict-free b128 reads

// Persistent solve of the tiles on anti-diagonals [K, L) by tile-column
// strips.  Each workgroup (one per CU) repeatedly takes a strip ticket and
// solves the strip's tiles in [K, L) top to bottom; strip J waits only for
// strips J-1 .. J-2, which hold smaller tickets.  Inside a strip the column
// dependencies are local: the last RING errors E of the strip stay in LDS, and
// so do L^A[J, J-k] for k = 1..knear.
//
// What bounds it: the chain of dependent element anti-diagonals (63 per tile,
// one tile after the other), so everything that is not on that chain is kept
// off the one wave that walks it.  Roles of the 12 waves:
//   solver (wave 0): the in-tile rounding, in registers.  Lanes 0..31 hold the
//     column sums G of rows 0..31, lanes 32..63 the row sums H; at step t lane
//     p is at entry (p, t - p).  A step adds the errors of the last SG to
//     2 SG - 1 anti-diagonals (below), exchanges G and H between the halves
//     (v_permlane32_swap), rounds, and writes E, F and x to LDS.
//   pull waves (8): one 16 x 16 block of G or H each, on fp32 MFMA
//     (v_mfma_f32_16x16x4f32).  Every SG anti-diagonals (a group) a barrier
//     hands them the errors of the group just finished; during the next group
//     they add its pushes into the whole tile and pass the entries of the
//     group after that to the solver through LDS.  So an entry's sources
//     within its own and the previous group are the solver's, all older ones
//     theirs.  In between they multiply the near-field sources of the next tile.
//   service waves (3): publish F of the finished tile, write codes, V and pre,
//     copy E to X, stage the next tile's operands in LDS.
// A wave alone issues about one operation per 6.5 cycles (measured), so the
// solver's time is its number of operations: per step 2 per source (a lane
// shift of the column half's history and a multiply-add that serves both
// halves) and about 25 others, 265 cycles at SG = 8.  A larger SG costs more
// sources, a smaller one more barriers and less time for the pull waves: SG = 7
// made the segments of the 4096 x 4096 layer 8% longer, SG = 4 37%.
// Measured against the kernel before it, in which all eight waves took turns
// at the rounding and met at a barrier per 4 anti-diagonals: 12.8 -> 10.5 us
// per tile anti-diagonal (4096 x 4096, kernel trace), 13.2 -> 11.4 (28672 x 8192), the
// 64 x 64 layer 34.5 -> 28.6 us in all.  Of a tile's 23000 cycles 2600 go to the sums
// of the block at its origin before the solver can start (flag and F of the
// left tile), 17100 to its steps, the rest to waiting for the pull waves of the
// blocks with the most pushes.
//
// Per tile I:
//  1. pull.  The sources at distance k >= 2 are complete while tile I-1 is
//     being rounded, up to the last of them; their operands are staged and
//     multiplied beside that (stage_index, use_group) once the left strips'
//     flags are up.  What was late is done here.  Then distance 1: F[I, J-1]
//     after its ready flag (device-coherent loads) and E(I-1) from the ring,
//     for the block at the origin before the solver starts, for the others
//     beside its first groups.
//  2. the 63 element anti-diagonals, in NGRP groups with a barrier each.
//  3. F -> Y with device-coherent (sc1) 16-byte stores of whole rows, rows 0 .. 15
//     as soon as they are complete (flag 1), the rest after the last group
//     (flag 2); E -> X (read by the node launches after this one); codes, V and
//     pre.  The service waves do this beside the next tile's start.
// GQ: scales per column group and/or per column (else one scale per row).
// ASYM: alphabet {qlo..qhi} (else the symmetric {-qhi..qhi}).
// LATE: a.late holds (a debug switch; one instance, for every quantiser).
constexpr int SEG_THREADS = 768;
constexpr int SG = 8;                                  // anti-diagonals per group
constexpr int NGRP = (2 * TS - 1 + SG - 1) / SG;       // groups per tile
constexpr int NSRC = 2 * SG - 1;                       // the solver's own source distances
constexpr int NV = (NSRC + 3) / 4;                     // in 16-byte pieces
constexpr int TROW = 4 * (NV | 1);                     // row stride of the coefficient tables:
                                                       // an odd number of 16-byte pieces
// The next tile's operands are staged in the order F[8], L^B[8], F[7], L^B[7],
// .., F[2], L^B[2], L^B[1] (by source distance), one tile per service wave and
// group; a group later they have landed, and in the group after that the pull
// waves may use them (use_group), one source per group.
__device__ constexpr int stage_index(int k, bool lb) { return k == 1 ? 14 : 2 * (KNEAR_MAX - k) + (lb ? 1 : 0); }
__device__ constexpr int use_group(int k, bool lb) { return 2 + stage_index(k, lb) / 3; }
constexpr int POLL_G = 2;                              // group in which the flag of (I + 1, J - 2) is polled
constexpr int PUB_G = (TS + TS / 2 - 1 + SG - 1) / SG; // rows 0 .. 15 are complete once this group begins
static_assert(2 * SG <= TS / 2 && PUB_G + 1 < NGRP && use_group(2, true) < NGRP && POLL_G % 2 == 0 &&
              POLL_G < stage_index(2, false) / 3, "group schedule");
// LDS layout (floats)
constexpr int S_RING = 0;                              // [RING][TS][RSTR]  E^T[q][i] per tile
constexpr int S_LA = S_RING + RING * TS * RSTR;        // [KNEAR_MAX] tiles L^A[J, J-k-1]
constexpr int S_LB = S_LA + KNEAR_MAX * TILE_ELEMS;    // [KNEAR_MAX] tiles L^B[I', I'-k-1]
constexpr int S_Y = S_LB + KNEAR_MAX * TILE_ELEMS;     // [KNEAR_MAX - 1] tiles F[I', J-k-2]
constexpr int S_F = S_Y + (KNEAR_MAX - 1) * TILE_ELEMS;   // [TS][RSTR] F of the tile
constexpr int S_X = S_F + TS * RSTR;                   // [TS][RSTR] x of the tile
constexpr int S_BASE = S_X + TS * RSTR;                // [2][SG][64] sums handed to the solver
constexpr int S_TA = S_BASE + 2 * SG * 64;             // [TS][TROW] L^A[q][q-k]
constexpr int S_TB = S_TA + TS * TROW;                 // [TS][TROW] L^B[p][p-k]
constexpr int S_END = S_TB + TS * TROW;
constexpr int S_SC = S_END;                            // GQ: [TS][TS + 1] scales, then reciprocals
constexpr int S_END_GQ = S_SC + 2 * TS * (TS + 1);
// the solver's lanes outside the tile read up to TS - 1 rows before and 2 TS - 1
// rows after the first row of S_TA; their results are masked
static_assert((TS - 1) * TROW <= S_TA && 2 * TS * TROW <= S_END - S_TA, "coefficient reads stay in LDS");
static_assert(S_END_GQ * 4 + 64 <= 160 * 1024, "LDS");

enum SegRole { SOLVER, PULL, SERVICE };
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;

// Workgroup barrier that orders LDS (also the writes the compiler does not see
// inside the solver's asm); global loads and stores stay in flight.
__device__ inline void seg_sync() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __syncthreads();
}

// The whole kernel for one role (the same statements and barriers for all
// three; what a role does not do is removed at compile time, so that the
// registers of the roles are not live at once).  W: the wave's number within
// its role.
template <bool GQ, bool ASYM, bool LATE, int ROLE>
__device__ __forceinline__ void seg_role(const SegArgs& a, float* sm, int& tk, volatile int* yready, int w, int W) {
    const int tid = threadIdx.x, l = tid & 63;
    const int hf = l >> 5, p = l & 31;
    const float qhi = a.q.qhi, qlo = ASYM ? a.q.qlo : -qhi;
    const int knear = a.knear;
    constexpr bool solver = ROLE == SOLVER, pull = ROLE == PULL;
    const int sv = ROLE == SERVICE ? W : -1;
    const int mb = W;                // pull block 0..7
    const bool roww = mb < 4;        // row-kind (C[q][p]) or column-kind (C[p][q]) block
    const int i16 = l & 15, ks = l >> 4;
    const int ra0 = 16 * ((mb & 3) >> 1), rb0 = 16 * (mb & 1), rb = rb0 + i16, ra = ra0 + i16;
    // the block at the tile's origin has all entries of the groups 0 and 1: its
    // two waves finish their sums before the solver starts; the others do it in
    // group 0, and the row-kind waves of the lower half, whose sources the left
    // strip publishes last, in group 1
    const bool lead = ra0 + rb0 == 0;
    const int base_g = lead ? -1 : roww && rb0 ? 1 : 0;
    // output items of the service waves 1 and 2: rows r0, r0 + 16, columns cb .. cb + 3
    const int ot = 64 * (sv - 1) + l, r0 = (ot >> 3) & 15, cb = 4 * (ot & 7);

    if (solver) __builtin_amdgcn_s_setprio(3);

    for (;;) {
        if (tid == 0) tk = atomicAdd(a.counter, 1);
        seg_sync();
        const int sidx = tk;
        if (sidx >= a.nstrips) break;   // uniform
        const int J = a.J_lo + sidx;
        const int I_first = a.K - J > 0 ? a.K - J : 0;
        const int I_last = a.L - 1 - J < a.mt - 1 ? a.L - 1 - J : a.mt - 1;
        const int kr = knear < J ? knear : J;   // row sources k = 1..kr of every tile of the strip
        const bool need_y = kr >= 2;

        // the column part of the scales of the thread's output columns
        ColScale cs[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            cs[v] = GQ && sv >= 1 ? col_scale_of(a.q, (int64_t)J * TS + cb + v, a.n) : ColScale{0, 1.0f};

        // inputs of a tile, loaded while the tile before it is solved:
        // pull waves their block of X or Y and, column kind, their rows of the
        // diagonal tile of L^B; the solver its rows' scales; service waves
        // the solver's L^B coefficients and the scales of their output entries
        float pfx[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        f32x4 pfl0 = {0.0f, 0.0f, 0.0f, 0.0f}, pfl1 = pfl0;
        float pfs = 0.0f, pft[8], pfo[2][GQ ? 4 : 1];
        auto prefetch = [&](int In) {
            const int64_t tb = ws_tile_offset(In, J, a.nt);
            const float* lbp = a.LB + packed_tile_offset(In, In);
            if (pull) {
                const float* src = (roww ? a.X : a.Y) + tb + (ra0 + 4 * ks) * TS + rb;
#pragma unroll
                for (int r = 0; r < 4; ++r) pfx[r] = src[r * TS];
                if (!roww && !a.b_ident) {
                    pfl0 = *reinterpret_cast<const f32x4*>(lbp + ra * TS + 8 * ks);
                    pfl1 = *reinterpret_cast<const f32x4*>(lbp + ra * TS + 8 * ks + 4);
                }
            } else if (solver) {
                if (!GQ) pfs = row_scale_of<GQ>(a.q, (int64_t)In * TS + p, ColScale{0, 1.0f}, a.m);
            } else {
                if (sv == 1) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int k = 8 * hf + j + 1;
                        pft[j] = (k <= p && !a.b_ident) ? lbp[p * TS + p - k] : 0.0f;
                    }
                }
                if (sv >= 1) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int v = 0; v < (GQ ? 4 : 1); ++v)
                            pfo[j][v] = row_scale_of<GQ>(a.q, (int64_t)In * TS + r0 + 16 * j, cs[v], a.m);
                }
            }
        };
        // issue the direct loads of one operand tile by the waves wi, wi + nw, ...
        auto stage_lb = [&](int It, int k, int wi, int nw) {   // L^B[It, It-k]
            for (int g = wi; g < 4; g += nw)   // uniform control flow
                stage_rows<0>(a.LB + packed_tile_offset(It, It - k), sm + S_LB + (k - 1) * TILE_ELEMS, g, l);
        };
        auto stage_y = [&](int It, int k, int wi, int nw) {    // F[It, J-k], k >= 2
            for (int g = wi; g < 4; g += nw)
                stage_rows<CPOL_SC1>(a.Y + ws_tile_offset(It, J - k, a.nt), sm + S_Y + (k - 2) * TILE_ELEMS, g, l);
        };

        // strip set-up: L^A[J, J-k], the coefficients of L^A[J, J], the ring with
        // the errors of the tiles above that were solved by earlier launches,
        // the first tile's inputs and its staged pull operands.  Every load is
        // issued before any is waited for: one memory round trip per strip.
        const int npre = a.b_ident ? 0 : (knear < I_first ? knear : I_first);
        const float* lad = a.LA + packed_tile_offset(J, J);
        {
            float2 rg[KNEAR_MAX];
#pragma unroll
            for (int k = 0; k < KNEAR_MAX; ++k)
                if (k < npre && tid < 512)
                    rg[k] = *reinterpret_cast<const float2*>(a.X + ws_tile_offset(I_first - 1 - k, J, a.nt) +
                                                              2 * tid);   // E^T, column-major E
            const int tq = tid / NSRC, tkk = tid - tq * NSRC + 1;
            float lac = 0.0f;
            static_assert(TS * NSRC <= SEG_THREADS, "one coefficient per thread");
            if (tq < TS && tkk <= tq) lac = lad[tq * TS + tq - tkk];
            for (int g = w; g < 4 * kr; g += SEG_THREADS / 64)
                stage_rows<0>(a.LA + packed_tile_offset(J, J - 1 - (g >> 2)), sm + S_LA + (g >> 2) * TILE_ELEMS, g & 3, l);
            prefetch(I_first);
            for (int g = w; g < 4 * npre; g += SEG_THREADS / 64) stage_lb(I_first, 1 + (g >> 2), g & 3, 4);
            if (need_y) {
                wait_ready(a.flags + I_first * a.nt + (J - 2), 2, a.status, a.spin_limit);
                for (int g = w; g < 4 * (kr - 1); g += SEG_THREADS / 64) stage_y(I_first, 2 + (g >> 2), g & 3, 4);
            }
            if (tq < TS) sm[S_TA + tq * TROW + tkk - 1] = lac;
#pragma unroll
            for (int k = 0; k < KNEAR_MAX; ++k)
                if (k < npre && tid < 512)
                    *reinterpret_cast<float2*>(&sm[S_RING + ((I_first - 1 - k) % RING) * (TS * RSTR) +
                                                   ((2 * tid) >> 5) * RSTR + ((2 * tid) & 31)]) = rg[k];
        }
        f32x4 lf0 = {0.0f, 0.0f, 0.0f, 0.0f}, lf1 = lf0;   // rows ra of the diagonal tile (L^A, or the tile's L^B)
        if (pull && roww) {
            lf0 = *reinterpret_cast<const f32x4*>(lad + ra * TS + 8 * ks);
            lf1 = *reinterpret_cast<const f32x4*>(lad + ra * TS + 8 * ks + 4);
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's direct loads landed
        seg_sync();

        // F[., J-k] of the tile staged for k = 2 and for k >= 3 (uniform; the
        // first tile's were staged above)
        bool y2 = true, y3 = true;
        // per wave: the next source distance to multiply, from the farthest down to 2
        int nk = roww ? kr : npre;
        f32x4 pacc = {0.0f, 0.0f, 0.0f, 0.0f};

        for (int I = I_first; I <= I_last; ++I) {
            const int kc = a.b_ident ? 0 : (knear < I ? knear : I);   // column sources k = 1..kc
            const bool has_next = I < I_last;
            const int kc_next = a.b_ident ? 0 : (knear < I + 1 ? knear : I + 1);
            const int slot = S_RING + (I % RING) * (TS * RSTR);

            // reads the operands of source distance k of tile It (row or column
            // kind), to be multiplied into pacc
            f32x4 a0, a1, b0, b1;
            auto pull_read = [&](int It, int k) {
                if (roww) {
                    const float* la = sm + S_LA + (k - 1) * TILE_ELEMS;
                    const float* y = sm + S_Y + (k - 2) * TILE_ELEMS;
                    a0 = lds_chunk(la, ra, 2 * ks);
                    a1 = lds_chunk(la, ra, 2 * ks + 1);
                    b0 = lds_chunk(y, rb, 2 * ks);
                    b1 = lds_chunk(y, rb, 2 * ks + 1);
                } else {
                    const float* lb = sm + S_LB + (k - 1) * TILE_ELEMS;
                    const float* e = sm + S_RING + ((It - k) % RING) * (TS * RSTR) + rb * RSTR + 8 * ks;
                    a0 = lds_chunk(lb, ra, 2 * ks);
                    a1 = lds_chunk(lb, ra, 2 * ks + 1);
                    b0 = *reinterpret_cast<const f32x4*>(e);
                    b1 = *reinterpret_cast<const f32x4*>(e + 4);
                }
            };
            // hands the entries of group g of this wave's block to the solver
            const int pd = ra0 + 4 * ks + rb;   // anti-diagonal of the lane's first entry
            float* const pb = sm + S_BASE + pd * 64 + (roww ? TS + rb : ra0 + 4 * ks);
            const int pstep = roww ? 64 : 65;   // the next entry is on the next anti-diagonal (column kind: and row)
            auto put = [&](int g, f32x4 v) {
                float* const b = pb - ((g >> 1) * 2 * SG) * 64;   // group g at parity g & 1
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if ((unsigned)(pd + r - g * SG) < (unsigned)SG) b[r * pstep] = v[r];
            };
            // service wave 0: stores rows 16 h .. + 15 of F (device-coherent, whole
            // rows); sets the tile's flag once its stores are complete; copies E to X
            auto publish = [&](int It, int h) {
                const __amdgpu_buffer_rsrc_t yr = tile_rsrc(a.Y + ws_tile_offset(It, J, a.nt));
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int r = 16 * h + 8 * j + (l >> 3), c = 4 * (l & 7);
                    const f32x4 v = *reinterpret_cast<const f32x4*>(&sm[S_F + r * RSTR + c]);
                    __builtin_amdgcn_raw_buffer_store_b128(v, yr, (r * TS + c) * 4, 0, CPOL_SC1);
                }
            };
            auto publish_flag = [&](int It, int level) {
                __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the stores are complete
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if (l == 0)
                    __hip_atomic_store(a.flags + It * a.nt + J, level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            };
            auto e_to_x = [&](int It) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 8 * j + (l >> 3), c = 4 * (l & 7);
                    *reinterpret_cast<f32x4*>(a.X + ws_tile_offset(It, J, a.nt) + r * TS + c) =
                        *reinterpret_cast<const f32x4*>(&sm[S_RING + (It % RING) * (TS * RSTR) + r * RSTR + c]);
                }
            };

            // 1. pull.  Row operands that were not ready during the previous
            // tile (a left strip that was late) are staged now.
            if (need_y && !(y2 && (y3 || kr < 3))) {   // uniform
                wait_ready(a.flags + I * a.nt + (J - 2), 2, a.status, a.spin_limit);
                for (int k = 2; k <= (y3 ? 2 : kr); ++k)
                    if (k > 2 || !y2) stage_y(I, k, w < 4 ? w : 4, 4);
                __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's direct loads landed
                seg_sync();
            }
            f32x4 base = {0.0f, 0.0f, 0.0f, 0.0f}, far = base;
            float s = 0.0f, inv_s = 0.0f;
            float so[2][GQ ? 4 : 1];
            // the wave's block of the tile's sums: distance 1, then the inputs
            auto finish_base = [&]() {
                if (roww) {
                    if (kr >= 1) {   // F[I, J-1] straight from memory after its flag (1: rows 0 .. 15 published)
                        wait_ready(a.flags + I * a.nt + (J - 1), rb0 ? 2 : 1, a.status, a.spin_limit);
                        const __amdgpu_buffer_rsrc_t r1 = tile_rsrc(a.Y + ws_tile_offset(I, J - 1, a.nt));
                        const f32x4 b0 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r1, (rb * TS + 8 * ks) * 4, 0, CPOL_SC1));
                        const f32x4 b1 = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r1, (rb * TS + 8 * ks + 4) * 4, 0, CPOL_SC1));
                        mfma_8(lds_chunk(sm + S_LA, ra, 2 * ks), lds_chunk(sm + S_LA, ra, 2 * ks + 1), b0, b1, pacc);
                    }
                } else {
                    if (kc >= 1) {   // E[I-1, J] from the ring
                        const float* e = sm + S_RING + ((I - 1) % RING) * (TS * RSTR) + rb * RSTR + 8 * ks;
                        mfma_8(lds_chunk(sm + S_LB, ra, 2 * ks), lds_chunk(sm + S_LB, ra, 2 * ks + 1),
                               *reinterpret_cast<const f32x4*>(e), *reinterpret_cast<const f32x4*>(e + 4), pacc);
                    }
                    lf0 = pfl0;
                    lf1 = pfl1;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) base[r] = pfx[r] + pacc[r];
                pacc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                nk = !has_next ? 0 : roww ? kr : kc_next;
            };
            if (pull) {
                for (; nk >= 2; --nk) {
                    pull_read(I, nk);
                    mfma_8(a0, a1, b0, b1, pacc);
                }
                if (lead) {
                    finish_base();
                    put(0, base);
                    put(1, base);
                }
            } else if (solver) {
                s = pfs;
                inv_s = s > 0.0f ? 1.0f / s : 0.0f;   // zero scale: alphabet {0}
            } else {
                if (sv == 1) {
                    float* t = sm + S_TB + p * TROW + 8 * hf;
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (8 * hf + j < NSRC) t[j] = pft[j];
                }
                if (sv >= 1) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int v = 0; v < (GQ ? 4 : 1); ++v) {
                            so[j][v] = pfo[j][v];
                            if (GQ) {
                                const int e = S_SC + (r0 + 16 * j) * (TS + 1) + cb + v;
                                sm[e] = so[j][v];
                                sm[e + TS * (TS + 1)] = so[j][v] > 0.0f ? 1.0f / so[j][v] : 0.0f;
                            }
                        }
                }
            }
            // can the next tile's row operands be staged?
            auto poll = [&](int k) {
                if (sv == 2 && l == 0)
                    yready[k - 2] = kr < k || __hip_atomic_load(a.flags + (I + 1) * a.nt + (J - k), __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT) >= 2 + (LATE ? a.late >> (k - 2) & 1 : 0);
            };
            if (has_next) poll(3);
            seg_sync();
            y3 = has_next && yready[1] != 0;

            // 2. the element anti-diagonals
            float V[2 * SG];   // solver: E (column half) and F (row half) of the last 2 SG steps
#pragma unroll
            for (int k = 0; k < 2 * SG; ++k) V[k] = 0.0f;
            // lane constants of the solver (byte addresses in LDS): the coefficient
            // row (column half: fixed), E or F and x of the lane's entry
            const uint32_t smb = (uint32_t)(uintptr_t)(lds_char*)sm;
            const lds_char* cp = (const lds_char*)sm + 4 * (hf ? S_TA - p * TROW : S_TB + p * TROW);
            const int cp_inc = hf ? 4 * TROW : 0;
            uint32_t ea = smb + 4 * (hf ? S_F + p * (RSTR - 1) : slot - p * (RSTR - 1));
            const uint32_t ea_inc = 4 * (hf ? 1 : RSTR);
            uint32_t xa = smb + 4 * (S_X + p * (RSTR - 1));
            // SG steps; H: which half of the history ring they fill
            auto group = [&](auto H, int g) {
                constexpr int N2 = 2 * SG, NC = 3;
                float b[SG], es[GQ ? SG : 1], ei[GQ ? SG : 1];
                f32x4 c[NC][NV];   // coefficients, two steps ahead
                auto coef = [&](int r) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) c[r % NC][v] = *(const lds_f32x4*)(cp + 16 * v);
                    cp += cp_inc;
                };
                coef(0);
                coef(1);
#pragma unroll
                for (int r = 0; r < SG; ++r) {
                    b[r] = sm[S_BASE + ((g & 1) * SG + r) * 64 + l];
                    if (GQ) {
                        es[r] = sm[S_SC + p * TS + g * SG + r];   // entry (p, t - p); other rows' outside the tile
                        ei[r] = sm[S_SC + TS * (TS + 1) + p * TS + g * SG + r];
                    }
                }
#pragma unroll
                for (int r = 0; r < SG; ++r) {
                    const int u = H.value * SG + r;   // ring slot of this step
                    if (r + 2 < SG) coef(r + 2);
                    // the column half's history moves one row down: lane p gets the
                    // errors of lane p - 1
#pragma unroll
                    for (int k = 1; k <= SG + r; ++k) {
                        float& h = V[(u - k + N2) % N2];
                        h = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(h), __float_as_int(h),
                                                                       0x138, 0x3, 0xf, true));
                    }
                    float x = b[r];
#pragma unroll
                    for (int k = NSRC; k >= 1; --k)
                        if (k <= SG + r) x = fmaf(V[(u - k + N2) % N2], c[r % NC][(k - 1) >> 2][(k - 1) & 3], x);
                    // G and H in both halves
                    const auto gh = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
                    const float gs = __uint_as_float(gh[0]), hs = __uint_as_float(gh[1]);
                    const float sr = GQ ? es[r] : s, ir = GQ ? ei[r] : inv_s;
                    const float acc = gs + hs;
                    const float xq = acc * ir;
                    const float rq = __builtin_amdgcn_fmed3f(rintf(xq), qlo, qhi);
                    const float e = fmaf(rq, sr, -acc);
                    const float f = gs + e;
                    // lanes with an entry on this anti-diagonal: max(0, t - 31) <= p <= min(t, 31)
                    const uint64_t in = (0x1fffffffeull << (g * SG + r)) >> 32;
                    float v = __builtin_amdgcn_inverse_ballot_w64(in) ? e : 0.0f;
                    v = __builtin_amdgcn_inverse_ballot_w64(in << 32) ? f : v;
                    V[u] = v;
                    // E or F, and x (the same in both halves), of the lanes in the tile
                    asm volatile("s_mov_b64 exec, %[m]\n\tds_write_b32 %[a], %[v]\n\t"
                                 "ds_write_b32 %[b], %[x] offset:%[o]\n\ts_mov_b64 exec, -1"
                                 :: [m] "s"(in | in << 32), [a] "v"(ea), [v] "v"(v), [b] "v"(xa), [x] "v"(xq),
                                    [o] "i"(4 * r)
                                 : "memory");
                    ea += ea_inc;
                }
                xa += 4 * SG;
            };
            // the pull waves' part of group g: the pushes of group g - 1, complete
            // since the last barrier, into the whole tile (older entries in the
            // block are stale by then and not used), then the sums of group g + 1
            auto push = [&](int g) {
                // the block has entries on the anti-diagonals ra0 + rb0 .. + 30 only,
                // its rows of the source tile on rb0 .. rb0 + 46 (all uniform)
                if (g < 1 || g + 1 >= NGRP || ra0 + rb0 + TS - 2 < (g + 1) * SG) return;
                if ((!roww && a.b_ident) || rb0 >= g * SG) {
                    if (ra0 + rb0 < (g + 2) * SG) put(g + 1, base + far);
                    return;
                }
                const float* src = sm + (roww ? S_F : slot) + rb * RSTR + 8 * ks;
                f32x4 b0 = *reinterpret_cast<const f32x4*>(src), b1 = *reinterpret_cast<const f32x4*>(src + 4);
                const int d0 = rb + 8 * ks - (g - 1) * SG;   // anti-diagonal of b0[0] within the group
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    b0[t] = (unsigned)(d0 + t) < (unsigned)SG ? b0[t] : 0.0f;
                    b1[t] = (unsigned)(d0 + 4 + t) < (unsigned)SG ? b1[t] : 0.0f;
                }
                mfma_8(lf0, lf1, b0, b1, far);
                if (ra0 + rb0 < (g + 2) * SG) put(g + 1, base + far);
            };
            auto others = [&](int g) {   // pull and service waves, beside group g of the solver
                if (pull) {
                    if (g == base_g) finish_base();
                    // one source of the next tile per group, two in the last; its
                    // operands are read before the pushes
                    auto ready = [&]() {   // uniform
                        return nk >= 2 && use_group(nk, !roww) <= g && (!roww || (y3 && (nk > 2 || y2)));
                    };
                    const bool one = ready();
                    if (one) pull_read(I + 1, nk);
                    push(g);
                    if (g == 1 && has_next) prefetch(I + 1);
                    if (one) {
                        mfma_8(a0, a1, b0, b1, pacc);
                        --nk;
                        if (g + 1 == NGRP && ready()) {
                            pull_read(I + 1, nk);
                            mfma_8(a0, a1, b0, b1, pacc);
                            --nk;
                        }
                    }
                } else {
                    if (g == 0 && sv == 0 && I > I_first) {   // the rest of the tile above
                        publish_flag(I - 1, 2);
                        e_to_x(I - 1);
                    }
                    if (has_next) {
                        if (g == POLL_G) poll(2);
                        __atomic_signal_fence(__ATOMIC_SEQ_CST);   // the F loads stay after the flag test
                        if (g < use_group(2, true)) {
                            if (g >= 1) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): the last group's direct loads landed
                            const int n = 3 * g + sv;             // stage_index of this wave's tile
                            const int k = n == 14 ? 1 : KNEAR_MAX - (n >> 1);
                            if (n <= 14) {
                                if (n == 14 || (n & 1)) {
                                    if (k <= kc_next) stage_lb(I + 1, k, 0, 1);
                                } else if (k <= kr && y3 && (k > 2 || y2)) {
                                    stage_y(I + 1, k, 0, 1);
                                }
                            }
                            if (g == 1) prefetch(I + 1);
                        }
                    }
                    if (g == PUB_G && sv == 0) {
                        publish(I, 0);
                        publish_flag(I, 1);
                    }
                }
            };
            if (solver && has_next) prefetch(I + 1);
            for (int g = 0; g < NGRP; g += 2) {
                if (solver) group(std::integral_constant<int, 0>{}, g);
                else others(g);
                seg_sync();
                if (g == POLL_G) y2 = y3 && yready[0] != 0;
                if (g + 1 < NGRP) {   // uniform
                    if (solver) group(std::integral_constant<int, 1>{}, g + 1);
                    else others(g + 1);
                    seg_sync();
                }
            }

            // 3. the rest of F, whose flag and the copy of E wait for the next
            // tile's group 0; outputs
            if (sv == 0) {
                publish(I, 1);
                if (!has_next) {
                    publish_flag(I, 2);
                    e_to_x(I);
                }
            } else if (sv >= 1) {
                const float nan = __builtin_nanf("");
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int r = r0 + 16 * j;
                    const int64_t orow = (int64_t)I * TS + r, ocol = (int64_t)J * TS + cb;
                    const f32x4 xq = *reinterpret_cast<const f32x4*>(&sm[S_X + r * RSTR + cb]);
                    float cv[4], vv[4], pv[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float sk = so[j][GQ ? k : 0];
                        cv[k] = __builtin_amdgcn_fmed3f(rintf(xq[k]), qlo, qhi);
                        vv[k] = cv[k] * sk;
                        pv[k] = sk > 0.0f ? xq[k] : nan;
                    }
                    if (orow < a.m) {
                        const int64_t o = orow * a.n + ocol;
                        if ((a.n & 3) == 0 && ocol + 3 < a.n) {   // aligned, inside the matrix
                            uint32_t packed = 0;
#pragma unroll
                            for (int k = 0; k < 4; ++k) packed |= (uint32_t)(uint8_t)(int8_t)(int)cv[k] << (8 * k);
                            *reinterpret_cast<uint32_t*>(a.codes + o) = packed;
                            *reinterpret_cast<f32x4*>(a.V + o) = f32x4{vv[0], vv[1], vv[2], vv[3]};
                            if (a.pre) *reinterpret_cast<f32x4*>(a.pre + o) = f32x4{pv[0], pv[1], pv[2], pv[3]};
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                if (ocol + k < a.n) {
                                    a.codes[o + k] = (int8_t)(int)cv[k];
                                    a.V[o + k] = vv[k];
                                    if (a.pre) a.pre[o + k] = pv[k];
                                }
                            }
                        }
                    }
                }
            }
        }
    }
}

// Wave i runs on SIMD i mod 4: the solver shares its SIMD with two service waves
// only (beside pull waves its steps took a third longer).
template <bool GQ, bool ASYM, bool LATE>
__global__ __launch_bounds__(SEG_THREADS) void k_seg(SegArgs a) {
    __shared__ __attribute__((aligned(16))) float sm[GQ ? S_END_GQ : S_END];
    __shared__ int tk, yready[2];
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (w == 0) seg_role<GQ, ASYM, LATE, SOLVER>(a, sm, tk, yready, w, 0);
    else if (w == 4 || w == 8 || w == 11) seg_role<GQ, ASYM, LATE, SERVICE>(a, sm, tk, yready, w, w >> 2 == 1 ? 0 : w == 8 ? 1 : 2);
    else seg_role<GQ, ASYM, LATE, PULL>(a, sm, tk, yready, w, w - 1 - (w > 4) - (w > 8));
}

// Fills n 32-bit words with v (a debug aid: poisoning the workspace before a
// solve shows that every word the solve reads was written by it first).
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = v;
}

// *bad <- 1 if any of the `count` scales at s is negative, NaN or infinite
// (the quantiser needs finite scales >= 0).  *bad is cleared by the caller.
__global__ __launch_bounds__(256) void k_check_scales(const float* __restrict__ s, int64_t count,
                                                       int* __restrict__ bad) {
    bool ok = true;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        const float v = s[i];
        ok = ok && v >= 0.0f && v <= 3.402823466e38f;
    }
    if (!ok) __hip_atomic_store(bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t check_scales(hipStream_t st, const float* s, int64_t count, int* bad) {
    if (count <= 0) return hipSuccess;
    const int64_t g = std::min<int64_t>((count + 255) / 256, 1024);
    hipLaunchKernelGGL(k_check_scales, dim3((unsigned)g), dim3(256), 0, st, s, count, bad);
    return hipGetLastError();
}

hipError_t fill_words(hipStream_t st, void* p, int64_t n, uint32_t v) {
    if (n <= 0) return hipSuccess;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)g), dim3(256), 0, st, static_cast<uint32_t*>(p), n, v);
    return hipGetLastError();
}

struct NodeArgs {
    int K, Mid;       // sources on tile anti-diagonals [K, Mid)
    int tlo, thi;     // targets on tile anti-diagonals [tlo, thi)
    int knear;
    int mt, nt;
    float* X;
    float* Y;
    const float* LA;
    const float* LB;
    const int4* items;  // work list of this launch (see NodeItem in common.h)
};

// Band push of one divide-and-conquer node, on the bf16 matrix cores with every
// fp32 operand split in three (split.h).
//
// Both pushes are computed as C[M][N] += sum_k A[M][k] * B[N][k] over source
// tiles kt (TS k's each, two chunks), with every operand tile stored [row][k]:
//   column push: C = Y[I, J] (row-major), A = L^B[I, kt], B = E[kt, J] read
//                from X, whose tiles are column-major (= E^T);
//   row push:    C = X[I, J] stored column-major, i.e. C^T[J][I]
//                = sum L^A[J, kt] * F[I, kt]^T, A = L^A[J, kt], B = F[I, kt]
//                read from Y (row-major).
// So every operand read is a 16-byte piece of a tile row and every output
// write is coalesced.  The (source, target) validity masks are separable, so
// invalid source tiles are staged as zeros and the sums stay exact.
//
// One workgroup per work-list item (MT x MT solver tiles): the host lists only
// items with a non-empty source range, longest first, so the long K loops
// start early.  What limits the large pushes (counters, <8> on the 28672 x 8192
// layer): no single unit.  The matrix cores are busy 54% of the cycles, the LDS 24%,
// HBM delivers 2.0 TB/s; the chip holds 1.9 GHz under this load (of 2.4), which is
// what a power limit looks like, and the one workgroup of a CU meets at a barrier per
// chunk.  Measured against fp32 MFMA: all pushes of that layer
// 65.0 -> 53.0 ms (129 -> 159 TFLOP/s of fp32 products), of 11008 x 4096 5.6 -> 5.0.
template <int MT>
__global__ __launch_bounds__(SplitShape<MT>::TH, 2) void k_node(NodeArgs a) {
    using C = SplitShape<MT>;
    __shared__ __attribute__((aligned(16))) uint16_t S[C::LDS];
    const int4 it = a.items[blockIdx.x];
    const int I0 = it.x, J0 = it.y;
    const bool colpush = (it.z & 1) == 0;
    const int klo = it.z >> 1, khi = it.w;

    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int wm = wv / C::WN, wn = wv % C::WN;

    // Operand tile of K tile kt as a buffer resource: a valid tile covers its
    // 4 KB, an invalid one (outside the matrix, outside the (source, target)
    // masks or past the item's range) has no records, so its loads return
    // zeros without touching memory.  Every chunk therefore issues the same
    // loads unconditionally, which lets the compiler wait only for the chunk
    // it stores.  A wave stages rows of one operand and, per pass, of one
    // tile, so base, stride and range are wave-uniform; consecutive K tiles
    // sit a fixed stride apart.
    //   column push: A = L^B[I0 + t, kt] (kt <= I - knear - 1), B = E[kt, J0 + t]
    //                (kt + J in [K, Mid)), read from X;
    //   row push:    A = L^A[J0 + t, kt] (kt <= J - knear - 1), B = F[I0 + t, kt]
    //                (I + kt in [K, Mid)), read from Y.
    const bool opb = wv >= C::TH / 128;
    const int th = tid & (C::TH / 2 - 1);
    const float* base[C::NU];
    int lo[C::NU], hi[C::NU];
    const int64_t stride = opb && colpush ? (int64_t)a.nt * TILE_ELEMS : TILE_ELEMS;
#pragma unroll
    for (int u = 0; u < C::NU; ++u) {
        const int t = u * (C::RP / TS) + __builtin_amdgcn_readfirstlane(th >> 7);
        if (!opb) {
            const int Ia = colpush ? I0 + t : J0 + t;   // factor tile row
            const bool in = colpush ? Ia < a.mt : Ia < a.nt;
            base[u] = in ? (colpush ? a.LB : a.LA) + packed_tile_offset(Ia, 0) : a.LA;
            lo[u] = 0;
            hi[u] = in ? min(khi, Ia - a.knear) : 0;
        } else {
            const int Ib = colpush ? J0 + t : I0 + t;   // fixed coordinate of the source tile
            const bool in = colpush ? Ib < a.nt : Ib < a.mt;
            base[u] = in ? (colpush ? a.X + ws_tile_offset(0, Ib, a.nt) : a.Y + ws_tile_offset(Ib, 0, a.nt))
                         : a.LA;
            lo[u] = max(a.K - Ib, 0);
            hi[u] = in ? min(khi, a.Mid - Ib) : 0;
        }
    }
    const int voff = (((th >> 2) & (TS - 1)) * TS + 4 * (th & 3)) * 4;
    f32x16 acc[C::WX][C::WY];
    split_gemm<MT>(S, 2 * (khi - klo), tid, [&](int c, int u) {
        // (an invalid tile's address may lie outside every allocation: with no
        // records nothing is read)
        const int kt = klo + (c >> 1);
        const int nrec = (kt >= lo[u] && kt < hi[u]) ? TILE_ELEMS * 4 : 0;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(base[u] + kt * stride), (short)0, nrec, 0x00020000);
        return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, (c & 1) * 64, 0));
    }, acc);

    // epilogue: block (x, y) of wave (wm, wn) is output solver tile
    // (M tile wm*WX+x, N tile wn*WY+y); C[M][N] row-major inside the tile.
    const int lr = l & 31, lk = l >> 5;
#pragma unroll
    for (int x = 0; x < C::WX; ++x)
#pragma unroll
        for (int y = 0; y < C::WY; ++y) {
            const int tm = wm * C::WX + x, tn = wn * C::WY + y;
            const int I = colpush ? I0 + tm : I0 + tn;
            const int J = colpush ? J0 + tn : J0 + tm;
            if (I >= a.mt || J >= a.nt || I + J < a.tlo || I + J >= a.thi) continue;
            float* out = (colpush ? a.Y : a.X) + ws_tile_offset(I, J, a.nt);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = (r >> 2) * 8 + lk * 4 + (r & 3);
                out[rr * TS + lr] += acc[x][y][r];
            }
        }
}

// The same push on fp32 MFMA, 64 x 64 per workgroup: for the nodes of at most
// NODE32_SPAN tile anti-diagonals.  Their source ranges are so short that the
// launch is bound by latency and operand bytes, and the split's conversions and
// the third more LDS bytes of its planes only add to it.  us per launch here / with
// k_node<2>: nodes of 15, 16, 31, 32 anti-diagonals of the 1024 x 1024 layer 6.9 /
// 7.8, 8.1 / 9.5, 12.9 / 14.5, 13.8 / 15.8, of the 4096 x 4096 layer 7.5 / 7.9, 10.2 /
// 11.1, 14.1 / 14.7, 26.1 / 27.5; from 58 to 64 anti-diagonals the two are within 6%
// (4096 x 4096: 29.1 / 30.5 and 77.7 / 77.4), and the split is the more exact one.
// 4 waves in a 2 x 2 arrangement; inside a K chunk
// the 32 k's are split between the two lane halves (half h takes k = 16h + s at
// step s), so each lane reads 16 consecutive floats per operand with four
// 16-byte LDS loads.  LDS is double buffered and the chunks two ahead are
// prefetched into registers while the current one is multiplied.
constexpr int LDS_STRIDE = TS + 4;   // 36 floats: 16-byte rows, no b128 bank conflicts
__global__ __launch_bounds__(256, 4) void k_node32(NodeArgs a) {
    constexpr int MT = 2, WB = MT / 2;   // 64 x 64 per workgroup, one 32x32 block per wave
    __shared__ __attribute__((aligned(16))) float As[2][MT * TS][LDS_STRIDE];
    __shared__ __attribute__((aligned(16))) float Bs[2][MT * TS][LDS_STRIDE];
    const int4 it = a.items[blockIdx.x];
    const int I0 = it.x, J0 = it.y;
    const bool colpush = (it.z & 1) == 0;
    const int klo = it.z >> 1, khi = it.w;

    const int tid = threadIdx.x;
    const int wv = tid >> 6, l = tid & 63;
    const int wm = wv >> 1, wn = wv & 1;
    const int lr = l & 31, lk = l >> 5;
    const int srow = tid >> 3, sk = (tid & 7) * 4;   // staging: one float4 of each tile

    // Operand tile t of K chunk kt as a buffer resource: a valid tile covers
    // its 4 KB, an invalid one (outside the matrix, outside the (source,
    // target) masks or past the item's range) has no records, so its loads
    // return zeros without touching memory.  Every chunk therefore issues the
    // same loads unconditionally, which lets the compiler wait only for the
    // chunk it stores (the two-ahead prefetch stays in flight).  Per operand
    // tile the valid chunks form one range [lo, hi) and consecutive chunks sit
    // a fixed stride apart, so the per-item set-up below leaves two compares
    // and an address per tile per chunk.
    //   column push: A = L^B[I0 + t, kt] (kt <= I - knear - 1), B = E[kt, J0 + t]
    //                (kt + J in [K, Mid)), read from X;
    //   row push:    A = L^A[J0 + t, kt] (kt <= J - knear - 1), B = F[I0 + t, kt]
    //                (I + kt in [K, Mid)), read from Y.
    const float* abase[MT];
    const float* bbase[MT];
    int alo[MT], ahi[MT], blo[MT], bhi[MT];
    const int64_t bstride = colpush ? (int64_t)a.nt * TILE_ELEMS : TILE_ELEMS;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int Ia = colpush ? I0 + t : J0 + t;   // factor tile row
        const bool arow = colpush ? Ia < a.mt : Ia < a.nt;
        abase[t] = arow ? (colpush ? a.LB : a.LA) + packed_tile_offset(Ia, 0) : a.LA;
        alo[t] = 0;
        ahi[t] = arow ? min(khi, Ia - a.knear) : 0;
        const int Ib = colpush ? J0 + t : I0 + t;   // fixed coordinate of the source tile
        const bool brow = colpush ? Ib < a.nt : Ib < a.mt;
        bbase[t] = brow ? (colpush ? a.X + ws_tile_offset(0, Ib, a.nt) : a.Y + ws_tile_offset(Ib, 0, a.nt))
                        : a.LA;
        blo[t] = max(a.K - Ib, 0);
        bhi[t] = brow ? min(khi, a.Mid - Ib) : 0;
    }
    // (an invalid tile's address may lie outside every allocation: with no
    // records nothing is read)
    auto rsrc = [](const float* base, int64_t stride, int kt, int lo, int hi) {
        const int nrec = (kt >= lo && kt < hi) ? TILE_ELEMS * 4 : 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base + kt * stride), (short)0, nrec,
                                                 0x00020000);
    };
    // two register sets: while chunk kt is multiplied from LDS, chunk kt + 1
    // (loaded one iteration earlier) waits in one set and chunk kt + 2 is in
    // flight into the other, so each global load has two chunks of MFMA work
    // to hide behind
    f32x4 ra[2][MT], rb[2][MT];
    auto load = [&](int kt, int r) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            ra[r][t] = __builtin_amdgcn_raw_buffer_load_b128(
                rsrc(abase[t], TILE_ELEMS, kt, alo[t], ahi[t]), tid * 16, 0, 0);
            rb[r][t] = __builtin_amdgcn_raw_buffer_load_b128(
                rsrc(bbase[t], bstride, kt, blo[t], bhi[t]), tid * 16, 0, 0);
        }
    };
    auto store = [&](int s, int r) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
            *reinterpret_cast<f32x4*>(&As[s][t * TS + srow][sk]) = ra[r][t];
            *reinterpret_cast<f32x4*>(&Bs[s][t * TS + srow][sk]) = rb[r][t];
        }
    };

    f32x16 acc[WB][WB];
#pragma unroll
    for (int x = 0; x < WB; ++x)
#pragma unroll
        for (int y = 0; y < WB; ++y) acc[x][y] = f32x16{0};

    // one K chunk: multiply LDS buffer s; issue the load of chunk kt + 2 into
    // register set r, then move chunk kt + 1 (set r ^ 1) into buffer s ^ 1
    auto chunk = [&](int kt, int s, int r) {
        load(kt + 2, r);   // past the range: no records, zeros
        f32x4 fa[WB][4], fb[WB][4];
#pragma unroll
        for (int x = 0; x < WB; ++x)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                fa[x][v] = *reinterpret_cast<const f32x4*>(
                    &As[s][(wm * WB + x) * TS + lr][lk * 16 + v * 4]);
#pragma unroll
        for (int y = 0; y < WB; ++y)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                fb[y][v] = *reinterpret_cast<const f32x4*>(
                    &Bs[s][(wn * WB + y) * TS + lr][lk * 16 + v * 4]);
#pragma unroll
        for (int st = 0; st < 16; ++st) {
#pragma unroll
            for (int x = 0; x < WB; ++x)
#pragma unroll
                for (int y = 0; y < WB; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[x][st >> 2][st & 3],
                                                                    fb[y][st >> 2][st & 3],
                                                                    acc[x][y], 0, 0, 0);
        }
        if (kt + 1 < khi) store(s ^ 1, r ^ 1);
        __syncthreads();
    };

    load(klo, 0);
    load(klo + 1, 1);
    store(0, 0);
    __syncthreads();
    // chunk klo + 2i uses buffer 0 and register set 0 for its prefetch,
    // chunk klo + 2i + 1 buffer 1 and set 1
    for (int kt = klo; kt < khi; kt += 2) {
        chunk(kt, 0, 0);
        if (kt + 1 < khi) chunk(kt + 1, 1, 1);
    }

    // epilogue: block (x, y) of wave (wm, wn) is output solver tile
    // (M tile wm*WB+x, N tile wn*WB+y); C[M][N] row-major inside the tile.
#pragma unroll
    for (int x = 0; x < WB; ++x)
#pragma unroll
        for (int y = 0; y < WB; ++y) {
            const int tm = wm * WB + x, tn = wn * WB + y;
            const int I = colpush ? I0 + tm : I0 + tn;
            const int J = colpush ? J0 + tn : J0 + tm;
            if (I >= a.mt || J >= a.nt || I + J < a.tlo || I + J >= a.thi) continue;
            float* out = (colpush ? a.Y : a.X) + ws_tile_offset(I, J, a.nt);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int rr = (r >> 2) * 8 + lk * 4 + (r & 3);
                out[rr * TS + lr] += acc[x][y][r];
            }
        }
}

// X <- W (tile-major, column-major inside each tile, zero padding), Y <- 0,
// ready flags <- 0 and ticket counters <- 0 (the give-up status word is left
// as it is: it is cleared only when the host reads it).  One workgroup per tile; the
// transpose goes through LDS so that both the read of W and the write of X
// are coalesced.
template <bool VEC>
__global__ __launch_bounds__(256) void k_prep(const float* __restrict__ W, int64_t m, int64_t n,
                                              int mt, int nt, float* __restrict__ X,
                                              float* __restrict__ Y, int* __restrict__ flags,
                                              int* __restrict__ counters, int ncounters) {
    __shared__ float T[TS][TS + 1];
    const int64_t tile = blockIdx.x;
    const int64_t I = tile / nt, J = tile - (tile / nt) * nt;
    const int tid = threadIdx.x;
    const int64_t base = tile * TILE_ELEMS;
    if (VEC) {
        // W rows as 16-byte chunks (n % 4 == 0, W 16-byte aligned), one per
        // thread; X (the tile transposed) and Y as contiguous 16-byte stores
        const int r = tid >> 3, c4 = (tid & 7) * 4;
        const int64_t gr = I * TS + r, gc = J * TS + c4;
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (gr < m && gc < n) v = *reinterpret_cast<const float4*>(W + gr * n + gc);
        T[r][c4] = v.x;
        T[r][c4 + 1] = v.y;
        T[r][c4 + 2] = v.z;
        T[r][c4 + 3] = v.w;
        __syncthreads();
        const int c = tid >> 3, r4 = (tid & 7) * 4;
        *reinterpret_cast<float4*>(X + base + 4 * tid) =
            make_float4(T[r4][c], T[r4 + 1][c], T[r4 + 2][c], T[r4 + 3][c]);
        *reinterpret_cast<float4*>(Y + base + 4 * tid) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
#pragma unroll
        for (int k = 0; k < TILE_ELEMS / 256; ++k) {
            const int e = k * 256 + tid;
            const int r = e >> 5, c = e & 31;
            const int64_t gr = I * TS + r, gc = J * TS + c;
            T[r][c] = (gr < m && gc < n) ? W[gr * n + gc] : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TILE_ELEMS / 256; ++k) {
            const int e = k * 256 + tid;
            const int c = e >> 5, r = e & 31;
            X[base + e] = T[r][c];
            Y[base + e] = 0.0f;
        }
    }
    if (tid == 0) flags[tile] = 0;
    if (tile == 0)
        for (int i = tid; i < ncounters; i += 256) counters[i] = 0;
}

// ---------------------------------------------------------------------------
// host launch driver

// Launches the plan: main ops on `st`, side ops on `side` (see Plan).
// ev_rel[i] is recorded on st after main op i when a side op waits for it;
// ev_side[c] on `side` after side op c.  tim (optional, profiling): an event
// pair around every launch, in enqueue order (prep first).
hipError_t run_plan(hipStream_t st, hipStream_t side, const Plan& plan, const float* W, int64_t m,
                    int64_t n, int mt, int nt, const Workspace& ws, const float* LA, const float* LB,
                    int b_ident, const QuantArgs& q, int8_t* codes, float* V, float* pre,
                    int knear, int spin_limit, int late, const int4* items, hipEvent_t* tim,
                    hipEvent_t* ev_rel, hipEvent_t* ev_side) {
    int ti = 0;
    auto t_begin = [&](hipStream_t s) { if (tim) (void)hipEventRecord(tim[2 * ti], s); };
    auto t_end = [&](hipStream_t s) { if (tim) (void)hipEventRecord(tim[2 * ti + 1], s); ++ti; };
    hipError_t e;
    t_begin(st);
    if (n % 4 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0)
        hipLaunchKernelGGL(k_prep<true>, dim3((unsigned)((int64_t)mt * nt)), dim3(256), 0, st, W, m,
                           n, mt, nt, ws.X, ws.Y, ws.flags, ws.counters, plan.nseg);
    else
        hipLaunchKernelGGL(k_prep<false>, dim3((unsigned)((int64_t)mt * nt)), dim3(256), 0, st, W, m,
                           n, mt, nt, ws.X, ws.Y, ws.flags, ws.counters, plan.nseg);
    t_end(st);
    if ((e = hipGetLastError()) != hipSuccess) return e;

    SegArgs sa{};
    sa.mt = mt; sa.nt = nt; sa.m = m; sa.n = n; sa.X = ws.X; sa.Y = ws.Y;
    sa.LA = LA; sa.LB = LB; sa.b_ident = b_ident; sa.q = q;
    sa.codes = codes; sa.V = V; sa.pre = pre; sa.knear = knear; sa.flags = ws.flags;
    sa.status = ws.status;
    sa.spin_limit = spin_limit;
    sa.late = late;
    NodeArgs nd{};
    nd.knear = knear; nd.mt = mt; nd.nt = nt; nd.X = ws.X; nd.Y = ws.Y; nd.LA = LA; nd.LB = LB;
    auto node = [&](const PlanOp& op, hipStream_t s) {
        nd.K = op.K;
        nd.Mid = op.Mid;
        nd.tlo = op.tlo;
        nd.thi = op.thi;
        nd.items = items + op.item_off;
        const dim3 grid((unsigned)op.item_cnt);
        if (op.macro == 8)
            hipLaunchKernelGGL(k_node<8>, grid, dim3(SplitShape<8>::TH), 0, s, nd);
        else if (op.fp32)
            hipLaunchKernelGGL(k_node32, grid, dim3(256), 0, s, nd);
        else if (op.macro == 4)
            hipLaunchKernelGGL(k_node<4>, grid, dim3(SplitShape<4>::TH), 0, s, nd);
        else
            hipLaunchKernelGGL(k_node<2>, grid, dim3(SplitShape<2>::TH), 0, s, nd);
    };
    int waited_side = 0, waited_rel = -1;
    for (const std::pair<int, int>& o : plan.order) {
        if (o.first == 0) {
            const PlanOp& op = plan.ops[o.second];
            if (op.need_side > waited_side) {
                if ((e = hipStreamWaitEvent(st, ev_side[op.need_side - 1], 0)) != hipSuccess) return e;
                waited_side = op.need_side;
            }
            t_begin(st);
            if (op.kind == 0) {
                sa.K = op.K;
                sa.L = op.L;
                sa.J_lo = op.strip_lo;
                sa.nstrips = op.nstrips;
                sa.counter = ws.counters + op.counter;
                const int grid = op.nstrips < SEG_GRID ? op.nstrips : SEG_GRID;
                const bool gq = q.gsize > 0 || q.col_scale, asym = q.qlo != -q.qhi;
                if (late)
                    hipLaunchKernelGGL((k_seg<true, true, true>), dim3((unsigned)grid), dim3(SEG_THREADS), 0, st, sa);
                else if (gq && asym)
                    hipLaunchKernelGGL((k_seg<true, true, false>), dim3((unsigned)grid), dim3(SEG_THREADS), 0, st, sa);
                else if (gq)
                    hipLaunchKernelGGL((k_seg<true, false, false>), dim3((unsigned)grid), dim3(SEG_THREADS), 0, st, sa);
                else if (asym)
                    hipLaunchKernelGGL((k_seg<false, true, false>), dim3((unsigned)grid), dim3(SEG_THREADS), 0, st, sa);
                else
                    hipLaunchKernelGGL((k_seg<false, false, false>), dim3((unsigned)grid), dim3(SEG_THREADS), 0, st, sa);
            } else {
                node(op, st);
            }
            t_end(st);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if (op.rec_rel && (e = hipEventRecord(ev_rel[o.second], st)) != hipSuccess) return e;
        } else {
            const PlanOp& op = plan.side[o.second];
            if (op.rel > waited_rel) {
                if ((e = hipStreamWaitEvent(side, ev_rel[op.rel], 0)) != hipSuccess) return e;
                waited_rel = op.rel;
            }
            t_begin(side);
            node(op, side);
            t_end(side);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if ((e = hipEventRecord(ev_side[o.second], side)) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

int plan_timed_launches(const Plan& plan) { return 1 + (int)plan.ops.size() + (int)plan.side.size(); }

}  // namespace bk
