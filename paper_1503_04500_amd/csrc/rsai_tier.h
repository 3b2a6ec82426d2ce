// Size-tiered fused RSAI(tol) column kernel (gfx950, one wave per workgroup).
//
// A wave holds 64/G columns; each column is owned by an aligned group of G lanes.
// The dense LS block A(I_k, J_k) of eq. (2.3) lives in registers, row i of the block
// in lane (i mod G), register slot (i / G): a column's block is at most
// MMAX = G * RPL rows by QMAX columns. Index sets are LDS hash sets (global index ->
// local position); rows and columns are numbered in insertion order, new ones in
// ascending global order, so the block grows by appending rows at the bottom and
// columns at the right and the Householder factor can be updated in place
// (Algorithm 1, step 7): stored reflectors are applied to the new columns only,
// then new reflectors are formed.
//
// What bounds it is the serial chain of one column's phases at two waves (small tier) or one
// wave per SIMD: index phases of dependent LDS and memory round trips, and reductions. So the
// index phases run without lane masks (absent entries go to slots past the arrays' ends),
// several columns' loads and insertions in flight together, new keys placed by ballots, and
// the local rows of the columns' first G entries kept as bytes, which the gathers and the
// residual read instead of probing the row hash. Measured against entry-by-entry insertion
// with look-ups: 512 x 512 grid, c = 3, eps = 0.4, 0.611 -> 0.585 ms in the small tier;
// 301 x 301, eps = 0.2, 3.84 -> 3.52 ms in the two group tiers; 64^3 grid 1.66 -> 1.65 ms
// (columns that outgrow the small tier pay 0.06 ms there and give 0.06 ms back after it);
// 400 000 power-law columns 19.6 -> 18.9 ms for the whole build.
//
// Every loop of Algorithm 1 runs in one pass of the wave's loop; groups that finish
// take the next column, so different groups of a wave may be at different loops.
// A column that outgrows the tier's caps is written to a spill record and resumed
// by the next larger tier.
#pragma once

#include "rsai_dev.h"

namespace rsai {

// Spill record: header of RHDR ints, then J (q), I (m), R (nR: dominant rows used so
// far), pending dominant rows (nRh). Header: [0] global column id, [1] matrix, [2] k,
// [3] l, [4] q, [5] m, [6] nR, [7] nRh, [8..9] flop count (double bits), [10] flags:
// bit 0 l is still to be advanced when the pending rows form J-hat, bit 1 the stored
// pattern is augmented but not yet solved, bit 2 dropping applies to that solve;
// [11] kept columns of the flop model of that solve, [12] the rows its kept factor
// was formed on.
constexpr int RHDR = 13;

template <int G_, int RPL_, int QMAX_, int STAGE_, int HSF_ = 2, int WPS_ = 2>
struct TierCfg {
    static constexpr int G = G_, RPL = RPL_, QMAX = QMAX_, STAGE = STAGE_;
    static constexpr int WPS = WPS_;  // waves per SIMD the register budget is cut for
    static constexpr int MMAX = G * RPL;
    static constexpr int GPW = 64 / G;
    static constexpr int LOGHSI = ilog2ceil(HSF_ * MMAX);  // row hash: HSF x MMAX slots
    static constexpr int HSI = 1 << LOGHSI;
    static constexpr int LOGHSJ = ilog2ceil(2 * QMAX);
    static constexpr int HSJ = 1 << LOGHSJ;
    static constexpr int NEWC = MMAX > QMAX ? MMAX : QMAX;
    static constexpr int RIN = HSI - MMAX - 1;  // candidates inserted per round (I)
    static constexpr int RJN = HSJ - QMAX - 1;  // (J)
    static constexpr int REC = RHDR + QMAX + MMAX + (MMAX + 1) + CMAX;  // spill record ints
    // keep the local rows of each column's first G entries (bytes in LDS): the column's wave
    // waits on its own chain of loads and look-ups, not on LDS space, so the gathers and the
    // residual read a byte instead of probing the row hash. The wave-wide tier's columns have
    // few entries per lane and its LDS decides the waves per CU; it looks the rows up.
    static constexpr bool CROW = G <= 16;
    // columns whose first G entries are inserted together (the row hash holds them all)
    static constexpr int CBN = (RIN / G < 1) ? 1 : (RIN / G > 6 ? 6 : RIN / G);
    // columns whose entries are loaded together for the residual of step 4
    static constexpr int SELB = QMAX <= 12 ? 6 : 4;
    static_assert(RPL <= 32 && QMAX <= 32, "bit masks");
    static_assert(RIN >= 1 && RJN >= 1, "hash sizes");
    static_assert(QMAX <= MMAX, "row j of the block must exist for every column j");
};

// Record layout (int32): [0] global column id, [1] matrix, [2] k, [3] l, [4] q, [5] m,
// [6] |R| (rows used as dominant rows, incl. k), [7] |R-hat| pending, [8..9] the
// column's flop count so far (double), [10] flags (bit 0: the loop counter is still
// to be advanced for the pending R-hat), then J[q], I[m], R[|R|], R-hat[|R-hat|].
// q = 0 and no pending R-hat means "start from scratch".
struct TierArgs {
    const MatDev *mats;
    int nmat;
    const int64_t *col_base;  // [nmat + 1]
    BuildParams P;
    ColOut out;
    int64_t arena_base;       // first arena slot of this tier
    int64_t qlen;             // tier 0: number of columns (all matrices)
    const int32_t *rec_in;    // tier >= 1: input records
    int rec_in_stride;
    const int32_t *rec_in_count;
    int64_t rec_in_cap;
    // Record queues of the later classes a spilled column may go to (index 0: the
    // next class). A column goes to the first class whose limits hold the estimated
    // |I_k| and |J_k| of its next augmentation, else to the last queue; nq = 0 means
    // no later class (a spill is then a cap error).
    static constexpr int MAXQ = 4;
    int nq;
    int32_t *q_rec[MAXQ];
    int q_stride[MAXQ];
    int32_t *q_count[MAXQ];
    int64_t q_cap[MAXQ];
    int q_mmax[MAXQ], q_qmax[MAXQ];
    int32_t *err;             // global error flags (bit 0: internal)
    int one_loop;             // 1: park every column after one loop (plain schedule)
    int sync_refill;          // 1: groups take new columns only when the whole wave is idle
};

// Per-group LDS. The staging tile doubles as scratch for the phase-local arrays:
// the new-entry lists and segment tables of the augmentation phases, and the
// residual accumulator and column order of the dominant-row phase.
template <class C>
struct alignas(16) GLds {
    // (arrays that the index phases read and write without a lane mask have room past their
    // end: lanes with nothing to do read what is there and write to the last element)
    static constexpr int TILE = C::STAGE * C::MMAX;
    static constexpr int CP = C::QMAX + (C::STAGE > 6 ? C::STAGE : 6);
    double stage[TILE + 2];
    double mt[C::QMAX];       // solution of the last LS solve, by column slot
    int cb[CP + 1];           // first entry of the column in each slot of J (CSC of A; nnz < 2^31)
    int cl[CP + 1];           // its length
    int Ilist[C::MMAX + 1];
    alignas(16) int Jlist[C::QMAX + 4];  // (INT_MAX in the four entries after the last column)
    int hI[C::HSI + 1];
    int hJ[C::HSJ + 1];
    int Rh[CMAX];             // pending dominant rows
    int cnt;
    int fo_lo, fo_hi;         // factor record of a finished column (kept R)
    int pad;
    unsigned char hIv[C::HSI + 1];  // local row of each key in hI
    // local rows of the first G entries of each column of J (entry gl of a column belongs to
    // lane gl), so that the gathers and the residual look no row up (groups of up to 16
    // lanes; the wave-wide tier looks them up)
    unsigned char crow[C::CROW ? (CP + 1) * C::G : 1];

    // augmentation phases (K, C, D)
    static constexpr int NEWP = (C::NEWC + 4 + 3) / 4 * 4;  // keys with room for the padding
    __device__ int *newk() { return reinterpret_cast<int *>(stage); }
    __device__ int *news() { return newk() + NEWP; }
    // dominant-row phase (J)
    __device__ double *racc() { return stage; }  // MMAX rows and one for lanes without an entry
    __device__ int *ord() { return reinterpret_cast<int *>(stage + C::MMAX + 1); }

    static_assert(NEWP * 8 <= C::STAGE * C::MMAX * 8, "scratch fits the tile");
    static_assert((C::MMAX + 1) * 8 + C::QMAX * 4 <= C::STAGE * C::MMAX * 8, "scratch fits the tile");
    static_assert(C::MMAX < 256 && C::HSI <= 256, "local rows and row-hash slots fit a byte");
};


// ----------------------------------------------------------------- tiers
// t0: up to 24 x 12 blocks (2D 5-point stencils), 8 columns per wave
// t1: up to 64 x 24 blocks (3D 7-point stencils), 4 columns per wave; one wave per
//     SIMD so that the fully unrolled QR keeps its 96 block entries per lane in
//     registers
// t2: up to 128 x 32 blocks, a whole wave per column (two rows per lane, the group
//     reductions crossing the 16-lane rows by permlane swaps): fully unrolled, its 64
//     block entries per lane stay in registers at one wave per SIMD
#ifndef RSAI_T0_STAGE
#define RSAI_T0_STAGE 6
#endif
#ifndef RSAI_T0_HSF
#define RSAI_T0_HSF 2
#endif
using Tier0 = TierCfg<8, 3, 12, RSAI_T0_STAGE, RSAI_T0_HSF>;
// tier 0 with hash tables of four times its row and column capacity (a tile choice of
// the autotuner: fewer probes per insertion, more slots cleared per column)
using Tier0H4 = TierCfg<8, 3, 12, RSAI_T0_STAGE, 4>;
using Tier1 = TierCfg<16, 4, 24, 8, 2, 1>;
using Tier2 = TierCfg<64, 2, 32, 8, 2, 1>;
void launch_tier2(const TierArgs &a, int waves, hipStream_t s);
void launch_tier0_h4(const TierArgs &a, int waves, hipStream_t s);

}  // namespace rsai
