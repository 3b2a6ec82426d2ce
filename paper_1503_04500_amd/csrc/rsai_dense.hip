// First level of the dense class of the RSAI(tol) build: one 256-thread workgroup per
// column for LS blocks A(I_k, J_k) of up to DENSE_MMAX = 128 rows and DENSE_QMAX = 63
// columns, most of whose rows are shared by several columns (small eps on grids). Same
// steps as the other classes (Algorithm 1 with the dropping of Section 4); a column that
// outgrows this level goes on to the second one (rsai_big.hip).
//
// Layout. The block lives in registers, lane c of every wave holding column c (the
// right-hand side e_k is column q) and row i in wave i mod 4, slot i / 4: a Householder
// step then needs no lane reduction. The products of column j with every column are one
// FMA per row and lane (the entries of column j read from lane j into scalar registers),
// summed over the four waves through LDS; the same sums hold ||column j||^2 in lane j.
// One barrier per step. The rows are ordered by the first column that holds them, so a
// step ends at the last row that its column and the earlier ones reach (on grids about
// 5 + 1.5 j of the 88 rows at step j). The slots are addressed at compile time: the steps run in
// rounds of 32 rows, after which the registers move up by 8 slots, so the code is one
// round long whatever |J_k| is. Finished rows of R go to LDS (packed by columns), where
// the back substitution and the re-solve after a drop read them: the kept columns of R
// are factored instead of the kept columns of A (A(:, kept) = Q R(:, kept), |J| rows
// instead of |I|, and nothing is gathered again).
//
// What bounds it: VALU issue (the vector units are busy about 70% of the time; a third of
// the instructions are the lane reads that broadcast column j) and the chain of a step's
// sums, square root and division, with four columns resident per CU to hide it (34 KB of
// LDS, 128 registers: 4 waves per SIMD). On a 100 x 100 grid at eps = 0.1 (9000 columns
// here, |I| about 85, |J| about 55, about 8 solves each) it takes 5.5 ms; the second
// level, one column per CU with its block in global memory, spent 62 ms on them. With the
// rows in insertion order instead of by first column, and column j read twice per step
// from its lane, it took 7.5 ms.
#include <climits>

#include "rsai_kernels.h"

namespace rsai {

namespace {
constexpr int NT = 256;
constexpr int NW = NT / 64;
constexpr int QM = DENSE_QMAX;           // columns of J
constexpr int MM = DENSE_MMAX;           // rows of I
constexpr int NS = MM / NW;              // register slots of a thread
constexpr int LOGHI = 9, HI = 1 << LOGHI;
constexpr int LOGHJ = 8, HJ = 1 << LOGHJ;
constexpr int TROWS = 32;                // rows of the gather tile (8 slots of the 4 waves)
constexpr int TILE = TROWS * 64;
constexpr int NE = 4;                    // entries of the block a thread keeps for the gather
constexpr int SG = 4;                    // slots a step takes or skips together
constexpr int XK = 12;                   // slots whose entries of column j stay in scalar registers
static_assert(QM * (QM + 1) / 2 <= TILE, "R packed by columns fits the gather tile");
static_assert(QM < 64 && QM <= MM, "a lane per column and one for the right-hand side");
static_assert(MM + NT < HI, "the row hash holds I and one round of new entries");

struct DLds {
    double R[TILE];            // gather tile; R (column c from c (c - 1) / 2); values by row
    double part[2][NW][64];    // products of a step, per wave; values by row where R is kept
    double piv[2][64];         // row j of the block
    double mt[64], mo[64];     // solution by slot, and in ascending column order
    double rd[64];             // diagonal of R
    double racc[MM];           // residual by row
    unsigned long long rmask[MM];  // columns (ascending positions) of each row
    int64_t cb[64];            // first entry of each column of J
    int cl[64], Jl[64], ord[64];
    int pre[65];               // prefix of the column lengths
    int Il[MM];
    int roff[MM];              // first value of each row
    int fc[MM];                // first column (slot) of J that holds each row
    int rnk[MM];               // its row of the block
    int top[64];               // rows of the block that columns 0..c touch
    int hI[HI], hJ[HJ];
    int newk[MM], news[MM];
    int Rh[CMAX];
    int cnt, misc, nsel, kR;
    unsigned char hIv[HI];
    unsigned char rfl[MM];     // row in R (used dominant rows)
};

// The matrix, read through a pointer whose value the compiler cannot see: its pointers
// are loaded where a phase uses them instead of being held in scalar registers across
// the solve.
using CMat = const __attribute__((address_space(4))) MatDev;
__device__ __forceinline__ CMat &matrix(CMat *p) {
    asm volatile("" : "+s"(p));
    return *p;
}
__device__ __forceinline__ int rcol(int c) { return c * (c - 1) / 2; }

// prefix of the lengths of the first n columns, by one wave
__device__ __forceinline__ void prefix_lengths(DLds &S, int n, int lane) {
    int x = (lane < n) ? S.cl[lane] : 0;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 0) S.pre[0] = 0;
    S.pre[lane + 1] = x;
}
// the column of [lo, hi) holding flattened entry u
__device__ __forceinline__ int column_of(const DLds &S, int lo, int hi, int u) {
    --hi;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (S.pre[mid] <= u) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// One Householder step: column j, its head row in slot PS of wave w4. rows: rows from the
// round's first one that column j can reach. Lane c > j gets its column updated and, in
// wave w4, stores R(j, c).
template <int PS>
__device__ __forceinline__ void hstep(double (&b)[NS], int j, int w4, int qn, int rows, int w, int lane, DLds &S,
                                      bool &singular) {
    const int buf = j & 1;
    double x[XK];
    double a0, a1 = 0.0;
    {
        // (rows above j of the head slot are finished)
        x[PS] = (w < w4) ? 0.0 : readlane_f64(b[PS], j);
        a0 = x[PS] * b[PS];
    }
#pragma unroll
    for (int g = 0; g < NS / SG; ++g) {
        if (NW * SG * g < rows) {
#pragma unroll
            for (int u = 0; u < SG; ++u) {
                const int t = SG * g + u;
                if (t > PS) {
                    const double xt = readlane_f64(b[t], j);
                    if (t < XK) x[t] = xt;
                    if (u & 1) a1 += xt * b[t]; else a0 += xt * b[t];
                }
            }
        }
    }
    S.part[buf][w][lane] = a0 + a1;
    if (w == w4) S.piv[buf][lane] = b[PS];
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int v = 0; v < NW; ++v) tot += S.part[buf][v][lane];
    const double bj = S.piv[buf][lane];
    const double s2 = readlane_f64(tot, j), x0 = readlane_f64(bj, j);
    double nx, be;
    hh_scalars(s2, x0, nx, be);
    const double alpha = (x0 >= 0.0) ? -nx : nx;
    if (!(nx > 0.0)) singular = true;
    // v = x with the head x0 - alpha: v . b = x . b - alpha b_j
    const double f = (lane > j && lane <= qn) ? be * (tot - alpha * bj) : 0.0;
    b[PS] -= f * ((w == w4) ? x0 - alpha : x[PS]);
    // (past the first XK slots column j, unchanged as f = 0 in lane j, is read again: its
    // scalar registers would not fit beside the rest)
    int j2 = j;
    asm volatile("" : "+s"(j2));
#pragma unroll
    for (int g = 0; g < NS / SG; ++g) {
        if (NW * SG * g < rows) {
#pragma unroll
            for (int u = 0; u < SG; ++u) {
                const int t = SG * g + u;
                if (t > PS) b[t] -= f * (t < XK ? x[t < XK ? t : 0] : readlane_f64(b[t], j2));
            }
        }
    }
    if (w == w4) {
        if (lane > j && lane <= qn) S.R[rcol(lane) + j] = b[PS];
        if (lane == j) S.rd[j] = alpha;
    }
}

template <int PS>
__device__ __forceinline__ void hround(double (&b)[NS], int r0, int top, int qn, int w, int lane, DLds &S,
                                       bool &singular) {
    if constexpr (PS < 8) {
#pragma unroll 1
        for (int w4 = 0; w4 < NW; ++w4) {
            const int j = r0 + NW * PS + w4;
            if (j < qn) hstep<PS>(b, j, w4, qn, __builtin_amdgcn_readlane(top, j) - r0, w, lane, S, singular);
        }
        hround<PS + 1>(b, r0, top, qn, w, lane, S, singular);
    }
}

// Householder QR of the block of qn columns in b (column qn: the right-hand side), back
// substitution into S.mt. top, in lane c: one past the last row that columns 0..c touch
// (the reflectors of column c and the earlier ones are zero from there on). Returns the
// sum of squares of the right-hand side below row qn; singular is set when a column has
// no norm left. Begins with the block loaded and S.R free, ends after a barrier.
__device__ __forceinline__ double factor_solve(double (&b)[NS], int top, int qn, int w, int lane, DLds &S,
                                               bool &singular) {
    int r0 = 0;
#pragma unroll 1
    for (;;) {
        hround<0>(b, r0, top, qn, w, lane, S, singular);
        if (r0 + 32 >= qn) break;
        r0 += 32;
#pragma unroll
        for (int t = 0; t < NS; ++t) b[t] = (t + 8 < NS) ? b[t + 8] : 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < NS; ++t)
        if (r0 + NW * t + w >= qn) s += b[t] * b[t];
    __syncthreads();
    S.part[0][w][lane] = s;
    __syncthreads();
    double r2 = 0.0;
#pragma unroll
    for (int v = 0; v < NW; ++v) r2 += S.part[0][v][qn];
    if (w == 0 && !singular) {
        // back substitution: lane i holds (Q^T e)_i, m_j broadcast from lane j
        // (a step divides by multiplying with the reciprocal and correcting the quotient by
        // its residual: the divisions of all steps are done beforehand, a lane each)
        double y = (lane < qn) ? S.R[rcol(qn) + lane] : 0.0;
        const double rdl = (lane < qn) ? S.rd[lane] : 1.0;
        const double ril = 1.0 / rdl;
        double mine = 0.0;
        for (int j = qn - 1; j >= 0; --j) {
            const double rj = (lane < j) ? S.R[rcol(j) + lane] : 0.0;
            const double yj = readlane_f64(y, j), ri = readlane_f64(ril, j);
            const double mj = div_by(yj, readlane_f64(rdl, j), ri);
            if (lane == j) mine = mj;
            y -= rj * mj;
        }
        S.mt[lane] = mine;
    }
    __syncthreads();
    return r2;
}
}  // namespace

__global__ __launch_bounds__(NT, 4) void dense_kernel(DenseArgs args) {
    __shared__ DLds S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (*args.err & ERR_SKIP) return;
    const BuildParams P = args.P;
    const int64_t Q = min((int64_t)(*args.rec_count), args.rec_cap);

    for (int64_t pos = blockIdx.x; pos < Q; pos += gridDim.x) {
        int32_t *rec = args.rec + pos * (int64_t)args.rec_stride;
        const int ucol = rec[0], mat = __builtin_amdgcn_readfirstlane(rec[1]), k = rec[2];
        int l = rec[3];
        int q = __builtin_amdgcn_readfirstlane(rec[4]), m = __builtin_amdgcn_readfirstlane(rec[5]);
        const int nR0 = rec[6];
        int nRh = __builtin_amdgcn_readfirstlane(rec[7]);
        double fl = __longlong_as_double(((long long)rec[9] << 32) | (long long)(unsigned)rec[8]);
        const int flags = rec[10];
        bool linc = (flags & 1) != 0;
        if (q > QM || m > MM || nRh > CMAX || (q == 0 && nRh == 0)) {
            // larger than this level on arrival (or a column not started yet, whose own
            // rows outgrew every earlier class): the record stays as it is
            if (tid == 0) args.next_list[atomicAdd(args.next_count, 1)] = (int32_t)pos;
            continue;
        }
        CMat *const Ac = (CMat *)(args.mats + mat);
        const int32_t *RJ = rec + RHDR, *RI = RJ + q, *RR = RI + m, *RHp = RR + nR0;
        int status = ST_OK;
        bool spill = false, lookup_fail = false;
        double rn = 0.0;
        int kidx;
        bool kR;

        // ---------------------------------------------------------- state from the record
        for (int t = tid; t < HI; t += NT) S.hI[t] = HEMPTY;
        for (int t = tid; t < HJ; t += NT) S.hJ[t] = HEMPTY;
        if (tid < m) S.newk[tid] = RI[tid];
        if (tid == 0) { S.misc = -1; S.kR = 0; }
        __syncthreads();
        if (tid < q) {
            CMat &A = matrix(Ac);
            const int col = RJ[tid];
            S.Jl[tid] = col;
            const int64_t b0 = A.colptr[col];
            S.cb[tid] = b0;
            S.cl[tid] = (int)(A.colptr[col + 1] - b0);
            int sl;
            hinsert<LOGHJ>(S.hJ, col, sl);
        }
        if (tid < nRh) S.Rh[tid] = RHp[tid];
        if (tid < m) {
            // rows of I numbered in ascending order (records may list them in any order)
            const int key = S.newk[tid];
            int rank = 0;
            for (int t = 0; t < m; ++t) rank += (S.newk[t] < key) ? 1 : 0;
            S.Il[rank] = key;
            S.rfl[rank] = 0;
            int sl;
            hinsert<LOGHI>(S.hI, key, sl);
            if (sl >= 0) S.hIv[sl] = (unsigned char)rank;
            if (key == k) S.misc = rank;
        }
        __syncthreads();
        for (int t = tid; t < nR0; t += NT) {
            const int row = RR[t];
            const int sl = hfind<LOGHI>(S.hI, row);
            if (sl >= 0) S.rfl[S.hIv[sl]] = 1;
            else if (row == k) S.kR = 1;  // k used as a dominant row while k is not in I
        }
        __syncthreads();
        kidx = S.misc;
        kR = S.kR != 0;
        __syncthreads();

        bool first = true, need_solve = true, dropok = false;
        int qmod = -1, mmod = 0, p = 0;
        if (flags & 2) {
            // augmented pattern handed over before its solve
            dropok = (flags & 4) != 0;
            qmod = rec[11];
            mmod = rec[12];
        }

        while (status == ST_OK && !spill) {
            // ================= J-hat: columns of the pending dominant rows not in J (step 5)
            if (nRh > 0) {
                if (linc) ++l;  // step 6
                linc = false;
                CMat &A = matrix(Ac);
                int64_t sb[CMAX];
                int sp[CMAX + 1];
                sp[0] = 0;
#pragma unroll
                for (int t = 0; t < CMAX; ++t) {
                    int64_t b0 = 0, e0 = 0;
                    if (t < nRh) {
                        const int rt = S.Rh[t];
                        b0 = A.rowptr[rt];
                        e0 = A.rowptr[rt + 1];
                    }
                    sb[t] = b0;
                    sp[t + 1] = sp[t] + (int)(e0 - b0);
                }
                if (tid == 0) S.cnt = 0;
                __syncthreads();
                bool ovf = false;
                for (int u = tid; u < sp[CMAX]; u += NT) {
                    int64_t b0 = sb[0];
                    int o0 = 0;
#pragma unroll
                    for (int t = 1; t < CMAX; ++t)
                        if (u >= sp[t]) { b0 = sb[t]; o0 = sp[t]; }
                    const int col = A.colidx[b0 + (u - o0)];
                    int sl;
                    if (hinsert<LOGHJ>(S.hJ, col, sl)) {
                        const int ps = atomicAdd(&S.cnt, 1);
                        if (q + ps < QM) S.newk[ps] = col; else ovf = true;
                    } else if (sl < 0) {
                        ovf = true;  // table full
                    }
                }
                if (__syncthreads_or(ovf)) { spill = true; break; }
                p = __builtin_amdgcn_readfirstlane(S.cnt);
                if (tid < p) {
                    const int key = S.newk[tid];
                    int rank = 0;
                    for (int t = 0; t < p; ++t) rank += (S.newk[t] < key) ? 1 : 0;
                    S.Jl[q + rank] = key;
                    const int64_t b0 = A.colptr[key];
                    S.cb[q + rank] = b0;
                    S.cl[q + rank] = (int)(A.colptr[key + 1] - b0);
                }
                need_solve = !(p == 0 && !first);  // empty J-hat: the loop ends without a solve
                dropok = (p > 0);
                qmod = (p > 0) ? q : (first ? -1 : q);
                mmod = m;
                __syncthreads();
            }
            if (need_solve) {
                if (w == 0) prefix_lengths(S, q + p, lane);
                if (tid == 0) { S.cnt = 0; S.misc = -1; }
                __syncthreads();
            }
            // ================= I-hat: rows of the new columns not in I (step 5)
            if (need_solve && p > 0) {
                CMat &A = matrix(Ac);
                const int e1 = S.pre[q + p];
                for (int base = S.pre[q]; base < e1; base += NT) {
                    const int u = base + tid;
                    if (u < e1) {
                        const int c = column_of(S, q, q + p, u);
                        const int row = A.rowidx[S.cb[c] + (u - S.pre[c])];
                        int sl;
                        if (hinsert<LOGHI>(S.hI, row, sl)) {
                            const int ps = atomicAdd(&S.cnt, 1);
                            if (ps < MM) { S.newk[ps] = row; S.news[ps] = sl; }
                        }
                    }
                    __syncthreads();
                    if (m + S.cnt > MM) { spill = true; break; }
                    __syncthreads();
                }
                if (spill) break;
                const int nn = __builtin_amdgcn_readfirstlane(S.cnt);
                if (tid < nn) {
                    const int key = S.newk[tid];
                    int rank = 0;
                    for (int t = 0; t < nn; ++t) rank += (S.newk[t] < key) ? 1 : 0;
                    S.Il[m + rank] = key;
                    S.hIv[S.news[tid]] = (unsigned char)(m + rank);
                    S.rfl[m + rank] = 0;
                    if (key == k) S.misc = m + rank;
                }
                __syncthreads();
                if (S.misc >= 0) {
                    kidx = S.misc;
                    if (kR) {
                        // k entered I: its flag moves to its row
                        if (tid == 0) S.rfl[kidx] = 1;
                        kR = false;
                    }
                }
                m += nn;
                q += p;
                p = 0;
            }
            nRh = 0;  // pending rows consumed
            first = false;

            // ================= LS solve(s) on (I, J) (2.3): the augmented pattern, then the
            // pattern kept after dropping (Section 4)
            if (need_solve) {
                double b[NS];
                // ---- rows of the block: ordered by the first column of J that holds them,
                // so that column c and its reflector end at row top[c] and a Householder
                // step passes over the rows below. The entries found once and kept, up to
                // NE per thread.
                CMat &A = matrix(Ac);
                const int nent = S.pre[q];
                int eat[NE];
                double ev[NE];
                auto locate = [&](int u, int &c, double &v) -> int {
                    c = column_of(S, 0, q, u);
                    const int64_t e = S.cb[c] + (u - S.pre[c]);
                    const int sl = hfind<LOGHI>(S.hI, A.rowidx[e]);
                    v = A.val[e];
                    if (sl < 0) { lookup_fail = true; return -1; }
                    return S.hIv[sl];
                };
                if (tid < MM) S.fc[tid] = 64;
                __syncthreads();
#pragma unroll
                for (int s = 0; s < NE; ++s) {
                    eat[s] = -1;
                    ev[s] = 0.0;
                    if (tid + s * NT < nent) {
                        int c;
                        const int id = locate(tid + s * NT, c, ev[s]);
                        if (id >= 0) {
                            atomicMin(&S.fc[id], c);
                            eat[s] = id * 64 + c;
                        }
                    }
                }
                for (int u = tid + NE * NT; u < nent; u += NT) {
                    int c;
                    double v;
                    const int id = locate(u, c, v);
                    if (id >= 0) atomicMin(&S.fc[id], c);
                }
                __syncthreads();
                if (tid < m) {
                    const int key = S.fc[tid] * MM + tid;
                    int rank = 0;
                    for (int t = 0; t < m; ++t) rank += (S.fc[t] * MM + t < key) ? 1 : 0;
                    S.rnk[tid] = rank;
                } else if (tid >= NT - 64) {
                    int n = 0;
                    for (int t = 0; t < m; ++t) n += (S.fc[t] <= tid - (NT - 64)) ? 1 : 0;
                    S.top[tid - (NT - 64)] = n;
                }
                __syncthreads();
#pragma unroll
                for (int s = 0; s < NE; ++s)
                    if (eat[s] >= 0) eat[s] = S.rnk[eat[s] >> 6] * 64 + (eat[s] & 63);
                const int krow = kidx >= 0 ? S.rnk[kidx] : -1;
                // ---- gather: 32 rows at a time through the tile
#pragma unroll
                for (int g = 0; g < NS / 8; ++g) {
                    if (TROWS * g < m) {
                        for (int t = tid; t < TILE; t += NT) S.R[t] = 0.0;
                        __syncthreads();
#pragma unroll
                        for (int s = 0; s < NE; ++s)
                            if (eat[s] >= 0 && eat[s] / TILE == g) S.R[eat[s] % TILE] = ev[s];
                        for (int u = tid + NE * NT; u < nent; u += NT) {
                            int c;
                            double v;
                            const int id = locate(u, c, v);
                            if (id >= 0 && S.rnk[id] / TROWS == g) S.R[(S.rnk[id] % TROWS) * 64 + c] = v;
                        }
                        __syncthreads();
#pragma unroll
                        for (int s = 0; s < 8; ++s) b[8 * g + s] = S.R[(NW * s + w) * 64 + lane];
                        __syncthreads();
                    } else {
#pragma unroll
                        for (int s = 0; s < 8; ++s) b[8 * g + s] = 0.0;
                    }
                }
                if (lane == q) {
#pragma unroll
                    for (int t = 0; t < NS; ++t) b[t] = (NW * t + w == krow) ? 1.0 : 0.0;
                }
                int top = S.top[lane];
                double tail = (kidx < 0) ? 1.0 : 0.0;  // r(k) = -1 when k is not in I
                for (int pass = 0; pass < 2; ++pass) {
                    bool singular = false;
                    tail += factor_solve(b, top, q, w, lane, S, singular);
                    if (singular) { status = ST_SINGULAR; break; }
                    rn = sqrt(tail);
                    if (qmod >= 0) fl += solve_flops(mmod, m, qmod, q);
                    // ---- dropping (Section 4), after the augment solve only
                    if (pass == 1 || !dropok || P.drop == DROP_NONE) break;
                    const double th = (P.drop == DROP_FIXED)
                                          ? P.tol
                                          : P.eps / ((double)q * __longlong_as_double((long long)*matrix(Ac).norm1_bits));
                    // kept columns as a lane mask (each wave forms the same one); with none
                    // above the threshold, the largest |m_j| stays (the smaller column index
                    // on ties)
                    const bool inq = lane < q;
                    const double am = inq ? fabs(S.mt[lane]) : -1.0;
                    const int jg = inq ? S.Jl[lane] : INT_MAX;
                    unsigned long long keepm = __ballot(inq && am > th);
                    if (__popcll(keepm) == q) break;
                    if (keepm == 0ull) {
                        double ba = am;
                        int bg = jg;
                        gargmax<64>(ba, bg);
                        keepm = __ballot(inq && jg == bg);
                    }
                    const int qo = q, nk = __popcll(keepm);
                    __syncthreads();
                    if (w == 0) {
                        // compaction of the slots in order; ord: the old slot of each kept one
                        const bool kc = inq && ((keepm >> lane) & 1ull);
                        const int64_t cbv = inq ? S.cb[lane] : 0;
                        const int clv = inq ? S.cl[lane] : 0;
                        const int d = __popcll(keepm & ((1ull << lane) - 1ull));
                        wave_sync();
                        if (kc) {
                            S.Jl[d] = jg;
                            S.cb[d] = cbv;
                            S.cl[d] = clv;
                            S.ord[d] = lane;
                        }
                        wave_sync();
                        prefix_lengths(S, nk, lane);
                    }
                    for (int t = tid; t < HJ; t += NT) S.hJ[t] = HEMPTY;
                    __syncthreads();
                    if (tid < nk) {
                        int sl;
                        hinsert<LOGHJ>(S.hJ, S.Jl[tid], sl);
                    }
                    // the kept columns of R and (Q^T e) as the block of the re-solve
                    const int oc = lane < nk ? S.ord[lane] : (lane == nk ? qo : -1);
                    const double rdo = (oc >= 0 && oc < qo) ? S.rd[oc] : 0.0;
#pragma unroll
                    for (int t = 0; t < NS; ++t) {
                        const int i = NW * t + w;
                        b[t] = 0.0;
                        if (t < 64 / NW && i < qo && oc >= 0) {
                            if (i < oc) b[t] = S.R[rcol(oc) + i];
                            else if (i == oc) b[t] = rdo;
                        }
                    }
                    top = oc + 1;
                    q = nk;
                    qmod = 0;
                    __syncthreads();
                }
                if (status != ST_OK) break;
            }
            need_solve = false;

            // ================= stop test (step 3)
            if (rn <= P.eps || l >= P.lmax) break;

            // ================= dominant rows of r = A(I,J) m - e_k (step 4): every row
            // sums its columns in ascending global order, so exact ties reach the
            // smaller-index rule. The entries are sorted by row in LDS: the columns
            // (ascending positions) of each row as a mask, a value's place its rank there.
            __syncthreads();
            if (tid < MM) S.rmask[tid] = 0ull;
            if (tid < q) {
                const int jc = S.Jl[tid];
                int rank = 0;
                for (int t = 0; t < q; ++t) rank += (S.Jl[t] < jc) ? 1 : 0;
                S.ord[tid] = rank;
                S.mo[rank] = S.mt[tid];
            }
            __syncthreads();
            CMat &A = matrix(Ac);
            const int nent = S.pre[q];
            auto entry = [&](int u, int &c, int64_t &e) -> int {
                c = column_of(S, 0, q, u);
                e = S.cb[c] + (u - S.pre[c]);
                const int sl = hfind<LOGHI>(S.hI, A.rowidx[e]);
                if (sl < 0) { lookup_fail = true; return -1; }
                return S.hIv[sl];
            };
            int eli[NE], epos[NE];
            double ev[NE];
#pragma unroll
            for (int s = 0; s < NE; ++s) {
                const int u = tid + s * NT;
                eli[s] = -1;
                epos[s] = 0;
                ev[s] = 0.0;
                if (u < nent) {
                    int c;
                    int64_t e;
                    eli[s] = entry(u, c, e);
                    epos[s] = S.ord[c];
                    ev[s] = A.val[e];
                    if (eli[s] >= 0) atomicOr(&S.rmask[eli[s]], 1ull << epos[s]);
                }
            }
            for (int u = tid + NE * NT; u < nent; u += NT) {
                int c;
                int64_t e;
                const int li = entry(u, c, e);
                if (li >= 0) atomicOr(&S.rmask[li], 1ull << S.ord[c]);
            }
            __syncthreads();
            if (w == 0) {
                // first value of each row: prefix of the row lengths
                const int n0 = __popcll(S.rmask[lane]), n1 = __popcll(S.rmask[lane + 64]);
                int x0 = n0, x1 = n1;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int y0 = __shfl_up(x0, d), y1 = __shfl_up(x1, d);
                    if (lane >= d) { x0 += y0; x1 += y1; }
                }
                const int h = __builtin_amdgcn_readlane(x0, 63);
                S.roff[lane] = x0 - n0;
                S.roff[lane + 64] = h + x1 - n1;
            }
            __syncthreads();
            // The values' buffer: the gather tile. Where R is kept for the adjoint it has to
            // outlive this phase (the column may end without another solve): the part of the
            // tile past R, or the steps' products if they are the larger, hold the values. A
            // block with more entries than the buffer goes as many rows at a time as fit (a
            // row has at most q).
            double *vals = S.R;
            int vcap = TILE;
            if (args.out.fac != nullptr) {
                constexpr int PART = 2 * NW * 64;
                const int tail = TILE - rcol(q);
                vals = tail >= PART ? S.R + rcol(q) : &S.part[0][0][0];
                vcap = tail >= PART ? tail : PART;
            }
            const int rstep = nent <= vcap ? MM : min(vcap / q, MM);
            for (int lo = 0; lo < m; lo += rstep) {
                const int base = S.roff[lo];
                auto put = [&](int li, int ps, double v) {
                    if (li >= lo && li < lo + rstep)
                        vals[S.roff[li] - base + __popcll(S.rmask[li] & ((1ull << ps) - 1ull))] = v;
                };
#pragma unroll
                for (int s = 0; s < NE; ++s)
                    if (eli[s] >= 0) put(eli[s], epos[s], ev[s]);
                for (int u = tid + NE * NT; u < nent; u += NT) {
                    int c;
                    int64_t e;
                    const int li = entry(u, c, e);
                    if (li >= 0) put(li, S.ord[c], A.val[e]);
                }
                __syncthreads();
                const int i = lo + tid;
                if (tid < rstep && i < m) {
                    double acc = 0.0;
                    int at = S.roff[i] - base;
                    for (unsigned long long mk = S.rmask[i]; mk != 0ull; mk &= mk - 1ull)
                        acc = __fma_rn(vals[at++], S.mo[__builtin_ctzll(mk)], acc);
                    S.racc[i] = acc - ((i == kidx) ? 1.0 : 0.0);
                }
                __syncthreads();
            }
            if (w == 0) {
                double ra[2];
                int gi[2], li[2];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = lane + 64 * r;
                    const double ri = i < m ? S.racc[i] : 0.0;
                    const bool cand = i < m && ri != 0.0 && !S.rfl[i];
                    ra[r] = cand ? fabs(ri) : -1.0;
                    gi[r] = cand ? S.Il[i] : INT_MAX;
                    li[r] = i;
                }
                bool kcand = kidx < 0 && !kR;
                int nsel = 0;
                for (int t = 0; t < P.c; ++t) {
                    double a = ra[0];
                    int g = gi[0];
                    if (ra[1] > a || (ra[1] == a && gi[1] < g)) { a = ra[1]; g = gi[1]; }
                    gargmax<64>(a, g);
                    if (kcand && (1.0 > a || (1.0 == a && k < g))) { a = 1.0; g = k; }
                    if (a < 0.0) break;
                    if (lane == 0) S.Rh[t] = g;
                    nsel = t + 1;
                    if (kcand && g == k) {
                        kcand = false;
                        if (lane == 0) S.kR = 1;
                    } else {
#pragma unroll
                        for (int r = 0; r < 2; ++r)
                            if (gi[r] == g && ra[r] >= 0.0) {
                                ra[r] = -1.0;
                                gi[r] = INT_MAX;
                                S.rfl[li[r]] = 1;
                            }
                    }
                }
                if (lane == 0) S.nsel = nsel;
            }
            __syncthreads();
            kR = kidx < 0 && S.kR != 0;
            nRh = __builtin_amdgcn_readfirstlane(S.nsel);
            __syncthreads();
            if (nRh == 0) break;  // no candidate row left: r = 0 (Section 3)
            linc = true;
        }
        if (lookup_fail) atomicOr(args.err, 16);

        if (spill) {
            // ---- on to the second level: the record is rewritten in place
            __syncthreads();
            if (tid == 0) S.cnt = 0;
            __syncthreads();
            int32_t *J = rec + RHDR, *I = J + q, *R = I + m;
            if (tid < q) J[tid] = S.Jl[tid];
            if (tid < m) {
                I[tid] = S.Il[tid];
                if (S.rfl[tid]) R[atomicAdd(&S.cnt, 1)] = S.Il[tid];
            }
            __syncthreads();
            const int nR = S.cnt + (kR ? 1 : 0);
            if (tid == 0 && kR) R[S.cnt] = k;
            if (tid < nRh) R[nR + tid] = S.Rh[tid];
            if (tid == 0) {
                rec[3] = l;
                rec[4] = q;
                rec[5] = m;
                rec[6] = nR;
                rec[7] = nRh;
                const long long fb = __double_as_longlong(fl);
                rec[8] = (int32_t)(fb & 0xffffffffLL);
                rec[9] = (int32_t)(fb >> 32);
                rec[10] = linc ? 1 : 0;
                args.next_list[atomicAdd(args.next_count, 1)] = (int32_t)pos;
            }
            __syncthreads();
            continue;
        }

        // ---------------------------------------------------------- output (rows ascending)
        const int qq = (status == ST_OK) ? q : 0;
        const int64_t slot = args.arena_base + pos * BQMAX_BIG;  // one slot per record
        if (tid < qq) {
            const int jc = S.Jl[tid];
            int rank = 0;
            for (int t = 0; t < qq; ++t) rank += (S.Jl[t] < jc) ? 1 : 0;
            args.out.arenaJ[slot + rank] = jc;
            args.out.arenaV[slot + rank] = S.mt[tid];
        }
        if (tid == 0) {
            args.out.off[ucol] = slot;
            args.out.nJ[ucol] = qq;
            args.out.nI[ucol] = m;
            args.out.loops[ucol] = l;
            args.out.status[ucol] = status;
            args.out.resnorm[ucol] = rn;
            args.out.flops[ucol] = fl;
        }
        if (args.out.fac != nullptr) {
            // R of the final solve (R^T R = A(I,J)^T A(I,J))
            if (tid == 0) {
                const long long fo = (qq > 0) ? fac_reserve(args.out, qq) : -1LL;
                args.out.foff[ucol] = fo;
                S.cnt = (int)(fo & 0xffffffffLL);
                S.misc = (int)(fo >> 32);
            }
            __syncthreads();
            const long long fo = ((long long)S.misc << 32) | (long long)(unsigned)S.cnt;
            if (fo >= 0) {
                double *F = args.out.fac + fo;
                if (tid < qq) F[tid] = (double)S.Jl[tid];
                for (int t = tid; t < qq * qq; t += NT) {
                    const int i = t / qq, c = t % qq;
                    if (c >= i) F[fac_row(qq, i) + (c - i)] = (c == i) ? S.rd[i] : S.R[rcol(c) + i];
                }
            }
        }
        __syncthreads();
    }
}

int dense_blocks_per_cu() { return 4; }

void launch_dense_kernel(const DenseArgs &a, int blocks, hipStream_t s) {
    hipLaunchKernelGGL(dense_kernel, dim3(blocks), dim3(NT), 0, s, a);
}

}  // namespace rsai
