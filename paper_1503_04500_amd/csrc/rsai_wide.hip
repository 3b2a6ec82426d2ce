// Sparse-block size class of the RSAI(tol) build: one workgroup (128 or 256 threads) per
// column, for LS blocks A(I_k, J_k) that outgrow the register tiers but are mostly
// structurally empty (long sparse columns with few rows in common, as in matrices
// with power-law column lengths). Up to 8192 rows and WIDE_QMAX columns.
//
// The LS problem (2.3) is solved on an orthogonally equivalent compressed block.
// A row of I_k met by exactly one column j of J_k (a private row of j) adds to
// column j only; an orthogonal transformation of the private rows of j turns them
// into one row holding their 2-norm s_j, and the part of e_k on them into
// a_kj / s_j on that row (when k is one of them) plus a constant part
// (s_j^2 - a_kj^2) / s_j^2 of ||r||^2 that no choice of m_k can reduce. The rows
// met by two or more columns (shared rows) stay as they are. Householder QR of the
// (shared + |J_k|) x |J_k| block then gives m_k and ||A m_k - e_k||.
//
// Everything else follows the register tiers step for step (Algorithm 1 with the
// dropping of Section 4): I_k is an LDS hash set whose entries carry the number of
// columns of J_k that hold the row and a flag for rows already used as dominant
// rows; the residual for step 4 is formed from the sparse columns with the columns
// taken in ascending global order, so exact ties reach the smaller-index rule.
//
// What bounds it is the latency of a column's dependent phases at the few columns that a CU's
// LDS holds (four in level 0): a mean column has 600 entries, 17 columns of J and 3 shared
// rows, so neither bandwidth nor arithmetic is near its limit. Hence the entries of J's
// columns lie side by side over all lanes (not a wave per column), loaded once, and their
// rows' hash slots stay in registers for the sums, the drop and the residual; steps that a
// wave can do alone take no workgroup barrier; and the compressed solve eliminates the columns
// of one shared row in closed form. 400 000 power-law columns (2 to 200 entries), c = 3,
// eps = 0.4: a wave per column, every entry looked up again per phase and all columns stepped
// through, 15.6 ms in levels 0 to 3; now 9.1 ms.
//
// Columns arrive as spill records of the previous class. A column whose |I_k| or
// compressed block outgrows this class moves on to the next one.
#include <cfloat>
#include <climits>
#include <type_traits>

#include "rsai_kernels.h"

namespace rsai {

namespace {
constexpr int QM = WIDE_QMAX;
constexpr int LOGHJ = 8;                // column hash: 256 slots
constexpr int HJ = 1 << LOGHJ;

// Three instances: rows of I up to 1024 (2048-slot row hash, four workgroups per CU),
// up to 2048 (three per CU) and up to 8192 (one per CU, larger compressed blocks).
//   BLK  doubles of the compressed block, (S + q) x (q + 1), row-major
//   SHV  doubles of the shared rows' values, S x q
//   SMAX shared rows
template <int NT, int LOGH, int BLK, int SHV, int SMAX, int KE>
struct WLds {
    static constexpr int NW = NT / 64;  // waves
    static constexpr int HS = 1 << LOGH;
    int hk[HS + 1];         // row keys (one more slot for lanes without a key)
    unsigned hv[HS / 4];    // one byte per slot: bits 0-6 columns of J holding the row, bit 7 row in R
    int hJ[HJ];             // J as a set
    double blk[BLK];        // also the entries' squares while the private sums are formed
    double shv[SHV];
    double s2[64];          // private rows of each column: sum of squares
    double mt[64], rd[64];  // solution by slot, diagonal of R
    unsigned long long start[NW * KE];  // bit u: entry u of J's columns is a column's first
    int cb[64];             // first entry of each column of J (nnz < 2^31)
    int clen[64];
    int pre[65];            // entries of the columns before it, side by side in slot order
    int cbo[64];            // cb - pre
    int Jl[64];             // J, slot order
    int ord[64];            // slots in ascending column order
    int srow[SMAX];         // shared rows, ascending
    unsigned long long shm[SMAX];  // columns (slots) of J holding each shared row
    int stmp[SMAX];
    int slist[SMAX];        // rows whose holder count reached 2 since the last scan, plus
                            // the shared rows of that scan (slovf: the list overflowed)
    int newc[64];           // columns of J-hat
    int Rh[CMAX];           // pending dominant rows
    double cva[NW];
    int cvg[NW];
    double akv;             // a_kj when k is a private row of column slot kcol
    int kcol;
    int cnt, nsh, flag, nsl, slovf, nsh2, madd;
    double rn;
};

template <class L>
__device__ __forceinline__ unsigned hget(const L &S, int sl) {
    return (S.hv[sl >> 2] >> ((sl & 3) * 8)) & 0xFFu;
}
template <class L>
__device__ __forceinline__ void now_shared(L &S, int row) {
    const int ps = atomicAdd(&S.nsl, 1);
    if (ps < (int)(sizeof(S.slist) / sizeof(int))) S.slist[ps] = row; else S.slovf = 1;
}
// one more column holds the row of slot sl; a row that becomes shared (two holders)
// joins the candidate list of the next shared-row scan
template <class L>
__device__ __forceinline__ void hinc(L &S, int sl, int row) {
    const unsigned old = atomicAdd(&S.hv[sl >> 2], 1u << ((sl & 3) * 8));
    if (((old >> ((sl & 3) * 8)) & 0x7Fu) == 1u) now_shared(S, row);
}
template <class L>
__device__ __forceinline__ void hdec(L &S, int sl) { atomicSub(&S.hv[sl >> 2], 1u << ((sl & 3) * 8)); }
template <class L>
__device__ __forceinline__ void hsetR(L &S, int sl) { atomicOr(&S.hv[sl >> 2], 0x80u << ((sl & 3) * 8)); }

// The matrix's pointers and the kernel's arguments, read through pointers whose value the
// compiler cannot see: loaded where a phase uses them instead of being held in scalar
// registers across the solve.
using CMat = const __attribute__((address_space(4))) MatDev;
__device__ __forceinline__ CMat &matrix(CMat *p) {
    asm volatile("" : "+s"(p));
    return *p;
}
using CArgs = const __attribute__((address_space(4))) WideArgs;
__device__ __forceinline__ CArgs &kargs() {
    CArgs *p = (CArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *p;
}

// wave-wide sum; every lane gets the bitwise-same value
__device__ __forceinline__ double wsum(double x) { return gsum<64>(x); }

// (a desc, g asc) order of dominant-row candidates
__device__ __forceinline__ bool better(double a, int g, double b, int h) { return a > b || (a == b && g < h); }

// index of row in the ascending shared-row list, or -1
__device__ __forceinline__ int sfind(const int *srow, int nsh, int row) {
    int lo = 0, hi = nsh - 1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int v = srow[mid];
        if (v == row) return mid;
        if (v < row) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}
// inclusive prefix sum over the wave
__device__ __forceinline__ int wscan(int x, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d);
        x += lane >= d ? y : 0;
    }
    return x;
}

// Householder steps of the compressed block's columns cm by one wave: lane c holds column c's
// entries of the SU shared rows in b, the right-hand side in lane q; the diagonal of column c
// is sjl, row kc of the right-hand side rk. The reflector of step j is read from lane j.
// Lanes with upd (behind j) get their column updated and store its entry of row j. Returns
// whether a column had no norm left.
template <int SU, class L>
__device__ __forceinline__ bool steps(L &S, double (&b)[SU], unsigned long long cm, double sjl, int lane, int q, int kc,
                                      double rk, bool upd) {
    const int ld = q + 1;
    bool sing = false;
    for (unsigned long long left = cm; left; left &= left - 1ull) {
        const int j = __ffsll((long long)left) - 1;
        double u[SU];
#pragma unroll
        for (int t = 0; t < SU; ++t) u[t] = readlane_f64(b[t], j);
        const double x0 = readlane_f64(sjl, j);
        double s0 = x0 * x0, s1 = 0.0;
#pragma unroll
        for (int t = 0; t < SU; t += 2) {
            s0 += u[t] * u[t];
            s1 += u[t + 1] * u[t + 1];
        }
        double nx, be;
        hh_scalars(s0 + s1, x0, nx, be);
        const double alpha = (x0 >= 0.0) ? -nx : nx;
        const double v0 = x0 - alpha;
        if (!(nx > 0.0)) sing = true;
        if (lane > j && lane <= q && upd) {
            const double bj = (lane == q && j == kc) ? rk : 0.0;
            double w0 = v0 * bj, w1 = 0.0;
#pragma unroll
            for (int t = 0; t < SU; t += 2) {
                w0 += u[t] * b[t];
                w1 += u[t + 1] * b[t + 1];
            }
            const double w = (w0 + w1) * be;
            S.blk[j * ld + lane] = bj - w * v0;
#pragma unroll
            for (int t = 0; t < SU; ++t) b[t] -= w * u[t];
        }
        if (lane == 0) S.rd[j] = alpha;
    }
    return sing;
}
}  // namespace

template <int NT, int LOGH, int BLK, int SHV, int SMAX, int KE, int WPC>
__global__ __launch_bounds__(NT, WPC * NT / 256) void wide_kernel(WideArgs args) {
    constexpr int HS = 1 << LOGH;
    constexpr int MM = HS / 2;  // row hash load at most one half
    constexpr int KU = KE * NT;  // entries of J's columns held in registers
    constexpr int SU = 8;        // shared rows of the one-wave QR and drop
    static_assert(KU <= BLK && KE % 4 == 0 && KE <= 64 && HS <= 1 << 16, "entry registers");
    constexpr int NW = NT / 64;  // waves
    static_assert(SMAX <= NT && QM < NT, "a thread per shared row and per column");
    __shared__ WLds<NT, LOGH, BLK, SHV, SMAX, KE> S;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    if (*args.err & ERR_SKIP) return;
    const BuildParams P = args.P;
    const int64_t Q = min((int64_t)(*args.rec_in_count), args.rec_in_cap);

    for (int64_t pos = blockIdx.x; pos < Q; pos += gridDim.x) {
        const int32_t *rec = args.rec_in + pos * (int64_t)args.rec_in_stride;
        // (the record's header is the same for every lane: scalar registers)
        auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
        const int ucol = uni(rec[0]), mat = uni(rec[1]), k = uni(rec[2]);
        int l = uni(rec[3]), q = uni(rec[4]), m = uni(rec[5]);
        const int nR0 = uni(rec[6]);
        int nRh = uni(rec[7]);
        double fl = __longlong_as_double(((long long)rec[9] << 32) | (long long)(unsigned)rec[8]);
        bool linc = (uni(rec[10]) & 1) != 0;
        CMat *const Am = (CMat *)(args.mats + mat);
        const int32_t *RJ = rec + RHDR, *RI = RJ + q, *RR = RI + m, *RHp = RR + nR0;
        int status = ST_OK;
        bool spill = false, pend = false, pend_drop = false;
        int pend_qmod = -1, pend_mmod = 0;
        int blk_nsh = -1;         // shared rows when the compressed block did not fit
        bool lookup_fail = false;
        double rn = 0.0;

        // ---------------------------------------------------------- state from the record
        for (int t = tid; t < HS; t += NT) S.hk[t] = HEMPTY;
        for (int t = tid; t < HS / 4; t += NT) S.hv[t] = 0u;
        for (int t = tid; t < HJ; t += NT) S.hJ[t] = HEMPTY;
        if (tid == 0) { S.flag = 0; S.nsl = 0; S.slovf = 0; S.madd = 0; S.hk[HS] = HEMPTY; }
        __syncthreads();
        if (q > QM || m > MM || nRh > CMAX) status = ST_CAP;  // larger than any register tier
        if (status == ST_OK) {
            for (int t = tid; t < q; t += NT) {
                const int col = RJ[t];
                S.Jl[t] = col;
                S.cb[t] = (int)matrix(Am).colptr[col];
                S.clen[t] = (int)matrix(Am).colptr[col + 1] - S.cb[t];
                int sl;
                hinsert<LOGHJ>(S.hJ, col, sl);
            }
            for (int t = tid; t < m; t += NT) {
                int sl;
                hinsert<LOGH>(S.hk, RI[t], sl);
            }
            if (tid < nRh) S.Rh[tid] = RHp[tid];
        }
        __syncthreads();
        if (status == ST_OK) {
            for (int t = tid; t < nR0; t += NT) {
                const int row = RR[t];
                const int sl = hfind<LOGH>(S.hk, row);
                if (sl >= 0) hsetR(S, sl);
                else if (row == k) S.flag = 1;  // k used as a dominant row while k is not in I
            }
        }
        __syncthreads();
        bool kR = S.flag != 0;
        __syncthreads();

        // The entries of J's columns, side by side in slot order: entry u = 64 (wid + NW i) +
        // lane in this lane's registers i < KE (row, or -1; slot of the row in the hash and
        // column; value). Entries from KU on are loaded where they are used.
        int erow[KE], esc[KE];
        double ev[KE];
        int total = 0;      // entries of J's columns
        bool held = false;  // the registers hold them
        // column, row and value of entry u
        auto load = [&](int u, int &c, int &row, double &v) {
            int lo = 0, hi = q - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (S.pre[mid] <= u) lo = mid; else hi = mid - 1;
            }
            c = lo;
            const int e = S.cbo[lo] + u;
            row = matrix(Am).rowidx[e];
            v = matrix(Am).val[e];
        };

        bool first = true, need_solve = true, dropok = false;
        int qmod = -1, mmod = 0;
        int p = 0;
        if (uni(rec[10]) & 2) {
            // augmented pattern handed over before its solve
            dropok = (uni(rec[10]) & 4) != 0;
            qmod = uni(rec[11]);
            mmod = uni(rec[12]);
        }
        if (status == ST_OK && q == 0 && nRh == 0) {
            // a column whose own rows exceed the register tiers: J = {k}, loop 0
            if (tid == 0) {
                S.Jl[0] = k;
                S.cb[0] = (int)matrix(Am).colptr[k];
                S.clen[0] = (int)matrix(Am).colptr[k + 1] - S.cb[0];
                int sl;
                hinsert<LOGHJ>(S.hJ, k, sl);
            }
            __syncthreads();
            p = 1;
            dropok = true;
            qmod = 0;
        }

        while (status == ST_OK && !spill) {
            // ================= J-hat: columns of the pending dominant rows not in J (step 5)
            if (nRh > 0) {
                if (linc) ++l;  // step 6
                linc = false;
                int sb[CMAX], sp[CMAX + 1];
                sp[0] = 0;
#pragma unroll
                for (int t = 0; t < CMAX; ++t) {
                    int b0 = 0, e0 = 0;
                    if (t < nRh) {
                        const int rt = S.Rh[t];
                        b0 = (int)matrix(Am).rowptr[rt];
                        e0 = (int)matrix(Am).rowptr[rt + 1];
                    }
                    sb[t] = b0;
                    sp[t + 1] = sp[t] + (e0 - b0);
                }
                if (tid == 0) S.cnt = 0;
                __syncthreads();
                bool ovf = false;
                for (int u = tid; u < sp[CMAX]; u += NT) {
                    int at = sb[0] + u;
#pragma unroll
                    for (int t = 1; t < CMAX; ++t) at = u >= sp[t] ? sb[t] - sp[t] + u : at;
                    const int col = matrix(Am).colidx[at];
                    int sl;
                    if (hinsert<LOGHJ>(S.hJ, col, sl)) {
                        const int ps = atomicAdd(&S.cnt, 1);
                        if (q + ps < QM) S.newc[ps] = col; else ovf = true;
                    } else if (sl < 0) {
                        ovf = true;  // table full
                    }
                }
                if (__syncthreads_or(ovf)) { spill = true; break; }
                p = uni(S.cnt);
                if (tid < p) {
                    const int key = S.newc[tid];
                    const int b0 = (int)matrix(Am).colptr[key], b1 = (int)matrix(Am).colptr[key + 1];
                    int rank = 0;
                    for (int t = 0; t < p; ++t) rank += (S.newc[t] < key) ? 1 : 0;
                    S.Jl[q + rank] = key;
                    S.cb[q + rank] = b0;
                    S.clen[q + rank] = b1 - b0;
                }
                need_solve = !(p == 0 && !first);  // empty J-hat: the loop ends without a solve
                dropok = (p > 0);
                qmod = (p > 0) ? q : (first ? -1 : q);
                mmod = m;
                __syncthreads();
            }
            // ================= I-hat: rows of the new columns not in I (step 5)
            if (need_solve && (p > 0 || first)) {
                const int qa = q + p;
                // prefix of the columns' lengths (each wave forms it, and the same words)
                const int lenl = lane < qa ? S.clen[lane] : 0;
                const int incl = wscan(lenl, lane), exl = incl - lenl;
                total = __builtin_amdgcn_readlane(incl, 63);
                if (m + total - __builtin_amdgcn_readlane(exl, q) > MM) { spill = true; break; }  // may outgrow the row hash
                if (lane < KE) S.start[wid + NW * lane] = 0ull;
                if (lane < qa) {
                    S.pre[lane] = exl;
                    S.cbo[lane] = S.cb[lane] - exl;
                }
                if (lane == 0) S.pre[qa] = total;
                wave_sync();
                // (a wave's entries: its own words)
                if (lane < qa && exl < KU && ((exl >> 6) & (NW - 1)) == wid)
                    atomicOr(&S.start[exl >> 6], 1ull << (exl & 63));
                wave_sync();
#pragma unroll
                for (int i = 0; i < KE; ++i) {
                    const int w = wid + NW * i, u = 64 * w + lane;
                    const bool in = u < total;
                    // columns that start up to entry u
                    const int c0 = __popcll(__ballot(lane < qa && exl < 64 * w)) - 1;
                    const int c = in ? c0 + __popcll(S.start[w] & ((2ull << lane) - 1ull)) : 0;
                    const int e = in ? S.cbo[c] + u : 0;
                    const int row = matrix(Am).rowidx[e];
                    ev[i] = matrix(Am).val[e];
                    erow[i] = in ? row : -1;
                    esc[i] = c << 16;
                }
                // rows into I; one more holder for the rows of the columns not counted yet
                const int cinc = first ? 0 : q;
                int added = 0;
#pragma unroll
                for (int b = 0; b < KE; b += 4) {
                    int key[4];
                    unsigned sl[4], od[4];
                    bool fresh[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) key[t] = erow[b + t];
                    hinsert_many<LOGH, 4>(S.hk, key, sl, fresh);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        od[t] = 0u;
                        const int sh = (int)(sl[t] & 3u) * 8;
                        if (key[t] >= 0 && (esc[b + t] >> 16) >= cinc)
                            od[t] = (atomicAdd(&S.hv[sl[t] >> 2], 1u << sh) >> sh) & 0x7Fu;
                        added += __popcll(__ballot(fresh[t]));
                        esc[b + t] |= (int)(sl[t] & 0xFFFFu);
                    }
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (od[t] == 1u) now_shared(S, key[t]);
                }
                q = qa;  // (load() searches all of J)
                for (int u = KU + tid; u < total; u += NT) {
                    int c, row, sl;
                    double v;
                    load(u, c, row, v);
                    added += __popcll(__ballot(hinsert<LOGH>(S.hk, row, sl)));
                    if (sl < 0) lookup_fail = true;
                    else if (c >= cinc) hinc(S, sl, row);
                }
                if (lane == 0 && added) atomicAdd(&S.madd, added);
                __syncthreads();
                m += uni(S.madd);
                if (kR) {
                    // k entered I: its flag moves into the hash entry
                    const int sl = hfind<LOGH>(S.hk, k);
                    if (sl >= 0) {
                        if (tid == 0) hsetR(S, sl);
                        kR = false;
                    }
                }
                held = total <= KU;
                p = 0;
            }
            nRh = 0;  // pending rows consumed
            first = false;

            // ================= LS solve(s) on (I, J) (2.3): pass 0 the augmented pattern,
            // pass 1 the pattern kept after dropping (Section 4)
            // (after a drop, the drop step leaves the kept columns' compressed data in
            // LDS: shared rows, their values, private sums and the row of k; the re-solve
            // forms its block from them instead of gathering every column again)
            bool reuse_next = false;
            for (int pass = 0; pass < 2 && need_solve && status == ST_OK; ++pass) {
                const bool reuse = reuse_next;
                reuse_next = false;
                // ---- shared rows (held by two or more columns of J), ascending: every row with
                // two or more holders is in the candidate list (it was shared at the last scan
                // or reached two holders since), unless that overflowed
                int nsh;
                if (reuse) {
                    nsh = uni(S.nsh);
                } else {
                    const int nl = uni(S.nsl);
                    const bool slovf = S.slovf != 0;
                    if (nl <= 64 && !slovf) {
                        // each wave forms the same list
                        const int key = lane < nl ? S.slist[lane] : 0;
                        bool sh = false;
                        if (lane < nl) {
                            const int sl = hfind<LOGH>(S.hk, key);
                            sh = sl >= 0 && (hget(S, sl) & 0x7Fu) >= 2u;
                        }
                        const unsigned long long bal = __ballot(sh);
                        nsh = __popcll(bal);
                        int rank = 0;
                        for (unsigned long long b = bal; b; b &= b - 1ull)
                            rank += __builtin_amdgcn_readlane(key, __ffsll((long long)b) - 1) < key ? 1 : 0;
                        if (wid == 0 && sh && rank < SMAX) S.srow[rank] = key;
                    } else {
                        if (tid == 0) S.nsh = 0;
                        __syncthreads();
                        const int nt = slovf ? HS : nl;
                        for (int t = tid; t < nt; t += NT) {
                            const int key = slovf ? S.hk[t] : S.slist[t];
                            const int sl = slovf ? (key != HEMPTY ? t : -1) : hfind<LOGH>(S.hk, key);
                            if (sl >= 0 && (hget(S, sl) & 0x7Fu) >= 2u) {
                                const int ps = atomicAdd(&S.nsh, 1);
                                if (ps < SMAX) S.stmp[ps] = key;
                            }
                        }
                        __syncthreads();
                        nsh = uni(S.nsh);
                        if (nsh <= SMAX && tid < nsh) {
                            const int key = S.stmp[tid];
                            int rank = 0;
                            for (int t = 0; t < nsh; ++t) rank += (S.stmp[t] < key) ? 1 : 0;
                            S.srow[rank] = key;
                        }
                    }
                }
                const int ld = q + 1, mp = nsh + q;
                if (nsh > SMAX || nsh * q > SHV || mp * ld > BLK) {
                    // the compressed block does not fit: hand the unsolved pattern over
                    spill = true;
                    blk_nsh = nsh;
                    pend = true;
                    pend_drop = dropok && pass == 0;
                    pend_qmod = qmod;
                    pend_mmod = mmod;
                    break;
                }
                if (!reuse) {
                    for (int t = tid; t < nsh * q; t += NT) S.shv[t] = 0.0;
                    for (int t = tid; t < nsh; t += NT) S.shm[t] = 0ull;
                    if (tid == 0) { S.kcol = -1; S.akv = 0.0; }
                    __syncthreads();
                    // (every wave has read the list and the counts)
                    if (tid < nsh && S.slovf == 0) S.slist[tid] = S.srow[tid];  // no row enters it twice
                    if (tid == 0) {
                        if (S.slovf == 0) S.nsl = nsh;
                        S.nsh = nsh;
                        S.flag = 0;
                        S.madd = 0;
                    }
                    // ---- gather: shared entries' values; private entries' squares, summed
                    // per column (8 lanes each, in the entries' order)
                    auto visit = [&](int u, int c, int row, int sl, double v) {
                        const unsigned cn = sl >= 0 ? (hget(S, sl) & 0x7Fu) : 0u;
                        double a2 = 0.0;
                        if (cn == 1u) {
                            a2 = v * v;
                            if (row == k) { S.kcol = c; S.akv = v; }
                        } else if (cn >= 2u) {
                            const int si = sfind(S.srow, nsh, row);
                            if (si >= 0) {
                                S.shv[si * q + c] = v;
                                atomicOr(&S.shm[si], 1ull << c);
                            } else {
                                lookup_fail = true;
                            }
                        } else {
                            lookup_fail = true;
                        }
                        S.blk[u] = a2;
                    };
#pragma unroll
                    for (int i = 0; i < KE; ++i)
                        if (erow[i] >= 0)
                            visit(64 * (wid + NW * i) + lane, esc[i] >> 16, erow[i], esc[i] & 0xFFFF, ev[i]);
                    for (int base = 0;;) {
                        __syncthreads();
                        for (int c = tid >> 3; c < q; c += NT / 8) {
                            const int lo = max(S.pre[c], base), hi = min(S.pre[c + 1], base + KU);
                            double x = 0.0;
                            for (int u = lo + (tid & 7); u < hi; u += 8) x += S.blk[u - base];
                            x = gsum<8>(x);
                            if ((tid & 7) == 0) S.s2[c] = (base ? S.s2[c] : 0.0) + x;
                        }
                        __syncthreads();
                        base += KU;
                        if (base >= total) break;
                        // the next KU entries, loaded again
                        for (int u = base + tid; u < min(total, base + KU); u += NT) {
                            int c, row;
                            double v;
                            load(u, c, row, v);
                            visit(u - base, c, row, hfind<LOGH>(S.hk, row), v);
                        }
                    }
                }
                // ---- the row of row k: shared (right-hand side 1), private (compressed), or
                // outside the pattern (a constant 1 in ||r||^2). Private in column j: the
                // collapsed row carries beta = a_kj / s_j and ||r||^2 gains 1 - beta^2.
                const int ksl = uni(hfind<LOGH>(S.hk, k));
                const int kcn = ksl >= 0 ? uni((int)(hget(S, ksl) & 0x7Fu)) : -1;
                double kconst = (kcn <= 0) ? 1.0 : 0.0;
                if (kcn == 1 && S.kcol >= 0) {
                    const double sk = sqrt(S.s2[S.kcol]);
                    const double bk = sk > 0.0 ? S.akv / sk : 0.0;
                    kconst = fmax(0.0, 1.0 - bk * bk);
                }
                // the collapsed row's right-hand side, and the shared row of k
                double rk = 0.0;
                if (kcn == 1 && S.kcol >= 0) {
                    const double sj = sqrt(S.s2[S.kcol]);
                    if (sj > 0.0) rk = S.akv / sj;
                }
                const int kc = (kcn == 1) ? uni(S.kcol) : -1;
                const int ksi = (kcn >= 2) ? uni(sfind(S.srow, nsh, k)) : -1;
                if (nsh > SU) {
                    // rows 0..q-1: the collapsed private rows (diagonal), rows q..q+S-1: shared
                    for (int t = tid; t < q * ld; t += NT) {
                        const int i = t / ld, c = t - i * ld;
                        S.blk[t] = i == c ? sqrt(S.s2[c]) : (c == q && i == kc) ? rk : 0.0;
                    }
                    for (int t = tid; t < nsh * ld; t += NT) {
                        const int si = t / ld, c = t - si * ld;
                        S.blk[q * ld + t] = c < q ? S.shv[si * q + c] : si == ksi ? 1.0 : 0.0;
                    }
                    __syncthreads();
                }
                // ---- Householder QR of the compressed block and Q^T e (wave 0: lane c
                // holds column c, lane q the right-hand side). Column j has nonzeros only
                // in row j and the shared rows (the reflectors of earlier columns touch
                // exactly those rows), so each reflector has 1 + S entries.
                if (wid == 0) {
                    bool singular = false;
                    // back substitution over the columns cm: lane i holds (Q^T e)_i; m_j
                    // broadcast by readlane (the divisions by the diagonal prepared
                    // beforehand, a lane each; the next column's entries loaded ahead)
                    auto back_substitute = [&](unsigned long long left) {
                        const bool in = (left >> lane) & 1ull;
                        double y = in ? S.blk[lane * ld + q] : 0.0;
                        const double rdl = in ? S.rd[lane] : 1.0;
                        const double ril = 1.0 / rdl;
                        double mine = 0.0;
                        auto rcol = [&](int j) { return (in && lane < j) ? S.blk[lane * ld + j] : 0.0; };
                        int j = left ? 63 - __clzll((long long)left) : 0;
                        double rj = left ? rcol(j) : 0.0;
                        while (left) {
                            left ^= 1ull << j;
                            const int jn = left ? 63 - __clzll((long long)left) : 0;
                            const double rjn = left ? rcol(jn) : 0.0;
                            const double mj =
                                div_by(readlane_f64(y, j), readlane_f64(rdl, j), readlane_f64(ril, j));
                            if (lane == j) mine = mj;
                            y -= rj * mj;
                            j = jn;
                            rj = rjn;
                        }
                        return mine;
                    };
                    // columns that take a step of the two loops below
                    unsigned long long cm = (1ull << q) - 1ull;
                    // Few shared rows: lane c keeps the shared-row entries of column c in
                    // registers; the reflector of step j is read from lane j. Row j of
                    // column c > j is zero before step j, except the right-hand side of
                    // the collapsed row of the column where k is private. SU slots: 4 when
                    // the column set has at most 4 shared rows (the common case), else 8.
                    // The slots past nsh hold zeros, but the two instances fuse their
                    // sums of products differently, so their results agree only to
                    // rounding level, not bit for bit.
                    //
                    // The columns of J-hat are those of a few dominant rows, so most meet the
                    // others in one shared row only. The columns c with one entry b_c in the
                    // shared rows, all in row t, are eliminated together, before the others:
                    // their q reflectors leave row t scaled by 1 / sqrt(T), T = 1 + sum of
                    // (b_c / s_c)^2, and given the other columns' part f of row t's right-hand
                    // side they have m_c = (b_c / s_c^2) z, z = f / T (k private in one of
                    // them: d = its right-hand side, f less d b / s, and m = (d (T - (b / s)^2)
                    // + f b / s) / (T s), T - (b / s)^2 summed without it). What is left takes
                    // the steps: 1.2k cycles each, q = 17 of them before the drop, about 3 now.
                    auto qr_regs = [&](auto ns) {
                        constexpr int SU = decltype(ns)::value;
                        double b[SU];
                        int own = -1, nown = 0;  // the last shared row of this lane's column, their number
#pragma unroll
                        for (int t = 0; t < SU; ++t) {
                            b[t] = (lane < q && t < nsh) ? S.shv[t * q + lane] : 0.0;
                            if (b[t] != 0.0) {
                                own = t;
                                ++nown;
                            }
                            if (lane == q && t == ksi) b[t] = 1.0;
                        }
                        const bool inq = lane < q;
                        const double sjl = inq ? sqrt(S.s2[lane]) : 0.0;
                        double bo = 0.0;
#pragma unroll
                        for (int t = 0; t < SU; ++t) bo = own == t ? b[t] : bo;
                        const bool alone = inq && nown <= 1 && sjl > 0.0 && sjl <= DBL_MAX &&
                                           fabs(bo) <= 1e60 * sjl;
                        cm = __ballot(inq && !alone);
                        const double ci = alone ? bo / sjl : 0.0;
                        const bool kin = kc >= 0 && !((cm >> kc) & 1ull);  // k private in one of them
                        const double ck = kin ? readlane_f64(ci, kc) : 0.0;
                        double Tl = 1.0, Tx = 1.0;  // T of this lane's row, without the column of k
#pragma unroll
                        for (int t = 0; t < SU; ++t) {
                            if (t >= nsh) continue;
                            const double x = 1.0 + wsum(own == t && lane != kc ? ci * ci : 0.0);
                            const bool kt = kin && __builtin_amdgcn_readlane(own, kc) == t;
                            const double T = kt ? x + ck * ck : x;
                            if (own == t) {
                                Tl = T;
                                Tx = x;
                            }
                            // the other columns and the right-hand side (lane q)
                            if (lane == q && kt) b[t] = -ck * rk;
                            if (!alone) b[t] *= 1.0 / sqrt(T);
                        }
                        const bool sing = steps(S, b, cm, sjl, lane, q, kc, rk, !alone);
                        // the right-hand side left in the shared rows (lane q)
                        double r2 = 0.0;
#pragma unroll
                        for (int t = 0; t < SU; ++t) r2 += b[t] * b[t];
                        r2 = readlane_f64(r2, q);
                        if (lane == 0) S.rn = sqrt(r2 + kconst);
                        wave_sync();
                        singular = sing;
                        if (sing) return;
                        double mine = back_substitute(cm);
                        if (cm != (1ull << q) - 1ull) {
                            // the others, from what those leave of their row
                            double f = 0.0;
#pragma unroll
                            for (int t = 0; t < SU; ++t) {
                                if (t >= nsh) continue;
                                const double bt = inq && !alone ? S.shv[t * q + lane] : 0.0;
                                const double x = (t == ksi ? 1.0 : 0.0) - wsum(bt * mine);
                                if (own == t) f = x;
                            }
                            if (alone) {
                                const bool kl = lane == kc;
                                const double d = kl ? rk : 0.0;
                                const double fk = (kin && !kl && own == __builtin_amdgcn_readlane(own, kc)) ? f - ck * rk : f;
                                mine = (d * Tx + ci * fk) / Tl / sjl;
                            }
                        }
                        if (inq) S.mt[lane] = mine;
                    };
                    if (nsh <= 4) {
                        qr_regs(std::integral_constant<int, 4>{});
                    } else if (nsh <= SU) {
                        qr_regs(std::integral_constant<int, SU>{});
                    } else {
                    for (int j = 0; j < q; ++j) {
                        // the reflector's entries (row j and the first shared rows) and this
                        // lane's column, loaded together
                        double u[SU], b[SU];
                        const bool act = lane > j && lane <= q;
                        const double x0 = S.blk[j * ld + j];
                        const double bj = act ? S.blk[j * ld + lane] : 0.0;
#pragma unroll
                        for (int t = 0; t < SU; ++t) {
                            u[t] = (t < nsh) ? S.blk[(q + t) * ld + j] : 0.0;
                            b[t] = (act && t < nsh) ? S.blk[(q + t) * ld + lane] : 0.0;
                        }
                        double s0 = x0 * x0, s1 = 0.0;
#pragma unroll
                        for (int t = 0; t < SU; t += 2) {
                            s0 += u[t] * u[t];
                            s1 += u[t + 1] * u[t + 1];
                        }
                        double s = s0 + s1;
                        if (nsh > SU) {
                            double r = 0.0;
                            for (int t = SU + lane; t < nsh; t += 64) {
                                const double x = S.blk[(q + t) * ld + j];
                                r += x * x;
                            }
                            s += wsum(r);
                        }
                        double nx, be;
                        hh_scalars(s, x0, nx, be);
                        const double alpha = (x0 >= 0.0) ? -nx : nx;
                        const double v0 = x0 - alpha;
                        if (!(nx > 0.0)) singular = true;
                        if (act) {
                            double w0 = v0 * bj, w1 = 0.0;
#pragma unroll
                            for (int t = 0; t < SU; t += 2) {
                                w0 += u[t] * b[t];
                                w1 += u[t + 1] * b[t + 1];
                            }
                            for (int t = SU; t < nsh; ++t) w0 += S.blk[(q + t) * ld + j] * S.blk[(q + t) * ld + lane];
                            const double w = (w0 + w1) * be;
                            S.blk[j * ld + lane] = bj - w * v0;
#pragma unroll
                            for (int t = 0; t < SU; ++t)
                                if (t < nsh) S.blk[(q + t) * ld + lane] = b[t] - w * u[t];
                            for (int t = SU; t < nsh; ++t) S.blk[(q + t) * ld + lane] -= w * S.blk[(q + t) * ld + j];
                        }
                        if (lane == 0) S.rd[j] = alpha;
                        wave_sync();
                    }
                    // the right-hand side left in the shared rows
                    double r2 = 0.0;
                    for (int t = lane; t < nsh; t += 64) {
                        const double x = S.blk[(q + t) * ld + q];
                        r2 += x * x;
                    }
                    r2 = wsum(r2);
                    if (lane == 0) S.rn = sqrt(r2 + kconst);
                    wave_sync();
                    if (!singular) {
                        const double mine = back_substitute(cm);
                        if (lane < q) S.mt[lane] = mine;
                    }
                    }
                    if (singular && lane == 0) S.flag = 1;
                }
                __syncthreads();
                if (S.flag) { status = ST_SINGULAR; break; }
                rn = S.rn;
                if (qmod >= 0) fl += solve_flops(mmod, m, qmod, q);
                // ---- dropping (Section 4), after the augment solve only
                if (pass == 0 && dropok && P.drop != DROP_NONE) {
                    const double th = (P.drop == DROP_FIXED)
                                          ? P.tol
                                          : P.eps / ((double)q * __longlong_as_double((long long)*matrix(Am).norm1_bits));
                    // kept columns as a lane mask (q <= 63: one lane per column, each wave
                    // forms the same mask); with none above the threshold, the largest |m_j|
                    // stays (the smaller column index on ties)
                    const bool inq = lane < q;
                    const double am = inq ? fabs(S.mt[lane]) : -1.0;
                    unsigned long long keepm = __ballot(inq && am > th);
                    const int nk = __popcll(keepm);
                    if (nk == 0) {
                        const int jg = inq ? S.Jl[lane] : INT_MAX;
                        double ba = am;
                        int bg = jg;
#pragma unroll
                        for (int off = 32; off >= 1; off >>= 1) {
                            const double a2 = __shfl_xor(ba, off);
                            const int g2 = __shfl_xor(bg, off);
                            if (a2 > ba || (a2 == ba && g2 < bg)) { ba = a2; bg = g2; }
                        }
                        keepm = __ballot(inq && jg == bg);
                        // (every wave has read J before the first one compacts it)
                        __syncthreads();
                    }
                    if (nk < q) {
                        // rows of the dropped columns lose one holder; the others keep their
                        // entries under their column's new slot
                        auto slot = [&](int c) { return __popcll(keepm & ((1ull << c) - 1ull)); };
#pragma unroll
                        for (int i = 0; i < KE; ++i) {
                            const int c = esc[i] >> 16;
                            if (erow[i] < 0) continue;
                            if ((keepm >> c) & 1ull) {
                                esc[i] = (esc[i] & 0xFFFF) | (slot(c) << 16);
                            } else {
                                hdec(S, esc[i] & 0xFFFF);
                                erow[i] = -1;
                            }
                        }
                        for (int u = KU + tid; u < total; u += NT) {
                            int c, row;
                            double v;
                            load(u, c, row, v);
                            if ((keepm >> c) & 1ull) continue;
                            const int sl = hfind<LOGH>(S.hk, row);
                            if (sl >= 0) hdec(S, sl); else lookup_fail = true;
                        }
                        if (nsh <= SU) {
                            // few shared rows: the first wave makes the compressed data of the
                            // kept columns (as below), lane c for column c
                            if (wid == 0) {
                                const int qn = __popcll(keepm), d = slot(lane);
                                const bool kept = inq && ((keepm >> lane) & 1ull);
                                double b[SU], acc = inq ? S.s2[lane] : 0.0, ka = 0.0;
                                int kcn2 = -1, jl = 0, cl = 0, cbv = 0;
#pragma unroll
                                for (int t = 0; t < SU; ++t) b[t] = (inq && t < nsh) ? S.shv[t * q + lane] : 0.0;
                                if (kept) {
                                    jl = S.Jl[lane];
                                    cl = S.clen[lane];
                                    cbv = S.cb[lane];
                                }
                                if (kc >= 0 && ((keepm >> kc) & 1ull)) {
                                    kcn2 = slot(kc);
                                    ka = S.akv;
                                }
#pragma unroll
                                for (int t = 0; t < SU; ++t) {
                                    if (t >= nsh) continue;
                                    const unsigned long long hm = S.shm[t] & keepm;
                                    if (hm == (1ull << lane)) acc += b[t] * b[t];
                                    if (t == ksi && __popcll(hm) == 1) {
                                        const int c = __ffsll((long long)hm) - 1;
                                        kcn2 = slot(c);
                                        ka = readlane_f64(b[t], c);
                                    }
                                }
                                for (int t = lane; t < HJ; t += 64) S.hJ[t] = HEMPTY;
                                wave_sync();
                                int ns = 0;
#pragma unroll
                                for (int t = 0; t < SU; ++t) {
                                    if (t >= nsh || __popcll(S.shm[t] & keepm) < 2) continue;
                                    if (kept) S.shv[ns * qn + d] = b[t];
                                    if (lane == 0) {
                                        const int row = S.srow[t];
                                        S.srow[ns] = row;
                                        if (S.slovf == 0) S.slist[ns] = row;
                                    }
                                    ++ns;
                                }
                                if (kept) {
                                    S.s2[d] = acc;
                                    S.Jl[d] = jl;
                                    S.cb[d] = cbv;
                                    S.clen[d] = cl;
                                    int sl;
                                    hinsert<LOGHJ>(S.hJ, jl, sl);
                                }
                                if (lane == 0) {
                                    S.kcol = kcn2;
                                    S.akv = ka;
                                    S.nsh = ns;
                                    if (S.slovf == 0) S.nsl = ns;
                                }
                            }
                            held = total <= KU;
                            q = __popcll(keepm);
                            qmod = 0;
                            reuse_next = true;
                            __syncthreads();
                            continue;  // solve on the kept pattern
                        }
                        __syncthreads();
                        // the kept columns' compressed data for the re-solve (old slots
                        // here): a shared row keeps its place among the rows still held by
                        // two or more kept columns; a row held by one kept column joins that
                        // column's private sum (after the sum it had, rows ascending); the
                        // row of k is private, shared or gone as its holders are
                        {
                            const int qo = q, nso = nsh;
                            const int qn = __popcll(keepm);
                            if (wid == 0) {
                                int base = 0;
                                for (int s0 = 0; s0 < nso; s0 += 64) {
                                    const int si = s0 + lane;
                                    const bool kr = si < nso && __popcll(S.shm[si] & keepm) >= 2;
                                    const unsigned long long bal = __ballot(kr);
                                    if (si < nso) S.stmp[si] = kr ? base + __popcll(bal & ((1ull << lane) - 1ull)) : -1;
                                    base += __popcll(bal);
                                }
                                if (lane == 0) S.nsh2 = base;
                            }
                            int kc2 = -1;
                            double ka = 0.0;
                            if (tid == 0) {
                                const int ksl2 = hfind<LOGH>(S.hk, k);
                                const unsigned kcn2 = ksl2 >= 0 ? (hget(S, ksl2) & 0x7Fu) : 0u;
                                if (kcn2 == 1u) {
                                    if (S.kcol >= 0 && ((keepm >> S.kcol) & 1ull)) {
                                        kc2 = slot(S.kcol);
                                        ka = S.akv;
                                    } else {
                                        const int si = sfind(S.srow, nso, k);
                                        if (si >= 0) {
                                            const unsigned long long hm = S.shm[si] & keepm;
                                            if (__popcll(hm) == 1) {
                                                const int c = __ffsll((long long)hm) - 1;
                                                kc2 = slot(c);
                                                ka = S.shv[si * qo + c];
                                            }
                                        }
                                    }
                                }
                            }
                            __syncthreads();
                            // kept shared values (staged in blk, free until the re-solve
                            // forms its block) and the kept columns' private sums (in rd)
                            for (int t = tid; t < nso * qo; t += NT) {
                                const int si = t / qo, c = t - si * qo;
                                const int ns = S.stmp[si];
                                if (ns >= 0 && ((keepm >> c) & 1ull)) S.blk[ns * qn + slot(c)] = S.shv[t];
                            }
                            if (tid < qo && ((keepm >> tid) & 1ull)) {
                                double acc = S.s2[tid];
                                const unsigned long long me = 1ull << tid;
                                for (int si = 0; si < nso; ++si)
                                    if ((S.shm[si] & keepm) == me) {
                                        const double v = S.shv[si * qo + tid];
                                        acc += v * v;
                                    }
                                S.rd[slot(tid)] = acc;
                            }
                            const int myrow = tid < nso ? S.srow[tid] : 0;
                            const int mynew = tid < nso ? S.stmp[tid] : -1;
                            __syncthreads();
                            const int nsn = S.nsh2;
                            if (mynew >= 0) S.srow[mynew] = myrow;
                            for (int t = tid; t < nsn * qn; t += NT) S.shv[t] = S.blk[t];
                            if (tid < qn) S.s2[tid] = S.rd[tid];
                            if (tid == 0) {
                                S.kcol = kc2;
                                S.akv = ka;
                                S.nsh = nsn;
                            }
                            __syncthreads();
                            if (S.slovf == 0) {
                                // the candidate list keeps the shared rows only
                                for (int t = tid; t < nsn; t += NT) S.slist[t] = S.srow[t];
                                if (tid == 0) S.nsl = nsn;
                            }
                        }
                        if (wid == 0) {
                            // compaction of the slots in order: lane c moves to the number of
                            // kept slots below it
                            const bool kept = inq && ((keepm >> lane) & 1ull);
                            int jl = 0, cl = 0, cbv = 0;
                            if (kept) {
                                jl = S.Jl[lane];
                                cbv = S.cb[lane];
                                cl = S.clen[lane];
                            }
                            const int d = __popcll(keepm & ((1ull << lane) - 1ull));
                            wave_sync();
                            if (kept) {
                                S.Jl[d] = jl;
                                S.cb[d] = cbv;
                                S.clen[d] = cl;
                            }
                            if (lane == 0) S.cnt = __popcll(keepm);
                        }
                        for (int t = tid; t < HJ; t += NT) S.hJ[t] = HEMPTY;
                        __syncthreads();
                        q = uni(S.cnt);
                        for (int c = tid; c < q; c += NT) {
                            int sl;
                            hinsert<LOGHJ>(S.hJ, S.Jl[c], sl);
                        }
                        qmod = 0;
                        reuse_next = true;
                        __syncthreads();
                        continue;  // solve on the kept pattern
                    }
                }
                break;
            }
            if (status != ST_OK || spill) break;
            need_solve = false;

            // ================= stop test (step 3)
            if (rn <= P.eps || l >= P.lmax) break;

            // ================= dominant rows of r = A(I,J) m - e_k (step 4)
            const int nsh = uni(S.nsh);
            if (tid < q) {
                const int jc = S.Jl[tid];
                int rank = 0;
                for (int t = 0; t < q; ++t) rank += (S.Jl[t] < jc) ? 1 : 0;
                S.ord[rank] = tid;
            }
            __syncthreads();
            double ta[CMAX];
            int tg[CMAX];
#pragma unroll
            for (int s = 0; s < CMAX; ++s) { ta[s] = -1.0; tg[s] = INT_MAX; }
            auto offer = [&](double a, int g) {
#pragma unroll
                for (int s = 0; s < CMAX; ++s) {
                    if (better(a, g, ta[s], tg[s])) {
                        const double a1 = ta[s];
                        const int g1 = tg[s];
                        ta[s] = a;
                        tg[s] = g;
                        a = a1;
                        g = g1;
                    }
                }
            };
            // shared rows: the columns in ascending global order, fused multiply-adds
            if (tid < nsh) {
                double acc = 0.0;
                for (int t = 0; t < q; ++t) {
                    const int c = S.ord[t];
                    const double a = S.shv[tid * q + c];
                    if (a != 0.0) acc = __fma_rn(a, S.mt[c], acc);
                }
                const int row = S.srow[tid];
                const double ri = acc - ((row == k) ? 1.0 : 0.0);
                const int sl = hfind<LOGH>(S.hk, row);
                if (ri != 0.0 && sl >= 0 && !(hget(S, sl) & 0x80u)) offer(fabs(ri), row);
            }
            // private rows: one product each
            auto product = [&](int c, int row, int sl, double v) {
                const unsigned hvv = sl >= 0 ? hget(S, sl) : 0u;
                if ((hvv & 0x7Fu) == 1u && !(hvv & 0x80u)) {
                    const double ri = __fma_rn(v, S.mt[c], 0.0) - ((row == k) ? 1.0 : 0.0);
                    if (ri != 0.0) offer(fabs(ri), row);
                }
            };
            if (held) {
#pragma unroll
                for (int i = 0; i < KE; ++i)
                    if (erow[i] >= 0) product(esc[i] >> 16, erow[i], esc[i] & 0xFFFF, ev[i]);
            } else {
                // more entries than the registers hold, and their columns may have moved
                const int lenl = lane < q ? S.clen[lane] : 0;
                const int incl = wscan(lenl, lane);
                if (lane < q) {
                    S.pre[lane] = incl - lenl;
                    S.cbo[lane] = S.cb[lane] - (incl - lenl);
                }
                const int tq = __builtin_amdgcn_readlane(incl, 63);
                wave_sync();
                for (int u = tid; u < tq; u += NT) {
                    int c, row;
                    double v;
                    load(u, c, row, v);
                    product(c, row, hfind<LOGH>(S.hk, row), v);
                }
            }
            // row k outside the columns of J: r(k) = -1
            if (tid == 0) {
                const int ksl = hfind<LOGH>(S.hk, k);
                if (ksl >= 0) {
                    const unsigned hvv = hget(S, ksl);
                    if ((hvv & 0x7Fu) == 0u && !(hvv & 0x80u)) offer(1.0, k);
                } else if (!kR) {
                    offer(1.0, k);
                }
            }
            int nsel = 0;
            for (int t = 0; t < P.c; ++t) {
                double a = ta[0];
                int g = tg[0];
                gargmax<16>(a, g);
#pragma unroll
                for (int off = 16; off <= 32; off <<= 1) {
                    const double a2 = __shfl_xor(a, off);
                    const int g2 = __shfl_xor(g, off);
                    if (better(a2, g2, a, g)) { a = a2; g = g2; }
                }
                if (lane == 0) { S.cva[wid] = a; S.cvg[wid] = g; }
                __syncthreads();
                a = S.cva[0];
                g = S.cvg[0];
#pragma unroll
                for (int w = 1; w < NW; ++w)
                    if (better(S.cva[w], S.cvg[w], a, g)) { a = S.cva[w]; g = S.cvg[w]; }
                __syncthreads();
                if (a < 0.0) break;
                // the holder of the winner drops it from its list
                if (tg[0] == g && ta[0] == a) {
#pragma unroll
                    for (int s = 0; s < CMAX - 1; ++s) { ta[s] = ta[s + 1]; tg[s] = tg[s + 1]; }
                    ta[CMAX - 1] = -1.0;
                    tg[CMAX - 1] = INT_MAX;
                }
                if (tid == 0) {
                    S.Rh[t] = g;
                    const int sl = hfind<LOGH>(S.hk, g);
                    if (sl >= 0) hsetR(S, sl);
                }
                if (g == k && hfind<LOGH>(S.hk, k) < 0) kR = true;
                nsel = t + 1;
            }
            __syncthreads();
            if (nsel == 0) break;  // no candidate row left: r = 0 (Section 3)
            nRh = nsel;
            linc = true;
        }
        if (lookup_fail) atomicOr(kargs().err, 16);

        if (spill) {
            // ---- hand the column over to a later class: the next one, or for a block
            // that did not fit, the first level with a larger block, or the dense class
            // when most of its rows are shared
            int32_t *qo = kargs().rec_out, *qc = kargs().rec_out_count;
            int qs = kargs().rec_out_stride;
            int64_t qcap = kargs().rec_out_cap;
            if (blk_nsh >= 0) {
                const int d = (kargs().rec_alt[1] != nullptr && 2 * blk_nsh >= m) ? 1 : (kargs().rec_alt[0] != nullptr ? 0 : -1);
                if (d >= 0) {
                    qo = kargs().rec_alt[d];
                    qc = kargs().rec_alt_count[d];
                    qs = kargs().rec_alt_stride[d];
                    qcap = kargs().rec_alt_cap[d];
                }
            }
            // (every wave has read the counters that thread 0 reuses here)
            __syncthreads();
            if (tid == 0) {
                int ps = INT_MAX;
                if (qo) ps = atomicAdd(qc, 1);
                S.cnt = ps;
                S.nsh = 0;  // R rows written
                S.flag = 0; // I rows written
            }
            __syncthreads();
            const int ps = S.cnt;
            if (qo != nullptr && (int64_t)ps < qcap) {
                int32_t *R = qo + (int64_t)ps * qs;
                int32_t *RJo = R + RHDR, *RIo = RJo + q, *RRo = RIo + m;
                for (int t = tid; t < q; t += NT) RJo[t] = S.Jl[t];
                // I (hash order; the receiver numbers its rows in ascending order) and R
                for (int t = tid; t < HS; t += NT) {
                    const int key = S.hk[t];
                    if (key != HEMPTY) {
                        RIo[atomicAdd(&S.flag, 1)] = key;
                        if (hget(S, t) & 0x80u) {
                            const int r = atomicAdd(&S.nsh, 1);
                            if (r < WIDE_RCAP) RRo[r] = key;
                        }
                    }
                }
                __syncthreads();
                int nR = S.nsh;
                if (tid == 0 && kR && nR < WIDE_RCAP) RRo[nR] = k;
                nR += kR ? 1 : 0;
                nR = min(nR, WIDE_RCAP);
                if (tid < nRh) RRo[nR + tid] = S.Rh[tid];
                if (tid == 0) {
                    R[0] = ucol; R[1] = mat; R[2] = k; R[3] = l;
                    R[4] = q; R[5] = m; R[6] = nR; R[7] = nRh;
                    const long long fb = __double_as_longlong(fl);
                    R[8] = (int32_t)(fb & 0xffffffffLL);
                    R[9] = (int32_t)(fb >> 32);
                    R[10] = (linc ? 1 : 0) | (pend ? 2 : 0) | (pend_drop ? 4 : 0);
                    R[11] = pend_qmod;
                    R[12] = pend_mmod;
                }
                __syncthreads();
                continue;
            }
            __syncthreads();  // (every wave has read its place before the output reuses the counter)
            status = ST_CAP;  // no room in the next class
            if (tid == 0 && qo != nullptr) atomicOr(kargs().err, 32);  // queue full
        }

        // ---------------------------------------------------------- output (rows ascending)
        const int qq = (status == ST_OK) ? q : 0;
        const int64_t slot = kargs().arena_base + (int64_t)ucol * 64;
        for (int c = tid; c < qq; c += NT) {
            const int jc = S.Jl[c];
            int rank = 0;
            for (int t = 0; t < qq; ++t) rank += (S.Jl[t] < jc) ? 1 : 0;
            kargs().out.arenaJ[slot + rank] = jc;
            kargs().out.arenaV[slot + rank] = S.mt[c];
        }
        if (tid == 0) {
            kargs().out.off[ucol] = slot;
            kargs().out.nJ[ucol] = qq;
            kargs().out.nI[ucol] = m;
            kargs().out.loops[ucol] = l;
            kargs().out.status[ucol] = status;
            kargs().out.resnorm[ucol] = rn;
            kargs().out.flops[ucol] = fl;
        }
        if (kargs().out.fac != nullptr) {
            // R of the final (compressed) solve: R^T R = A(I,J)^T A(I,J); rows 0..q-1 of
            // the block hold its strict upper part, rd the diagonal. With few shared rows
            // the solve left most columns' rows out (see above): every column takes its step
            // here, on the compressed data of the final pattern, and M keeps the values that it
            // has without kept factors. Once a column instead of in every solve: a build of
            // 100 000 power-law columns with kept factors 5.90 -> 5.46 ms (5.07 without).
            if (qq > 0 && wid == 0 && S.nsh <= SU) {
                const int nsh = S.nsh;
                double b[SU];
#pragma unroll
                for (int t = 0; t < SU; ++t) b[t] = (lane < qq && t < nsh) ? S.shv[t * qq + lane] : 0.0;
                steps(S, b, (1ull << qq) - 1ull, lane < qq ? sqrt(S.s2[lane]) : 0.0, lane, qq, -1, 0.0, lane < qq);
            }
            __syncthreads();
            if (tid == 0) {
                const long long fo = (qq > 0) ? fac_reserve(kargs().out, qq) : -1LL;
                kargs().out.foff[ucol] = fo;
                S.cnt = (int)(fo & 0xffffffffLL);
                S.nsh = (int)(fo >> 32);
            }
            __syncthreads();
            const long long fo = ((long long)S.nsh << 32) | (long long)(unsigned)S.cnt;
            if (fo >= 0) {
                double *F = kargs().out.fac + fo;
                const int ld = qq + 1;
                for (int c = tid; c < qq; c += NT) F[c] = (double)S.Jl[c];
                for (int t = tid; t < qq * qq; t += NT) {
                    const int i = t / qq, c = t % qq;
                    if (c >= i) F[fac_row(qq, i) + (c - i)] = (c == i) ? S.rd[i] : S.blk[i * ld + c];
                }
            }
        }
        __syncthreads();
    }
}

namespace {
// Level 2 takes level 0's columns whose compressed block does not fit (many shared
// rows, as in the columns that pick a relatively dense row) at two workgroups per CU
// instead of sending them to the one-per-CU level 3.
// Threads: two waves in level 0, whose columns have about 600 entries (256 registers a lane
// against 128 and scratch spills with four waves: a build of 400 000 columns 16.8 against
// 17.1 ms); four in level 1, with 1024 to 2048 entries (16.8 against 17.4 ms with two).
constexpr int kWideLogH[WIDE_LEVELS] = {11, 12, 11, 14};
constexpr int kWideNT[WIDE_LEVELS] = {128, 256, 256, 256};
constexpr int kWidePerCU[WIDE_LEVELS] = {4, 3, 2, 1};
// KE: the registers hold as many entries as the level's rows, up to 4096
#define RSAI_WIDE(L, BLK, SHV, SMAX, KE) kWideNT[L], kWideLogH[L], BLK, SHV, SMAX, KE / kWideNT[L], kWidePerCU[L]
#define RSAI_WIDE0 RSAI_WIDE(0, 2048, 768, 128, 1024)
#define RSAI_WIDE1 RSAI_WIDE(1, 2048, 768, 128, 2048)
#define RSAI_WIDE2 RSAI_WIDE(2, 4096, 1536, 128, 2048)
#define RSAI_WIDE3 RSAI_WIDE(3, 6144, 1536, 256, 4096)
}  // namespace

int wide_max_rows(int level) { return (1 << kWideLogH[level]) / 2; }
int wide_rec_stride(int level) { return RHDR + 64 + wide_max_rows(level) + WIDE_RCAP + CMAX; }
int wide_queue_stride(int queue) {
    // rows of the largest record a writer of the queue can hand over
    static const int writer_level[WIDE_LEVELS] = {0, 0, 1, 3};
    return wide_rec_stride(writer_level[queue]);
}
int wide_blocks_per_cu(int level) { return kWidePerCU[level]; }

void launch_wide_kernel(int level, const WideArgs &a, int blocks, hipStream_t s) {
    const dim3 nt(kWideNT[level]);
    if (level == 0)
        hipLaunchKernelGGL((wide_kernel<RSAI_WIDE0>), dim3(blocks), nt, 0, s, a);
    else if (level == 1)
        hipLaunchKernelGGL((wide_kernel<RSAI_WIDE1>), dim3(blocks), nt, 0, s, a);
    else if (level == 2)
        hipLaunchKernelGGL((wide_kernel<RSAI_WIDE2>), dim3(blocks), nt, 0, s, a);
    else
        hipLaunchKernelGGL((wide_kernel<RSAI_WIDE3>), dim3(blocks), nt, 0, s, a);
}

}  // namespace rsai
