// Fused, size-tiered RSAI(tol) kernel: the whole loop of Algorithm 1 (Section 3)
// with the dropping of Section 4, for every column of one or more matrices.
// Included by the files that instantiate it for the size tiers (each tier's file is
// compiled with the unrolling it needs).
#pragma once
#include <climits>
#include <type_traits>

#include "rsai_kernels.h"
#include "rsai_tier.h"

namespace rsai {


// The kernel's argument block in the kernarg segment, read through a pointer whose
// value the compiler cannot see: the fields the column loop needs only now and then
// (refill, spill, output) are loaded where they are used instead of being held in
// scalar registers across the loop.
__device__ __forceinline__ const __attribute__((address_space(4))) TierArgs *kargs() {
    const __attribute__((address_space(4))) TierArgs *p =
        (const __attribute__((address_space(4))) TierArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}

// MULTI = false: one matrix, whose pointers stay in scalar registers.
template <class C, bool MULTI>
__global__ __launch_bounds__(64, C::WPS) void tier_kernel(TierArgs args) {
    constexpr int G = C::G, RPL = C::RPL, QMAX = C::QMAX, MMAX = C::MMAX, GPW = C::GPW;
    constexpr int STAGE = C::STAGE;
    // columns per chunk of the QR update: the small first tier keeps one (a chunk may
    // reach past the wave's last column, which costs more there than the interleaving
    // saves)
    constexpr int QCB = QMAX <= 12 ? 1 : 4;
    constexpr int NRI = (C::RIN + G - 1) / G;   // per-lane candidates per I round
    constexpr int NRJ = (C::RJN + G - 1) / G;   // per-lane candidates per J round
    constexpr int NNEW = (C::NEWC + G - 1) / G;

    __shared__ GLds<C> lds[GPW];
    __shared__ FacChunk fch;
    const int lane = threadIdx.x;
    const int gl = lane % G;
    const int grp = lane / G;
    GLds<C> &S = lds[grp];
    const BuildParams P = args.P;
    if (*args.err & ERR_SKIP) return;  // the CSC contract failed: process nothing
    fac_chunk_init(fch);

    // ---- static, XCD-aware schedule: each of the 8 XCDs takes a contiguous range
    const bool first_tier = (args.rec_in == nullptr);
    const int64_t Q = first_tier ? args.qlen : min((int64_t)(*args.rec_in_count), args.rec_in_cap);
    const int nblk = gridDim.x;
    const int xcd = blockIdx.x % 8;
    const int widx = blockIdx.x / 8;
    const int nw = (nblk - xcd + 7) / 8;
    const int64_t chunk = (Q + 7) / 8;
    const int64_t qlo_range = (int64_t)xcd * chunk;
    const int64_t qhi_range = min(Q, qlo_range + chunk);
    const int64_t gstride = (int64_t)nw * GPW;
    int64_t u_next = qlo_range + (int64_t)widx * GPW + grp;

    // ---- per-group state (uniform inside a group)
    S.hI[C::HSI] = HEMPTY;  // (what an absent key probes)
    S.hJ[C::HSJ] = HEMPTY;
    bool busy = false, fin = false;
    int64_t pos = 0;          // position in this launch's queue
    int64_t ucol = 0;         // global column id
    int mat = 0, k = 0;
    int q = 0, m = 0, l = 0, p = 0, qlo = 0;
    int qmod = 0;             // kept columns for the flop model of the next solve
    int mmod = 0;             // rows the kept factor of that model was formed on
    int kidx = -1;            // local row of k in I, or -1
    bool kR = false;          // k used as a dominant row while k is not in I
    int nRh = 0;
    bool solve = false, dropok = false, linc = true;
    bool park = false;        // plain schedule: write the state out after this loop
    int status = ST_OK;
    double rn = 0.0, fl = 0.0;
    // (a group without a column still loads: element 0 of the first matrix's arrays)
    MatDev A = args.mats[0];
    // ---- per-lane block rows
    double b[RPL][QMAX];
    double y[RPL];
    double rd[RPL], bt[RPL];  // R(i,i) and beta_i of the reflectors of this lane's rows
    unsigned rflag = 0u;      // bit r: local row r*G+gl is in R (used dominant rows)

#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        y[r] = 0.0;
        rd[r] = 1.0;
        bt[r] = 0.0;
#pragma unroll
        for (int c = 0; c < QMAX; ++c) b[r][c] = 0.0;
    }

    while (true) {
        // ============================================================ A. refill
        bool start = false;
        // with sync_refill, groups of a wave start their columns together, so they
        // stay at the same loop and the wave's QR is only as wide as its work
        const bool may_refill = kargs()->sync_refill ? wave_all(!busy) : true;
        if (!busy && !fin && may_refill) {
            if (u_next < qhi_range) {
                pos = u_next;
                u_next += gstride;
                start = true;
            } else {
                fin = true;
            }
        }
        if (wave_all(fin)) break;

        const int32_t *rec = nullptr;
        if (start) {
            if (first_tier) {
                ucol = pos;
                if constexpr (MULTI) {
                    int lo = 0, hi = kargs()->nmat - 1;  // matrix with col_base[mat] <= ucol
                    while (lo < hi) {
                        int mid = (lo + hi + 1) / 2;
                        if (kargs()->col_base[mid] <= ucol) lo = mid; else hi = mid - 1;
                    }
                    mat = lo;
                    k = (int)(ucol - kargs()->col_base[mat]);
                } else {
                    mat = 0;
                    k = (int)ucol;
                }
            } else {
                rec = kargs()->rec_in + pos * (int64_t)kargs()->rec_in_stride;
                ucol = rec[0];
                mat = rec[1];
                k = rec[2];
            }
            if constexpr (MULTI) A = kargs()->mats[mat];
            busy = true;
            status = ST_OK;
            fl = 0.0;
            kR = false;
            kidx = -1;
            rn = 0.0;
            rflag = 0u;
            nRh = 0;
            for (int t = gl; t < C::HSI; t += G) S.hI[t] = HEMPTY;
            for (int t = gl; t < C::HSJ; t += G) S.hJ[t] = HEMPTY;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                y[r] = 0.0;
#pragma unroll
                for (int c = 0; c < QMAX; ++c) b[r][c] = 0.0;
            }
        }
        wave_sync();
        bool resumed = false;
        if (start) {
            int rq = 0, rm = 0, rl = 0, rnR = 0, rnRh = 0;
            if (rec) { rl = rec[3]; rq = rec[4]; rm = rec[5]; rnR = rec[6]; rnRh = rec[7]; }
            if (rq == 0 && rnRh == 0) {
                // fresh column: J = {k}, pending; I from column k (Algorithm 1, steps 1-2)
                q = 0; m = 0; l = 0; p = 1; qlo = 0; qmod = 0;
                solve = true; dropok = true; linc = true;
                if (gl == 0) {
                    S.Jlist[0] = k;
                    int sl;
                    hinsert<C::LOGHSJ>(S.hJ, k, sl);
                }
            } else {
                resumed = true;
                q = rq; m = rm; l = rl; p = 0; qlo = 0;
                linc = (rec[10] & 1) != 0;
                fl = __longlong_as_double(((long long)rec[9] << 32) | (long long)(unsigned)rec[8]);
                const int32_t *RJ = rec + RHDR;
                const int32_t *RI = RJ + rq;
                for (int t = gl; t < rq; t += G) {
                    int col = RJ[t];
                    S.Jlist[t] = col;
                    const int b0 = (int)A.colptr[col];
                    S.cb[t] = b0;
                    S.cl[t] = (int)A.colptr[col + 1] - b0;
                    int sl;
                    hinsert<C::LOGHSJ>(S.hJ, col, sl);
                }
                for (int t = gl; t < rm; t += G) {
                    int row = RI[t];
                    S.Ilist[t] = row;
                    int sl;
                    hinsert<C::LOGHSI>(S.hI, row, sl);
                    if (sl >= 0) S.hIv[sl] = t;
                    if (row == k) kidx = t;
                }
                kidx = gmax_i<G>(kidx);
                nRh = rnRh;
                for (int t = gl; t < rnRh; t += G) S.Rh[t] = RI[rm + rnR + t];
            }
        }
        wave_sync();
        if (resumed) {
            // rows of R (the dominant rows used so far) -> flags of their local rows
            const int32_t *RR = rec + RHDR + q + m;
            const int nR = rec[6];
            for (int t = 0; t < nR; ++t) {
                int row = RR[t];
                int sl = hfind<C::LOGHSI>(S.hI, row);
                int li = sl >= 0 ? S.hIv[sl] : -1;
                if (li < 0 && row == k) kR = true;
                if (li >= 0 && (li % G) == gl) rflag |= 1u << (li / G);
            }
            // a resumed column is re-solved on its stored pattern
            solve = true;
            dropok = false;
        }
        if constexpr (C::CROW) {
            // local rows of the stored columns' entries
            constexpr int RB = 4;
            for (int t0 = 0; wave_any(resumed && t0 < q); t0 += RB) {
                int rw[RB];
#pragma unroll
                for (int u = 0; u < RB; ++u) {
                    rw[u] = -1;
                    if (resumed && t0 + u < q && gl < S.cl[t0 + u]) rw[u] = A.rowidx[S.cb[t0 + u] + gl];
                }
#pragma unroll
                for (int u = 0; u < RB; ++u)
                    if (rw[u] >= 0) {
                        const int sl = hfind<C::LOGHSI>(S.hI, rw[u]);
                        if (sl >= 0) S.crow[(t0 + u) * G + gl] = S.hIv[sl];
                        else atomicOr(kargs()->err, 16);
                    }
            }
        }

        // ====================================== K. J-hat from pending dominant rows
        // (Algorithm 1, step 5: columns of A(R-hat, :) not in J)
        bool spill = park;          // parked by the plain schedule: hand over as is
        int est_m = m, est_q = q;   // size estimate of a spilled column (routing)
        const bool parked = park;
        park = false;
        {
            const bool doK = busy && nRh > 0 && !spill;
            // start and prefix length of each pending row's pattern, held in registers
            // by every lane of the group (the loads are independent)
            int sb[CMAX], sp[CMAX + 1];
            sp[0] = 0;
#pragma unroll
            for (int t = 0; t < CMAX; ++t) {
                sb[t] = 0;
                sp[t + 1] = sp[t];
                if (t >= P.c) continue;  // (no column has more pending rows)
                const bool in = doK && t < nRh;
                const int rt = in ? S.Rh[t] : 0;
                const int b0 = (int)A.rowptr[rt], e0 = (int)A.rowptr[rt + 1];
                sb[t] = b0;
                sp[t + 1] = sp[t] + (in ? e0 - b0 : 0);
            }
            const int total = doK ? sp[CMAX] : 0;
            est_m = m;
            int kcnt = 0;  // new columns found
            bool ovf = false;
            for (int base = 0; wave_any(doK && !ovf && base < total); base += C::RJN) {
                int cand[NRJ];
#pragma unroll
                for (int s = 0; s < NRJ; ++s) {
                    const int uu = base + s * G + gl;
                    const bool in = doK && !ovf && uu < total && uu < base + C::RJN;
                    int at = sb[0] + uu;
#pragma unroll
                    for (int t = 1; t < CMAX; ++t) {
                        if (t >= P.c) continue;
                        at = uu >= sp[t] ? sb[t] - sp[t] + uu : at;
                    }
                    const int col = A.colidx[in ? at : 0];
                    cand[s] = in ? col : -1;
                }
                unsigned h[NRJ];
                bool isnew[NRJ];
                hinsert_many<C::LOGHSJ, NRJ>(S.hJ, cand, h, isnew);
#pragma unroll
                for (int s = 0; s < NRJ; ++s) {
                    const int ps = group_place<G>(isnew[s], lane, gl, kcnt);
                    S.newk()[(isnew[s] && ps < C::NEWC) ? ps : GLds<C>::NEWP - 1] = cand[s];
                }
                if (doK && !ovf && q + kcnt > QMAX) {
                    // |J-hat| extrapolated from the share of new columns seen so far
                    ovf = true;
                    est_q = q + (int)ceilf((float)kcnt * (float)total / (float)min(base + C::RJN, total));
                }
                wave_sync();
            }
            const int nnew = (doK && !ovf) ? kcnt : 0;
            if (nnew > 0 && gl < 4) S.newk()[nnew + gl] = INT_MAX;
            wave_sync();
            if (doK) {
                constexpr int NJ = (QMAX + G - 1) / G;
                int key[NJ], rank[NJ];
#pragma unroll
                for (int s = 0; s < NJ; ++s) key[s] = (s * G + gl < nnew) ? S.newk()[s * G + gl] : INT_MIN;
                ranks_in<NJ>(S.newk(), nnew, key, rank);
#pragma unroll
                for (int s = 0; s < NJ; ++s)
                    if (s * G + gl < nnew) S.Jlist[q + rank[s]] = key[s];
                if (linc) ++l;  // step 6
                if (ovf) {
                    spill = true;
                } else {
                    p = nnew;
                    if (linc && !resumed) {
                        // empty J-hat: the loop is consumed without a solve (step 6)
                        solve = (p > 0);
                        qlo = q;
                        qmod = q;
                        mmod = m;
                        dropok = true;
                    } else if (linc) {
                        // resumed by the plain schedule: the factor is rebuilt from the
                        // stored pattern; an empty J-hat still needs r for the next loop
                        solve = true;
                        qlo = 0;
                        dropok = (p > 0);
                        qmod = (p > 0) ? q : -1;
                        mmod = m;
                    } else {
                        // resumed column: its block is refactored from scratch here, but
                        // the method's work is the update from the stored pattern
                        solve = true;
                        qlo = 0;
                        dropok = (p > 0);
                        qmod = (p > 0) ? q : -1;
                        mmod = m;
                    }
                }
            }
            wave_sync();
        }

        // ================================ C. I-hat: rows of the new columns not in I
        {
            const bool doC = busy && !spill && p > 0;
            // pending columns the wave has at most: the unrolled batches stop there
            const int pmaxw = wave_max_i(doC ? p : 0);
            // pending columns in parallel: start and length -> LDS
            int ctot = 0;
#pragma unroll
            for (int s = 0; s < (QMAX + G - 1) / G; ++s) {
                const int t = s * G + gl;
                const bool in = doC && t < p;
                const int j = in ? S.Jlist[q + t] : 0;
                const int b0 = (int)A.colptr[j], len = (int)A.colptr[j + 1] - b0;
                S.cb[in ? q + t : GLds<C>::CP] = b0;  // kept by slot for the gathers and the residual
                S.cl[in ? q + t : GLds<C>::CP] = len;
                ctot += in ? len : 0;
            }
            const int total = gsum_i<G>(ctot);
            wave_sync();
            bool ovf = false;
            int ccnt = 0;   // new rows found
            int seen = 0;   // entries inserted
            // new rows of one insertion: appended to the list in lane order
            auto take = [&](int row, unsigned slot, bool fresh) {
                const int ps = group_place<G>(fresh, lane, gl, ccnt);
                // (room for one more entry past the last)
                const int at = (fresh && ps < C::NEWC) ? ps : GLds<C>::NEWP - 1;
                S.newk()[at] = row;
                S.news()[at] = (int)slot;
            };
            auto full = [&]() {
                if (doC && !ovf && m + ccnt > MMAX) {
                    // |I-hat| extrapolated from the share of new rows seen so far
                    ovf = true;
                    est_m = m + (int)ceilf((float)ccnt * (float)total / (float)min(seen, total));
                    est_q = q + p;
                }
            };
            if constexpr (C::CROW) {
                // entry gl of CBN columns at a time (the insertions of one lane's entries in
                // flight together), then the rest of the longer ones
                bool longer = false;
                auto batch = [&](auto nb, int t0) {
                    constexpr int NB = decltype(nb)::value;
                    int rw[NB];
                    unsigned h[NB];
                    bool isnew[NB];
#pragma unroll
                    for (int u = 0; u < NB; ++u) {
                        // (a slot past the last column: its length counts as 0)
                        const int c = min(q + t0 + u, GLds<C>::CP);
                        const int len = (doC && !ovf && t0 + u < p) ? S.cl[c] : 0;
                        const int row = A.rowidx[gl < len ? S.cb[c] + gl : 0];
                        rw[u] = gl < len ? row : -1;
                        longer |= len > G;
                        seen += min(len, G);
                    }
                    hinsert_many<C::LOGHSI, NB>(S.hI, rw, h, isnew);
#pragma unroll
                    for (int u = 0; u < NB; ++u) {
                        S.crow[(rw[u] >= 0 ? q + t0 + u : GLds<C>::CP) * G + gl] = (unsigned char)h[u];
                        take(rw[u], h[u], isnew[u]);
                    }
                    full();
                };
                // (a wave whose columns are all at loop 0 has one each: no batch for that)
                if (pmaxw == 1) batch(std::integral_constant<int, 1>{}, 0);
                else
                    for (int t0 = 0; wave_any(doC && !ovf && t0 < p); t0 += C::CBN)
                        batch(std::integral_constant<int, C::CBN>{}, t0);
                if (wave_any(longer && !ovf)) {
                    for (int t = 0; wave_any(longer && !ovf && t < p); ++t) {
                        const int e1 = (longer && !ovf && t < p) ? S.cl[q + t] : 0;
                        for (int e = G; wave_any(!ovf && e < e1); e += G) {
                            int rw[1];
                            unsigned h[1];
                            bool isnew[1];
                            rw[0] = (!ovf && e + gl < e1) ? A.rowidx[S.cb[q + t] + e + gl] : -1;
                            seen += (!ovf && e < e1) ? min(e1 - e, G) : 0;
                            hinsert_many<C::LOGHSI, 1>(S.hI, rw, h, isnew);
                            take(rw[0], h[0], isnew[0]);
                            full();
                        }
                    }
                }
            } else {
                // a wave per column of the build: the entries of all pending columns side by
                // side, found by their prefix
                int cpx[QMAX + 1];
                cpx[0] = 0;
#pragma unroll
                for (int t = 0; t < QMAX; ++t) cpx[t + 1] = cpx[t] + ((doC && t < p) ? S.cl[q + t] : 0);
                for (int base = 0; wave_any(doC && !ovf && base < total); base += C::RIN) {
                    int rw[NRI];
                    unsigned h[NRI];
                    bool isnew[NRI];
#pragma unroll
                    for (int s = 0; s < NRI; ++s) {
                        const int uu = base + s * G + gl;
                        rw[s] = -1;
                        if (doC && !ovf && uu < total && uu < base + C::RIN) {
                            int seg = 0, o0 = 0;
#pragma unroll
                            for (int t = 1; t < QMAX; ++t)
                                if (uu >= cpx[t]) { seg = t; o0 = cpx[t]; }
                            rw[s] = A.rowidx[S.cb[q + seg] + (uu - o0)];
                        }
                    }
                    seen = base + C::RIN;
                    hinsert_many<C::LOGHSI, NRI>(S.hI, rw, h, isnew);
#pragma unroll
                    for (int s = 0; s < NRI; ++s) take(rw[s], h[s], isnew[s]);
                    full();
                }
            }
            wave_sync();
            if (doC && ovf) spill = true;
            // ============================ D. number the new rows (ascending order)
            const int nnew = (doC && !ovf) ? ccnt : 0;
            int kpos = -1;
            if (nnew > 0 && gl < 4) S.newk()[nnew + gl] = INT_MAX;
            wave_sync();
            if (nnew > 0) {
                int key[NNEW], rank[NNEW];
#pragma unroll
                for (int s = 0; s < NNEW; ++s) key[s] = (s * G + gl < nnew) ? S.newk()[s * G + gl] : INT_MIN;
                ranks_in<NNEW>(S.newk(), nnew, key, rank);
#pragma unroll
                for (int s = 0; s < NNEW; ++s) {
                    const bool in = s * G + gl < nnew;
                    const int li = in ? m + rank[s] : MMAX;
                    const int sl = S.news()[s * G + gl];
                    S.Ilist[li] = key[s];
                    S.hIv[in ? sl : C::HSI] = (unsigned char)li;
                    kpos = (in && key[s] == k) ? li : kpos;
                }
            }
            kpos = gmax_i<G>(kpos);
            wave_sync();
            if constexpr (C::CROW) {
                // hash slots of the new columns' entries -> their local rows
                auto batch = [&](auto nb, int t0) {
                    constexpr int NB = decltype(nb)::value;
                    int sl[NB], at[NB];
#pragma unroll
                    for (int u = 0; u < NB; ++u) {
                        at[u] = ((doC && !ovf && t0 + u < p) ? q + t0 + u : GLds<C>::CP) * G + gl;
                        // (a lane without an entry there reads any slot of the table)
                        sl[u] = S.crow[at[u]] & (C::HSI - 1);
                    }
#pragma unroll
                    for (int u = 0; u < NB; ++u) sl[u] = S.hIv[sl[u]];
#pragma unroll
                    for (int u = 0; u < NB; ++u) S.crow[at[u]] = (unsigned char)sl[u];
                };
                if (pmaxw == 1) batch(std::integral_constant<int, 1>{}, 0);
                else
                    for (int t0 = 0; wave_any(doC && !ovf && t0 < p); t0 += C::CBN)
                        batch(std::integral_constant<int, C::CBN>{}, t0);
            }
            if (doC && !ovf) {
                if (kpos >= 0) {
                    kidx = kpos;
                    if (kR) {
                        if ((kpos % G) == gl) rflag |= 1u << (kpos / G);
                        kR = false;
                    }
                }
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    int i = r * G + gl;
                    if (i >= m && i < m + nnew) {
                        y[r] = (i == kidx) ? 1.0 : 0.0;
                    }
                }
                m += nnew;
            }
        }

        // ================================================ spill to the next tier
        if (wave_any(spill)) {
            int ps = 0;
            // destination class: the first whose limits hold the estimate
            int d = kargs()->nq - 1;
#pragma unroll
            for (int i = TierArgs::MAXQ - 2; i >= 0; --i)
                if (i < kargs()->nq - 1 && est_m <= kargs()->q_mmax[i] && est_q <= kargs()->q_qmax[i]) d = i;
            int32_t *qrec = kargs()->q_rec[0];
            int qstr = kargs()->q_stride[0];
            int64_t qcap = kargs()->q_cap[0];
            if (spill && gl == 0) ps = INT_MAX;
#pragma unroll
            for (int i = 0; i < TierArgs::MAXQ; ++i) {
                if (i > 0 && d == i) { qrec = kargs()->q_rec[i]; qstr = kargs()->q_stride[i]; qcap = kargs()->q_cap[i]; }
                // one counter address per pass, so that the lanes' increments combine
                const bool mine = spill && gl == 0 && d == i && i < kargs()->nq;
                if (wave_any(mine) && mine) ps = atomicAdd(kargs()->q_count[i], 1);
            }
            if (kargs()->nq <= 0) qrec = nullptr;
            ps = gbcast_i<G>(ps, gl == 0);
            // (the plain schedule parks every column that fits after each loop in queue
            // 0; a column that outgrew the class goes on to a later one)
            const bool ok = spill && qrec != nullptr && (int64_t)ps < qcap &&
                            (parked || !kargs()->one_loop || d > 0);
            int nR = __popc(rflag);
            nR = gsum_i<G>(nR) + (kR ? 1 : 0);
            if (spill && gl == 0) S.cnt = 0;
            wave_sync();
            if (ok) {
                int32_t *R = qrec + (int64_t)ps * qstr;
                if (gl == 0) {
                    R[0] = (int32_t)ucol; R[1] = mat; R[2] = k; R[3] = l;
                    R[4] = q; R[5] = m; R[6] = nR; R[7] = nRh;
                    const long long fb = __double_as_longlong(fl);
                    R[8] = (int32_t)(fb & 0xffffffffLL);
                    R[9] = (int32_t)(fb >> 32);
                    R[10] = parked ? 1 : 0;
                }
                for (int t = gl; t < q; t += G) R[RHDR + t] = S.Jlist[t];
                for (int t = gl; t < m; t += G) R[RHDR + q + t] = S.Ilist[t];
                int32_t *RR = R + RHDR + q + m;
#pragma unroll
                for (int r = 0; r < RPL; ++r)
                    if (rflag & (1u << r)) RR[atomicAdd(&S.cnt, 1)] = S.Ilist[r * G + gl];
                if (kR && gl == 0) RR[atomicAdd(&S.cnt, 1)] = k;
#pragma unroll
                for (int t = 0; t < CMAX; ++t)
                    if (t < nRh && gl == 0) RR[nR + t] = S.Rh[t];
            }
            if (spill && !ok) {
                // no larger tier can take the column
                status = ST_CAP;
                if (gl == 0 && qrec != nullptr && (int64_t)ps >= qcap) atomicOr(kargs()->err, 32);  // queue full
            }
            if (spill && ok) busy = false;
            wave_sync();
        }
        if (busy && !spill) nRh = 0;  // pending rows consumed

        // ============================================ LS solve(s): gather + QR
        // pass 0: the augmented pattern (or the stored pattern of a resumed column);
        // pass 1: the pattern kept after dropping (Section 4).
        bool singular = false;
        bool redo = false;
#pragma unroll 1
        for (int pass = 0; pass < 2; ++pass) {
            const bool act = busy && status == ST_OK && (pass == 0 ? solve : redo);
            if (!wave_any(act)) continue;
            const int qn = q + p;
            if (act && qlo == 0) {
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    int i = r * G + gl;
                    y[r] = (i < m && i == kidx) ? 1.0 : 0.0;
#pragma unroll
                    for (int c = 0; c < QMAX; ++c) b[r][c] = 0.0;
                }
            }
            const int qmaxw = wave_max_i(act ? qn : 0);
            // ---- gather columns [qlo, qn) of A(I, J) through LDS staging
            bool lookup_fail = false;
            for (int it = 0; wave_any(act && qlo + it * STAGE < qn); ++it) {
                const int c0 = qlo + it * STAGE;
                const bool ract = act && c0 < qn;
                const int nstage = wave_max_i(ract ? qn - c0 : 0);  // columns staged at most
                // first G entries of each staged column: all loads issued together, a lane
                // without an entry loads the first one and writes past the tile
                bool more = false;
                auto put = [&](auto nb) {
                    constexpr int NB = decltype(nb)::value;
#pragma unroll
                    for (int s = 0; s < NB; ++s)
#pragma unroll
                        for (int r = 0; r < RPL; ++r) S.stage[s * MMAX + r * G + gl] = 0.0;
                    wave_sync();
                    int ce0[NB], cln[NB], li[NB];
                    double vv[NB];
#pragma unroll
                    for (int s = 0; s < NB; ++s) {
                        const int c = min(c0 + s, GLds<C>::CP);
                        ce0[s] = S.cb[c];
                        cln[s] = (ract && c < qn) ? S.cl[c] : 0;
                        if constexpr (C::CROW) li[s] = S.crow[c * G + gl];
                    }
#pragma unroll
                    for (int s = 0; s < NB; ++s) {
                        more |= cln[s] > G;
                        const int e = gl < cln[s] ? ce0[s] + gl : 0;
                        vv[s] = A.val[e];
                        if constexpr (!C::CROW) li[s] = A.rowidx[e];
                    }
#pragma unroll
                    for (int s = 0; s < NB; ++s) {
                        if constexpr (C::CROW) {
                            S.stage[gl < cln[s] ? s * MMAX + li[s] : GLds<C>::TILE] = vv[s];
                        } else if (gl < cln[s]) {
                            const int sl = hfind<C::LOGHSI>(S.hI, li[s]);
                            const int l2 = sl >= 0 ? S.hIv[sl] : MMAX;
                            if (l2 < MMAX) S.stage[s * MMAX + l2] = vv[s];
                            else lookup_fail = true;
                        }
                    }
                };
                if (nstage == 1) put(std::integral_constant<int, 1>{});
                else put(std::integral_constant<int, STAGE>{});
                // entries beyond the first G (long columns)
                if (wave_any(more)) {
#pragma unroll 1
                    for (int s = 0; s < STAGE; ++s) {
                        const int c = c0 + s;
                        const bool in = ract && c < qn;
                        const int b0 = in ? S.cb[c] : 0, e1 = in ? b0 + S.cl[c] : 0;
                        for (int e = b0 + G + gl; e < e1; e += G) {
                            const int sl = hfind<C::LOGHSI>(S.hI, A.rowidx[e]);
                            const int l2 = sl >= 0 ? S.hIv[sl] : -1;
                            if (l2 >= 0 && l2 < MMAX) S.stage[s * MMAX + l2] = A.val[e];
                            else lookup_fail = true;
                        }
                    }
                }
                wave_sync();
                // (columns outside the wave's staged ranges are passed over; a group whose
                // range does not hold column c keeps what it has)
                const int cfirst = -wave_max_i(ract ? -c0 : -QMAX), clast = wave_max_i(ract ? c0 : -STAGE) + STAGE;
#pragma unroll
                for (int c = 0; c < QMAX; ++c) {
                    if (c < cfirst || c >= clast || c >= qmaxw) continue;
                    const int s = c - c0;
                    const bool in = ract && s >= 0 && s < STAGE && c < qn;
                    const int at = (in ? s * MMAX : 0) + gl;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) {
                        const double x = S.stage[at + r * G];
                        b[r][c] = in ? x : b[r][c];
                    }
                }
                wave_sync();
            }
            if (lookup_fail) atomicOr(kargs()->err, 16);

            // ---- Householder QR update: stored reflectors j < qlo act on the new
            // columns only; reflectors qlo..qn-1 are formed and applied. In the larger
            // tiers, columns below the smallest qlo of the wave's solving groups are
            // final for every group: no reflector is formed there and no stored one is
            // applied to them (the first tier's blocks are too narrow for the test to
            // pay).
            const int qloww = QMAX > 12 ? -wave_max_i(act ? -qlo : -QMAX) : 0;
#pragma unroll
            for (int j = 0; j < QMAX; ++j) {
                if (j >= qmaxw) continue;
                const bool ja = act && j < qn;
                const bool newr = j >= qlo;
                double bj;
                // the reflector's vector: column j from its head row down, exact zeros
                // above it (the entries of R there), so that the products with the
                // other columns need no per-row predicate
                double vr[RPL];
#pragma unroll
                for (int r = 0; r < RPL; ++r) vr[r] = (r * G + gl >= j) ? b[r][j] : 0.0;
                if (j < qloww) {
                    bj = bcast_lane<G>(bt[j / G], j % G);
                } else {
                    double s2 = 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) s2 += vr[r] * vr[r];
                    s2 = gsum<G>(s2);
                    const double x0 = bcast_lane<G>(b[j / G][j], j % G);
                    double nx, bnew;
                    hh_scalars(s2, x0, nx, bnew);
                    const double alpha = (x0 >= 0.0) ? -nx : nx;
                    const double vj = x0 - alpha;
                    if (ja && newr) {
                        if (!(nx > 0.0)) singular = true;
#pragma unroll
                        for (int r = 0; r < RPL; ++r)
                            if (r * G + gl == j) {
                                b[r][j] = vj;
                                vr[r] = vj;
                            }
#pragma unroll
                        for (int r = 0; r < RPL; ++r)
                            if (r * G + gl == j) {
                                rd[r] = alpha;
                                bt[r] = bnew;
                            }
                    }
                    double bold = 0.0;
                    if (wave_any(ja && !newr)) bold = bcast_lane<G>(bt[j / G], j % G);
                    bj = newr ? bnew : bold;
                }
                // groups that do not take part have f = 0 below (as have the zero columns
                // past qn), and the columns a stored reflector must leave: no lane masks
                bj = ja ? bj : 0.0;
                const int lo = newr ? 0 : qlo;
                // the columns right of j in chunks of QCB: the chunk's products and
                // group sums are independent chains the wave issues interleaved
#pragma unroll
                for (int c0 = 0; c0 < QMAX; c0 += QCB) {
                    if (c0 + QCB - 1 <= j) continue;
                    if (c0 >= qmaxw || c0 + QCB <= qloww) continue;
                    double w[QCB];
#pragma unroll
                    for (int u = 0; u < QCB; ++u) {
                        const int c = c0 + u;
                        w[u] = 0.0;
                        if (c > j && c < QMAX) {
#pragma unroll
                            for (int r = 0; r < RPL; ++r) w[u] += vr[r] * b[r][c];
                        }
                    }
#pragma unroll
                    for (int u = 0; u < QCB; ++u)
                        if (c0 + u > j && c0 + u < QMAX) w[u] = gsum<G>(w[u]);
#pragma unroll
                    for (int u = 0; u < QCB; ++u) {
                        const int c = c0 + u;
                        if (c > j && c < QMAX) {
                            const double f = (c >= lo) ? bj * w[u] : 0.0;
#pragma unroll
                            for (int r = 0; r < RPL; ++r) b[r][c] -= f * vr[r];
                        }
                    }
                }
                if (wave_any(ja && newr)) {
                    double w = 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) w += vr[r] * y[r];
                    w = gsum<G>(w);
                    const double f = newr ? bj * w : 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) y[r] -= f * vr[r];
                }
            }
            // ---- back substitution R m = (Q^T e)(0:qn)
            {
                // (every lane divides by the diagonal of its rows; the group takes the owner's)
                double z[RPL], ri[RPL];
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    z[r] = y[r];
                    ri[r] = 1.0 / rd[r];
                }
#pragma unroll
                for (int j = QMAX - 1; j >= 0; --j) {
                    if (j >= qmaxw) continue;
                    const bool ja = act && j < qn;
                    double mj = bcast_lane<G>(div_by(z[j / G], rd[j / G], ri[j / G]), j % G);
                    mj = ja ? mj : 0.0;
#pragma unroll
                    for (int r = 0; r < RPL; ++r) z[r] -= (r * G + gl < j ? b[r][j] : 0.0) * mj;
                }
                // (row j of z is final once step j has taken it)
#pragma unroll
                for (int r = 0; r < RPL; ++r)
                    if (act && r * G + gl < qn) S.mt[r * G + gl] = div_by(z[r], rd[r], ri[r]);
            }
            // ---- residual norm ||(Q^T e)(qn:m)||, plus r(k) = -1 if k is not in I
            {
                double s = 0.0;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    const int i = r * G + gl;
                    if (i >= qn && i < m) s += y[r] * y[r];
                }
                s = gsum<G>(s);
                if (act) {
                    rn = sqrt(s + (kidx < 0 ? 1.0 : 0.0));
                    if (qmod >= 0) fl += solve_flops(mmod, m, qmod, qn);
                    q = qn;
                    p = 0;
                    if (singular) status = ST_SINGULAR;
                }
            }
            // ---- dropping (Section 4): after the pass-0 solve only
            if (pass == 0) {
                bool dact = act && dropok && P.drop != DROP_NONE && status == ST_OK;
                unsigned keep = 0u;
                if (dact) {
                    const double t = (P.drop == DROP_FIXED)
                                         ? P.tol
                                         : P.eps / ((double)q * __longlong_as_double((long long)*A.norm1_bits));
#pragma unroll
                    for (int c = 0; c < QMAX; ++c)
                        if (c < q && fabs(S.mt[c]) > t) keep |= 1u << c;
                    if (__popc(keep) == q) dact = false;
                }
                if (wave_any(dact)) {
                    int jv[(QMAX + G - 1) / G], lv[(QMAX + G - 1) / G], bv0[(QMAX + G - 1) / G];
                    if (dact) {
                        if (keep == 0u) {
                            // keep the largest |m_j| (smaller column index on ties)
                            double bv = -1.0;
                            int bc = 0, bg = INT_MAX;
#pragma unroll
                            for (int c = 0; c < QMAX; ++c) {
                                if (c < q) {
                                    const double a = fabs(S.mt[c]);
                                    const int gj = S.Jlist[c];
                                    if (a > bv || (a == bv && gj < bg)) { bv = a; bc = c; bg = gj; }
                                }
                            }
                            keep = 1u << bc;
                        }
#pragma unroll
                        for (int s = 0; s < (QMAX + G - 1) / G; ++s) {
                            const int c = s * G + gl;
                            jv[s] = (c < q) ? S.Jlist[c] : 0;
                            bv0[s] = (c < q) ? S.cb[c] : 0;
                            lv[s] = (c < q) ? S.cl[c] : 0;
                        }
                    }
                    wave_sync();
                    if (dact) {
#pragma unroll
                        for (int s = 0; s < (QMAX + G - 1) / G; ++s) {
                            const int c = s * G + gl;
                            if (c < q && (keep & (1u << c))) {
                                const int d = __popc(keep & ((1u << c) - 1u));
                                S.Jlist[d] = jv[s];
                                S.cb[d] = bv0[s];
                                S.cl[d] = lv[s];
                            }
                        }
                        if constexpr (C::CROW) {
                            // (a lane's own bytes; a column only moves towards the front)
                            constexpr int RB = 6;
                            static_assert(QMAX % RB == 0, "batches of columns");
#pragma unroll
                            for (int c0 = 0; c0 < QMAX; c0 += RB) {
                                int rv[RB];
#pragma unroll
                                for (int u = 0; u < RB; ++u) rv[u] = S.crow[(c0 + u) * G + gl];
#pragma unroll
                                for (int u = 0; u < RB; ++u)
                                    if (c0 + u < q && (keep & (1u << (c0 + u))))
                                        S.crow[__popc(keep & ((1u << (c0 + u)) - 1u)) * G + gl] = (unsigned char)rv[u];
                            }
                        }
                        for (int t = gl; t < C::HSJ; t += G) S.hJ[t] = HEMPTY;
                    }
                    wave_sync();
                    if (dact) {
                        const int nk = __popc(keep);
                        for (int t = gl; t < nk; t += G) {
                            int sl;
                            hinsert<C::LOGHSJ>(S.hJ, S.Jlist[t], sl);
                        }
                        q = 0;
                        p = nk;
                        qlo = 0;
                        qmod = 0;
                        redo = true;
                    }
                    wave_sync();
                }
            }
        }

        // ============================================= I. stop test (step 3)
        bool finish = busy && (status != ST_OK || rn <= P.eps || l >= P.lmax);

        // ============================= J. dominant rows of the residual (step 4)
        const bool sel = busy && !finish;
        if (wave_any(sel)) {
            const int qmaxw = wave_max_i(sel ? q : 0);
            // r = A(I,J) m - e_k(I), eq. (2.4), formed from the sparse columns of A with
            // the columns taken in ascending global order. Rows whose coefficients tie
            // give bitwise-equal residuals, so exact ties reach the index tie-break.
            double *racc = S.racc();           // [MMAX] accumulator
            const double *mts = S.mt;          // [QMAX] solution values by slot
            int *ord = S.ord();                // [QMAX] slots in ascending column order
            if (sel && gl < 4) S.Jlist[q + gl] = INT_MAX;
            wave_sync();
            if (sel) {
                constexpr int NJ = (QMAX + G - 1) / G;
                int key[NJ], rank[NJ];
#pragma unroll
                for (int s = 0; s < NJ; ++s) key[s] = (s * G + gl < q) ? S.Jlist[s * G + gl] : INT_MIN;
                ranks_in<NJ>(S.Jlist, q, key, rank);
#pragma unroll
                for (int s = 0; s < NJ; ++s)
                    if (s * G + gl < q) ord[rank[s]] = s * G + gl;
#pragma unroll
                for (int r = 0; r < RPL; ++r) racc[r * G + gl] = 0.0;
            }
            wave_sync();
            bool lookup_fail2 = false;
            // SELB columns at a time, their first G entries' loads in flight together; the
            // accumulation keeps the ascending column order (rows of one column are
            // distinct; successive columns are ordered by the wave's in-order LDS execution)
            auto batch = [&](auto nb, int t0) {
                constexpr int NB = decltype(nb)::value;
                int cc[NB], lr[NB], cl[NB];
                double vv[NB], mc[NB];
                bool more = false;
#pragma unroll
                for (int u = 0; u < NB; ++u) cc[u] = (sel && t0 + u < q) ? ord[min(t0 + u, QMAX - 1)] : -1;
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const int c = cc[u] >= 0 ? cc[u] : 0;
                    cl[u] = cc[u] >= 0 ? S.cl[c] : 0;
                    mc[u] = mts[c];
                    more |= cl[u] > G;
                    const int e = gl < cl[u] ? S.cb[c] + gl : 0;
                    int r0;
                    if constexpr (C::CROW) r0 = S.crow[c * G + gl];
                    else r0 = A.rowidx[e];
                    lr[u] = gl < cl[u] ? r0 : -1;
                    vv[u] = A.val[e];
                }
                const bool wmore = wave_any(more);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    if constexpr (C::CROW) {
                        // (a lane without an entry accumulates past the rows)
                        const int l2 = lr[u] >= 0 ? lr[u] : MMAX;
                        racc[l2] = __fma_rn(vv[u], mc[u], racc[l2]);
                    } else if (lr[u] >= 0) {
                        const int sl = hfind<C::LOGHSI>(S.hI, lr[u]);
                        const int l2 = sl >= 0 ? S.hIv[sl] : MMAX;
                        if (l2 < MMAX) racc[l2] = __fma_rn(vv[u], mc[u], racc[l2]);
                        else lookup_fail2 = true;
                    }
                    if (wmore && cl[u] > G) {
                        const int e1 = S.cb[cc[u]] + cl[u];
                        for (int e = S.cb[cc[u]] + G + gl; e < e1; e += G) {
                            const int sl = hfind<C::LOGHSI>(S.hI, A.rowidx[e]);
                            const int l2 = sl >= 0 ? S.hIv[sl] : -1;
                            if (l2 >= 0 && l2 < MMAX) racc[l2] = __fma_rn(A.val[e], mc[u], racc[l2]);
                            else lookup_fail2 = true;
                        }
                    }
                }
            };
            if (qmaxw == 1) batch(std::integral_constant<int, 1>{}, 0);
            else
                for (int t0 = 0; t0 < qmaxw; t0 += C::SELB) batch(std::integral_constant<int, C::SELB>{}, t0);
            wave_sync();
            if (lookup_fail2) atomicOr(kargs()->err, 16);
            double ra[RPL];
            int gi[RPL];
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const int i = r * G + gl;
                const double ri = racc[i] - ((i == kidx) ? 1.0 : 0.0);
                const bool cand = sel && i < m && ri != 0.0 && !(rflag & (1u << r));
                ra[r] = cand ? fabs(ri) : -1.0;
                gi[r] = cand ? S.Ilist[i] : INT_MAX;
            }
            bool kcand = sel && kidx < 0 && !kR;  // r(k) = -1 when k is not in I
            unsigned chosen = 0u;
            int nsel = 0;
#pragma unroll
            for (int t = 0; t < CMAX; ++t) {
                if (t >= P.c) continue;
                double a = -1.0;
                int g = INT_MAX;
#pragma unroll
                for (int r = 0; r < RPL; ++r) {
                    if (!(chosen & (1u << r)) && ra[r] >= 0.0 && (ra[r] > a || (ra[r] == a && gi[r] < g))) {
                        a = ra[r];
                        g = gi[r];
                    }
                }
                gargmax<G>(a, g);
                if (kcand && (1.0 > a || (1.0 == a && k < g))) { a = 1.0; g = k; }
                if (sel && a >= 0.0) {
                    if (gl == 0) S.Rh[t] = g;
                    nsel = t + 1;
                    if (kcand && g == k) {
                        kcand = false;
                        kR = true;
                    } else {
#pragma unroll
                        for (int r = 0; r < RPL; ++r)
                            if (gi[r] == g && ra[r] >= 0.0) chosen |= 1u << r;
                    }
                }
            }
            if (sel) {
                rflag |= chosen;
                nRh = nsel;
                if (nsel == 0) finish = true;  // no candidate row left: r = 0 (Section 3)
                linc = true;
                dropok = true;
                if (kargs()->one_loop && nsel > 0) park = true;
            }
        }

        // ================================================== output of a column
        if (finish && gl < 4) S.Jlist[q + gl] = INT_MAX;
        wave_sync();
        if (finish) {
            const int64_t slot = kargs()->arena_base + ucol * (int64_t)QMAX;
            const int qq = (status == ST_OK) ? q : 0;
            // m_k with its rows in ascending order (rank of each entry in the group)
            {
                constexpr int NJ = (QMAX + G - 1) / G;
                int key[NJ], rank[NJ];
#pragma unroll
                for (int s = 0; s < NJ; ++s) key[s] = (s * G + gl < qq) ? S.Jlist[s * G + gl] : INT_MIN;
                ranks_in<NJ>(S.Jlist, qq, key, rank);
#pragma unroll
                for (int s = 0; s < NJ; ++s)
                    if (s * G + gl < qq) {
                        kargs()->out.arenaJ[slot + rank[s]] = key[s];
                        kargs()->out.arenaV[slot + rank[s]] = S.mt[s * G + gl];
                    }
            }
            if (gl == 0) {
                kargs()->out.off[ucol] = slot;
                kargs()->out.nJ[ucol] = qq;
                kargs()->out.nI[ucol] = m;
                kargs()->out.loops[ucol] = l;
                kargs()->out.status[ucol] = status;
                kargs()->out.resnorm[ucol] = rn;
                kargs()->out.flops[ucol] = fl;
            }
            // R of the final solve for the adjoint: row i of R is held by the owner lane
            // of row i (diagonal in rd, the rest in the block). Small tiers pack it in the
            // staging tile first, so the global stores need no per-entry addressing.
            if (kargs()->out.fac != nullptr) {
                const long long fo = fac_take(kargs()->out, fch, (gl == 0 && qq > 0) ? qq + qq * (qq + 1) / 2 : 0);
                if (gl == 0) {
                    kargs()->out.foff[ucol] = fo;
                    S.fo_lo = (int)(fo & 0xffffffffLL);
                    S.fo_hi = (int)(fo >> 32);
                }
                if constexpr (QMAX * (QMAX + 1) / 2 <= C::STAGE * MMAX) {
#pragma unroll
                    for (int r = 0; r < RPL; ++r) {
                        const int i = r * G + gl;
                        if (i < qq) {
                            const int base = (int)fac_row(qq, i) - qq;
                            S.stage[base] = rd[r];
#pragma unroll
                            for (int c = 0; c < QMAX; ++c)
                                if (c > i && c < qq) S.stage[base + c - i] = b[r][c];
                        }
                    }
                    wave_sync();
                    const long long fo = ((long long)S.fo_hi << 32) | (long long)(unsigned)S.fo_lo;
                    if (fo >= 0) {
                        double *F = kargs()->out.fac + fo;
                        const int tot = qq + qq * (qq + 1) / 2;
                        for (int t = gl; t < tot; t += G) F[t] = (t < qq) ? (double)S.Jlist[t] : S.stage[t - qq];
                    }
                } else {
                    wave_sync();
                    const long long fo = ((long long)S.fo_hi << 32) | (long long)(unsigned)S.fo_lo;
                    if (fo >= 0) {
                        double *F = kargs()->out.fac + fo;
                        for (int c = gl; c < qq; c += G) F[c] = (double)S.Jlist[c];
#pragma unroll
                        for (int r = 0; r < RPL; ++r) {
                            const int i = r * G + gl;
                            if (i < qq) {
                                double *Fr = F + fac_row(qq, i);
                                Fr[0] = rd[r];
#pragma unroll
                                for (int c = 0; c < QMAX; ++c)
                                    if (c > i && c < qq) Fr[c - i] = b[r][c];
                            }
                        }
                    }
                }
            }
            busy = false;
        }
        wave_sync();
    }
}

template <class C>
static void launch_tier(const TierArgs &a, int waves, hipStream_t s) {
    if (a.nmat > 1) hipLaunchKernelGGL((tier_kernel<C, true>), dim3(waves), dim3(64), 0, s, a);
    else hipLaunchKernelGGL((tier_kernel<C, false>), dim3(waves), dim3(64), 0, s, a);
}

}  // namespace rsai
