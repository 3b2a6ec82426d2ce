// Preprocessing, scan, assembly and SpMV kernels.
//
// These steps are bandwidth- and latency-bound index work: one thread per column or
// per entry, coalesced over the CSC arrays.
#include <algorithm>

#include <climits>

#include "rsai_kernels.h"

namespace rsai {

// ---------------------------------------------------------------- entries of a CSC matrix
//
// A wave takes EC neighbouring columns, whose entries lie side by side, and its lanes the
// entries in turn, EU windows of 64 at a time: with a column per lane a wave waits for its
// longest column (200 entries against a mean of 7 in a power-law matrix), and a small matrix
// fills few waves. The column of an entry is the number of columns of the wave that start up
// to it: one bit per start in LDS words of 64 entries. Where all columns of a wave are short,
// a column per lane is kept: its atomics go to 64 neighbouring rows, the entries side by side
// to the same few rows over and over (512 x 512 grid: counts 6.7 us, entries side by side
// 12.1; row pattern 9.1 against 13.3).
// Measured, a column per lane and now: 400 000 power-law columns (2 to 200 entries), check and
// counts 155 -> 101 us, row pattern 230 -> 125 us; 100 000 of them with values 129 -> 41 us;
// 21^3 grid with values 19.2 -> 5.9 us; 150 x 150 grid 4.3 -> 3.6 and 5.7 -> 4.3 us.
constexpr int EU = 4;           // windows in flight
constexpr int EWORDS = 16;      // windows whose starts are noted together
constexpr int EWAVES = 4;       // waves of a workgroup
constexpr int ESHORT = 8;       // longest column of the column-per-lane form
// Columns of a wave: 64, or 16 where 64 would leave SIMDs without a wave (1024 SIMDs).
constexpr int64_t ENARROW = 64 * 1024;
struct ELds {
    unsigned long long start[EWORDS];
    int col[64];
};
// The columns of this wave: from j in steps up to end, each XCD's workgroups on a contiguous
// eighth of them: the hardware deals workgroups to the eight XCDs round robin (block b on XCD
// b % 8), so a plain grid stride would spread neighbouring columns, and the rows they touch,
// over all eight L2s. Grids of fewer than eight blocks keep the plain stride.
struct ESpan {
    int64_t j, end, step;
};
template <int EC>
__device__ __forceinline__ ESpan entry_span(int64_t n) {
    const int64_t groups = (n + EC - 1) / EC;
    const int nb = gridDim.x, w = threadIdx.x >> 6;
    if (nb < 8) return {(blockIdx.x * (int64_t)EWAVES + w) * EC, n, (int64_t)nb * EWAVES * EC};
    const int x = blockIdx.x % 8, bw = blockIdx.x / 8, nw = (nb - x + 7) / 8;
    const int64_t chunk = (groups + 7) / 8, lo = x * chunk, hi = min(groups, lo + chunk);
    return {(lo + (int64_t)bw * EWAVES + w) * EC, min(n, hi * EC), (int64_t)nw * EWAVES * EC};
}
static inline int entry_blocks(int64_t n) {
    const int64_t EC = n < ENARROW ? 16 : 64;
    // (a multiple of 8, so that every XCD's blocks cover its chunk of the columns)
    const int64_t b = (n + EC * EWAVES - 1) / (EC * EWAVES);
    return (int)std::min<int64_t>(b < 8 ? b : (b + 7) / 8 * 8, 1048576);
}
// f(t, e, in, j, first) for every entry e of columns j0 .. j0 + EC - 1 (calls t = 0 .. EU - 1
// in a row, then done(); in: this lane has one there, j its column, first: the column's first
// entry). The extents are valid.
template <int EC, class F, class D>
__device__ __forceinline__ void each_entry(ELds &L, int64_t j0, int64_t jend, int64_t s, int64_t e, int lane, F &&f,
                                           D &&done) {
    if (EC == 64 && !wave_any(e - s > ESHORT)) {
#pragma unroll
        for (int b = 0; b < ESHORT; b += EU) {
#pragma unroll
            for (int t = 0; t < EU; ++t) f(t, s + b + t, s + b + t < e, j0 + lane, b + t == 0);
            done();
        }
        return;
    }
    const int last = (int)min((int64_t)EC, jend - j0) - 1;
    const int64_t b0 = __shfl(s, 0), b1 = __shfl(e, last);
    const bool some = lane <= last && e > s;
    const unsigned long long have = __ballot(some);
    if (some) L.col[__popcll(have & ((1ull << lane) - 1ull))] = lane;
    for (int64_t base = b0; base < b1; base += EWORDS * 64) {
        if (lane < EWORDS) L.start[lane] = 0ull;
        wave_sync();
        if (some && s >= base && s < base + EWORDS * 64)
            atomicOr(&L.start[(int)(s - base) >> 6], 1ull << ((s - base) & 63));
        wave_sync();
        for (int w = 0; w < EWORDS && base + 64 * w < b1; w += EU) {
#pragma unroll
            for (int t = 0; t < EU; ++t) {
                const int64_t w0 = base + 64 * (w + t);
                const unsigned long long m = L.start[w + t];
                const int before = __popcll(__ballot(some && s < w0));
                const int r = before + __popcll(m & ((2ull << lane) - 1ull)) - 1;
                const bool in = w0 + lane < b1;
                f(t, w0 + lane, in, j0 + L.col[in ? r : 0], (m >> lane) & 1ull);
            }
            done();
        }
        wave_sync();
    }
}

static inline int nblocks(int64_t work, int per_block) {
    int64_t b = (work + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > 1048576) b = 1048576;
    return (int)b;
}

// ---------------------------------------------------------------- fills

template <class T>
__global__ void k_fill(T *p, T v, int64_t count) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
void launch_fill_i32(int32_t *p, int32_t v, int64_t count, hipStream_t s) {
    if (count > 0) hipLaunchKernelGGL(k_fill<int32_t>, dim3(nblocks(count, 1024)), dim3(256), 0, s, p, v, count);
}
void launch_fill_i64(int64_t *p, int64_t v, int64_t count, hipStream_t s) {
    if (count > 0) hipLaunchKernelGGL(k_fill<int64_t>, dim3(nblocks(count, 1024)), dim3(256), 0, s, p, v, count);
}
void launch_fill_f64(double *p, double v, int64_t count, hipStream_t s) {
    if (count > 0) hipLaunchKernelGGL(k_fill<double>, dim3(nblocks(count, 1024)), dim3(256), 0, s, p, v, count);
}

// One launch for several int32 fills, p[i][0..count[i]) = v[i], which also writes the
// batch's matrix table from its arguments when ntab > 0 (no host-to-device copy).
struct FillMany {
    int32_t *p[FILL_SLOTS];
    int64_t count[FILL_SLOTS];
    int32_t v[FILL_SLOTS];
    MatDev *dtab;
    int64_t *dcolbase;
    int ntab;
    MatDev tab[FILL_TAB];
    int64_t colbase[FILL_TAB + 1];
};
__global__ void k_fill_many(FillMany f) {
    if (f.ntab > 0 && blockIdx.x == 0 && threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < FILL_TAB; ++i)
            if (i < f.ntab) f.dtab[i] = f.tab[i];
#pragma unroll
        for (int i = 0; i <= FILL_TAB; ++i)
            if (i <= f.ntab) f.dcolbase[i] = f.colbase[i];
    }
#pragma unroll
    for (int a = 0; a < FILL_SLOTS; ++a) {
        if (!f.p[a]) continue;
        for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < f.count[a];
             i += (int64_t)gridDim.x * blockDim.x)
            f.p[a][i] = f.v[a];
    }
}
void launch_fill_many(int32_t *const *p, const int64_t *count, const int32_t *v, int k, const MatDev *tab,
                      const int64_t *colbase, int ntab, MatDev *dtab, int64_t *dcolbase, hipStream_t s) {
    FillMany f{};
    int64_t mx = 1;
    for (int a = 0; a < k && a < FILL_SLOTS; ++a) {
        f.p[a] = p[a];
        f.count[a] = count[a];
        f.v[a] = v[a];
        mx = std::max(mx, count[a]);
    }
    if (ntab > 0 && ntab <= FILL_TAB) {
        f.ntab = ntab;
        f.dtab = dtab;
        f.dcolbase = dcolbase;
        for (int i = 0; i < ntab; ++i) f.tab[i] = tab[i];
        for (int i = 0; i <= ntab; ++i) f.colbase[i] = colbase[i];
    }
    hipLaunchKernelGGL(k_fill_many, dim3(nblocks(mx, 1024)), dim3(256), 0, s, f);
}

// longest column of a CSC matrix: atomic max into *out
__global__ void k_max_collen(int64_t n, const int64_t *colptr, int32_t *out) {
    int m = 0;
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        m = max(m, (int)(colptr[j + 1] - colptr[j]));
    for (int off = 32; off >= 1; off >>= 1) m = max(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) atomicMax(out, m);
}
void launch_max_collen(int64_t n, const int64_t *colptr, int32_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_max_collen, dim3(std::min(nblocks(n, 256), 1024)), dim3(256), 0, s, n, colptr, out);
}

// ---------------------------------------------------------------- CSC contract

__global__ void k_validate(int64_t n, int64_t nnz, const int64_t *colptr, const int32_t *rowidx, int32_t *err) {
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s = colptr[j], e = colptr[j + 1];
        if ((j == 0 && s != 0) || (j == n - 1 && e != nnz) || s < 0 || e > nnz || s > e) {
            atomicOr(err, 1);
            continue;
        }
        if (e == s) {
            atomicOr(err, 4);
            continue;
        }
        int prev = -1;
        for (int64_t t = s; t < e; ++t) {
            const int r = rowidx[t];
            if (r <= prev || r >= n) {
                atomicOr(err, 2);
                break;
            }
            prev = r;
        }
    }
}
void launch_validate(int64_t n, int64_t nnz, const int64_t *colptr, const int32_t *rowidx, int32_t *err,
                     hipStream_t s) {
    hipLaunchKernelGGL(k_validate, dim3(nblocks(n, 256)), dim3(256), 0, s, n, nnz, colptr, rowidx, err);
}

// The check above fused with the row counts of the row pattern: every entry of a column
// whose extent is valid and whose row is in range adds one to its row's count (the
// counts of a malformed matrix are never used: the later kernels skip their work).
template <int EC>
__global__ __launch_bounds__(EWAVES * 64) void k_validate_counts(int64_t n, int64_t nnz, const int64_t *colptr,
                                                                 const int32_t *rowidx, int32_t *cnt, int32_t *err) {
    __shared__ ELds lds[EWAVES];
    const int lane = threadIdx.x & 63;
    ELds &L = lds[threadIdx.x >> 6];
    for (ESpan sp = entry_span<EC>(n); sp.j < sp.end; sp.j += sp.step) {
        const int64_t j = sp.j + lane;
        const bool mine = lane < EC && j < sp.end;
        int64_t s = 0, e = 0;
        if (mine) {
            s = colptr[j];
            e = colptr[j + 1];
        }
        const bool off = mine && ((j == 0 && s != 0) || (j == n - 1 && e != nnz) || s < 0 || e > nnz || s > e);
        if (off) atomicOr(err, 1);
        if (mine && !off && e == s) atomicOr(err, 4);
        bool bad = false;
        if (wave_any(off)) {
            // columns whose entries may not lie side by side: one lane each
            int prev = -1;
            for (int64_t t = s; mine && !off && t < e; ++t) {
                const int r = rowidx[t];
                if (r < 0 || r >= n || r <= prev) bad = true;
                if (r < 0 || r >= n) break;
                prev = r;
            }
        } else {
            int r[EU];
            bool first[EU], has[EU];
            int carry = -1;  // the row before: of the window (side by side), of this lane
            const bool lanes = EC == 64 && !wave_any(e - s > ESHORT);
            each_entry<EC>(
                L, sp.j, sp.end, s, e, lane,
                [&](int t, int64_t at, bool in, int64_t, bool fst) {
                    r[t] = in ? rowidx[at] : -1;
                    has[t] = in;
                    first[t] = fst;
                },
                [&]() {
#pragma unroll
                    for (int t = 0; t < EU; ++t) {
                        int prev = carry;
                        if (!lanes) {
                            const int below = __shfl_up(r[t], 1);
                            if (lane > 0) prev = below;
                        }
                        carry = lanes ? r[t] : __builtin_amdgcn_readlane(r[t], 63);
                        if (has[t]) {
                            const bool range = r[t] >= 0 && r[t] < n;
                            bad |= !range || (!first[t] && r[t] <= prev);
                            if (range) atomicAdd(&cnt[r[t]], 1);
                        }
                    }
                });
        }
        if (bad) atomicOr(err, 2);
    }
}
void launch_validate_counts(int64_t n, int64_t nnz, const int64_t *colptr, const int32_t *rowidx, int32_t *cnt,
                            int32_t *err, hipStream_t s) {
    const auto k = n < ENARROW ? k_validate_counts<16> : k_validate_counts<64>;
    hipLaunchKernelGGL(k, dim3(entry_blocks(n)), dim3(EWAVES * 64), 0, s, n, nnz, colptr, rowidx, cnt, err);
}

// ---------------------------------------------------------------- row pattern

__global__ void k_row_counts(int64_t nnz, const int32_t *rowidx, int32_t *cnt, const int32_t *err) {
    if (*err) return;  // the CSC contract failed: touch nothing
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&cnt[rowidx[e]], 1);
}
void launch_row_counts(int64_t nnz, const int32_t *rowidx, int32_t *cnt, const int32_t *err, hipStream_t s) {
    if (nnz > 0) hipLaunchKernelGGL(k_row_counts, dim3(nblocks(nnz, 1024)), dim3(256), 0, s, nnz, rowidx, cnt, err);
}

// VAL: the values too (the transpose of a CSC matrix)
template <bool VAL, int EC>
__global__ __launch_bounds__(EWAVES * 64) void k_row_fill(int64_t n, const int64_t *colptr, const int32_t *rowidx,
                                                          const double *val, const int64_t *rowptr, int32_t *fillpos,
                                                          int32_t *colidx, double *valT, const int32_t *err) {
    __shared__ ELds lds[EWAVES];
    if (err && *err) return;
    const int lane = threadIdx.x & 63;
    ELds &L = lds[threadIdx.x >> 6];
    for (ESpan sp = entry_span<EC>(n); sp.j < sp.end; sp.j += sp.step) {
        const int64_t j = sp.j + lane;
        int64_t s = 0, e = 0;
        if (lane < EC && j < sp.end) {
            s = colptr[j];
            e = colptr[j + 1];
        }
        int r[EU], c[EU];
        double v[EU];
        each_entry<EC>(
            L, sp.j, sp.end, s, e, lane,
            [&](int t, int64_t at, bool in, int64_t col, bool) {
                r[t] = in ? rowidx[at] : -1;
                v[t] = (VAL && in) ? val[at] : 0.0;
                c[t] = (int)col;
            },
            [&]() {
                int64_t d[EU];
#pragma unroll
                for (int t = 0; t < EU; ++t) {
                    d[t] = 0;
                    if (r[t] >= 0) d[t] = rowptr[r[t]] + atomicAdd(&fillpos[r[t]], 1);
                }
#pragma unroll
                for (int t = 0; t < EU; ++t) {
                    if (r[t] < 0) continue;
                    colidx[d[t]] = c[t];
                    if (VAL) valT[d[t]] = v[t];
                }
            });
    }
}
void launch_row_fill(int64_t n, const int64_t *colptr, const int32_t *rowidx, const int64_t *rowptr,
                     int32_t *fillpos, int32_t *colidx, const int32_t *err, hipStream_t s) {
    const auto k = n < ENARROW ? k_row_fill<false, 16> : k_row_fill<false, 64>;
    hipLaunchKernelGGL(k, dim3(entry_blocks(n)), dim3(EWAVES * 64), 0, s, n, colptr, rowidx, nullptr, rowptr, fillpos,
                       colidx, nullptr, err);
}

// stats[0] = max row count (g of Theorem 4.1), stats[1] = bits of ||A||_1
// (max column absolute sum); block reduction, one atomic per block
__global__ void k_mat_stats(int64_t n, const int64_t *colptr, const double *val, const int32_t *rowcnt,
                            unsigned long long *stats, const int32_t *err) {
    if (*err) return;
    __shared__ unsigned long long sg[256], sn[256];
    unsigned long long gmax = 0, nmax = 0;
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int64_t e = colptr[j]; e < colptr[j + 1]; ++e) s += fabs(val[e]);
        unsigned long long bits = (unsigned long long)__double_as_longlong(s);  // s >= 0: order-preserving
        nmax = bits > nmax ? bits : nmax;
        unsigned long long g = (unsigned long long)rowcnt[j];
        gmax = g > gmax ? g : gmax;
    }
    sg[threadIdx.x] = gmax;
    sn[threadIdx.x] = nmax;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            sg[threadIdx.x] = max(sg[threadIdx.x], sg[threadIdx.x + w]);
            sn[threadIdx.x] = max(sn[threadIdx.x], sn[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicMax(&stats[0], sg[0]);
        atomicMax(&stats[1], sn[0]);
    }
}
void launch_mat_stats(int64_t n, const int64_t *colptr, const double *val, const int32_t *rowcnt,
                      unsigned long long *stats, const int32_t *err, hipStream_t s) {
    hipLaunchKernelGGL(k_mat_stats, dim3(std::min(nblocks(n, 256), 1024)), dim3(256), 0, s, n, colptr, val, rowcnt, stats, err);
}

// ---------------------------------------------------------------- exclusive scan
// Three passes: per-block sums, a single-block scan of the block sums, and the
// per-block scan with its offset. 2048 items per block.

constexpr int SCAN_T = 256, SCAN_PER = 8, SCAN_B = SCAN_T * SCAN_PER;

int64_t scan_tmp_elems(int64_t n) { return (n + SCAN_B - 1) / SCAN_B + 1; }

__global__ void k_scan_sums(const int32_t *in, int64_t n, int64_t *bsum) {
    __shared__ int64_t red[SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * SCAN_B;
    int64_t s = 0;
    for (int t = threadIdx.x; t < SCAN_B; t += SCAN_T) {
        int64_t i = base + t;
        if (i < n) s += in[i];
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = SCAN_T / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

__global__ void k_scan_final(const int32_t *in, int64_t n, int64_t nb, const int64_t *bsum, int64_t *out) {
    __shared__ int64_t sh[SCAN_T];
    // offset of this block: sum of the sums of all earlier blocks
    int64_t pre = 0;
    for (int64_t i = threadIdx.x; i < blockIdx.x; i += SCAN_T) pre += bsum[i];
    sh[threadIdx.x] = pre;
    __syncthreads();
    for (int w = SCAN_T / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    const int64_t boff = sh[0];
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SCAN_B + (int64_t)threadIdx.x * SCAN_PER;
    int64_t loc[SCAN_PER];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < SCAN_PER; ++t) {
        int64_t i = base + t;
        loc[t] = s;
        s += (i < n) ? in[i] : 0;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < SCAN_T; off <<= 1) {
        int64_t t = (threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    const int64_t pre2 = boff + sh[threadIdx.x] - s;
#pragma unroll
    for (int t = 0; t < SCAN_PER; ++t) {
        int64_t i = base + t;
        if (i < n) out[i] = pre2 + loc[t];
    }
    if (blockIdx.x == nb - 1 && threadIdx.x == SCAN_T - 1) out[n] = boff + sh[SCAN_T - 1];
}

// Single-pass form (decoupled look-back). A tile takes a ticket, so tiles start in
// ticket order and every tile one waits on is already running; it scans its items,
// publishes its sum, reads back through its predecessors' words until one holds an
// inclusive prefix, and publishes its own prefix. state[0] counts the tickets, state[1 + t]
// is tile t's word (bits 62-63: 1 sum, 2 prefix; bits 0-61 the value); all of it is zero
// before the launch. A ticket past the last tile or a wait past its bound (neither
// happens when the state was zeroed) sets err bit 64. With host_flags, the first tile
// copies the error flags as they stand at the launch to that host word.
constexpr unsigned long long SC_SUM = 1ull << 62, SC_PRE = 2ull << 62, SC_VAL = (1ull << 62) - 1;
int64_t scan1_state_elems(int64_t n) { return 1 + (n + SCAN_B - 1) / SCAN_B; }

// Sum of the tiles before `tile`, by its first wave; publishes the tile's sum and prefix.
// The wave reads 64 predecessors' words at a time (lane i: tile hi - i; a tile before the
// first counts as a prefix of 0) and sums those up to the nearest prefix; a window with a
// word not yet written is read again.
__device__ __forceinline__ int64_t look_back(unsigned long long *w, int64_t tile, int64_t tsum, int32_t *err) {
    const int lane = threadIdx.x & 63;
    if (lane == 0 && tile > 0)
        __hip_atomic_store(&w[tile], SC_SUM | (unsigned long long)tsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int64_t acc = 0;
    int64_t hi = tile - 1;
    unsigned spins = 0;
    while (hi >= 0) {
        const int64_t p = hi - lane;
        const unsigned long long v =
            p >= 0 ? __hip_atomic_load(&w[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : SC_PRE;
        const unsigned long long f = v >> 62;
        const unsigned long long pre = __ballot(f == 2);
        const int lim = pre ? __ffsll((long long)pre) - 1 : 63;  // lanes 0..lim are needed
        const unsigned long long need = lim == 63 ? ~0ull : ((2ull << lim) - 1);
        if (__ballot(f == 0) & need) {
            if (++spins > (1u << 22)) {
                if (lane == 0) atomicOr(err, 64);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        int64_t x = lane <= lim ? (int64_t)(v & SC_VAL) : 0;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
        acc += x;
        if (pre) break;
        hi -= 64;
    }
    if (lane == 0)
        __hip_atomic_store(&w[tile], SC_PRE | (unsigned long long)(acc + tsum), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return acc;
}

__global__ void k_scan1(const int32_t *in, int64_t n, int64_t *out, unsigned long long *state, int32_t *err,
                        int32_t *host_flags) {
    __shared__ int64_t sh[SCAN_T];
    __shared__ int64_t toff;
    __shared__ unsigned long long tk;
    if (threadIdx.x == 0) {
        tk = atomicAdd(&state[0], 1ull);
        if (host_flags && tk == 0)
            __hip_atomic_store(host_flags, __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __syncthreads();
    const int64_t nb = (n + SCAN_B - 1) / SCAN_B;
    const int64_t tile = (int64_t)tk;
    if (tile >= nb) {
        if (threadIdx.x == 0) atomicOr(err, 64);
        return;
    }
    const int64_t base = tile * SCAN_B + (int64_t)threadIdx.x * SCAN_PER;
    int64_t loc[SCAN_PER];
    int64_t s = 0;
#pragma unroll
    for (int t = 0; t < SCAN_PER; ++t) {
        const int64_t i = base + t;
        loc[t] = s;
        s += (i < n) ? in[i] : 0;
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < SCAN_T; off <<= 1) {
        const int64_t t = (threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    const int64_t tsum = sh[SCAN_T - 1];
    if (threadIdx.x < 64) {
        const int64_t acc = look_back(state + 1, tile, tsum, err);
        if (threadIdx.x == 0) toff = acc;
    }
    __syncthreads();
    const int64_t pre = toff + sh[threadIdx.x] - s;
#pragma unroll
    for (int t = 0; t < SCAN_PER; ++t) {
        const int64_t i = base + t;
        if (i < n) out[i] = pre + loc[t];
    }
    if (tile == nb - 1 && threadIdx.x == SCAN_T - 1) out[n] = toff + tsum;
}
void launch_scan1_i32(const int32_t *in, int64_t n, int64_t *out, unsigned long long *state, int32_t *err,
                      int32_t *host_flags, hipStream_t s) {
    const int64_t nb = (n + SCAN_B - 1) / SCAN_B;
    hipLaunchKernelGGL(k_scan1, dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, n, out, state, err, host_flags);
}

// exclusive scan with out[n] = total (n >= 1)
void launch_scan_i32(const int32_t *in, int64_t n, int64_t *out, int64_t *tmp, hipStream_t s) {
    const int64_t nb = (n + SCAN_B - 1) / SCAN_B;
    hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, n, tmp);
    hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, n, nb, tmp, out);
}

// ---------------------------------------------------------------- assembly
// The size classes leave each column's (row, value) pairs in ascending row order in its
// arena slot. One launch forms colptr of M (the exclusive scan of nJ) and compacts the
// slots: a tile of T columns is scanned by its block (single-pass look-back, as in
// k_scan1) and then copied, 16 lanes per column, 8 columns in flight. Bound by the
// look-back chain and the copy's latency: small tiles spread few columns over more CUs, large
// ones shorten the chain. Tiles of 256 columns up to ASM_TILES of them, of 1024 beyond; both
// measured on grids (build's event times, us, 256 / 1024): n = 1024 10.7 / 12.3, 16384
// 12.0 / 13.3, 32761 12.9 / 13.8, 40000 13.9 / 14.0, 50625 15.1 / 14.4, 65536 15.9 / 14.9,
// 131044 22.7 / 16.3, 262144 35.1 / 22.3. As two launches (scan, then copy) the assembly took
// 26.5 us on 262144 columns and 12.2 on 1024 where one launch took 19.2 and 8.2 (kernel times).
// state: asm_state_elems(n) zeroed words (k_scan1's layout). The same pass fills the
// summary the host reads after the build (zeroed at its start): sum[0] = nnz of M,
// sum[1] = error flags, sum[2..4] = columns with status singular / cap / anything else
// not ok.
constexpr int ASM_SMALL = 256, ASM_LARGE = 1024, ASM_TILES = 160;
int64_t asm_state_elems(int64_t n) { return 1 + (n + ASM_SMALL - 1) / ASM_SMALL; }

template <int ASM_T>
__global__ __launch_bounds__(ASM_T) void k_assemble(int64_t n, int qcap, const int64_t *off, const int32_t *nJ,
                                                    int64_t *colptrM, const int32_t *aJ, const double *aV,
                                                    int32_t *rowidxM, double *valM, const int32_t *status,
                                                    int32_t *err, unsigned long long *state, int64_t *sum) {
    __shared__ int loc[ASM_T + 1];  // offsets of the tile's columns in the tile
    __shared__ int64_t src[ASM_T];
    __shared__ int wsum[ASM_T / 64];
    __shared__ int64_t toff;
    __shared__ unsigned long long tk;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) tk = atomicAdd(&state[0], 1ull);
    __syncthreads();
    const int64_t nb = (n + ASM_T - 1) / ASM_T;
    const int64_t tile = (int64_t)tk;
    if (tile >= nb) {
        if (tid == 0) atomicOr(err, 64);
        return;
    }
    const int64_t k = tile * ASM_T + tid;
    const int cnt = k < n ? nJ[k] : 0;
    src[tid] = k < n ? off[k] : 0;
    const int st = k < n ? status[k] : 0;
    // columns that did not finish: one atomic per wave and kind that occurs
    const unsigned long long b3 = __ballot(st == 3), b6 = __ballot(st == 6), bx = __ballot(st != 0 && st != 3 && st != 6);
    if (lane == 0) {
        if (b3) atomicAdd((unsigned long long *)&sum[2], (unsigned long long)__popcll(b3));
        if (b6) atomicAdd((unsigned long long *)&sum[3], (unsigned long long)__popcll(b6));
        if (bx) atomicAdd((unsigned long long *)&sum[4], (unsigned long long)__popcll(bx));
    }
    int x = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int before = 0, tsum = 0;
#pragma unroll
    for (int u = 0; u < ASM_T / 64; ++u) {
        if (u < w) before += wsum[u];
        tsum += wsum[u];
    }
    loc[tid] = before + x - cnt;
    if (tid == 0) loc[ASM_T] = tsum;
    if (w == 0) {
        const int64_t acc = look_back(state + 1, tile, tsum, err);
        if (lane == 0) toff = acc;
    }
    __syncthreads();
    const int64_t base = toff;
    if (k < n) colptrM[k] = base + loc[tid];
    if (tile == nb - 1 && tid == 0) {
        colptrM[n] = base + tsum;
        sum[0] = base + tsum;
        sum[1] = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // (no copy of columns that the CSC check or a class left unwritten: their count is 0)
    // U columns of a 16-lane group at a time, their first 16 entries loaded together
    constexpr int U = 8;
    const int gl = tid & 15;
    for (int c0 = tid >> 4; c0 < ASM_T; c0 += U * (ASM_T / 16)) {
        int j[U], len[U];
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * (ASM_T / 16);
            len[u] = min(loc[c + 1] - loc[c], qcap);
            j[u] = 0;
            v[u] = 0.0;
            if (gl < len[u]) {
                j[u] = aJ[src[c] + gl];
                v[u] = aV[src[c] + gl];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * (ASM_T / 16);
            const int64_t d0 = base + loc[c];
            if (gl < len[u]) {
                rowidxM[d0 + gl] = j[u];
                valM[d0 + gl] = v[u];
            }
            for (int t = gl + 16; t < len[u]; t += 16) {
                rowidxM[d0 + t] = aJ[src[c] + t];
                valM[d0 + t] = aV[src[c] + t];
            }
        }
    }
}
void launch_assemble(int64_t n, int qcap, const int64_t *off, const int32_t *nJ, int64_t *colptrM,
                     const int32_t *arenaJ, const double *arenaV, int32_t *rowidxM, double *valM,
                     const int32_t *status, int32_t *err, unsigned long long *state, int64_t *summary,
                     hipStream_t s) {
    auto go = [&](auto kernel, int64_t t) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n + t - 1) / t)), dim3((unsigned)t), 0, s, n, qcap, off, nJ, colptrM,
                           arenaJ, arenaV, rowidxM, valM, status, err, state, summary);
    };
    if (n <= (int64_t)ASM_SMALL * ASM_TILES) go(k_assemble<ASM_SMALL>, ASM_SMALL);
    else go(k_assemble<ASM_LARGE>, ASM_LARGE);
}

// ---------------------------------------------------------------- SpMV

void launch_csc_transpose_fill(int64_t n, const int64_t *colptr, const int32_t *rowidx, const double *val,
                               const int64_t *rowptr, int32_t *fillpos, int32_t *colidxT, double *valT,
                               hipStream_t s) {
    const auto k = n < ENARROW ? k_row_fill<true, 16> : k_row_fill<true, 64>;
    hipLaunchKernelGGL(k, dim3(entry_blocks(n)), dim3(EWAVES * 64), 0, s, n, colptr, rowidx, val, rowptr, fillpos, colidxT,
                       valT, nullptr);
}

// one row by one thread: up to 32 entries in registers (each entry's place is the
// number of smaller column indices in the row, which are distinct), longer in place
__device__ __forceinline__ void sort_row_thread(int64_t s, int64_t e, int32_t *colidx, double *val) {
    constexpr int RS = 32;
    const int len = (int)(e - s);
    if (len <= RS) {
        int key[RS];
        double v[RS];
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            key[t] = (t < len) ? colidx[s + t] : INT_MAX;
            v[t] = (t < len && val) ? val[s + t] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            if (t < len) {
                int rank = 0;
#pragma unroll
                for (int u = 0; u < RS; ++u) rank += (key[u] < key[t]) ? 1 : 0;
                colidx[s + rank] = key[t];
                if (val) val[s + rank] = v[t];
            }
        }
        return;
    }
    for (int64_t a = s + 1; a < e; ++a) {
        int key = colidx[a];
        double v = val ? val[a] : 0.0;
        int64_t b = a - 1;
        while (b >= s && colidx[b] > key) {
            colidx[b + 1] = colidx[b];
            if (val) val[b + 1] = val[b];
            --b;
        }
        colidx[b + 1] = key;
        if (val) val[b + 1] = v;
    }
}

// number of keys in this lane's 16-lane row smaller than its own: the row rotated by
// D = 1..15 lanes (DPP row_ror), one comparison per rotation
template <int D>
__device__ __forceinline__ int row16_rank(int key, int acc) {
    if constexpr (D == 16) {
        return acc;
    } else {
        const int other = __builtin_amdgcn_mov_dpp(key, 0x120 + D, 0xF, 0xF, true);
        return row16_rank<D + 1>(key, acc + (other < key ? 1 : 0));
    }
}

// Two keys per lane (entries gl and gl + 16 of a row of up to 32): the ranks of both
// among all 32, counted over the rotations of both halves.
template <int D>
__device__ __forceinline__ void row32_rank(int ka, int kb, int &ca, int &cb) {
    if constexpr (D < 16) {
        const int ra = __builtin_amdgcn_mov_dpp(ka, 0x120 + D, 0xF, 0xF, true);
        const int rb = __builtin_amdgcn_mov_dpp(kb, 0x120 + D, 0xF, 0xF, true);
        ca += (ra < ka ? 1 : 0) + (rb < ka ? 1 : 0);
        cb += (ra < kb ? 1 : 0) + (rb < kb ? 1 : 0);
        row32_rank<D + 1>(ka, kb, ca, cb);
    }
}

// sort each row's (col, value) pairs by column so that row sums have a fixed order.
// Rows of up to 32 entries: a 16-lane row of the wave per matrix row, one or two
// entries per lane (contiguous loads), each entry's place its rank; longer rows by
// one lane.
constexpr int SORT_G = 16;
__global__ void k_sort_rows(int64_t n, const int64_t *rowptr, int32_t *colidx, double *val) {
    const int gl = threadIdx.x % SORT_G;
    const int64_t g0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / SORT_G;
    const int64_t gs = (int64_t)gridDim.x * blockDim.x / SORT_G;
    for (int64_t i = g0; i < n; i += gs) {
        const int64_t s = rowptr[i], e = rowptr[i + 1];
        const int len = (int)(e - s);
        if (len <= SORT_G) {
            const int key = gl < len ? colidx[s + gl] : INT_MAX;
            const double v = (gl < len && val) ? val[s + gl] : 0.0;
            const int rank = row16_rank<1>(key, 0);
            if (gl < len) {
                colidx[s + rank] = key;
                if (val) val[s + rank] = v;
            }
        } else if (len <= 2 * SORT_G) {
            const int ka = colidx[s + gl];  // gl < 16 < len
            const int kb = gl + SORT_G < len ? colidx[s + gl + SORT_G] : INT_MAX;
            const double va = val ? val[s + gl] : 0.0;
            const double vb = (gl + SORT_G < len && val) ? val[s + gl + SORT_G] : 0.0;
            int ca = kb < ka ? 1 : 0, cb = ka < kb ? 1 : 0;
            row32_rank<1>(ka, kb, ca, cb);
            colidx[s + ca] = ka;
            if (val) val[s + ca] = va;
            if (gl + SORT_G < len) {
                colidx[s + cb] = kb;
                if (val) val[s + cb] = vb;
            }
        } else if (gl == 0) {
            sort_row_thread(s, e, colidx, val);
        }
    }
}
void launch_sort_rows(int64_t n, const int64_t *rowptr, int32_t *colidx, double *val, hipStream_t s) {
    hipLaunchKernelGGL(k_sort_rows, dim3(nblocks(n * SORT_G, 256)), dim3(256), 0, s, n, rowptr, colidx, val);
}

// y = A x by rows: SG lanes per row take its entries side by side, SR neighbouring rows per
// group with their first SG entries in flight together, and their partial sums are added over
// the lanes. Bound by the entries' bytes (12 each) and the latency of the chain extents ->
// indices -> x; every wave the chip holds is needed, so no LDS staging: with the rows' entries
// staged (48 KB a workgroup, three on a CU, a second and nearly empty round of workgroups)
// M of a 512 x 512 grid (262144 rows of 7) took 18.9 us, now 11.2 us (38 MB; four rows
// a group 11.7, four lanes a row 14.4). Each XCD's
// workgroups take a contiguous eighth of the rows, so that neighbouring rows' x meet in one L2.
constexpr int SG = 8, SR = 2, SPMV_T = 256, SPMV_ROWS = SPMV_T / SG * SR;
__global__ __launch_bounds__(SPMV_T) void k_csr_spmv(int64_t n, const int64_t *rowptr, const int32_t *colidx,
                                                    const double *val, const double *x, double *y) {
    const int gl = threadIdx.x % SG, grp = threadIdx.x / SG;
    const int64_t blocks = (n + SPMV_ROWS - 1) / SPMV_ROWS;
    int64_t b = blockIdx.x, bend = blocks, bstep = gridDim.x;
    if (gridDim.x >= 8) {
        const int64_t chunk = (blocks + 7) / 8;
        b = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
        bend = min(blocks, (int64_t)(blockIdx.x % 8 + 1) * chunk);
        bstep = gridDim.x / 8;
    }
    for (; b < bend; b += bstep) {
        const int64_t r0 = b * SPMV_ROWS + (int64_t)grp * SR;
        const int64_t mine = rowptr[min(r0 + gl, n)];  // SR + 1 extents of the group's rows
        int64_t e[SR + 1];
        double sum[SR];
        int c[SR];
        double v[SR];
#pragma unroll
        for (int t = 0; t <= SR; ++t) e[t] = __shfl(mine, t, SG);
#pragma unroll
        for (int t = 0; t < SR; ++t) {
            const bool in = e[t] + gl < e[t + 1];
            c[t] = in ? colidx[e[t] + gl] : 0;
            v[t] = in ? val[e[t] + gl] : 0.0;
        }
#pragma unroll
        for (int t = 0; t < SR; ++t) sum[t] = e[t] + gl < e[t + 1] ? v[t] * x[c[t]] : 0.0;
#pragma unroll
        for (int t = 0; t < SR; ++t) {
            for (int64_t k = e[t] + SG + gl; k < e[t + 1]; k += SG) sum[t] += val[k] * x[colidx[k]];
            sum[t] = gsum<SG>(sum[t]);
        }
        double out = sum[0];
#pragma unroll
        for (int t = 1; t < SR; ++t) out = gl == t ? sum[t] : out;
        if (gl < SR && r0 + gl < n) y[r0 + gl] = out;
    }
}
void launch_csr_spmv(int64_t n, const int64_t *rowptr, const int32_t *colidx, const double *val, const double *x,
                     double *y, hipStream_t s) {
    const int b = nblocks(n, SPMV_ROWS);
    hipLaunchKernelGGL(k_csr_spmv, dim3(b < 8 ? b : (b + 7) / 8 * 8), dim3(SPMV_T), 0, s, n, rowptr, colidx, val, x, y);
}

// y = A^T x for CSC A: y_j = sum_i a_ij x_i, a column dot product in ascending row
// order; the columns of A in CSC are the rows of A^T in CSR, so the row kernel serves
// unchanged
void launch_csc_spmv_t(int64_t n, const int64_t *colptr, const int32_t *rowidx, const double *val, const double *x,
                       double *y, hipStream_t s) {
    launch_csr_spmv(n, colptr, rowidx, val, x, y, s);
}



// dval[e] += dy[row(e)] * x[col(e)]: a group of VG lanes per column walks its entries
// side by side (contiguous loads); every entry is updated by exactly one lane
constexpr int VG = 8;
__global__ void k_spmv_vjp(int64_t n, const int64_t *colptr, const int32_t *rowidx, const double *dy,
                           const double *x, double *dval) {
    const int gl = threadIdx.x % VG;
    const int64_t g0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / VG;
    const int64_t gs = (int64_t)gridDim.x * blockDim.x / VG;
    for (int64_t j = g0; j < n; j += gs) {
        const double xj = x[j];
        const int64_t e1 = colptr[j + 1];
        for (int64_t e = colptr[j] + gl; e < e1; e += VG) dval[e] += dy[rowidx[e]] * xj;
    }
}
void launch_spmv_vjp(int64_t n, const int64_t *colptr, const int32_t *rowidx, const double *dy, const double *x,
                     double *dval, hipStream_t s) {
    hipLaunchKernelGGL(k_spmv_vjp, dim3(nblocks(n * VG, 256)), dim3(256), 0, s, n, colptr, rowidx, dy, x, dval);
}

// FP64 FMA throughput probe: every lane runs FMA_CHAINS independent dependency chains
// of iters fused multiply-adds (enough in flight to cover the FMA latency at four
// waves per SIMD). The result is stored only if it takes a value it cannot reach, so
// the arithmetic stays while the stores do not.
constexpr int FMA_CHAINS = 8;
__global__ __launch_bounds__(256) void k_fma_probe(int64_t iters, double *out) {
    double a[FMA_CHAINS];
#pragma unroll
    for (int u = 0; u < FMA_CHAINS; ++u) a[u] = 1.0 + 1e-9 * (double)(threadIdx.x + u);
    const double mul = 0.9999999, add = 1e-7;
    for (int64_t i = 0; i < iters; ++i) {
#pragma unroll
        for (int u = 0; u < FMA_CHAINS; ++u) a[u] = __builtin_fma(a[u], mul, add);
    }
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < FMA_CHAINS; ++u) t += a[u];
    if (t == -1.0) out[blockIdx.x] = t;
}
int fma_probe_chains() { return FMA_CHAINS; }
void launch_fma_probe(int blocks, int64_t iters, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_fma_probe, dim3(blocks), dim3(256), 0, s, iters, out);
}

}  // namespace rsai
