// One Krylov cycle (Fig. 3) of a single 2-D grid in one resident launch
// (ch_resident.h): matvec, dot products, Gram-Schmidt coefficients, update and
// the phi tests of every Arnoldi iteration.
//
// The arithmetic, and the order in which every sum is added, are those of the
// separate launches (k_matvec_s, k_dots_reduce, k_dc_update, phi_test), so a
// cycle's basis and Hessenberg matrix are bit for bit theirs.
//
// Workgroups [0, G) own the strips of the 2-D kernels, one or two to a wave, in groups
// of four (a strip workgroup of the separate launches).  An iteration k:
//   1. a wave reads the rows of u_k around its strip (its neighbours' rows
//      once their flags say they are written), forms w = Ahat u_k and the dot
//      products of its own points with the columns before;
//   2. each group hands its partials out; waves all over the grid add up the
//      2k + 2 rows and hand out the sums;
//   3. wave 0 of every workgroup forms the iteration's coefficients from the
//      totals (H is kept in LDS by each);
//   4. every wave forms q_k and u_{k+1} at its own points.
// A partial and a total are their own flag: until written they hold a
// signalling NaN, which no arithmetic produces (two polls instead of two drains, two
// flags, two polls and two reads).  The first `lc` basis columns of a wave's
// points stay in registers and LDS; all go to the basis in memory, for the solution
// update.
//
// The last CYC_TESTS workgroups run the phi tests: each follows the totals to
// its own copy of H and tests every CYC_TESTS-th dimension, so a test (10-25 us)
// does not hold up the iterations; tests take effect in order (chain words).
// A cycle's iterations run ahead of its tests by two or three; what they
// write is not read by the finished cycle.
#pragma once

#include "ch_phi.h"
#include "ch_resident.h"
#include "ch_rows.h"

#include <algorithm>

struct CycleArgs {
    Ctl* ctl;
    Inst I;
    void* V;
    size_t ldv;
    const void* y;
    double* part;    // two buffers of CYC_PART partials
    double* tot;     // per iteration, CYC_WAVES rows of CYC_TOT wave sums
    int* words;      // flags, failure word, done word, chain words
    int* dflags;
    int epoch, G, m_max, lc;
    unsigned wait_us;
};

namespace {

constexpr unsigned long long RES_OPEN = 0x7FF4A5A5C3C35A5Aull;   // a value not yet written

constexpr int CYC_ROWS = 2 * CH_MSMALL + 2;   // dot-product rows of an iteration
constexpr int CYC_TOT = 128;                  // stride of the totals of an iteration (two per lane of a wave)
constexpr int CYC_LINE = 16;                  // rows of partials in a cache line
constexpr int CYC_LINES = (CYC_ROWS + CYC_LINE - 1) / CYC_LINE;
constexpr int CYC_GROUPS = 1280;              // most groups
constexpr int CYC_PART = CYC_LINES * CYC_GROUPS * CYC_LINE;   // partials of an iteration
constexpr int CYC_LDH = CH_MSMALL + 2;        // leading dimension of H in LDS

__device__ __forceinline__ bool is_open(double x) { return __builtin_bit_cast(unsigned long long, x) == RES_OPEN; }

// Coefficients of the current iteration and H, per workgroup.
struct CycCoef {
    double hs[CYC_LDH * (CH_MSMALL + 1)];   // h_{r, c} at hs[r + c CYC_LDH], zero where there is none
    double dt[CYC_TOT];
    double s[CH_MSMALL + 1];
    double h1[2][CH_MSMALL + 1];      // h' of the newest column, as Ctl::h1
    double2 ab[CH_MSMALL + 1];        // coefficients of column i in q_j and u_{j+1}
    double cbw, cq, rho;
    int stop;                         // the cycle has ended, or a wait ran out
};

// One wave: the coefficients of iteration j from the totals in C.dt, as
// dc_prepare forms them; column j - 1 of H.  fin: only that column.
__device__ __forceinline__ void cyc_prepare(CycCoef& C, int j, bool fin, double vscale0) {
    const int i = threadIdx.x & 63;
    const double si = i < j ? C.dt[i] : 0.0, ti = i < j ? C.dt[j + i] : 0.0;
    const double ss = wave_sum(product(si, si)), st = wave_sum(product(si, ti));
    const double rho2 = C.dt[2 * j] - ss;
    const double rho = rho2 > 0.0 ? sqrt(rho2) : (rho2 <= 0.0 ? 0.0 : rho2);   // NaN stays NaN
    if (i <= j && j >= 1) C.hs[i + (j - 1) * CYC_LDH] = i < j ? C.h1[j & 1][i] + si : rho;
    if (i <= j) C.s[i] = si;
    if (i == 0) C.rho = rho;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if (fin) return;
    double g = 0.0;   // (H_j s)_i; terms below the subdiagonal add zero
    for (int c0 = 0; c0 < j; c0 += 8) {   // eight columns' reads in flight; columns past j - 1 are zero
        double h[8], sc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            h[c] = C.hs[min(i, CYC_LDH - 1) + (c0 + c) * CYC_LDH];
            sc[c] = C.s[c0 + c];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) g = __builtin_fma(h[c], sc[c], g);
    }
    const double ir = 1.0 / rho;
    const double qw = (C.dt[2 * j + 1] - st) * ir;   // q_j^T w
    if (i <= j) {
        const double hp = product((i < j ? ti : qw) - g, ir);   // h'_i
        const double c = __builtin_fma(g, ir, hp);
        C.h1[(j + 1) & 1][i] = hp;
        if (i < j) {
            C.ab[i] = double2{-si * ir, -c};
        } else {
            C.ab[j].x = (j == 0 ? vscale0 : 1.0) * ir;
            C.cq = -c;
        }
    }
    if (i == 0) C.cbw = ir;
}

// Waits of a cycle end in one of three ways.
enum CycWait { CYC_OK = 0, CYC_END = 1 };

// True when a wait is to end: the cycle is done, another workgroup gave up,
// or the time ran out (which marks the run for a repeat).
__device__ __forceinline__ bool cyc_ended(const CycleArgs& A, unsigned spin, long long& t0) {
    if (spin & 7) return false;
    if (res_load(A.words + CH_RES_DONE) == A.epoch) return true;
    if (spin & 63) return false;
    if (!res_expired(spin, t0, A.words + CH_RES_FAIL, A.epoch, A.wait_us)) return false;
    A.ctl->status = CH_RES_RETRY;
    A.ctl->halted = 1;
    return true;
}

// sum_partials adds the partials of 256 threads wave by wave; a row's sum over
// each of those waves is formed by a wave of its own (cyc_reduce), and whoever needs the
// total adds the four.
constexpr int CYC_WAVES = CH_BLOCK / 64;
__device__ __forceinline__ int cyc_waves(const CycleArgs& A) { return min((A.I.wblk + 63) / 64, CYC_WAVES); }
__device__ __forceinline__ double* cyc_tot(const CycleArgs& A, int k, int w) {
    return A.tot + (size_t)(k * CYC_WAVES + w) * CYC_TOT;
}

// One wave: the totals of iteration k into C.dt.
__device__ __forceinline__ int cyc_totals(const CycleArgs& A, CycCoef& C, int k) {
    const int lane = threadIdx.x & 63, rows = 2 * k + 2, nw = cyc_waves(A);
#pragma unroll 1
    for (int h = 0; h < rows; h += 64) {
        const bool on = lane + h < rows;
        double v[CYC_WAVES];
        long long t0 = 0;
        for (unsigned spin = 0;; ++spin) {
            bool ok = true;
#pragma unroll
            for (int w = 0; w < CYC_WAVES; ++w) {
                v[w] = 0.0;
                if (on && w < nw) v[w] = res_load(cyc_tot(A, k, w) + lane + h);
                ok = ok && !is_open(v[w]);
            }
            if (__all(ok)) break;
            if (cyc_ended(A, spin, t0)) return CYC_END;
            __builtin_amdgcn_s_sleep(1);
        }
        double t = v[0];
#pragma unroll
        for (int w = 1; w < CYC_WAVES; ++w) t += v[w];
        C.dt[lane + h] = t;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    return CYC_OK;
}

// A group's partials of an iteration are whole cache lines of CYC_LINE rows, so
// that no line has two writers (a row of partials side by side took 7 us to be complete
// at 640 groups, whole lines 2.5).  g: the group's position in a launch of
// k_matvec_s.
__device__ __forceinline__ double* cyc_part(const CycleArgs& A, int k, int row, int g) {
    return A.part + (size_t)(k & 1) * CYC_PART + ((row / CYC_LINE) * CYC_GROUPS + g) * CYC_LINE + row % CYC_LINE;
}

// One wave: wave w's share of the sum over row `row` of iteration k, as
// sum_partials (k_dots_reduce) adds it.
__device__ __forceinline__ int cyc_reduce(const CycleArgs& A, int k, int row, int w) {
    constexpr int PER = CYC_GROUPS / CH_BLOCK;
    static_assert(PER * CH_BLOCK == CYC_GROUPS, "whole rounds of sum_partials");
    const int lane = threadIdx.x & 63, np = A.I.wblk, at = 64 * w + lane;
    double v[PER];
    long long t0 = 0;
    for (unsigned spin = 0;; ++spin) {
        bool ok = true;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            v[u] = 0.0;
            if (at + CH_BLOCK * u < np) v[u] = res_load(cyc_part(A, k, row, at + CH_BLOCK * u));
            ok = ok && !is_open(v[u]);
        }
        if (__all(ok)) break;
        if (cyc_ended(A, spin, t0)) return CYC_END;
        __builtin_amdgcn_s_sleep(1);
    }
    double s = v[0];
#pragma unroll
    for (int u = 1; u < PER; ++u) s += v[u];
    s = wave_sum(s);
    if (lane == 0) res_store(cyc_tot(A, k, w) + row, s);
    return CYC_OK;
}

// Strip i (of nt) of a neighbour at distance one or two, folded at the boundary.
__device__ __forceinline__ int fold_strip(int i, int nt, bool neu) {
    if (neu) {
        i = i < 0 ? -1 - i : (i >= nt ? 2 * nt - 1 - i : i);
        return min(max(i, 0), nt - 1);
    }
    i %= nt;
    return i < 0 ? i + nt : i;
}

// Every workgroup waits until all have raised their flags to v; call from
// every thread.
__device__ __forceinline__ void cyc_all(const CycleArgs& A, CycCoef& C, int v) {
    for (int i = threadIdx.x; i < A.G; i += blockDim.x) {
        long long t0 = 0;
        for (unsigned spin = 0; res_load(A.words + i * CH_RES_LINE) < v; ++spin) {
            if (cyc_ended(A, spin, t0)) {
                C.stop = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    __syncthreads();
}

// Basis columns a wave keeps in registers, by the waves of a workgroup (four
// waves leave 512 registers a lane, eight 256, twelve 168).  Four and eight waves
// spill no vector registers; twelve spill 28 to 35 with four columns, and eight
// columns are slower: 1290 us for three steps at 1024^2 FP32, 1050 with four.
// With two strips to a wave (ten waves, 168 registers, 32 to 57 of them spilled without any
// column) four columns cost more than they save; two columns fit in LDS, and the others come from the last-level cache
// at about 9 TB/s, which is what bounds a cycle at 1024^2 FP64 (three steps 2270 us
// as launches, 1860 here).  Five strips to each of four waves hold ten columns, but one
// wave per SIMD hides no latency: 3950.
constexpr int cyc_reg_cols(int NW, int S) { return S > 1 ? 0 : NW == 4 ? 16 : NW == 8 ? 8 : 4; }

// NW waves to a workgroup, S strips to a wave: wave v holds the workgroup's strips
// v, v + NW, ...
template <typename TV, int NW, int S, int VX, bool NEU, bool MOB>
__device__ __forceinline__ void cycle_main(const CycleArgs& A, CycCoef& C, double (*red)[NW * S], TV* rows, TV* cols) {
    constexpr int NU = SR + 4, ND = SR + 2, NS = NW * S, NG = NS / 4, T = 64 * NW, RC = cyc_reg_cols(NW, S), LANES = 64 * VX;
    static_assert(NS % 4 == 0, "whole groups");
    constexpr int bc = NEU ? CH_BC_NEUMANN : CH_BC_PERIODIC;
    const Inst& I = A.I;
    Ctl* ctl = A.ctl;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int r = xcd_remap(blockIdx.x, A.G);
    const int n = I.n, eyre = I.eyre, m_max = A.m_max;
    const int nsx = (n + strip_cols(VX) - 1) / strip_cols(VX), nsy = (n + SR - 1) / SR, ns = nsx * nsy;
    StripPos<VX> P[S];
    unsigned bo[S], bs[S], bd[S], bh[S];
    bool in[S][SR], above[S], below[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
        const int strip = r * NS + wv + q * NW;
        const bool live = strip < ns;
        const int at = live ? strip : ns - 1;
        P[q] = strip_pos<VX>(at, nsx, n, lane, bc);
        P[q].out = P[q].out && live;
        P[q].need = P[q].need && live;
        bo[q] = (unsigned)P[q].xl * (unsigned)sizeof(TV);
        bs[q] = P[q].need ? bo[q] : OFF_ROW;
        bd[q] = P[q].out ? bo[q] : OFF_ROW;
        bh[q] = P[q].need && !P[q].out ? bo[q] : OFF_ROW;
#pragma unroll
        for (int i = 0; i < SR; ++i) in[q][i] = P[q].out && P[q].r0 + i < n;
        // The strips above and below the wave's are other waves' of this workgroup
        // (strips nsx apart) or another workgroup's: the former hand their rows on
        // through LDS, the latter through memory, as do the halo columns.
        above[q] = wv + q * NW >= nsx;
        below[q] = wv + q * NW + nsx < NS && at + nsx < ns && P[q].r0 + 2 * SR - 1 < n;
    }
    TV* V = static_cast<TV*>(A.V) + I.off;
    const TV* Y = static_cast<const TV*>(A.y) + I.off;
    const TV ih2 = TV(I.inv_h2), e2ih2 = TV(I.eps2 * I.inv_h2);
    const Mob mob = mob_of(ctl, MOB);
    const double vscale0 = ctl->vscale[0];
    const int hv = wave_sum8_holder(lane);
    // the flag this lane waits for before u is read: the owners of the strips
    // around the wave's, 32 lanes to a strip (the second neighbour only across a fold, where
    // the strip between may be narrower than the halo)
    constexpr int NF = (S + 1) / 2;
    const int* nflag[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int l = lane & 31, q = 2 * f + (lane >> 5), at = min(r * NS + wv + q * NW, ns - 1);
        const int sx = at % nsx, sy = at / nsx, dx = l % 5 - 2, dy = l / 5 - 2;
        const bool near_x = dx >= -1 && dx <= 1, near_y = dy >= -1 && dy <= 1;
        nflag[f] = nullptr;
        if (l < 25 && q < S && (near_x || sx + dx < 0 || sx + dx >= nsx) && (near_y || sy + dy < 0 || sy + dy >= nsy)) {
            const int o = fold_strip(sy + dy, nsy, NEU) * nsx + fold_strip(sx + dx, nsx, NEU);
            nflag[f] = A.words + o / NS * CH_RES_LINE;
        }
    }
    int* flag = A.words + r * CH_RES_LINE;

    // mark the partials (both buffers) and the totals as not yet written
    const double open = __builtin_bit_cast(double, RES_OPEN);
    int gpos[NG];   // launch positions of the workgroup's groups (-1: none)
#pragma unroll
    for (int g = 0; g < NG; ++g) gpos[g] = r * NG + g < I.wblk ? xcd_unmap(r * NG + g, I.wblk) : -1;
    auto open_slots = [&](int k, int nrows) {
#pragma unroll
        for (int g = 0; g < NG; ++g)
            for (int i = threadIdx.x; i < nrows; i += T)
                if (gpos[g] >= 0) res_store(cyc_part(A, k, i, gpos[g]), open);
    };
    open_slots(0, 2 * m_max + 2);
    open_slots(1, 2 * m_max + 2);
    for (int i = blockIdx.x * T + threadIdx.x; i < (m_max + 1) * CYC_WAVES * CYC_TOT; i += A.G * T) res_store(A.tot + i, open);
    for (int i = threadIdx.x; i < CYC_LDH * (CH_MSMALL + 1); i += T) C.hs[i] = 0.0;
    for (int i = threadIdx.x; i <= CH_MSMALL; i += T) C.s[i] = 0.0;
    res_drain();
    __syncthreads();
    if (threadIdx.x == 0) res_store(flag, A.epoch + 1);

    TV rc[S][RC > 0 ? RC : 1][SR][VX];
#pragma unroll
    for (int q = 0; q < S; ++q)
#pragma unroll
        for (int c = 0; c < RC; ++c)
#pragma unroll
            for (int i = 0; i < SR; ++i)
#pragma unroll
                for (int e = 0; e < VX; ++e) rc[q][c][i][e] = TV(0);
    // u_k at a strip's points (k > 0)
    auto mine = [&](int q) { return rows + (wv + q * NW) * SR * LANES + lane * VX; };
    // columns [0, RC) are in registers, [RC, lc) in LDS, the rest in memory
    auto local_col = [&](int q, int c, int i) { return cols + (((c - RC) * NS + wv + q * NW) * SR + i) * LANES + lane * VX; };
    // column c of strip q from memory (zeros from column `end` on)
    auto fetch = [&](int q, int c, int end, TV (&v)[SR][VX]) {
        const TV* Q = V + (size_t)(c < end ? c : 0) * A.ldv;
        const unsigned o = c < end ? bd[q] : OFF_ROW;
#pragma unroll
        for (int i = 0; i < SR; ++i) load_row<TV, VX>(grid_row(Q, P[q].r0 + i, n, bc), o, v[i]);
    };
    auto fetch_local = [&](int q, int c, int end, TV (&v)[SR][VX]) {
#pragma unroll
        for (int i = 0; i < SR; ++i) {
            const TV* l = local_col(q, c, i);
#pragma unroll
            for (int e = 0; e < VX; ++e) v[i][e] = c < end ? l[e] : TV(0);
        }
    };
    const int lfull = RC + (A.lc - RC) / 4 * 4, gfirst = RC + (A.lc - RC + 3) / 4 * 4;   // blocks of four columns
    for (int k = 0;; ++k) {
        TV w[S][SR][VX];
#pragma unroll
        for (int q = 0; q < S; ++q) {
            if constexpr (S > 1) __builtin_amdgcn_sched_barrier(0);   // one strip's rows in registers at a time
            TV u[NU][VX];
            {
                const TV* U = V + (size_t)k * A.ldv;
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    const bool here = k > 0 && (j < 2 ? above[q] : j < 2 + SR ? P[q].r0 + j - 2 < n : below[q]);
                    load_row<TV, VX, RES_SC1>(grid_row(U, P[q].r0 - 2 + j, n, bc), here ? bh[q] : bs[q], u[j]);
                }
                TV y[ND][VX];
#pragma unroll
                for (int j = 0; j < ND; ++j) load_row<TV, VX>(grid_row(Y, P[q].r0 - 1 + j, n, bc), bs[q], y[j]);
#pragma unroll
                for (int j = 0; j < ND; ++j) flip_if<TV, VX>(P[q].rev, y[j]);
#pragma unroll
                for (int j = 0; j < NU; ++j) {
                    flip_if<TV, VX>(P[q].rev, u[j]);
                    if (k > 0 && (j < 2 ? above[q] : j < 2 + SR ? P[q].r0 + j - 2 < n : below[q])) {
                        const int d = j < 2 ? j - nsx * SR : (j < 2 + SR ? j - 2 : j - 2 - SR + nsx * SR);
#pragma unroll
                        for (int e = 0; e < VX; ++e) {
                            const TV l = mine(q)[d * LANES + e];
                            u[j][e] = P[q].out ? l : u[j][e];
                        }
                    }
                }
                matvec_rows<TV, VX, MOB>(u, y, TV(k > 0 ? 1.0 : vscale0), eyre, ih2, e2ih2, mob, w[q]);
            }
            // dot products of the strip's points (zero outside the grid), in FP64
            double ud[SR][VX], wd[SR][VX];
#pragma unroll
            for (int i = 0; i < SR; ++i)
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    ud[i][e] = in[q][i] ? double(u[i + 2][e]) : 0.0;
                    wd[i][e] = in[q][i] ? double(w[q][i][e]) : 0.0;
                }
            auto sum_col = [&](const TV (&v)[SR][VX], double* a) {
                double su = 0.0, sw = 0.0;
#pragma unroll
                for (int i = 0; i < SR; ++i)
#pragma unroll
                    for (int e = 0; e < VX; ++e) {
                        const double qv = double(v[i][e]);
                        su = __builtin_fma(ud[i][e], qv, su);
                        sw = __builtin_fma(wd[i][e], qv, sw);
                    }
                a[0] = su;
                a[1] = sw;
            };
            auto row_sums = [&](double (&a)[8], int c0) {
                const double tot = wave_sum8(a);
                const int c = c0 + (hv >> 1);   // column of the value this lane holds
                if (hv >= 0 && c < k) red[(hv & 1) ? k + c : c][wv + q * NW] = 0.0 + tot;
            };
            TV qa[SR][VX], qb[SR][VX];
#pragma unroll
            for (int b = 0; b < RC / 4; ++b)
                if (4 * b < k) {
                    double a[8];
#pragma unroll
                    for (int c = 0; c < 4; ++c) sum_col(rc[q][4 * b + c], a + 2 * c);
                    row_sums(a, 4 * b);
                }
            // Columns in memory come last to first, and the update reads them first to last: of
            // the columns a pass read last, the next one finds some in the L2.
            if (k > gfirst) {
                int c0 = gfirst + (k - 1 - gfirst) / 4 * 4;
                fetch(q, c0, k, qa);
                for (; c0 >= gfirst; c0 -= 4) {   // two buffers that alternate, as in k_matvec_s
                    double a[8];
                    fetch(q, c0 + 1, k, qb);
                    sum_col(qa, a);
                    fetch(q, c0 + 2, k, qa);
                    sum_col(qb, a + 2);
                    fetch(q, c0 + 3, k, qb);
                    sum_col(qa, a + 4);
                    fetch(q, c0 > gfirst ? c0 - 4 : k, k, qa);
                    sum_col(qb, a + 6);
                    row_sums(a, c0);
                }
            }
            for (int c0 = RC; c0 < min(k, lfull); c0 += 4) {
                double a[8];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    fetch_local(q, c0 + c, k, qa);
                    sum_col(qa, a + 2 * c);
                }
                row_sums(a, c0);
            }
            if (S > 1 && k > lfull && lfull < gfirst) {   // a block whose first columns are in LDS
                double a[8];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    __builtin_amdgcn_sched_barrier(0);
                    const bool here = lfull + c < A.lc;
                    fetch(q, here ? k : lfull + c, k, qa);
                    fetch_local(q, min(lfull + c, A.lc - 1), k, qb);
#pragma unroll
                    for (int i = 0; i < SR; ++i)
#pragma unroll
                        for (int e = 0; e < VX; ++e) qa[i][e] = here ? (lfull + c < k ? qb[i][e] : TV(0)) : qa[i][e];
                    sum_col(qa, a + 2 * c);
                }
                row_sums(a, lfull);
            }
            double b8[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < SR; ++i)
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    b8[0] = __builtin_fma(ud[i][e], ud[i][e], b8[0]);
                    b8[1] = __builtin_fma(ud[i][e], wd[i][e], b8[1]);
                }
            const double tot = wave_sum8(b8);
            if (hv == 0 || hv == 1) red[2 * k + hv][wv + q * NW] = 0.0 + tot;
        }
        __syncthreads();
        if (C.stop) return;
        const int nrows = 2 * k + 2;
#pragma unroll
        for (int g = 0; g < NG; ++g)
            for (int i = threadIdx.x - g * (T / NG); i < nrows; i += T) {   // each group's rows by its own waves first
                if (i < 0) continue;
                double t = red[i][4 * g];
#pragma unroll
                for (int x = 1; x < 4; ++x) t += red[i][4 * g + x];
                if (gpos[g] >= 0) res_store(cyc_part(A, k, i, gpos[g]), t);
            }
        if (k == 0) cyc_all(A, C, A.epoch + 1);   // nothing is read before everyone has marked it
        // the sums this wave forms
        const int nw = cyc_waves(A);
        for (int q = r + A.G * (NW - 1 - wv); q < nrows * nw && !C.stop; q += A.G * NW)
            if (cyc_reduce(A, k, q / nw, q % nw) != CYC_OK) C.stop = 1;
        if (k == m_max) return;   // the last totals are for the test
        if (wv == 0) {
            if (C.stop || cyc_totals(A, C, k) != CYC_OK) C.stop = 1;
            else cyc_prepare(C, k, false, vscale0);
        }
        __syncthreads();
        if (C.stop) return;
        // everyone has read this iteration's partials: open the slots for iteration k + 2
        open_slots(k, nrows);
        // q_k and u_{k+1} at the strips' points
        const double cu = C.ab[k].x, cw = C.cbw, cq = C.cq;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            if constexpr (S > 1) __builtin_amdgcn_sched_barrier(0);
            TV qa[SR][VX], qb[SR][VX];
            double xq[SR][VX], xu[SR][VX];
            if (k > A.lc) fetch(q, A.lc, k, qa);
            if (k == 0) {   // column 0 is not normalised: its values as stored
                fetch(q, 0, 1, qb);
            } else {
#pragma unroll
                for (int i = 0; i < SR; ++i)
#pragma unroll
                    for (int e = 0; e < VX; ++e) qb[i][e] = mine(q)[i * LANES + e];
            }
#pragma unroll
            for (int i = 0; i < SR; ++i)
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    xq[i][e] = product(cu, in[q][i] ? double(qb[i][e]) : 0.0);
                    xu[i][e] = product(cw, in[q][i] ? double(w[q][i][e]) : 0.0);
                }
            auto add_col = [&](const TV (&v)[SR][VX], int c) {
                const double2 ab = c < k ? C.ab[c] : double2{0.0, 0.0};
#pragma unroll
                for (int i = 0; i < SR; ++i)
#pragma unroll
                    for (int e = 0; e < VX; ++e) {
                        xq[i][e] = __builtin_fma(ab.x, double(v[i][e]), xq[i][e]);
                        xu[i][e] = __builtin_fma(ab.y, double(v[i][e]), xu[i][e]);
                    }
            };
#pragma unroll
            for (int b = 0; b < RC / 4; ++b)
                if (4 * b < k) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) add_col(rc[q][4 * b + c], 4 * b + c);
                }
            for (int c = RC; c < min(k, A.lc); ++c) {
                fetch_local(q, c, k, qb);
                add_col(qb, c);
            }
            for (int c = A.lc; c < k; c += 2) {
                fetch(q, c + 1, k, qb);
                add_col(qa, c);
                fetch(q, c + 2, k, qa);
                add_col(qb, c + 1);
            }
            TV* Q = V + (size_t)k * A.ldv;
            TV* U = V + (size_t)(k + 1) * A.ldv;
#pragma unroll
            for (int i = 0; i < SR; ++i) {
                TV qn[VX], un[VX];
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    qn[e] = TV(xq[i][e]);
                    un[e] = TV(__builtin_fma(cq, double(qn[e]), xu[i][e]));   // with q_k as stored
                }
                const unsigned o = in[q][i] ? bo[q] : OFF_ROW;
                store_row<TV, VX, RES_SC1>(grid_row(U, P[q].r0 + i, n, bc), o, un);
                store_row<TV, VX>(grid_row(Q, P[q].r0 + i, n, bc), o, qn);
                TV* l = mine(q) + i * LANES;
#pragma unroll
                for (int e = 0; e < VX; ++e) {
                    l[e] = un[e];
                    qn[e] = in[q][i] ? qn[e] : TV(0);
                }
#pragma unroll
                for (int c = 0; c < RC; ++c)
                    if (c == k) {
#pragma unroll
                        for (int e = 0; e < VX; ++e) rc[q][c][i][e] = qn[e];
                    }
                if (k >= RC && k < A.lc) {
                    TV* lq = local_col(q, k, i);
#pragma unroll
                    for (int e = 0; e < VX; ++e) lq[e] = qn[e];
                }
            }
        }
        res_drain();
        __syncthreads();
        if (threadIdx.x == 0) res_store(flag, A.epoch + 2 + k);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (!nflag[f]) continue;
            long long t0 = 0;
            for (unsigned spin = 0; res_load(nflag[f]) < A.epoch + 2 + k; ++spin) {
                if (cyc_ended(A, spin, t0)) {
                    C.stop = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        // The next reads of u are ordinary loads, which the relaxed polls do not order: the
        // compiler is to keep them behind (the hardware does; no instruction).
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// The tests of one test workgroup take effect after those of the others
// before them.
struct ChainGate {
    const CycleArgs& A;
    CycCoef& C;
    int j;
    bool* mine;
    __device__ bool enter() {
        if (threadIdx.x == 0) {
            long long t0 = 0;
            if (j > 1)
                for (unsigned spin = 0; res_load(A.words + CH_RES_CHAIN + j - 1) != A.epoch; ++spin) {
                    if (cyc_ended(A, spin, t0)) {
                        C.stop = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
        }
        __syncthreads();
        *mine = !C.stop;
        return !C.stop;
    }
    __device__ void pending(Ctl*, double) {
        if (threadIdx.x == 0) res_store(A.words + CH_RES_CHAIN + j, A.epoch);
        *mine = false;
    }
};

constexpr int CYC_TESTS = 4;
constexpr int CYC_NPS = 32;   // padded order of the tests of Krylov dimensions below it (51 KB of LDS; above, 113)

template <int NPM>
__device__ __forceinline__ void cycle_tests(const CycleArgs& A, CycCoef& C, PhiShared<NPM>& S, int p) {
    if (threadIdx.x >= CH_BLOCK) return;   // the tests are for one workgroup of CH_BLOCK threads
    Ctl* ctl = A.ctl;
    for (int i = threadIdx.x; i < CYC_LDH * (CH_MSMALL + 1); i += CH_BLOCK) C.hs[i] = 0.0;
    for (int i = threadIdx.x; i <= CH_MSMALL; i += CH_BLOCK) C.s[i] = 0.0;
    taylor_coefficients(S.c);
    for (int i = threadIdx.x; i < A.G; i += CH_BLOCK) {   // the totals are marked
        long long t0 = 0;
        for (unsigned spin = 0; res_load(A.words + i * CH_RES_LINE) < A.epoch + 1; ++spin) {
            if (cyc_ended(A, spin, t0)) {
                C.stop = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    }
    __syncthreads();
    for (int j = 0; j <= A.m_max; ++j) {
        if (threadIdx.x < 64) {
            if (C.stop || cyc_totals(A, C, j) != CYC_OK) C.stop = 1;
            else cyc_prepare(C, j, j == A.m_max, 1.0);
        }
        __syncthreads();
        if (C.stop) return;
        if (j == 0 || j % CYC_TESTS != p) continue;
        bool mine = false;
        if (phi_test<NPM>(S, ctl, A.dflags ? A.dflags + A.I.slot : nullptr, j, C.rho, nullptr, C.hs, CYC_LDH,
                          ChainGate{A, C, j, &mine})) {
            if (mine) {   // this test ended the cycle
                for (int i = threadIdx.x; i < j * (j + 1); i += CH_BLOCK) {
                    const int c = i / (j + 1), q = i - c * (j + 1);
                    if (q <= c + 1) ctl->H[q + c * CH_LDH] = C.hs[q + c * CYC_LDH];
                }
                if (threadIdx.x == 0) res_store(A.words + CH_RES_DONE, A.epoch);
            }
            return;
        }
        __syncthreads();
    }
}

template <typename TV, int NW, int S, int VX, bool NEU, bool MOB>
__global__ __launch_bounds__(64 * NW, 1) void k_cycle(const CycleArgs A) {
    extern __shared__ __align__(16) unsigned char lds[];
    if (A.ctl->done | A.ctl->halted) return;
    CycCoef& C = *reinterpret_cast<CycCoef*>(lds);
    unsigned char* rest = lds + (sizeof(CycCoef) + 15) / 16 * 16;
    if (threadIdx.x == 0) C.stop = 0;
    __syncthreads();
    if ((int)blockIdx.x >= A.G) {
        const int p = blockIdx.x - A.G;
        if (A.m_max < CYC_NPS) cycle_tests(A, C, *reinterpret_cast<PhiShared<CYC_NPS>*>(rest), p);
        else cycle_tests(A, C, *reinterpret_cast<PhiShared<NPMAX>*>(rest), p);
        return;
    }
    double(*red)[NW * S] = reinterpret_cast<double(*)[NW * S]>(rest);
    TV* rows = reinterpret_cast<TV*>(rest + sizeof(double) * CYC_ROWS * NW * S);
    cycle_main<TV, NW, S, VX, NEU, MOB>(A, C, red, rows, rows + NW * S * SR * 64 * VX);
}

constexpr size_t CYC_LDS = 160 * 1024;

template <typename TV, int NW, int S, int VX, bool NEU, bool MOB>
hipError_t launch_cycle_t(const Table& t, const CycleArgs& a0, hipStream_t s) {
    CycleArgs A = a0;
    const size_t head = (sizeof(CycCoef) + 15) / 16 * 16, red = sizeof(double) * CYC_ROWS * NW * S;
    const size_t col = sizeof(TV) * NW * S * SR * 64 * VX;
    constexpr int RC = cyc_reg_cols(NW, S);
    // u and the columns that fit beside it; with one strip to a wave whole blocks of four (a
    // mixed block costs registers: 41 spilled at twelve waves, 920 us a cycle instead of 700)
    constexpr int Q = S > 1 ? 1 : 4;
    const int lds_cols = std::min((int)((CYC_LDS - head - red) / col - 1) / Q * Q, std::max(0, (A.m_max - RC + 3) / 4 * 4));
    A.lc = RC + lds_cols;
    const size_t phi = A.m_max < CYC_NPS ? sizeof(PhiShared<CYC_NPS>) : sizeof(PhiShared<NPMAX>);
    const size_t bytes = head + std::max(red + (1 + lds_cols) * col, phi);
    const auto f = k_cycle<TV, NW, S, VX, NEU, MOB>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(f), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)CYC_LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(f, dim3(A.G + CYC_TESTS), dim3(64 * NW), bytes, s, A);
    return hipGetLastError();
}

template <typename TV, int NW, int S, int VX>
hipError_t launch_cycle_v(const Table& t, const CycleArgs& A, hipStream_t s) {
    if (t.hinst[0].mob) return launch_cycle_t<TV, NW, S, VX, false, true>(t, A, s);
    if (t.hinst[0].bc == CH_BC_NEUMANN) return launch_cycle_t<TV, NW, S, VX, true, false>(t, A, s);
    return launch_cycle_t<TV, NW, S, VX, false, false>(t, A, s);
}

template <typename TV, int NW, int S>
hipError_t launch_cycle_n(const Table& t, const CycleArgs& A, hipStream_t s) {
    const int vx = t.hinst[0].vx;
    if constexpr (sizeof(TV) == 4) {
        if (vx >= 4) return launch_cycle_v<TV, NW, S, 4>(t, A, s);
    }
    if (vx >= 2) return launch_cycle_v<TV, NW, S, 2>(t, A, s);
    return launch_cycle_v<TV, NW, S, 1>(t, A, s);
}

}  // namespace

// The kernels of one basis precision and number of strips to a workgroup each have a file of their
// own: they take most of a minute to compile together, and a first launch loads the code of
// its file only (a process's first call 15.4 -> 14.5 ms at 64^2, of kernels in two files).
hipError_t launch_cycle_64_4(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_64_8(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_64_12(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_64_20(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_32_4(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_32_8(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_32_12(const Table& t, const CycleArgs& A, hipStream_t s);
hipError_t launch_cycle_32_20(const Table& t, const CycleArgs& A, hipStream_t s);
