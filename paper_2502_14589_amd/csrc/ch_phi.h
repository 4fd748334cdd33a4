// The small-matrix phi of the Krylov algorithm: the exponential of the
// Hessenberg matrix on the FP64 matrix cores, the residual test and the
// residual-time trace (Fig. 3; eqs. rm, phi_stop).  One workgroup of CH_BLOCK
// threads.
#pragma once

#include "ch_common.h"

namespace {

// ---------------------------------------------------------------------------
// Small-matrix exponential.  exp([[X, b], [0, 0]]) = [[e^X, phi(X) b], [0, 1]]
// (phi of eq. phi), so with X = -s H_jj and b = s e_1 the last column holds
// u = s phi(-s H_jj) e_1 and the first column exp(-s H_jj) e_1 = du/ds.
//
// Scaling and squaring with the degree-19 Taylor polynomial T_19: the
// argument is scaled by 2^-q so that its 1-norm is at most theta_19 =
// 1.2603811, the largest theta for which the relative backward error of T_19
// is at most 2^-53 (the power series of log(e^-x T_19(x)) has coefficients
// c_k, k >= 20, with sum_k |c_k| theta^(k-1) <= 2^-53; the backward-error
// analysis of Al-Mohy and Higham, SIAM J. Matrix Anal. Appl. 31 (2009)
// 970-989, applied to a Taylor instead of a Pade approximant).  T_19 is a
// polynomial, so the evaluation is matrix products only -- no linear solve --
// and all of them run on the FP64 matrix cores:
//   X^2, X^3, X^4;  T_19 = B_0 + X^4 (B_1 + X^4 (B_2 + X^4 (B_3 + X^4 B_4))),
//   B_i = sum_{q=0..3} X^q / (4i + q)!     (7 products),
// then q squarings.  Everything stays in LDS, in FP64.
// ---------------------------------------------------------------------------
// Orders are padded to a multiple of 16 for the matrix cores; the padding is
// a zero block of the argument, whose exponential is an identity block.
constexpr int NPMAX = 48;          // largest padded order in LDS
constexpr int NPBIG = 112;         // largest padded order (device scratch)
static_assert(CH_MSMALL + 1 <= NPMAX, "augmented matrix exceeds the padded LDS order");
static_assert(CH_MMAX + 1 <= NPBIG, "augmented matrix exceeds the padded order");
constexpr double THETA19 = 1.2603811;
constexpr int NLVL = 80;

// LDS of one phi evaluation for padded orders up to NPM; rows of stride
// LD = NPM + 1 (odd: rows fall in different banks).
template <int NPM>
struct PhiShared {
    static constexpr int LD = NPM + 1;
    double B[6][NPM * LD];      // X, X^2, X^3, X^4, two Horner / squaring buffers
    double c[20];               // 1 / k!
    double lvl[NLVL];           // lvl[kk] = resnorm at s 2^-kk from the squaring chain
    double red;
    int nsq;                    // squarings of the last evaluation (order-16 path)
    double hcol[NPM];           // column j - 1 of H when it is not yet in the control block
};

typedef double dbl4 __attribute__((ext_vector_type(4)));

// C = A B (+ epi(r, c) elementwise) for padded order np (a multiple of 16) on
// the FP64 matrix cores: 16x16 output tiles spread over the waves, K in steps
// of 4.  Lanes of the 16x16x4 instruction: lane l supplies A(l % 16, l / 16)
// and B(l / 16, l % 16) of its 16x4 and 4x16 slices and receives
// C(4 v + l / 16, l % 16) in element v.
struct NoEpi {
    __device__ double operator()(int, int) const { return 0.0; }
};

// NT = np / 16 tiles per direction.  The K loop is unrolled: every A and B
// operand of a tile is read from LDS before the first product, and even and
// odd K steps accumulate separately (two independent chains).
template <int NT, int PLD, typename Epi = NoEpi>
__device__ void mm_t(double* __restrict__ C, const double* __restrict__ A, const double* __restrict__ B,
                     Epi epi = Epi()) {
    constexpr int NP = 16 * NT, KS = NP / 4;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
#pragma unroll 1
    for (int t = wid; t < NT * NT; t += CH_BLOCK / 64) {
        const int ti = t / NT, tj = t - ti * NT;
        const double* a = A + (16 * ti + li) * PLD + lk;
        const double* b = B + lk * PLD + 16 * tj + li;
        double av[KS], bv[KS];
#pragma unroll
        for (int q = 0; q < KS; ++q) {
            av[q] = a[4 * q];
            bv[q] = b[4 * q * PLD];
        }
        dbl4 acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < KS; q += 2) {
            acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q], bv[q], acc0, 0, 0, 0);
            if (q + 1 < KS) acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(av[q + 1], bv[q + 1], acc1, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 16 * ti + 4 * v + lk, c = 16 * tj + li;
            C[r * PLD + c] = (acc0[v] + acc1[v]) + epi(r, c);
        }
    }
    __syncthreads();
}

template <int NPM, typename Epi = NoEpi>
__device__ void mm(double* __restrict__ C, const double* __restrict__ A, const double* __restrict__ B, int np,
                   Epi epi = Epi()) {
    constexpr int PLD = NPM + 1;
    if (np <= 16) mm_t<1, PLD>(C, A, B, epi);
    else if (NPM >= 32 && np <= 32) mm_t<(NPM >= 32 ? 2 : 1), PLD>(C, A, B, epi);
    else if (NPM >= 48 && np <= 48) mm_t<(NPM >= 48 ? 3 : 1), PLD>(C, A, B, epi);
    else if (NPM >= 64 && np <= 64) mm_t<(NPM >= 64 ? 4 : 1), PLD>(C, A, B, epi);
    else if (NPM >= 80 && np <= 80) mm_t<(NPM >= 80 ? 5 : 1), PLD>(C, A, B, epi);
    else if (NPM >= 96 && np <= 96) mm_t<(NPM >= 96 ? 6 : 1), PLD>(C, A, B, epi);
    else if (NPM >= 112) mm_t<(NPM >= 112 ? 7 : 1), PLD>(C, A, B, epi);
}

// B_i(r, c) = sum_{q=0..3} X^q(r, c) / (4i + q)!
template <int PLD>
struct TaylorBlock {
    const double* X[4];   // X^1 .. X^3 in X[1..3]
    const double* cf;
    int i;
    __device__ double operator()(int r, int c) const {
        const int o = r * PLD + c;
        const double* f = cf + 4 * i;
        return (r == c ? f[0] : 0.0) + f[1] * X[1][o] + f[2] * X[2][o] + f[3] * X[3][o];
    }
};

// ---------------------------------------------------------------------------
// Padded order 16: the whole exponential in the registers of wave 0.  A
// 16 x 16 matrix M is held in the layout the matrix cores return it in
// ("C layout": lane l, element v holds M(4 v + l / 16, l % 16)), which is
// also the layout of a right operand's K slices; a left operand is wanted
// transposed ("A layout": lane l, element q holds M(l % 16, 4 q + l / 16)),
// made by a round trip through a block of LDS that only wave 0 touches (one
// wave's LDS accesses complete in order, so no barrier is needed).  Same
// products, epilogue and accumulation order as mm_t, without a workgroup
// barrier per product.
// ---------------------------------------------------------------------------
__device__ __forceinline__ dbl4 mm16(const dbl4& a, const dbl4& b) {
    dbl4 c0 = {0.0, 0.0, 0.0, 0.0}, c1 = {0.0, 0.0, 0.0, 0.0};
    c0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], b[0], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], b[1], c1, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], b[2], c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], b[3], c1, 0, 0, 0);
    return c0 + c1;
}

// C layout -> A layout through T (16 rows of stride 17)
__device__ __forceinline__ dbl4 to_a(const dbl4& c, double* T) {
    const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) T[(4 * v + lk) * 17 + li] = c[v];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    dbl4 a;
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = T[li * 17 + 4 * q + lk];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    return a;
}

__device__ __forceinline__ double elem(const dbl4& e, int v) {
    return v == 0 ? e[0] : (v == 1 ? e[1] : (v == 2 ? e[2] : e[3]));
}

// As expm_aug for n = j + 1 <= 16.  Call from every thread.
template <int NPM>
__device__ const double* expm16(PhiShared<NPM>& S, const double* __restrict__ H, int ldh, const double* hlast,
                                int j, double s, double hnext, int* nsq_out) {
    constexpr int PLD = PhiShared<NPM>::LD;
    static_assert(16 * 17 <= NPM * PLD, "transpose block");
    double* E = S.B[4];
    __syncthreads();   // every wave's reads of the previous evaluation are done
    if (threadIdx.x < 64) {
        const int l = threadIdx.x, li = l & 15, lk = l >> 4;
        double* T = S.B[5];
        dbl4 x;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int r = 4 * v + lk, c = li;
            double val = 0.0;
            if (r < j && c < j) val = -s * (hlast && c == j - 1 ? hlast[r] : H[r + c * ldh]);
            else if (r == 0 && c == j) val = s;
            x[v] = val;
        }
        // 1-norm: column sums (rows over v and the four lane groups), max over columns
        double cs = (fabs(x[0]) + fabs(x[1])) + (fabs(x[2]) + fabs(x[3]));
        cs += __shfl_xor(cs, 16, 64);
        cs += __shfl_xor(cs, 32, 64);
        const double nrm = wave_max(cs);
        int nsq = 0;
        if (nrm > THETA19 && nrm < __builtin_inf()) nsq = (int)ceil(log2(nrm / THETA19));
        if (nsq > 1100) nsq = 1100;
        const double scale = ldexp(1.0, -nsq);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] *= scale;
        const dbl4 xa = to_a(x, T);
        const dbl4 x2 = mm16(xa, x);
        const dbl4 x2a = to_a(x2, T);
        const dbl4 x3 = mm16(x2a, x);
        const dbl4 x4a = to_a(mm16(x2a, x2), T);
        // T_19 = B_0 + X^4 (B_1 + X^4 (B_2 + X^4 (B_3 + X^4 B_4))),
        // B_i = sum_{q=0..3} X^q / (4i + q)!
        auto blk = [&](int i) {
            const double* f = S.c + 4 * i;
            dbl4 b;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                b[v] = ((4 * v + lk == li ? f[0] : 0.0) + f[1] * x[v] + f[2] * x2[v]) + f[3] * x3[v];
            return b;
        };
        dbl4 R = blk(4);
        for (int i = 3; i >= 0; --i) R = mm16(x4a, R) + blk(i);
        // resnorm at every dyadic level: element (j - 1, j)
        const int lr = j + 16 * ((j - 1) & 3), vr = (j - 1) >> 2;
        if (nsq < NLVL) {
            const double rv = hnext * fabs(readlane_d(elem(R, vr), lr));
            if (l == 0) S.lvl[nsq] = rv;
        }
        for (int i = 1; i <= nsq; ++i) {
            R = mm16(to_a(R, T), R);
            const int kk = nsq - i;
            if (kk < NLVL) {
                const double rv = hnext * fabs(readlane_d(elem(R, vr), lr));
                if (l == 0) S.lvl[kk] = rv;
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) E[(4 * v + lk) * PLD + li] = R[v];
        if (l == 0) S.nsq = nsq;
    }
    __syncthreads();
    *nsq_out = S.nsq;
    return E;
}

// exp(s [[-H_jj, e_1], [0, 0]]); returns the LDS matrix holding it and the
// number of squarings in *nsq_out.  Records resnorm at every dyadic level of
// the squaring chain in S.lvl.  Column j - 1 of H comes from hlast when it is
// given (not yet in the control block), else from H.
template <int NPM>
__device__ const double* expm_aug(PhiShared<NPM>& S, const double* __restrict__ H, int ldh, const double* hlast,
                                  int j, double s, double hnext, int* nsq_out) {
    constexpr int PLD = PhiShared<NPM>::LD;
    const int n = j + 1;
    if (n <= 16) return expm16<NPM>(S, H, ldh, hlast, j, s, hnext, nsq_out);
    const int np = (n + 15) & ~15;
    double* X1 = S.B[0];
    for (int idx = threadIdx.x; idx < np * np; idx += CH_BLOCK) {
        const int r = idx / np, c = idx - r * np;
        double v = 0.0;
        if (r < j && c < j) v = -s * (hlast && c == j - 1 ? hlast[r] : H[r + c * ldh]);
        else if (r == 0 && c == j) v = s;
        X1[r * PLD + c] = v;
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        double cs = 0.0;
        if ((int)threadIdx.x < n)
            for (int r = 0; r < n; ++r) cs += fabs(X1[r * PLD + threadIdx.x]);
        cs = wave_max(cs);
        if (threadIdx.x == 0) S.red = cs;
    }
    __syncthreads();
    const double nrm = S.red;
    int nsq = 0;
    if (nrm > THETA19 && nrm < __builtin_inf()) nsq = (int)ceil(log2(nrm / THETA19));
    if (nsq > 1100) nsq = 1100;
    const double scale = ldexp(1.0, -nsq);
    for (int idx = threadIdx.x; idx < n * n; idx += CH_BLOCK) {
        const int r = idx / n, c = idx - r * n;
        X1[r * PLD + c] *= scale;
    }
    __syncthreads();
    mm<NPM>(S.B[1], X1, X1, np);         // X^2
    mm<NPM>(S.B[2], S.B[1], X1, np);     // X^3
    mm<NPM>(S.B[3], S.B[1], S.B[1], np); // X^4
    // T_19 = B_0 + X^4 (B_1 + X^4 (B_2 + X^4 (B_3 + X^4 B_4)))
    TaylorBlock<PLD> tb{{nullptr, S.B[0], S.B[1], S.B[2]}, S.c, 4};
    double* R = S.B[4];
    double* R2 = S.B[5];
    for (int idx = threadIdx.x; idx < np * np; idx += CH_BLOCK) {
        const int r = idx / np, c = idx - r * np;
        R[r * PLD + c] = tb(r, c);
    }
    __syncthreads();
    for (int i = 3; i >= 0; --i) {
        tb.i = i;
        mm<NPM>(R2, S.B[3], R, np, tb);
        double* t = R;
        R = R2;
        R2 = t;
    }
    double* X = R;
    double* Y = R2;
    if (threadIdx.x == 0 && nsq < NLVL) S.lvl[nsq] = hnext * fabs(X[(j - 1) * PLD + j]);
    for (int i = 1; i <= nsq; ++i) {
        mm<NPM>(Y, X, X, np);
        double* tmp = X;
        X = Y;
        Y = tmp;
        const int kk = nsq - i;
        if (threadIdx.x == 0 && kk < NLVL) S.lvl[kk] = hnext * fabs(X[(j - 1) * PLD + j]);
    }
    __syncthreads();
    *nsq_out = nsq;
    return X;
}

__device__ void taylor_coefficients(double* c) {
    if (threadIdx.x == 0) {   // 1 / k!, k = 0..19
        double f = 1.0;
        c[0] = 1.0;
        for (int i = 1; i < 20; ++i) {
            f /= double(i);
            c[i] = f;
        }
    }
}

template <int PLD>
__device__ void store_u(Ctl* ctl, const double* E, int j) {
    for (int i = threadIdx.x; i < j; i += CH_BLOCK) ctl->u[i] = E[i * PLD + j];
}

// ---------------------------------------------------------------------------
// phi of the Hessenberg matrix after an Arnoldi iteration, convergence test
// and residual-time trace (Fig. 3; eqs. rm, phi_stop).  One workgroup.
// MGS iteration k: dimension j = k + 1, h_{j+1,j} from the norm
// partials.  DCGS2 (DC) iteration k >= 1: dimension j = k, H final up to
// column j - 1 (written by the update launch of the same iteration).
//
// Trace: the squaring chain of the evaluation at tau0 gives resnorm at every
// s = tau0 2^-kk; the largest passing one brackets the crossing in
// [tau0 2^-kk, tau0 2^(1-kk)] (further halvings are evaluated if the chain is
// too short).  The crossing resnorm(s) = tol_phi is then located by Newton's
// method on log resnorm against log s, using d resnorm/ds =
// h_{j+1,j} |e_j^T exp(-s H) e_1| from the same exponential, safeguarded by the
// bracket, to a relative precision of about 1e-14.
// ---------------------------------------------------------------------------
// One phi test of Krylov dimension j (h_{j+1,j} = hnext, H columns 0..j-1
// final): returns true when the Krylov cycle is finished (converged, traced
// at the last dimension, or failed).
// H: columns 0 .. j - 1, leading dimension ldh.  gate: what happens once the
// residual at tau0 is known, before anything is written for the cycle: enter()
// is false when an earlier test has ended the cycle, pending() takes the
// residual of a test that does not end it.
struct OpenGate {
    __device__ bool enter() { return true; }
    __device__ void pending(Ctl* ctl, double r) {
        if (threadIdx.x == 0) ctl->resnorm = r;
    }
};

template <int NPM, typename Gate = OpenGate>
__device__ __forceinline__ bool phi_test(PhiShared<NPM>& S, Ctl* ctl, int* dflag, int j, double hnext,
                                         const double* hlast, const double* H, int ldh, Gate gate = Gate()) {
    constexpr int PLD = PhiShared<NPM>::LD;
    // One exponential per pass of the loop below (a single call site keeps
    // the register footprint of one evaluation).  Phases: 0 the test at
    // tau0; 1 dyadic steps below the squaring chain, until one passes; 2
    // Newton inside the bracket; 3 the final evaluation at the chosen step.
    const double tau0 = ctl->tau0, tol = ctl->tol_phi, tau_min = ctl->tau_min;
    int phase = 0, kk = 0, it = 0, kchain = 0;   // kchain: deepest level of the first squaring chain
    double s = tau0, lo = -1.0, hi = 0.0, rlo = 0.0, rhi = 0.0, prev = 0.0, step_prev = 1.0;
    int fail = 0;   // ch_status of a failed cycle
    auto finish = [&](const double* E, double sf, double res, int conv) {
        store_u<PLD>(ctl, E, j);
        if (threadIdx.x == 0) {
            ctl->tau_acc = sf;
            ctl->resnorm = res;
            ctl->converged = conv;
            if (!conv) ctl->traced = 1;
            ctl->done = 1;
            if (dflag) *dflag = ctl->cyc;
            ctl->j = j;
        }
    };
    // first Newton iterate inside [lo, hi]: log resnorm against log2(s / lo)
    // through the chain's values at lo / 2, lo and hi (quadratic) when they
    // are at hand, else through lo and hi
    auto first_guess = [&](bool chain) {
        double g = -1.0;
        if (rlo > 0.0 && rhi > rlo) {
            const double y0 = log(rlo), y1 = log(rhi), yt = log(tol);
            double x = (yt - y0) / (y1 - y0);
            const int kl = (int)lrint(log2(tau0 / lo));   // lo = tau0 2^-kl
            if (chain && kl + 1 <= kchain && S.lvl[kl + 1] > 0.0 && S.lvl[kl + 1] < rlo) {
                const double ym = log(S.lvl[kl + 1]);
                const double bq = 0.5 * (y1 - ym), cq = 0.5 * (y1 + ym) - y0;
                const double disc = __builtin_fma(bq, bq, -product(4.0 * cq, y0 - yt));
                if (fabs(cq) > 1e-12 * fabs(bq) && disc >= 0.0) {
                    const double xq = (-bq + sqrt(disc)) / (2.0 * cq);
                    if (xq > 0.0 && xq < 1.0) x = xq;
                }
            }
            g = lo * exp2(x);
        }
        if (!(g > lo && g < hi)) g = 0.5 * (lo + hi);
        return g;
    };
    for (;;) {
        int nsq = 0;
        const double* E = expm_aug<NPM>(S, H, ldh, hlast, j, s, hnext, &nsq);
        const double uj = E[(j - 1) * PLD + j];
        const double r = hnext * fabs(uj);
        if (phase == 0) {
            if (!gate.enter()) return true;
            if (!(r < __builtin_inf())) {
                fail = CH_ENONFINITE;
                break;
            }
            if (r <= tol) {
                finish(E, tau0, r, 1);
                return true;
            }
            if (j < ctl->m_max) {
                gate.pending(ctl, r);
                return false;
            }
            // ---- trace: largest passing dyadic step below tau0 ----
            const int kmax = nsq < NLVL - 1 ? nsq : NLVL - 1;
            kchain = kmax;
            for (int q = 1; q <= kmax; ++q) {
                if (S.lvl[q] <= tol) {
                    lo = ldexp(tau0, -q);
                    rlo = S.lvl[q];
                    hi = 2.0 * lo;
                    rhi = S.lvl[q - 1];
                    break;
                }
            }
            if (lo < 0.0) {   // below the chain: more halvings, one evaluation each
                prev = S.lvl[kmax];
                kk = kmax + 1;
                s = ldexp(tau0, -kk);
                if (kk > 1100 || s == 0.0 || s < tau_min) {
                    fail = CH_ETAU_UNDERFLOW;
                    break;
                }
                phase = 1;
                continue;
            }
            if (lo < tau_min) {
                fail = CH_ETAU_UNDERFLOW;
                break;
            }
            s = first_guess(true);
            phase = 2;
            continue;
        }
        if (phase == 1) {
            if (r <= tol) {
                lo = s;
                rlo = r;
                hi = 2.0 * s;
                rhi = prev;
                if (lo < tau_min) {
                    fail = CH_ETAU_UNDERFLOW;
                    break;
                }
                s = first_guess(false);
                phase = 2;
                continue;
            }
            prev = r;
            ++kk;
            s = ldexp(tau0, -kk);
            if (kk > 1100 || s == 0.0 || s < tau_min) {
                fail = CH_ETAU_UNDERFLOW;
                break;
            }
            continue;
        }
        if (phase == 2) {
            // Newton on log resnorm against log s, d resnorm / ds =
            // h_{j+1,j} |e_j^T exp(-s H) e_1| from the same exponential; it
            // converges quadratically, so a Newton step below 1e-7 s after
            // one below 1e-3 s leaves the next iterate within about 1e-14 of
            // the crossing.  Bisection steps (Newton iterate outside the
            // bracket) say nothing about convergence and reset that count.
            const double dr = hnext * (uj >= 0.0 ? 1.0 : -1.0) * E[(j - 1) * PLD + 0];
            if (r <= tol) {
                lo = s;
                rlo = r;
            } else {
                hi = s;
                rhi = r;
            }
            double sn = -1.0;
            if (r > 0.0 && dr > 0.0) sn = s * exp(-log(r / tol) * r / (s * dr));
            bool stop;
            if (hi - lo <= 0x1p-47 * lo) {
                sn = lo;
                stop = true;
            } else if (sn > 0.0 && fabs(sn - s) <= 1e-14 * s) {
                // s is the crossing to rounding (from the passing side the
                // Newton iterate may round onto lo itself); passing, it is
                // the step, and this exponential its result
                if (r <= tol) {
                    finish(E, s, r, 0);
                    return true;
                }
                stop = true;
            } else {
                const bool newton = sn > lo && sn < hi;
                if (!newton) sn = 0.5 * (lo + hi);
                const double step = fabs(sn - s) / s;
                stop = (newton && step <= 1e-7 && step_prev <= 1e-3) || ++it >= 60;
                step_prev = newton ? step : 1.0;
            }
            s = sn;
            if (stop) phase = 3;
            continue;
        }
        finish(E, s, r, 0);   // phase 3
        return true;
    }
    if (threadIdx.x == 0) {
        ctl->status = fail;
        ctl->halted = 1;
        ctl->done = 1;
        if (dflag) *dflag = ctl->cyc;
        ctl->j = 0;
    }
    return true;
}

}  // namespace
