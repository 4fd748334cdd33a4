// Row-wise stencil arithmetic of the 2-D kernels (row strips, ch_strip.hip;
// resident LIM stages, ch_resident.hip; resident Krylov cycles, ch_cycle.h): a
// lane holds VX consecutive columns of each row it touches.
#pragma once

#include "ch_common.h"

namespace {

// Raw buffer resource over one grid row (wave-uniform base; lanes address it
// by byte offset; an offset past the row reads zero and drops a store).  The
// last word is the gfx9 data-format word.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

using u32x2 = unsigned __attribute__((ext_vector_type(2)));
using u32x4 = unsigned __attribute__((ext_vector_type(4)));

// VX consecutive values of type T at byte offset `bo` of row resource r.
// AUX: the cache-policy bits of the access (16: agent scope, ch_resident.h).
template <typename T, int VX, int AUX = 0>
__device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t r, unsigned bo, T (&v)[VX]) {
    constexpr unsigned so = 0;
    constexpr int B = VX * (int)sizeof(T);
    if constexpr (B == 4) {
        v[0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, bo, so, AUX));
    } else if constexpr (B == 8) {
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, bo, so, AUX);
        struct P { T e[VX]; };
        const P p = __builtin_bit_cast(P, x);
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = p.e[e];
    } else if constexpr (B == 16) {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, bo, so, AUX);
        struct P { T e[VX]; };
        const P p = __builtin_bit_cast(P, x);
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = p.e[e];
    } else {
        static_assert(B == 32, "row chunk of 4, 8, 16 or 32 bytes");
        constexpr int H = VX / 2;
        T a[H], c[H];
        load_row<T, H, AUX>(r, bo, a);
        load_row<T, H, AUX>(r, bo + 16u, c);
#pragma unroll
        for (int e = 0; e < H; ++e) {
            v[e] = a[e];
            v[H + e] = c[e];
        }
    }
}

template <typename T, int VX, int AUX = 0>
__device__ __forceinline__ void store_row(__amdgpu_buffer_rsrc_t r, unsigned bo, const T (&v)[VX]) {
    constexpr unsigned so = 0;
    constexpr int B = VX * (int)sizeof(T);
    struct P { T e[VX]; };
    P p;
#pragma unroll
    for (int e = 0; e < VX; ++e) p.e[e] = v[e];
    if constexpr (B == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, p), r, bo, so, AUX);
    } else if constexpr (B == 8) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, p), r, bo, so, AUX);
    } else if constexpr (B == 16) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, p), r, bo, so, AUX);
    } else {
        static_assert(B == 32, "row chunk of 4, 8, 16 or 32 bytes");
        constexpr int H = VX / 2;
        T a[H], c[H];
#pragma unroll
        for (int e = 0; e < H; ++e) {
            a[e] = v[e];
            c[e] = v[H + e];
        }
        store_row<T, H, AUX>(r, bo, a);
        store_row<T, H, AUX>(r, bo + 16u, c);
    }
}

// Whole-wave DPP shifts: lane L receives lane L - 1 (from_left) or L + 1
// (from_right); the wave's end lanes receive 0 (only halo lanes read them).
enum { DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138 };

template <int CTRL>
__device__ __forceinline__ float wave_shift(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ double wave_shift(double x) {
    const unsigned long long v = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Unscaled -Laplacian (4 c - (l + r) - (u + d)) at element e of row `c`,
// with rows `up` and `dn` above and below.  The x neighbours across the
// lane boundary arrive by DPP (xl: the left lane's last element, xr: the
// right lane's first).
template <typename T, int VX>
__device__ __forceinline__ T lap5(const T (&up)[VX], const T (&c)[VX], const T (&dn)[VX], T xl, T xr, int e) {
    const T l = e > 0 ? c[e - 1] : xl;
    const T r = e < VX - 1 ? c[e + 1] : xr;
    const T nb = (l + r) + (up[e] + dn[e]);
    return T(4) * c[e] - nb;
}

// Flux form of the variable-mobility operator (Section 2, Remark 1),
// unscaled: sum over the four neighbours k of (m_c + m_k)/2 (q_c - q_k), the
// mobilities m laid out as the values q (mxl, mxr: the lane neighbours' m).
// With m = 1 it equals lap5.
template <typename T, int VX>
__device__ __forceinline__ T lap5m(const T (&up)[VX], const T (&c)[VX], const T (&dn)[VX], T xl, T xr,
                                   const T (&mup)[VX], const T (&mc)[VX], const T (&mdn)[VX], T mxl, T mxr, int e) {
    const T l = e > 0 ? c[e - 1] : xl, r = e < VX - 1 ? c[e + 1] : xr;
    const T ml = e > 0 ? mc[e - 1] : mxl, mr = e < VX - 1 ? mc[e + 1] : mxr;
    const T q = c[e], m = mc[e];
    const T fx = (m + ml) * (q - l) + (m + mr) * (q - r);
    const T fy = (m + mup[e]) * (q - up[e]) + (m + mdn[e]) * (q - dn[e]);
    return T(0.5) * (fx + fy);
}

// The outer operator at element e of row c: A (MOB false) or A_M (MOB true,
// mobility rows m), both unscaled.
template <bool MOB, typename T, int VX>
__device__ __forceinline__ T outer_op(const T (&up)[VX], const T (&c)[VX], const T (&dn)[VX], T xl, T xr,
                                      const T (&mup)[VX], const T (&mc)[VX], const T (&mdn)[VX], T mxl, T mxr, int e) {
    if constexpr (MOB) return lap5m<T, VX>(up, c, dn, xl, xr, mup, mc, mdn, mxl, mxr, e);
    else return lap5<T, VX>(up, c, dn, xl, xr, e);
}

// Mobility coefficients (from the control block) of a MOB launch.
struct Mob {
    double m0, m1;
};
__device__ __forceinline__ Mob mob_of(const Ctl* ctl, bool on) { return on ? Mob{ctl->mob0, ctl->mob1} : Mob{0.0, 0.0}; }

// Mobility rows of a block of state rows (MOB), or nothing.
template <bool MOB, typename T, int VX, int NR>
struct MobRows {
    T m[MOB ? NR : 1][VX];
    __device__ __forceinline__ void set(int j, const T (&y)[VX], T m0, T m1) {
        if constexpr (MOB) {
#pragma unroll
            for (int e = 0; e < VX; ++e) m[j][e] = mobility_of(y[e], m0, m1);
        }
    }
    __device__ __forceinline__ const T (&row(int j) const)[VX] { return m[MOB ? j : 0]; }
    __device__ __forceinline__ T left(int j) const {
        if constexpr (MOB) return wave_shift<DPP_WAVE_SHR1>(m[j][VX - 1]);
        else return T(0);
    }
    __device__ __forceinline__ T right(int j) const {
        if constexpr (MOB) return wave_shift<DPP_WAVE_SHL1>(m[j][0]);
        else return T(0);
    }
};

template <typename T>
__device__ __forceinline__ T dcoef(T y, int eyre) {
    return T(3) * y * y - T(1) + T(eyre);
}
template <typename T>
__device__ __forceinline__ T ccoef(T y, int eyre) {
    return T(2) * y * y * y + (eyre ? y : T(0));
}

constexpr int SR = CH_STRIP_ROWS;

// Strip geometry of one wave.
template <int VX>
struct StripPos {
    int r0;         // first row
    int xl;         // lane's first column, in [0, n)
    bool out;       // the lane's columns are outputs of this strip
    bool need;      // ... or the halo of one
    bool rev;       // the lane's values are those of its columns in reverse (Neumann mirror)
};

// Grid column of the first of the VX columns [c, c + VX) of a lane (c a
// multiple of VX, VX dividing n, -n < c < 2n): periodic wrap, or, past a
// Neumann boundary, the mirror chunk [-c - VX, -c) or [2n - c - VX, 2n - c),
// whose values the lane then takes in reverse order (rev).
template <int VX>
__device__ __forceinline__ int chunk_col(int c, int n, int bc, bool& rev) {
    rev = false;
    if (bc == CH_BC_NEUMANN && (c < 0 || c >= n)) {
        rev = VX > 1;
        const int x = c < 0 ? -c - VX : 2 * n - c - VX;
        return x < 0 ? 0 : x;   // lanes past the halo (never read) stay in bounds
    }
    const int x = c % n;
    return x < 0 ? x + n : x;
}

// Reverse the VX values of a lane when `rev`, without a branch.
template <typename T, int VX>
__device__ __forceinline__ void flip_if(bool rev, T (&v)[VX]) {
    if constexpr (VX > 1) {
        T t[VX];
#pragma unroll
        for (int e = 0; e < VX; ++e) t[e] = v[VX - 1 - e];
#pragma unroll
        for (int e = 0; e < VX; ++e) v[e] = rev ? t[e] : v[e];
    }
}

// A lane offset past every row: the load returns zeros without a memory
// access (lanes that neither own nor border an output column).
constexpr unsigned OFF_ROW = 0x80000000u;

template <int VX>
__device__ __forceinline__ StripPos<VX> strip_pos(int s, int nsx, int n, int lane, int bc) {
    constexpr int HL = CH_STRIP_HALO(VX), OW = strip_cols(VX);
    StripPos<VX> p;
    const int sx = s % nsx;
    p.r0 = (s / nsx) * SR;
    const int c = sx * OW + (lane - HL) * VX;     // first column, before the boundary fold
    p.xl = chunk_col<VX>(c, n, bc, p.rev);
    p.out = lane >= HL && lane < 64 - HL && c < n;
    p.need = c < n + HL * VX;
    return p;
}

// Row r (r in [-n, 2n): periodic wrap or Neumann mirror) of an instance's
// field of n x n values of type T.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t grid_row(const T* f, int r, int n, int bc) {
    return row_rsrc(f + (size_t)bc_index(r, n, bc) * n, (unsigned)n * (unsigned)sizeof(T));
}

// ---------------------------------------------------------------------------
// Arithmetic of one LIM stage at one point (Fig. 1).  Which products are fused
// into sums is written out, and the stage's result is rounded, so that every
// kernel that forms a stage gives the same bits whether the stage before it
// came from memory or from a register of the same launch.
// ---------------------------------------------------------------------------
// d z + eps^2 A z - c; lap: the unscaled A z, e2ih2 = eps^2 / h^2.
__device__ __forceinline__ double lim_inner(double d, double z, double e2ih2, double lap, double c) {
#pragma clang fp contract(off)
    return __builtin_fma(d, z, e2ih2 * lap) - c;
}

// (y + ta z - tau h^-2 op) inv; op: the unscaled outer operator of the inner expression.
__device__ __forceinline__ double lim_next(double y, double ta, double z, double tau, double inv_h2, double op,
                                           double inv) {
#pragma clang fp contract(off)
    return __builtin_fma(-tau, inv_h2 * op, __builtin_fma(ta, z, y)) * inv;
}

// outer_op of a LIM stage.
template <bool MOB, int VX>
__device__ __forceinline__ double lim_outer(const double (&up)[VX], const double (&c)[VX], const double (&dn)[VX],
                                            double xl, double xr, const double (&mup)[VX], const double (&mc)[VX],
                                            const double (&mdn)[VX], double mxl, double mxr, int e) {
#pragma clang fp contract(off)
    const double l = e > 0 ? c[e - 1] : xl, r = e < VX - 1 ? c[e + 1] : xr;
    if constexpr (MOB) {
        const double ml = e > 0 ? mc[e - 1] : mxl, mr = e < VX - 1 ? mc[e + 1] : mxr;
        const double q = c[e], m = mc[e];
        const double fx = __builtin_fma(m + ml, q - l, (m + mr) * (q - r));
        const double fy = __builtin_fma(m + mup[e], q - up[e], (m + mdn[e]) * (q - dn[e]));
        return 0.5 * (fx + fy);
    } else {
        return __builtin_fma(4.0, c[e], -((l + r) + (up[e] + dn[e])));
    }
}

__device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

// w = Ahat (sc u) on a strip's rows r0 .. r0 + SR - 1 from the operand's rows
// r0 - 2 .. (scaled in place) and the state's rows r0 - 1 ...  Which products are fused
// into sums is written out, so that every kernel that forms a matvec gives the
// same bits: of two neighbours the outer row's, or the one nearer the lane's
// middle, enters unscaled with its scaling fused.
template <typename TV, int VX, bool MOB>
__device__ __forceinline__ void matvec_rows(TV (&u)[SR + 4][VX], const TV (&y)[SR + 2][VX], TV sc, int eyre, TV ih2,
                                            TV e2ih2, Mob mob, TV (&w)[SR][VX]) {
#pragma clang fp contract(off)
    constexpr int NU = SR + 4, ND = SR + 2;
    TV raw[NU][VX];
#pragma unroll
    for (int j = 0; j < NU; ++j)
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            raw[j][e] = u[j][e];
            u[j][e] *= sc;
        }
    MobRows<MOB, TV, VX, ND> mb;
#pragma unroll
    for (int j = 0; j < ND; ++j) mb.set(j, y[j], TV(mob.m0), TV(mob.m1));
    // inner expression d u + eps^2 A u on rows r0 - 1 .. r0 + SR
    TV q[ND][VX];
#pragma unroll
    for (int j = 0; j < ND; ++j) {
        const TV xl = wave_shift<DPP_WAVE_SHR1>(u[j + 1][VX - 1]), xr = wave_shift<DPP_WAVE_SHL1>(u[j + 1][0]);
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const TV l = e > 0 ? u[j + 1][e - 1] : xl, r = e < VX - 1 ? u[j + 1][e + 1] : xr;
            TV nx;
            if (VX == 1) nx = l + r;
            else if (2 * e < VX) nx = fma_of(sc, raw[j + 1][e < VX - 1 ? e + 1 : e], l);
            else nx = fma_of(sc, raw[j + 1][e > 0 ? e - 1 : e], r);
            const TV ny = 2 * j < ND ? fma_of(sc, raw[j][e], u[j + 2][e]) : fma_of(sc, raw[j + 2][e], u[j][e]);
            const TV lap = fma_of(TV(4), u[j + 1][e], -(nx + ny));
            const TV d = fma_of(y[j][e], TV(3) * y[j][e], TV(-1)) + TV(eyre);
            if (VX == 4 && (e == 1 || e == 2)) q[j][e] = fma_of(lap, e2ih2, d * u[j + 1][e]);
            else q[j][e] = fma_of(d, u[j + 1][e], lap * e2ih2);
        }
    }
    // w = A q (A_M q with mobility) on rows r0 .. r0 + SR - 1
#pragma unroll
    for (int i = 0; i < SR; ++i) {
        const TV xl = wave_shift<DPP_WAVE_SHR1>(q[i + 1][VX - 1]), xr = wave_shift<DPP_WAVE_SHL1>(q[i + 1][0]);
        const TV ml = mb.left(i + 1), mr = mb.right(i + 1);
#pragma unroll
        for (int e = 0; e < VX; ++e) {
            const TV c = q[i + 1][e];
            const TV l = e > 0 ? q[i + 1][e - 1] : xl, r = e < VX - 1 ? q[i + 1][e + 1] : xr;
            if constexpr (MOB) {
                const TV m = mb.row(i + 1)[e];
                const TV a = m + (e > 0 ? mb.row(i + 1)[e - 1] : ml), b = m + (e < VX - 1 ? mb.row(i + 1)[e + 1] : mr);
                const TV fx = 2 * e + 1 < VX ? fma_of(b, c - r, a * (c - l)) : fma_of(a, c - l, b * (c - r));
                const TV fy = fma_of(m + mb.row(i)[e], c - q[i][e], (m + mb.row(i + 2)[e]) * (c - q[i + 2][e]));
                w[i][e] = ih2 * (TV(0.5) * (fx + fy));
            } else {
                w[i][e] = ih2 * fma_of(TV(4), c, -((l + r) + (q[i][e] + q[i + 2][e])));
            }
        }
    }
}

}  // namespace
