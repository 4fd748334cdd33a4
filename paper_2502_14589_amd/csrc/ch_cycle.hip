// Resident Krylov cycles (ch_cycle.h): which grids take them, and their launch.
#include "ch_cycle.h"

size_t cycle_doubles() { return (size_t)2 * CYC_PART + (size_t)(CH_MSMALL + 1) * CYC_WAVES * CYC_TOT; }

// The cycle is resident where every strip of the launches has a wave of its own there
// (at most CH_WBLK_MAX groups of four), the groups fit on the CUs one, two, three
// (a strip to a wave) or five (two to a wave) to a workgroup, and the phi tests fit
// in LDS.  The fewest per workgroup: most of a small grid's columns then stay on the
// chip.  Three steps of 30 iterations as launches and resident, us: 64^2 FP64
// 1040, 590; 512^2 1155, 690; 640^2 1290, 730; 701^2 (five groups) 1505, 1190; 1024^2
// 2270, 1860; FP32 1024^2 1520, 1030; 1400^2 2200, 2020.  Dimensions 32 to 47 take the
// tests' larger padded order: 64^2 FP64 at 40 1670, 900.
CycleShape cycle_shape(const Table& t, int m_max, int cus) {
    const Inst& I = t.hinst[0];
    const int most = std::min(cus, CH_RES_MAX + CYC_TESTS) - CYC_TESTS;
    CycleShape c{0, 0};
    if (t.dim != 2 || t.ninst != 1 || m_max > CH_MSMALL) return c;
    if (strip_count(I.n, I.vx) > 4ll * I.wblk || I.wblk > CYC_GROUPS) return c;   // one strip per wave of the launches
    for (int ng : {1, 2, 3, 5}) {
        const int g = (I.wblk + ng - 1) / ng;
        if (g <= most) return {4 * ng, g + CYC_TESTS};
    }
    return c;
}

hipError_t launch_cycle(const Table& t, int prec, const DevBuffers& b, const CycleShape& c, int epoch, const double* y,
                        int m_max, hipStream_t s) {
    CycleArgs A{};
    A.ctl = b.ctl + t.hinst[0].slot;
    A.I = t.hinst[0];
    A.V = b.V;
    A.ldv = b.ldv;
    A.part = b.cyc;
    A.tot = b.cyc + (size_t)2 * CYC_PART;
    A.words = b.flags;
    A.dflags = b.dflag;
    A.epoch = epoch;
    A.G = c.workgroups - CYC_TESTS;
    A.m_max = m_max;
    A.wait_us = b.wait_us;
    const bool wide = prec == CH_FP64;
    A.y = wide ? static_cast<const void*>(y) : b.y32;
    switch (c.strips) {
        case 4: return wide ? launch_cycle_64_4(t, A, s) : launch_cycle_32_4(t, A, s);
        case 8: return wide ? launch_cycle_64_8(t, A, s) : launch_cycle_32_8(t, A, s);
        case 12: return wide ? launch_cycle_64_12(t, A, s) : launch_cycle_32_12(t, A, s);
        case 20: return wide ? launch_cycle_64_20(t, A, s) : launch_cycle_32_20(t, A, s);
        default: return hipErrorInvalidValue;
    }
}
