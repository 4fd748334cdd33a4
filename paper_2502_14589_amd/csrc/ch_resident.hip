// The stages of a LIM step of a single 2-D grid in one resident launch
// (ch_resident.h): the previous stage stays in registers, and only the edges
// of each workgroup's tile travel between workgroups.
#include "ch_resident.h"
#include "ch_rows.h"

#include <algorithm>

namespace {

constexpr int LIM_WAVES = 8, LIM_ROWS_MAX = 8;

// ---------------------------------------------------------------------------
// LIM stages (one iteration of Fig. 1 each):
//   y_next = (y^n + tau a_m z + tau (ghat - Ahat z)) / (1 + tau a_m)
// with the expressions of the strip kernels, in the same order, so the result
// is bit for bit theirs.
//
// A workgroup owns a tile of grid points and holds it with a halo of H = 2 S
// cells around it (S: stages per exchange; a stage reaches two cells) in the
// registers of NW waves: wave w has rows [w K, w K + K) of the region, lane L
// its columns 2L and 2L + 1.  Within a stage the x neighbours come by DPP
// whole-wave shifts and the rows of the waves above and below through LDS (two
// rows each way, one barrier per stage).  Each stage makes two more cells at
// the region's rim stale; after S stages the tile's own rim of H cells is
// written out, the neighbours' flags are awaited, and the halo is read back.
//
// What bounds it, per stage at 1024^2 (10 x 24 tiles, K = 8, S = 5: 2.4 us;
// two stages per launch took 4.7-5.1): about 2 us of the region's own work (FP64
// arithmetic 0.9, DPP shifts 0.3 and the waves' rows through LDS 0.3 at full overlap, the
// barriers), and a fifth of the 3 us that a round of stores, flag, wait and
// loads between neighbouring workgroups takes there.  At 64^2 (8 tiles) a
// stage takes 1.5 us, at 512^2 1.6 us; the launches 4.6 and 5.0.
// Rims packed through LDS into runs of whole lines were slower (two more
// barriers: 2.5 -> 3.3 us at 64^2), and so was polling the cells themselves instead of a flag (its
// loads compete with the stores they wait for: 3.1 -> 4.3 us at 1024^2).
// ---------------------------------------------------------------------------
// First row (column) of tile t of `nt` over n.
__device__ __forceinline__ int tile_first(int t, int nt, int n) { return (int)((long long)t * n / nt); }

template <int NW, int K, bool MOB>
__global__ __launch_bounds__(64 * NW, 1) void k_lim_run(Ctl* __restrict__ ctls, const Inst I, int ntx, int nty, int S,
                                                        const double* __restrict__ ybase, double* youtbase,
                                                        double* zbufbase, const double* __restrict__ coefs,
                                                        int* flags, int epoch, unsigned wait_us) {
    const int H = 2 * S;
    __shared__ double2 edge[2][NW][4][64];   // rows 0, 1, K - 2, K - 1 of each wave, two stages in turn
    __shared__ int dead;
    Ctl* ctl = ctls + I.slot;
    if (ctl->halted) return;
    const int n = I.n, bc = I.bc, eyre = I.eyre;
    const int stages = 2 * ctl->p - 1;
    const double tau = ctl->tau0;
    const double inv_h2 = I.inv_h2, e2ih2 = I.eps2 * I.inv_h2;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int tx = tile % ntx, ty = tile / ntx;
    const int x0 = tile_first(tx, ntx, n), tw = tile_first(tx + 1, ntx, n) - x0;
    const int y0 = tile_first(ty, nty, n), th = tile_first(ty + 1, nty, n) - y0;
    const double* Y = ybase + I.off;
    double* out = youtbase + I.off;
    double* zb = zbufbase + I.off;
    if (threadIdx.x == 0) dead = 0;

    // the wave's rows and the lane's columns: grid offsets of the cells of
    // the region (folded at the boundary), and which of them are the tile's own
    const int r0 = wv * K;
    int ro[K], co[2];
    bool ci[2], ce[2], cn[2];
#pragma unroll
    for (int a = 0; a < K; ++a) {
        const int i = r0 + a;
        ro[a] = i < th + 2 * H ? bc_index(y0 - H + i, n, bc) * n : 0;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int c = 2 * lane + e;
        cn[e] = c < tw + 2 * H;
        ci[e] = c >= H && c < H + tw;
        ce[e] = ci[e] && (c < 2 * H || c >= tw);
        co[e] = cn[e] ? bc_index(x0 - H + c, n, bc) : 0;
    }
    auto row_in = [&](int i) { return i >= H && i < H + th; };
    auto row_edge = [&](int i) { return i < 2 * H || i >= th; };
    // both columns of every lane of one kind, and neighbours in the grid: 16-byte accesses
    const bool pairs = __all(cn[0] == cn[1] && ci[0] == ci[1] && ce[0] == ce[1] && (!cn[0] || co[1] == co[0] + 1));

    // y^n, and d, c of Ahat_n and ghat^n on rows -1 .. K
    double z[K][2], y[K][2], d[K + 2][2], c[K + 2][2];
    MobRows<MOB, double, 2, K + 2> mb;
    const Mob mob = mob_of(ctl, MOB);
#pragma unroll
    for (int j = 0; j < K + 2; ++j) {
        const int i = r0 + j - 1;
        const bool in = i >= 0 && i < th + 2 * H;
        const int o = in ? bc_index(y0 - H + i, n, bc) * n : 0;
        double v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            v[e] = in && cn[e] ? Y[o + co[e]] : 0.0;
            d[j][e] = dcoef(v[e], eyre);
            c[j][e] = ccoef(v[e], eyre);
            if (j >= 1 && j <= K) z[j - 1][e] = y[j - 1][e] = v[e];
        }
        mb.set(j, v, mob.m0, mob.m1);
    }

    const double* cf = coefs + (size_t)I.slot * 2 * CH_PMAX * 2;
    // coefficients of 64 stages, one per lane, and of the next 64 on their way
    double cta = lane < stages ? cf[2 * lane] : 0.0, cinv = lane < stages ? cf[2 * lane + 1] : 0.0, nta, ninv;
    auto fetch = [&](int p0) {
        nta = p0 + lane < stages ? cf[2 * (p0 + lane)] : 0.0;
        ninv = p0 + lane < stages ? cf[2 * (p0 + lane) + 1] : 0.0;
    };
    fetch(64);
    auto stage = [&](int pos) {
        if (pos && (pos & 63) == 0) {
            cta = nta;
            cinv = ninv;
            fetch(pos + 64);
        }
        const double ta = readlane_d(cta, pos & 63), inv = readlane_d(cinv, pos & 63);
        double2(*E)[4][64] = edge[pos & 1];
        E[wv][0][lane] = double2{z[0][0], z[0][1]};
        E[wv][1][lane] = double2{z[1][0], z[1][1]};
        E[wv][2][lane] = double2{z[K - 2][0], z[K - 2][1]};
        E[wv][3][lane] = double2{z[K - 1][0], z[K - 1][1]};
        __syncthreads();
        double zr[K + 4][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            // the waves at the region's ends take any rows: theirs are stale there
            const double2 up = E[wv > 0 ? wv - 1 : wv][2 + r][lane], dn = E[wv < NW - 1 ? wv + 1 : wv][r][lane];
            zr[r][0] = up.x;
            zr[r][1] = up.y;
            zr[K + 2 + r][0] = dn.x;
            zr[K + 2 + r][1] = dn.y;
        }
#pragma unroll
        for (int a = 0; a < K; ++a)
#pragma unroll
            for (int e = 0; e < 2; ++e) zr[a + 2][e] = z[a][e];
        double q[K + 2][2];
#pragma unroll
        for (int j = 0; j < K + 2; ++j) {
            const double xl = wave_shift<DPP_WAVE_SHR1>(zr[j + 1][1]), xr = wave_shift<DPP_WAVE_SHL1>(zr[j + 1][0]);
#pragma unroll
            for (int e = 0; e < 2; ++e)
                q[j][e] = lim_inner(d[j][e], zr[j + 1][e], e2ih2,
                                    lap5<double, 2>(zr[j], zr[j + 1], zr[j + 2], xl, xr, e), c[j][e]);
        }
#pragma unroll
        for (int a = 0; a < K; ++a) {
            const double xl = wave_shift<DPP_WAVE_SHR1>(q[a + 1][1]), xr = wave_shift<DPP_WAVE_SHL1>(q[a + 1][0]);
            const double ml = mb.left(a + 1), mr = mb.right(a + 1);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const double op = lim_outer<MOB, 2>(q[a], q[a + 1], q[a + 2], xl, xr, mb.row(a), mb.row(a + 1),
                                                    mb.row(a + 2), ml, mr, e);
                z[a][e] = lim_next(y[a][e], ta, zr[a + 2][e], tau, inv_h2, op, inv);
            }
        }
    };

    // the neighbour this thread waits for (threads 0..8, the tile itself among
    // them; at a Neumann boundary the mirrored cells are the tile's own)
    const int* nflag = flags;
    if (threadIdx.x < 9) {
        int nx = tx + (int)threadIdx.x % 3 - 1, ny = ty + (int)threadIdx.x / 3 - 1;
        if (bc == CH_BC_NEUMANN) {
            nx = min(max(nx, 0), ntx - 1);
            ny = min(max(ny, 0), nty - 1);
        } else {
            nx = nx < 0 ? ntx - 1 : (nx == ntx ? 0 : nx);
            ny = ny < 0 ? nty - 1 : (ny == nty ? 0 : ny);
        }
        nflag = flags + (ny * ntx + nx) * CH_RES_LINE;
    }
    const int last = (stages + S - 1) / S - 1;   // exchanges
    const unsigned bytes = (unsigned)I.N * 8u;
    int pos = 0;
    for (int g = 1;; ++g) {
        for (int s = 0; s < S && pos < stages; ++s) stage(pos++);
        if (pos == stages) break;
        // Exchange g through zbuf and yout in turn, the last one through zbuf:
        // a workgroup that is done writes yout while a neighbour may still
        // read exchange `last`.  Before that, a buffer is written again only after
        // the neighbours' next flag, which they raise once they have read it.
        const __amdgpu_buffer_rsrc_t X = row_rsrc(((last - g) & 1) ? out : zb, bytes);
#pragma unroll
        for (int a = 0; a < K; ++a) {
            const int i = r0 + a;
            if (!row_in(i)) continue;
            if (pairs) {
                if (ci[0] && (row_edge(i) || ce[0])) res_store_pair(X, (unsigned)(ro[a] + co[0]) * 8u, z[a]);
            } else {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (ci[e] && (row_edge(i) || ce[e])) res_store_one(X, (unsigned)(ro[a] + co[e]) * 8u, z[a][e]);
            }
        }
        res_drain();
        __syncthreads();
        if (threadIdx.x == 0) res_store(flags + tile * CH_RES_LINE, epoch + g);
        if (threadIdx.x < 9 && !res_wait(nflag, epoch + g, flags + CH_RES_FAIL, epoch, wait_us)) dead = 1;
        __syncthreads();
        if (dead) {   // the host repeats the step: nothing here is kept
            if (threadIdx.x == 0) {
                ctl->status = CH_RES_RETRY;
                ctl->halted = 1;
            }
            return;
        }
#pragma unroll
        for (int a = 0; a < K; ++a) {
            const int i = r0 + a;
            if (i >= th + 2 * H) continue;
            if (pairs) {
                if (cn[0] && !(row_in(i) && ci[0])) res_load_pair(X, (unsigned)(ro[a] + co[0]) * 8u, z[a]);
            } else {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (cn[e] && !(row_in(i) && ci[e])) z[a][e] = res_load_one(X, (unsigned)(ro[a] + co[e]) * 8u);
            }
        }
    }
#pragma unroll
    for (int a = 0; a < K; ++a)
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (row_in(r0 + a) && ci[e]) out[ro[a] + co[e]] = z[a][e];
}

template <int K>
void launch_lim_run_k(const Table& t, const DevBuffers& b, const LimTiles& g, int epoch, const double* yin,
                      double* yout, hipStream_t s) {
    const dim3 grid(g.ntx * g.nty), block(64 * LIM_WAVES);
    if (mobility(t))
        hipLaunchKernelGGL((k_lim_run<LIM_WAVES, K, true>), grid, block, 0, s, b.ctl, t.hinst[0], g.ntx, g.nty, g.stages,
                           yin, yout, b.zbuf, b.lcoef, b.flags, epoch, b.wait_us);
    else
        hipLaunchKernelGGL((k_lim_run<LIM_WAVES, K, false>), grid, block, 0, s, b.ctl, t.hinst[0], g.ntx, g.nty, g.stages,
                           yin, yout, b.zbuf, b.lcoef, b.flags, epoch, b.wait_us);
}

}  // namespace

// The tiles with the smallest predicted time per stage among those that fit
// the device, one workgroup per CU: taller tiles (K) cost their rows, more
// stages per exchange (S) amortise it and widen the halo.  Fitted to a sweep of all
// (K, S) that fit at fifteen sides from 48 to 1300; the choice was the
// measured best or within 5% of it at each (1024^2: K = 8, S = 5 predicted 2.55 us,
// measured 2.44; K = 6, S = 2: 3.03 and 3.08).  Larger grids (from about 1310^2) do not fit
// and take the strip launches.
LimTiles lim_tiles(const Inst& I, int cus) {
    const int n = I.n, most = std::min(cus, CH_RES_MAX);
    LimTiles best{0, 0, 0, 0};
    double best_us = 0.0;
    for (int K = 2; K <= LIM_ROWS_MAX; ++K)
        for (int S = 1; S <= 8; ++S) {
            const int H = 2 * S, tw = 128 - 2 * H, th = LIM_WAVES * K - 2 * H;
            if (th < 1) continue;
            const int ntx = (n + tw - 1) / tw, nty = (n + th - 1) / th;
            if (n / ntx < H || n / nty < H || ntx * nty > most) continue;   // a neighbour's rim is one tile deep
            const double us = 0.45 + 0.19 * K + (1.7 + 1.3 * (ntx * nty) / 256.0) / S;
            if (best.rows == 0 || us < best_us) {
                best = {K, S, ntx, nty};
                best_us = us;
            }
        }
    return best;
}

hipError_t launch_lim_run(const Table& t, const DevBuffers& b, const LimTiles& g, int epoch, const double* yin,
                          double* yout, hipStream_t s) {
    switch (g.rows) {
        case 2: launch_lim_run_k<2>(t, b, g, epoch, yin, yout, s); break;
        case 3: launch_lim_run_k<3>(t, b, g, epoch, yin, yout, s); break;
        case 4: launch_lim_run_k<4>(t, b, g, epoch, yin, yout, s); break;
        case 5: launch_lim_run_k<5>(t, b, g, epoch, yin, yout, s); break;
        case 6: launch_lim_run_k<6>(t, b, g, epoch, yin, yout, s); break;
        case 7: launch_lim_run_k<7>(t, b, g, epoch, yin, yout, s); break;
        case 8: launch_lim_run_k<8>(t, b, g, epoch, yin, yout, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
