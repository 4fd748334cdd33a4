// Launches whose workgroups are all resident at once and exchange data while
// they run ("resident" launches), instead of one launch per exchange.
//
// The eight XCDs' L2 caches are not coherent with each other inside a launch.
// What one workgroup hands to another is therefore written and read with
// relaxed agent-scope atomics (write-through stores, loads that bypass stale
// lines); a workgroup waits until its stores are acknowledged, then raises
// its flag, and the reader polls the flag before it reads.  No cache is written back
// or invalidated, which is what makes a fence-based grid barrier slow here:
// measured per exchange, with all workgroups waiting for all others' flags,
// 0.9 us at 16 workgroups and 1.6 us at 256; cooperative-groups grid.sync()
// takes 26 us at 256; a kernel boundary 2.4-3 us plus the next launch's ramp.
//
// Every wait ends: after `wait_us` of waiting a workgroup gives up, raises
// the launch's failure word (which ends the others' waits) and the launch
// marks the run as not done; the host then repeats the cycle or step with ordinary
// launches, and keeps to them for a while (ch_pause.h).  The workgroups of a launch fit the
// device together because its host call holds a lease on that many CUs (ch_lease.h).
// The leases are this process's: another process on the device can make a wait run out.
#pragma once

#include "ch_internal.h"

// Most workgroups of a resident launch (one per CU).
#define CH_RES_MAX 256
// Words of a context that workgroups poll, each in a cache line of its own:
// one flag per workgroup, the failure word, the word that ends a Krylov cycle.
// Nothing clears them between launches: a launch owns the values above its
// `epoch`, up to the next launch's.
#define CH_RES_LINE 32
#define CH_RES_FAIL (CH_RES_MAX * CH_RES_LINE)
#define CH_RES_DONE (CH_RES_FAIL + CH_RES_LINE)
#define CH_RES_CHAIN (CH_RES_DONE + CH_RES_LINE)    // CH_MSMALL + 1 words: phi tests that did not end the cycle
#define CH_RES_WORDS (CH_RES_CHAIN + 2 * CH_RES_LINE)
// Status a resident launch leaves in the control block (with halted set)
// when a wait ran out: never returned to a caller.
#define CH_RES_RETRY 1000
#define CH_RES_WAIT_US 100000     // some fifty cycles
#define CH_RES_WAIT_MAX_US 10000000

#ifdef __HIPCC__
namespace {

__device__ __forceinline__ int res_load(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_store(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double res_load(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void res_store(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every store of this wave has reached the point where other XCDs see it.
__device__ __forceinline__ void res_drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// True when a wait that has polled `spin` times is to end: `wait_us` ran out
// since its first poll (t0) or another workgroup gave up.  Sets the failure
// word to the launch's epoch.
__device__ __forceinline__ bool res_expired(unsigned spin, long long& t0, int* fail, int epoch, unsigned wait_us) {
    if (spin & 63) return false;
    const long long now = (long long)wall_clock64();   // 100 MHz
    if (spin == 0) t0 = now;
    if (res_load(fail) != epoch && now - t0 < 100ll * wait_us) return false;
    res_store(fail, epoch);
    return true;
}

// Waits until *flag >= v; false when the wait expired.
__device__ __forceinline__ bool res_wait(const int* flag, int v, int* fail, int epoch, unsigned wait_us) {
    long long t0 = 0;
    for (unsigned spin = 0; res_load(flag) < v; ++spin) {
        if (res_expired(spin, t0, fail, epoch, wait_us)) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    return true;
}

// 16- and 8-byte accesses of a field as agent-scope stores and loads (bit 4 of
// the cache policy: sc1).  A 16-byte pair is not one atomic access: its
// reader waits for the writer's flag.
constexpr int RES_SC1 = 16;
__device__ __forceinline__ void res_store_pair(__amdgpu_buffer_rsrc_t r, unsigned bo, const double (&v)[2]) {
    using u32x4r = unsigned __attribute__((ext_vector_type(4)));
    struct P { double e[2]; };
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4r, P{{v[0], v[1]}}), r, bo, 0u, RES_SC1);
}
__device__ __forceinline__ void res_load_pair(__amdgpu_buffer_rsrc_t r, unsigned bo, double (&v)[2]) {
    struct P { double e[2]; };
    const P p = __builtin_bit_cast(P, __builtin_amdgcn_raw_buffer_load_b128(r, bo, 0u, RES_SC1));
    v[0] = p.e[0];
    v[1] = p.e[1];
}
__device__ __forceinline__ void res_store_one(__amdgpu_buffer_rsrc_t r, unsigned bo, double v) {
    using u32x2r = unsigned __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2r, v), r, bo, 0u, RES_SC1);
}
__device__ __forceinline__ double res_load_one(__amdgpu_buffer_rsrc_t r, unsigned bo) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, bo, 0u, RES_SC1));
}

}  // namespace
#endif

// Tiles of a resident LIM step: ntx x nty workgroups, `rows` rows of a tile's
// region per wave, `stages` stages per exchange; rows = 0: the grid does not fit.
struct LimTiles {
    int rows, stages, ntx, nty;
};
LimTiles lim_tiles(const Inst& I, int cus);
// All 2p - 1 stages of a LIM step of a single 2-D grid in one launch, from
// y^n (yin) to yout, p and the stage coefficients from the plan launch.  Uses
// LIM_EPOCHS values above `epoch`.
#define LIM_EPOCHS (2 * CH_PMAX)
hipError_t launch_lim_run(const Table& t, const DevBuffers& b, const LimTiles& g, int epoch, const double* yin,
                          double* yout, hipStream_t s);

// Resident Krylov cycle (ch_cycle.hip) of a single 2-D grid: strips per
// workgroup, workgroups in all; strips = 0: the grid or m_max does not fit.
struct CycleShape {
    int strips, workgroups;
};
CycleShape cycle_shape(const Table& t, int m_max, int cus);
size_t cycle_doubles();   // of DevBuffers::cyc
// All DCGS2 iterations and phi tests of a cycle begun by launch_after_resid or
// launch_step_end.  Uses CYCLE_EPOCHS values above `epoch`.
#define CYCLE_EPOCHS 128
hipError_t launch_cycle(const Table& t, int prec, const DevBuffers& b, const CycleShape& c, int epoch, const double* y,
                        int m_max, hipStream_t s);
