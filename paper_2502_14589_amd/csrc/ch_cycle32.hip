// Resident Krylov cycles (ch_cycle.h): the kernels of an FP32 basis.
#include "ch_cycle.h"

hipError_t launch_cycle_32(const Table& t, int strips, const CycleArgs& A, hipStream_t s) {
    return launch_cycle_p<float>(t, strips, A, s);
}
