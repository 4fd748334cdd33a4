// Resident Krylov cycles (ch_cycle.h): FP32 basis, twenty strips to a workgroup of ten waves.
#include "ch_cycle.h"

hipError_t launch_cycle_32_20(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<float, 10, 2>(t, A, s); }
