// Resident Krylov cycles (ch_cycle.h): FP32 basis, eight strips to a workgroup of eight waves.
#include "ch_cycle.h"

hipError_t launch_cycle_32_8(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<float, 8, 1>(t, A, s); }
