// Resident Krylov cycles (ch_cycle.h): FP32 basis, twelve strips to a workgroup of twelve waves.
#include "ch_cycle.h"

hipError_t launch_cycle_32_12(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<float, 12, 1>(t, A, s); }
