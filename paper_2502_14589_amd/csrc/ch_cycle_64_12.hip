// Resident Krylov cycles (ch_cycle.h): FP64 basis, twelve strips to a workgroup of twelve waves.
#include "ch_cycle.h"

hipError_t launch_cycle_64_12(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<double, 12, 1>(t, A, s); }
