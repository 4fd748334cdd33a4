// Resident Krylov cycles (ch_cycle.h): FP64 basis, eight strips to a workgroup of eight waves.
#include "ch_cycle.h"

hipError_t launch_cycle_64_8(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<double, 8, 1>(t, A, s); }
