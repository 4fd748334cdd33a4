// Resident Krylov cycles (ch_cycle.h): FP64 basis, four strips to a workgroup of four waves.
#include "ch_cycle.h"

hipError_t launch_cycle_64_4(const Table& t, const CycleArgs& A, hipStream_t s) { return launch_cycle_n<double, 4, 1>(t, A, s); }
