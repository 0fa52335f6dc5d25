// GEMM of more than 64 rows: gate/up projection.
#include "gemm_direct.h"

template void gemm::launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const SwigluEpi&, hipStream_t);
