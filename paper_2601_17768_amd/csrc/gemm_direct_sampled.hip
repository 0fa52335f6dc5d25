// GEMM of more than 64 rows: LM head, sampled.
#include "gemm_direct.h"

template void gemm::launch_direct(int, const bf16x8*, const bf16x8*, int, const Range&, const Workspace&, const LogitsEpi<true>&, hipStream_t);
