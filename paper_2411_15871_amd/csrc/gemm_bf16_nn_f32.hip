// The bf16 GEMM kernels, A [M,K] and B [K,N], float32 result (a source for each layout and result, so that they compile side by side).
#include "gemm_bf16.h"
template int launch_out<false, false, true>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
