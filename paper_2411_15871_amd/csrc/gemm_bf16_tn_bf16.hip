// The bf16 GEMM kernels, A [K,M] and B [K,N], bf16 result (a source for each layout and result, so that they compile side by side).
#include "gemm_bf16.h"
template int launch_out<true, false, false>(const GemmArgs&, int, int, hipStream_t, int, int, int, const GemmAr*);
