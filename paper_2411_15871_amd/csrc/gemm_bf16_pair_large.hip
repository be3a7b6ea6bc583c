// The two gradient products of a linear layer in one launch, large tiles.
#include "gemm_bf16.h"
template int launch_pair<2>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
template int launch_pair<5>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
