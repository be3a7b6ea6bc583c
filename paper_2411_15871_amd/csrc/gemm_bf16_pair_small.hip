// The two gradient products of a linear layer in one launch, small tiles.
#include "gemm_bf16.h"
template int launch_pair<3>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
template int launch_pair<7>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
template int launch_pair<8>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
