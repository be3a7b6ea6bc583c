// The two gradient products of a linear layer in one launch, mid tiles.
#include "gemm_bf16.h"
template int launch_pair<1>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
template int launch_pair<4>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
template int launch_pair<6>(const GemmArgs&, const GemmArgs&, bool, hipStream_t, int, const BiasGrad*, bool*);
