// Persistent kernel of the pipelined MLP.
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_mlp.hip.h"

AMP_PERSISTENT_KERNEL(mlp, role_mlp_lin(D, W);)
