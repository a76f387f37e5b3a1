// Persistent kernel of the pipelined MLP.  256 threads: a message is one small matrix-vector product, most of whose
// instructions every wave executes whatever its share, so one wave per SIMD gets through it sooner than two.
#define AMP_THREADS 256
#define AMP_BOUNDED_FETCHED
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_mlp.hip.h"
#include "amp_mlp_one.hip.h"

AMP_PERSISTENT_KERNEL(mlp, mlp_one_fits(D), if (W->role == ROLE_CTRL) role_mlp_whole(D, W); else role_mlp_lin(D, W);)
