// Persistent kernel of the variable-length RNN.
#include <hip/hip_runtime.h>
#include "amp_worker.hip.h"
#include "amp_batch.hip.h"
#include "amp_tree.hip.h"
#include "amp_rnn.hip.h"

static __device__ __forceinline__ void rnn_worker(const GQ AmpDev* D, const GQ WorkerDev* W) {
  if (W->role == ROLE_RNN_CELL) {
    // hidden = emb = 128 (8 row blocks, 16 column groups) has products with fixed trip counts
    if (D->node[1].rows == 128 && D->node[1].cols == 256 && D->node[1].seg0 == 128)
      role_rnn_cell<8, 16>(D, W);
    else
      role_rnn_cell<0, 0>(D, W);
  } else {
    role_rnn_out(D, W);
  }
}

AMP_PERSISTENT_KERNEL(rnn, rnn_worker(D, W);)
